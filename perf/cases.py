"""The work this library is used for, as cases that can be timed and checked.

Every case goes through the public entry points of ``efgpu`` on seeded
synthetic graphs of the families the tests and the benchmark use:
Erdos-Renyi, Barabasi-Albert, R-MAT, Watts-Strogatz and the erased
configuration model. The kinds of work:

  score_new   a graph the program has just read (host CSR, validated, or a
              host edge list): load it, score every node, results on the host
  score       a graph kept in device memory: score every node, device outputs
  seeds       exact EF of chosen nodes of a kept graph, results on the host
  batch       many small graphs kept as one batch, replayed, device outputs
  topk        the k key nodes from EF already on the device, on the host
  predict     the learned surrogate's EF of every node, device output
  train       a new surrogate fitted to labelled rows; its weights
  sir         simulated outbreaks and the spreading power of every node
  j3          EF with three transmission events, device outputs
"""
import math

import numpy as np
import torch

from paper_2306_00606_amd import efgpu, gen

# about this many event sequences can be listed in double precision in a few
# seconds; larger graphs have no reference value here
EXACT_EVENTS = 1_500_000_000
EXACT_EVENTS_J3 = 60_000_000


def listed():
    return [
        # one contact network of a study, read as an edge list and scored once
        # (the Erdos-Renyi workload: n = 1000, mean degree 8), in double precision
        {"name": "new_er1000", "op": "score_new", "family": "er", "n": 1000, "k": 8.0,
         "source": "edges", "algo": "cluster", "prec": "fp64"},
        # a network of 10^6 edges, read as CSR, checked, loaded and scored once
        {"name": "new_ba200k", "op": "score_new", "family": "ba", "n": 200_003, "m": 5,
         "source": "csr", "algo": "cluster", "prec": "fp32c"},
        # a small network kept on the device and scored again and again: the
        # latency of a call
        {"name": "score_er1000", "op": "score", "family": "er", "n": 1000, "k": 8.0,
         "algo": "cluster", "prec": "fp32c"},
        # the Barabasi-Albert workload, 5 * 10^6 edges, in double precision
        {"name": "score_ba1m_fp64", "op": "score", "family": "ba", "n": 1_000_000, "m": 5,
         "algo": "cluster", "prec": "fp64"},
        # the benchmark's graph: R-MAT scale 22, 4 * 10^7 edges, hubs of 10^5
        # neighbours
        {"name": "score_rmat22", "op": "score", "family": "rmat", "scale": 22, "ef": 10,
         "algo": "cluster", "prec": "fp32c"},
        # exact scores of nodes somebody asks about, or of another method's
        # candidates (the original per-seed formulation)
        {"name": "seeds_rmat18", "op": "seeds", "family": "rmat", "scale": 18, "ef": 10,
         "seeds": 1000, "prec": "fp32c"},
        # an ensemble of sampled networks scored together
        {"name": "batch_64", "op": "batch", "graphs": 64, "n_lo": 1000, "n_hi": 20_000,
         "prec": "fp32c"},
        # the key nodes of a large network from its scores
        {"name": "topk_4m", "op": "topk", "n": 4_000_000, "top": 1000},
        # quick ranking of a large network by the surrogate (BA, m = 8)
        {"name": "predict_ba1m", "op": "predict", "n": 1_000_000, "m": 8},
        # a surrogate fitted to a labelled sample, two epochs of the default batch
        {"name": "train_100k", "op": "train", "rows": 100_000, "batch": 4096, "epochs": 2},
        # spreading checked by simulation at the paper's calibration
        {"name": "sir_ba100k", "op": "sir", "n": 100_000, "m": 5, "sims": 100},
        # three transmission events on a graph of moderate degrees
        {"name": "j3_ba100k", "op": "j3", "family": "ba", "n": 100_000, "m": 5,
         "prec": "fp32c"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["score_new", "score_new", "score", "score", "score", "seeds", "batch", "topk",
                     "predict", "train", "sir", "j3"])
    if op == "score_new":
        c = _draw_graph(rng, 300, 200_000)
        return {"op": op, **c, "source": rng.choice(["csr", "edges"]), "algo": "cluster",
                "prec": rng.choice(["fp32c", "fp64"])}
    if op == "score":
        algo = rng.choice(["cluster", "cluster", "cluster", "per_seed", "cluster_agg"])
        c = _draw_graph(rng, 300, 50_000 if algo == "per_seed" else 1_000_000)
        return {"op": op, **c, "algo": algo, "prec": rng.choice(["fp32c", "fp32c", "fp64"])}
    if op == "seeds":
        return {"op": op, **_draw_graph(rng, 2000, 250_000), "seeds": _log(rng, 1, 4096),
                "prec": rng.choice(["fp32c", "fp64"])}
    if op == "batch":
        lo = _log(rng, 200, 5000)
        return {"op": op, "graphs": _log(rng, 2, 64), "n_lo": lo, "n_hi": 4 * lo,
                "prec": rng.choice(["fp32c", "fp32c", "fp64"])}
    if op == "topk":
        n = _log(rng, 1000, 4_000_000)
        return {"op": op, "n": n, "top": min(_log(rng, 10, 40_000), n)}
    if op == "predict":
        return {"op": op, "n": _log(rng, 2000, 1_000_000), "m": rng.randint(2, 10)}
    if op == "train":
        return {"op": op, "rows": _log(rng, 3000, 100_000),
                "batch": rng.choice([1024, 2048, 4096]), "epochs": rng.randint(1, 2)}
    if op == "sir":
        return {"op": op, "n": _log(rng, 1000, 100_000), "m": rng.randint(2, 8),
                "sims": rng.randint(10, 100)}
    n, prec = _log(rng, 500, 100_000), rng.choice(["fp32c", "fp32c", "fp64"])
    if rng.random() < 0.5:
        return {"op": op, "family": "er", "n": n, "k": round(rng.uniform(4, 12), 2), "prec": prec}
    return {"op": op, "family": "ba", "n": n, "m": rng.randint(2, 5), "prec": prec}


def _draw_graph(rng, lo, hi):
    family = rng.choice(["er", "ba", "rmat", "rmat"])
    if family == "er":
        return {"family": family, "n": _log(rng, lo, hi), "k": round(rng.uniform(4, 16), 2)}
    if family == "ba":
        return {"family": family, "n": _log(rng, lo, hi), "m": rng.randint(2, 10)}
    return {"family": family, "scale": rng.randint(int(math.log2(lo)), int(math.log2(hi))),
            "ef": rng.randint(4, 16)}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _rmat(scale, ef, seed):
    """R-MAT (a .57, b .19, c .19, d .05) with shuffled ids as a simple
    undirected CSR, drawn on the device (the host generator takes many
    seconds at scale 22)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    n, e = 1 << scale, ef << scale
    src = torch.zeros(e, dtype=torch.int32, device="cuda")
    dst = torch.zeros_like(src)
    for _ in range(scale):
        u = torch.rand(e, generator=g, device="cuda")
        src = 2 * src + (u >= 0.76).int()
        dst = 2 * dst + (((u >= 0.57) & (u < 0.76)) | (u >= 0.95)).int()
    perm = torch.randperm(n, generator=g, device="cuda", dtype=torch.int64)
    src, dst = perm[src.long()], perm[dst.long()]
    keep = src != dst
    src, dst = src[keep], dst[keep]
    key = torch.unique(torch.cat([src * n + dst, dst * n + src]))
    rp = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rp[1:] = torch.cumsum(torch.bincount(key // n, minlength=n), 0).int()
    return rp, (key % n).int()


def _seed(seed):
    """A seed for the host generators: theirs of neighbouring seeds are one
    stream, a draw apart."""
    return int(np.random.default_rng(seed).integers(1, 2 ** 62))


def _graph(case, seed):
    """(row_ptr, col_idx): int32, on the device for R-MAT, else on the host."""
    if case["family"] == "rmat":
        return _rmat(case["scale"], case["ef"], seed)
    if case["family"] == "er":
        return gen.erdos_renyi(case["n"], case["k"] / (case["n"] - 1), _seed(seed))
    return gen.barabasi_albert(case["n"], case["m"], _seed(seed))


def _host(rp, ci):
    return tuple(x.cpu().numpy() if torch.is_tensor(x) else x for x in (rp, ci))


def _outputs(n):
    return (torch.empty(n, dtype=torch.float64, device="cuda"),
            torch.empty(n, dtype=torch.int64, device="cuda"),
            torch.empty(n, dtype=torch.int64, device="cuda"))


def _batch_graphs(case, seed):
    """Half Watts-Strogatz, half configuration model, as the batch workload
    (the sizes go with the case)."""
    rs, size = np.random.default_rng(seed), np.random.default_rng(case["graphs"])
    out = []
    for i in range(case["graphs"]):
        n = int(size.integers(case["n_lo"], case["n_hi"] + 1))
        s = int(rs.integers(1, 2 ** 62))
        if i % 2 == 0:
            out.append(gen.watts_strogatz(n, int(rs.choice([4, 6, 8, 10])),
                                          float(rs.uniform(0.01, 0.3)), s))
        else:
            out.append(gen.config_model(n, float(rs.uniform(2.1, 3.0)), s))
    return out


def _ef_values(n, seed):
    """EF-like scores: a bell of ln-sized values, some of them shared by many
    nodes of the same neighbourhood, and zeros for nodes without clusters."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    v = 6.0 + 1.2 * torch.randn(n, generator=g, device="cuda", dtype=torch.float64)
    u = torch.rand(n, generator=g, device="cuda")
    v = torch.where(u < 0.3, torch.round(v * 64) / 64, v)
    return torch.where(u > 0.95, torch.zeros_like(v), v).clamp_(min=0.0)


def _train_rows(case, seed):
    """Feature rows and targets shaped like the labelled sets: correlated
    log-degree features and a smooth positive residual with noise."""
    rs = np.random.default_rng(seed)
    base = rs.normal(0, 1, (case["rows"], 4))
    X = base @ rs.normal(0, 1, (4, 16)) + 0.3 * rs.normal(0, 1, (case["rows"], 16))
    X += rs.uniform(0, 8, 16)
    y = np.abs(0.2 + 0.1 * np.sin(base[:, 0]) + 0.05 * base[:, 1]) + 0.01 * rs.normal(0, 1, case["rows"])
    return X.astype(np.float32), y.astype(np.float32)


def prepare(case, seed):
    op = case["op"]
    st = {"case": case, "seed": seed}
    if op == "score_new":
        rp, ci = _host(*_graph(case, seed))
        if case["source"] == "edges":
            src = np.repeat(np.arange(rp.size - 1, dtype=np.int32), np.diff(rp))
            once = src < ci
            order = np.random.default_rng(seed).permutation(int(once.sum()))
            st["n"], st["src"], st["dst"] = rp.size - 1, src[once][order], ci[once][order]
        else:
            st["rp"], st["ci"] = rp, ci
    elif op in ("score", "seeds", "j3"):
        rp, ci = _graph(case, seed)
        st["graph"] = efgpu.Graph(rp, ci, validate=False)
        if op == "seeds":
            st["seeds"] = np.random.default_rng(seed).integers(0, st["graph"].n, case["seeds"]).astype(np.int32)
        else:
            st["out"] = _outputs(st["graph"].n)
    elif op == "batch":
        st["batch"] = efgpu.Batch(_batch_graphs(case, seed))
        st["batch"].autotune(case["prec"])
        st["out"] = _outputs(st["batch"].n)
    elif op == "topk":
        st["ef"] = _ef_values(case["n"], seed)
        # a handle of a graph of n nodes; the selection reads the scores alone
        rp = np.zeros(case["n"] + 1, np.int32)
        st["graph"] = efgpu.Graph(rp, np.zeros(0, np.int32), validate=False)
    elif op == "predict":
        rp, ci = gen.barabasi_albert(case["n"], case["m"], _seed(seed))
        st["graph"] = efgpu.Graph(rp, ci, validate=False)
        st["sur"] = efgpu.Surrogate()
        st["sur"].set_params(*_weights(rp, ci, seed))
        st["out"] = torch.empty(case["n"], dtype=torch.float64, device="cuda")
    elif op == "train":
        st["X"], st["y"] = _train_rows(case, seed)
    elif op == "sir":
        rp, ci = gen.barabasi_albert(case["n"], case["m"], _seed(seed))
        st["graph"] = efgpu.Graph(rp, ci, validate=False)
        st["beta"] = 1.3 / (3.0 * ci.size / case["n"])
    return st


def _weights(rp, ci, seed):
    """Random weights (He-normal), features standardised as training leaves
    them: (params, mean, inv_std)."""
    X, _ = _exact_features(_Plain(rp, ci))
    std = X.std(0, unbiased=False).clamp(min=1e-6)
    rs = np.random.default_rng(seed)
    p = np.concatenate([rs.normal(0, (2 / 16) ** 0.5, 1024), np.zeros(64),
                        rs.normal(0, (2 / 64) ** 0.5, 4096), np.zeros(64),
                        rs.normal(0, (1 / 64) ** 0.5, 64), np.zeros(1)])
    return tuple(t.astype(np.float32) for t in (p, X.mean(0).cpu().numpy(), (1.0 / std).cpu().numpy()))


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(st):
    case = st["case"]
    op = case["op"]
    if op == "score_new":
        if case["source"] == "edges":
            g = efgpu.Graph.from_edges(st["n"], st["src"], st["dst"])
        else:
            g = efgpu.Graph(st["rp"], st["ci"])
        with g:
            return g.compute(algo=case["algo"], prec=case["prec"])
    if op == "score":
        return st["graph"].compute(algo=case["algo"], prec=case["prec"], out=st["out"])
    if op == "seeds":
        return st["graph"].compute(prec=case["prec"], seeds=st["seeds"])
    if op == "batch":
        return st["batch"].compute(prec=case["prec"], out=st["out"])
    if op == "topk":
        return st["graph"].topk_values(st["ef"], case["top"])
    if op == "predict":
        return st["sur"].predict(st["graph"], out=st["out"])
    if op == "train":
        sur = efgpu.Surrogate(seed=st["seed"])
        rep = sur.train(st["X"], st["y"], batch=case["batch"], epochs=case["epochs"], seed=st["seed"])
        out = sur.params()
        sur.close()
        return {"params": out[0], "mean": out[1], "inv_std": out[2],
                "train_loss": np.float32(rep["train_loss"]), "val_loss": np.float32(rep["val_loss"])}
    if op == "sir":
        return st["graph"].sir(st["beta"], 1.0 / 3.0, st["seed"], case["sims"])
    return st["graph"].compute(prec=case["prec"], j=3, out=st["out"])


# ---------------------------------------------------------------------------
# what one pass cannot do without
# ---------------------------------------------------------------------------
def _size(case):
    """Nodes, arcs and clusters (pairs of neighbours of a node) to expect."""
    fam = case.get("family", "ba")
    if fam == "rmat":
        n, e = 1 << case["scale"], float(case["ef"] << case["scale"])
        # sum of squared endpoint probabilities is 0.6352^scale; about a
        # third of the pairs go with the repeated edges
        return n, 1.93 * e, max(2.0 * e, 1.3 * e * e * 0.6352 ** case["scale"])
    if fam == "er":
        return case["n"], case["n"] * case["k"], 0.5 * case["n"] * case["k"] ** 2
    n, m = case["n"], case["m"]
    return n, 2.0 * n * m, 0.55 * n * m * (m + 1) * math.log(n)


def work(case):
    op = case["op"]
    if op == "topk":
        return {"bytes": 8.0 * case["n"] + 12.0 * case["top"], "flops": 0.0}
    if op == "train":  # every row read once an epoch; forward and backward
        rows = case["rows"] * case["epochs"]
        return {"bytes": 68.0 * rows, "flops": 6.0 * 5184 * rows}
    if op == "batch":
        n = 0.5 * case["graphs"] * (case["n_lo"] + case["n_hi"])
        return {"bytes": 4.0 * (n + 5.5 * n) + 24.0 * n, "flops": 5.0 * 40.0 * n}
    n, nnz, w = _size(case)
    csr = 4.0 * (n + 1 + nnz)
    if op == "seeds":  # two-hop walks: 4 clusters' event sequences a cluster
        share = min(1.0, case["seeds"] / n)
        return {"bytes": share * (4.0 * w * 4) + 28.0 * case["seeds"], "flops": share * 20.0 * w}
    if op == "predict":
        return {"bytes": csr + 8.0 * n, "flops": 2.0 * 5184 * n + 40.0 * nnz}
    if op == "sir":  # an outbreak walks the arcs of those it infects, about three steps each
        return {"bytes": 0.15 * case["sims"] * 3 * csr + 40.0 * n, "flops": 0.15 * case["sims"] * 3 * 54.0 * nnz}
    if op == "j3":
        return {"bytes": csr + 24.0 * n, "flops": 40.0 * w * math.sqrt(w / n)}
    return {"bytes": csr + 24.0 * n, "flops": 5.0 * w}


# ---------------------------------------------------------------------------
# the same in 64 bits, from the definitions
# ---------------------------------------------------------------------------
class _Plain:
    """A CSR as int64 tensors with an adjacency test."""

    def __init__(self, rp, ci):
        dev = "cuda" if torch.cuda.is_available() else "cpu"
        self.rp = torch.as_tensor(rp).to(dev).long()
        self.ci = torch.as_tensor(ci).to(dev).long()
        self.n = self.rp.numel() - 1
        self.k = self.rp[1:] - self.rp[:-1]
        self.src = torch.repeat_interleave(torch.arange(self.n, device=dev), self.k)
        self.keys = self.src * self.n + self.ci
        self.dev = dev

    def adjacent(self, a, b):
        q = a * self.n + b
        i = torch.searchsorted(self.keys, q).clamp_(max=max(self.keys.numel() - 1, 0))
        return self.keys[i] == q

    def expand(self, x):
        """Every (i, y): y a neighbour of x[i]."""
        k = self.k[x]
        i = torch.repeat_interleave(torch.arange(x.numel(), device=self.dev), k)
        off = torch.arange(i.numel(), device=self.dev) - (torch.cumsum(k, 0) - k)[i]
        return i, self.ci[self.rp[x[i]] + off]


def _segments(x, lengths):
    """Row-wise sums over consecutive segments of x (rows x entries, float64)."""
    return torch.stack([torch.segment_reduce(r.contiguous(), "sum", lengths=lengths, initial=0.0)
                        for r in x])


def _sums(d, on, lengths):
    """Per segment: number of clusters, sum of their degrees d, sum of d ln d
    (rows; whole numbers below 2^53 are exact)."""
    d = torch.where(on, d, torch.zeros_like(d)).double()
    return _segments(torch.stack([on.double(), d, d * torch.log(d.clamp(min=1.0))]), lengths)


def _eq1(N, D, S):
    """(EF, D, N) from the sums."""
    ef = torch.log(D.clamp(min=1.0)) - S / D.clamp(min=1.0)
    ef = torch.where((D > 0) & (N > 1), ef.clamp(min=0.0), torch.zeros_like(ef))
    return ef, D.long(), N.long()


def _exact_ef(P, seeds=None):
    """EF, D and N of two events, by listing every event sequence."""
    pos = torch.arange(P.n, device=P.dev) if seeds is None else torch.arange(len(seeds), device=P.dev)
    node = pos if seeds is None else torch.as_tensor(seeds, device=P.dev).long()
    i, a = P.expand(node)
    ksum = P.k[node][i] + P.k[a]
    if float(ksum.double().sum()) > EXACT_EVENTS:
        return None
    # per arc of a seed first, then per seed: the sequences of an arc s -> a
    # whose second infection is by s, and by a
    arcs = []
    ends = torch.cumsum(ksum, 0)
    lo = 0
    while lo < i.numel():
        base = int(ends[lo - 1]) if lo else 0
        hi = max(lo + 1, int(torch.searchsorted(ends, base + (1 << 26), right=True)))
        aa = a[lo:hi]
        s = node[i[lo:hi]]
        by_arc = 0
        for centre, other in ((s, aa), (aa, s)):
            j, b = P.expand(centre)
            on = (b != s[j]) & (b != aa[j])
            d = P.k[s[j]] + P.k[aa[j]] + P.k[b] - 4 - 2 * P.adjacent(b, other[j]).long()
            by_arc = by_arc + _sums(d, on, P.k[centre])
        arcs.append(by_arc)
        lo = hi
    if not arcs:
        return _eq1(*_sums(node, node < 0, torch.zeros_like(node)).unbind())
    return _eq1(*_segments(torch.cat(arcs, 1), P.k[node]).unbind())


def _exact_j3(P):
    """EF, D and N of three events, by listing every event sequence."""
    # arcs, then second events, then third events
    e = torch.arange(P.src.numel(), device=P.dev)
    s, y = P.src, P.ci
    parts = []
    for x in (s, y):
        j, z = P.expand(x)
        keep = (z != s[j]) & (z != y[j])
        parts.append((e[j[keep]], z[keep]))
    e = torch.cat([p[0] for p in parts])
    z = torch.cat([p[1] for p in parts])
    s, y = s[e], y[e]
    if float((P.k[s] + P.k[y] + P.k[z]).double().sum()) > EXACT_EVENTS_J3:
        return None
    e3 = 1 + P.adjacent(s, z).long() + P.adjacent(y, z).long()
    total = torch.zeros(3, P.n, dtype=torch.float64, device=P.dev)
    for x in (s, y, z):
        j, w = P.expand(x)
        on = (w != s[j]) & (w != y[j]) & (w != z[j])
        inner = e3[j] + sum(P.adjacent(t[j], w).long() for t in (s, y, z))
        d = P.k[s[j]] + P.k[y[j]] + P.k[z[j]] + P.k[w] - 2 * inner
        total.index_add_(1, s, _sums(d, on, P.k[x]))
    return _eq1(*total.unbind())


def _exact_features(P):
    """The surrogate's 16 features and ln N, closed forms per arc in float64."""
    n, k = P.n, P.k.double()

    def nbr(x):
        return _segments(x[None], P.k)[0]

    s, a = P.src, P.ci
    ks, ka = k[s], k[a]
    m = [nbr(ka ** j) for j in (1, 2, 3, 4)]
    A, B, Q = m[0], m[1], nbr(m[0][a])
    N = k * k - 2 * k + A
    D = k * (k - 1) * (k - 4) + 2 * (k - 1) * A + (k - 4) * (A - k) + (B - A) + (Q - k * k)
    c, cnt = ks + ka - 4, ks + ka - 2
    p = [m[j][s] - ka ** (j + 1) + m[j][a] - ks ** (j + 1) for j in range(4)]
    r = [nbr(cnt * c ** 2 + 2 * c * p[0] + p[1]),
         nbr(cnt * c ** 3 + 3 * c ** 2 * p[0] + 3 * c * p[1] + p[2]),
         nbr(cnt * c ** 4 + 4 * c ** 3 * p[0] + 6 * c ** 2 * p[1] + 4 * c * p[2] + p[3])]
    ok = (N > 0) & (D > 0)
    q = torch.where(ok, N / D.clamp(min=1), torch.ones_like(N))
    r = [r[j] * q ** (j + 2) / N.clamp(min=1) for j in range(3)]
    zero = torch.zeros_like(N)
    m2 = torch.where(ok, r[0] - 1, zero)
    m3 = torch.where(ok, r[1] - 3 * r[0] + 2, zero)
    m4 = torch.where(ok, r[2] - 4 * r[1] + 6 * r[0] - 3, zero)
    lk = torch.log(ka)
    has, kk = k > 0, k.clamp(min=1)
    mx = torch.where(has, torch.segment_reduce(lk, "max", lengths=P.k), zero)
    mn = torch.where(has, torch.segment_reduce(lk, "min", lengths=P.k), zero)
    mean = nbr(lk) / kk
    std = torch.sqrt((nbr(lk * lk) / kk - mean * mean).clamp(min=0))
    F = [torch.log1p(k), torch.log1p(A), torch.log1p(B), torch.asinh(m3), torch.asinh(m4),
         torch.log1p(A - k), torch.log1p(N), torch.log1p(D),
         torch.where(ok, torch.log(D.clamp(min=1) / N.clamp(min=1)), zero), mx, mn, mean, std,
         torch.log1p(Q), nbr((ka == 1).double()) / kk, torch.log1p(m2.clamp(min=0))]
    return torch.stack(F, 1), torch.where(N > 0, torch.log(N.clamp(min=1)), zero)


def _exact_predict(P, params, mean, inv_std):
    X, lnN = _exact_features(P)
    p, mean, inv_std = (torch.as_tensor(t).to(P.dev).double() for t in (params, mean, inv_std))
    W1, b1, W2, b2, w3, b3 = (t for t in torch.split(p, [1024, 64, 4096, 64, 64, 1]))
    gelu = torch.nn.functional.gelu
    h = gelu((X - mean) * inv_std @ W1.view(16, 64) + b1, approximate="tanh")
    h = gelu(h @ W2.view(64, 64) + b2, approximate="tanh")
    return (lnN - h @ w3 - b3).clamp(min=0.0)


def exact(case, seed):
    op = case["op"]
    if op in ("train", "sir"):  # a trajectory of 16-bit steps; whole numbers only
        return None
    if op == "topk":
        v = _ef_values(case["n"], seed)
        order = torch.sort(v, descending=True, stable=True)[1][:case["top"]]
        return order.int(), v[order]
    if op in ("score", "score_new", "seeds") and 4 * _size(case)[2] * (
            min(1.0, case["seeds"] / _size(case)[0]) if op == "seeds" else 1.0) > EXACT_EVENTS:
        return None
    if op == "j3" and 3 * _size(case)[1] * (case["k"] if case["family"] == "er" else case["m"]) ** 2 > EXACT_EVENTS_J3:
        return None
    if op == "batch":
        _, rp, ci = efgpu.union_csr(_batch_graphs(case, seed))
        return _exact_ef(_Plain(rp, ci))
    if op == "predict":
        rp, ci = gen.barabasi_albert(case["n"], case["m"], _seed(seed))
        return _exact_predict(_Plain(rp, ci), *_weights(rp, ci, seed))
    P = _Plain(*_graph(case, seed))
    if op == "j3":
        return _exact_j3(P)
    if op == "seeds":
        return _exact_ef(P, np.random.default_rng(seed).integers(0, P.n, case["seeds"]))
    return _exact_ef(P)
