"""FP64 scores from tables (needs an MI355X): centres of every bin whose
cluster degrees lie below, across and above the 8192 table entries, against
the CPU oracle; and the same sums when there is no memory for the table."""
import os

import numpy as np
import pytest

import oracle
from paper_2306_00606_amd import efgpu, gen

pytestmark = pytest.mark.gpu


def hubs_graph(hub_degrees, centre_degree, seed):
    """Hubs with leaves of their own, all joined to one centre that has further
    leaves up to centre_degree, some of which are joined to each other."""
    rs = np.random.default_rng(seed)
    src, dst = [], []
    nxt = 1
    for k in hub_degrees:
        h = nxt
        nxt += 1
        src.append(0)
        dst.append(h)
        src += [h] * (k - 1)
        dst += range(nxt, nxt + k - 1)
        nxt += k - 1
    rest = list(range(nxt, nxt + max(centre_degree - len(hub_degrees), 0)))
    src += [0] * len(rest)
    dst += rest
    nxt += len(rest)
    for _ in range(len(rest)):
        a, b = rs.integers(0, len(rest), 2)
        if a != b:
            src.append(rest[a])
            dst.append(rest[b])
    return gen.from_edges(nxt, np.array(src), np.array(dst))


CASES = [((4000, 4100), 5), ((4090, 4091), 7), ((4100, 4200), 12), ((8100, 8300), 40),
         ((4090, 4093), 64), ((4000, 4100, 20), 65), ((5000, 3000, 200), 130), ((3500, 4600), 300),
         ((9000,), 700), ((4000, 4200), 1025), ((2500, 6500, 40), 2100)]


@pytest.mark.parametrize("hubs,k", CASES)
def test_table_edges(hubs, k):
    rp, ci = hubs_graph(hubs, k, k)
    oN, oD, oE = oracle.ef(rp, ci, threads=4)
    with efgpu.Graph(rp, ci) as g:
        for algo in ("cluster", "per_seed"):
            ef, D, N = g.compute(algo=algo, prec="fp64")
            assert np.array_equal(N, oN) and np.array_equal(D, oD), algo
            assert np.all(np.abs(ef - oE) <= 1e-9 * np.abs(oE)), algo
    with efgpu.Batch([(rp, ci)]) as b:
        for design in ("phased", "persistent"):
            ef, D, N = b.compute(prec="fp64", design=design)
            assert np.array_equal(N, oN) and np.array_equal(D, oD), design
            assert np.all(np.abs(ef - oE) <= 1e-9 * np.abs(oE)), design


def test_without_memory_for_the_table():
    """The smallest EF_MAX_DEVICE_BYTES that a call fits leaves no room for
    the table: same sums, from logs."""
    rp, ci = gen.rmat(11, 8, 3, perm_seed=4)
    old = os.environ.get("EF_MAX_DEVICE_BYTES")

    def run(limit):
        os.environ["EF_MAX_DEVICE_BYTES"] = str(limit)
        try:
            with efgpu.Graph(rp, ci) as g:
                return g.compute(prec="fp64")
        except efgpu.EFError as e:
            assert e.name == "EF_ERR_NOMEM"
            return None
    try:
        want = run(1 << 40)
        lo, hi = 0, 1 << 28
        assert run(hi) is not None
        while hi - lo > 1:
            mid = (lo + hi) // 2
            if run(mid) is None:
                lo = mid
            else:
                hi = mid
        tight = run(hi)
    finally:
        if old is None:
            os.environ.pop("EF_MAX_DEVICE_BYTES", None)
        else:
            os.environ["EF_MAX_DEVICE_BYTES"] = old
    assert np.array_equal(tight[1], want[1]) and np.array_equal(tight[2], want[2])
    assert np.allclose(tight[0], want[0], rtol=1e-12, atol=0)
