"""Seeds cut into pieces (needs an MI355X): hubs of every per-seed bin whose
2-hop work is one piece, just more, and many, several chunks of neighbours,
among a seed list and over all nodes; and uncut, for want of memory."""
import os

import numpy as np
import pytest

import oracle
from paper_2306_00606_amd import efgpu, gen

pytestmark = pytest.mark.gpu

POOL = 10_000


def pool_graph(hubs, pool_degree, seed):
    """Random nodes 0 .. POOL-1 of average degree pool_degree, and hubs joined to
    so many of them each."""
    rs = np.random.default_rng(seed)
    m = POOL * pool_degree // 2
    src, dst = [rs.integers(0, POOL, m)], [rs.integers(0, POOL, m)]
    for i, k in enumerate(hubs):
        src.append(np.full(k, POOL + i))
        dst.append(rs.choice(POOL, k, replace=False))
    return gen.from_edges(POOL + len(hubs), np.concatenate(src), np.concatenate(dst))


# (hub degrees, average degree of the rest): at degree 32 the pieces of 16384
# and 32768 entries start near 512 and 1024 neighbours; 8193 has a bitmap
CASES = [((500, 512, 513, 1024, 1025, 1100), 32), ((64, 511, 2048, 2049, 4096, 4097), 60),
         ((8192, 8193, 9999, 60), 40)]


@pytest.mark.parametrize("hubs,deg", CASES)
def test_pieces(hubs, deg):
    rp, ci = pool_graph(hubs, deg, len(hubs))
    oN, oD, oE = oracle.ef(rp, ci, threads=4)
    rs = np.random.default_rng(1)
    seeds = np.concatenate([rs.integers(0, POOL, 200), POOL + np.arange(len(hubs)), [POOL, 3]])
    rs.shuffle(seeds)
    seeds = seeds.astype(np.int32)
    # the repository's bounds against the oracle
    for prec, rel in (("fp64", 1e-9), ("fp32c", 1e-5)):
        with efgpu.Graph(rp, ci) as g:
            # whole-graph pieces are kept while other calls use the buffer
            for sd in (None, seeds, None, seeds[:7]):
                ef, D, N = g.compute(algo="per_seed", prec=prec, seeds=sd)
                idx = slice(None) if sd is None else sd
                assert np.array_equal(N, oN[idx]) and np.array_equal(D, oD[idx]), prec
                assert np.all(np.abs(ef - oE[idx]) <= rel * np.abs(oE[idx])), prec


def test_without_memory_for_the_pieces():
    """Under the smallest EF_MAX_DEVICE_BYTES that a call fits no seed is cut.
    The FP32 sums of a round are the same; only double or double-float sums are
    taken in another order (some 700 adds of 2^-46 each, about ten times that in
    EF): 1e-10."""
    rp, ci = pool_graph((600, 3000), 40, 9)
    seeds = np.array([POOL, POOL + 1, 5], np.int32)
    old = os.environ.get("EF_MAX_DEVICE_BYTES")

    def run(limit):
        os.environ["EF_MAX_DEVICE_BYTES"] = str(limit)
        try:
            with efgpu.Graph(rp, ci) as g:
                return g.compute(prec="fp32c", seeds=seeds)
        except efgpu.EFError as e:
            assert e.name == "EF_ERR_NOMEM"
            return None
    try:
        want = run(1 << 40)
        lo, hi = 0, 1 << 28
        assert want is not None and run(hi) is not None
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
    assert np.allclose(tight[0], want[0], rtol=1e-10, atol=0)
