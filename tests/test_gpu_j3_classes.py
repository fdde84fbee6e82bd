"""Three-event sums by classes of equal degree (needs an MI355X): lists whose
members fall into few classes, into more than the class table holds, and of
the sizes where the bins change; one item per edge in whole-graph calls against
one per arc for chosen seeds."""
import numpy as np
import pytest

import oracle
from paper_2306_00606_amd import efgpu, gen

pytestmark = pytest.mark.gpu


def broom(distinct, same):
    """Hub 0 whose neighbours have degrees 1 .. distinct (a leaf fan each), and
    `same` more neighbours that are leaves."""
    src, dst, nxt = [], [], 1
    for d in range(1, distinct + 1):
        v = nxt
        src.append([0])
        dst.append([v])
        src.append(np.full(d - 1, v))
        dst.append(np.arange(nxt + 1, nxt + d))
        nxt += d
    src.append(np.zeros(same, np.int64))
    dst.append(np.arange(nxt, nxt + same))
    nxt += same
    return gen.from_edges(nxt, np.concatenate(src), np.concatenate(dst))


@pytest.mark.parametrize("distinct,same", [(1, 63), (2, 64), (60, 5), (200, 60), (250, 20),
                                           (255, 900), (1020, 8), (1023, 0), (1024, 3), (1026, 0),
                                           (1200, 500)])
def test_class_table_sizes(distinct, same):
    rp, ci = broom(distinct, same)
    # the hub's first, middle and last fan centres, and a leaf of the hub's
    hub = ci[rp[0]:rp[1]]
    seeds = np.unique(hub[[0, len(hub) // 2, -1]])[:3]
    oN, oD, oE = oracle.ef(rp, ci, seeds=seeds, threads=4, j=3)
    with efgpu.Graph(rp, ci) as g:
        for prec, tol in (("fp64", 1e-9), ("fp32c", 1e-5)):
            ef, D, N = g.compute(prec=prec, j=3, seeds=seeds)
            assert np.array_equal(N, oN) and np.array_equal(D, oD), prec
            assert np.all(np.abs(ef - oE) <= tol * np.abs(oE)), prec


@pytest.mark.parametrize("make", [lambda: gen.barabasi_albert(3000, 4, 77),
                                  lambda: gen.rmat(10, 6, 5, perm_seed=3),
                                  lambda: gen.watts_strogatz(500, 8, 0.1, 9)])
def test_edge_items_equal_arc_items(make):
    rp, ci = make()
    n = rp.size - 1
    with efgpu.Graph(rp, ci) as g:
        for prec in ("fp64", "fp32c"):
            ef, D, N = g.compute(prec=prec, j=3)
            efs, Ds, Ns = g.compute(prec=prec, j=3, seeds=np.arange(n, dtype=np.int32))
            assert np.array_equal(N, Ns) and np.array_equal(D, Ds)
            assert np.allclose(ef, efs, rtol=1e-12 if prec == "fp64" else 2e-7, atol=0)
