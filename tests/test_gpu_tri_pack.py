"""The packed triangle kernel (needs an MI355X): nodes of at most 16 upper
neighbours, 12 per wavefront, 64 of their segments at a time. Graphs at the
edges of those sizes against the CPU oracle, both precisions."""
import numpy as np
import pytest

import oracle
from paper_2306_00606_amd import efgpu, gen

pytestmark = pytest.mark.gpu


def ring_of_cliques(c, size):
    """c cliques of `size` nodes, neighbouring cliques joined by an edge."""
    src, dst = [], []
    for i in range(c):
        b = i * size
        for x in range(size):
            for y in range(x + 1, size):
                src.append(b + x)
                dst.append(b + y)
        src.append(b)
        dst.append((b + size) % (c * size) if c > 1 else b + 1)
    return gen.from_edges(c * size, np.array(src), np.array(dst))


GRAPHS = {
    # the middle node of a clique of 12 has its largest walk within 64 tests;
    # from 13 on some nodes leave the packed bin
    **{f"cliques_{c}x{s}": (lambda c=c, s=s: ring_of_cliques(c, s))
       for c, s in ((1, 3), (1, 12), (1, 13), (1, 17), (1, 18), (12, 3), (13, 3), (40, 12), (5, 17))},
    "ws_11": lambda: gen.watts_strogatz(11, 4, 0.1, 5),
    "ws_13": lambda: gen.watts_strogatz(13, 4, 0.1, 5),
    "ws_3000": lambda: gen.watts_strogatz(3000, 10, 0.05, 7),
    "er_dense": lambda: gen.erdos_renyi(200, 0.12, 3),
    "rmat": lambda: gen.rmat(11, 4, 9, perm_seed=2),
}


@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_packed_triangles(name):
    rp, ci = GRAPHS[name]()
    oN, oD, oE = oracle.ef(rp, ci)
    with efgpu.Graph(rp, ci) as g:
        for prec, tol in (("fp64", 1e-9), ("fp32c", 1e-5)):
            ef, D, N = g.compute(prec=prec)
            assert np.array_equal(N, oN) and np.array_equal(D, oD), prec
            assert np.all(np.abs(ef - oE) <= tol * np.abs(oE) + 1e-300), prec
            again = g.compute(prec=prec)
            assert np.array_equal(ef.view(np.int64), again[0].view(np.int64)), prec
