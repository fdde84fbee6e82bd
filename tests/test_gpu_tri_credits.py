"""FP64 credits to the middle node of a triangle are summed in double (needs an
MI355X). A node that is the middle one of a single triangle has one such
credit, so that every design holds the same double: the single-graph pass,
which packs the segments of several nodes on a wavefront, gives the bits of the
persistent batch kernel, which takes a node per lane. (The single-graph call is
a captured one: like the batch kernel it computes its scores, where an eager
call reads them from a table that holds them rounded.)"""
import numpy as np
import pytest

from paper_2306_00606_amd import efgpu, gen

pytestmark = pytest.mark.gpu


def _triangles(count, seed):
    """`count` triangles a, b, c, each node with its own number of leaves, so
    that the ranks are a < b < c; the ids of the middle nodes."""
    r = np.random.default_rng(seed)
    src, dst, mid, n = [], [], [], 0
    for _ in range(count):
        la = int(r.integers(0, 7))
        lb = int(r.integers(7, 25))  # 9 to 26 neighbours: both sum those on 8 lanes
        lc = lb + int(r.integers(1, 6))
        a, b, c = n, n + 1, n + 2
        n += 3
        src += [a, a, b]
        dst += [b, c, c]
        for v, leaves in ((a, la), (b, lb), (c, lc)):
            src += [v] * leaves
            dst += range(n, n + leaves)
            n += leaves
        mid.append(b)
    return gen.from_edges(n, np.array(src, np.int32), np.array(dst, np.int32)), np.array(mid)


@pytest.mark.parametrize("count", [1, 12, 13, 4000])  # nodes of a wavefront: 12
def test_middle_node_credits(count):
    torch = pytest.importorskip("torch")
    (rp, ci), mid = _triangles(count, count)
    with efgpu.Graph(rp, ci) as g:
        out = (torch.empty(g.n, dtype=torch.float64, device="cuda"),
               *(torch.empty(g.n, dtype=torch.int64, device="cuda") for _ in range(2)))
        g.compute(prec="fp64", out=out)
        torch.cuda.synchronize()
        graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        with torch.cuda.graph(graph, stream=stream):
            g.compute(prec="fp64", out=out, stream=stream.cuda_stream)
        graph.replay()
        torch.cuda.synchronize()
        ef0, D0, N0 = (t.cpu().numpy() for t in out)
    with efgpu.Batch([(rp, ci)]) as b:
        ef1, D1, N1 = b.compute(prec="fp64", design="persistent")
    assert np.array_equal(N0, N1) and np.array_equal(D0, D1)
    assert np.array_equal(ef0[mid], ef1[mid])
