"""A graph that the caller captured keeps the workspace it was captured with
(needs an MI355X): a later call that needs more takes a block of its own, and
the replays still give the captured call's results."""
import numpy as np
import pytest

import oracle
from paper_2306_00606_amd import efgpu, gen

pytestmark = pytest.mark.gpu

REL = {"fp64": 1e-9, "fp32c": 1e-5}


@pytest.mark.parametrize("algo,prec", [("per_seed", "fp64"), ("cluster", "fp32c")])
def test_outgrown_block(algo, prec):
    torch = pytest.importorskip("torch")
    # 2.6M arcs: an FP64 cluster-centric call needs more than these two take
    rp, ci = gen.barabasi_albert(260_000, 5, 11)
    oN, oD, oE = oracle.ef(rp, ci, threads=8)
    with efgpu.Graph(rp, ci) as g:
        out = (torch.empty(g.n, dtype=torch.float64, device="cuda"),
               *(torch.empty(g.n, dtype=torch.int64, device="cuda") for _ in range(2)))
        g.compute(algo=algo, prec=prec, out=out)  # sizes the workspace
        torch.cuda.synchronize()
        graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        with torch.cuda.graph(graph, stream=stream):
            g.compute(algo=algo, prec=prec, out=out, stream=stream.cuda_stream)
        for i in range(3):
            for t in out:
                t.zero_()
            graph.replay()
            torch.cuda.synchronize()
            ef, D, N = (t.cpu().numpy() for t in out)
            assert np.array_equal(N, oN) and np.array_equal(D, oD), i
            assert np.all(np.abs(ef - oE) <= REL[prec] * np.abs(oE)), i
            ef, D, N = g.compute(prec="fp64")  # outgrows the block at first
            assert np.array_equal(N, oN) and np.array_equal(D, oD), i
            assert np.all(np.abs(ef - oE) <= REL["fp64"] * np.abs(oE)), i
