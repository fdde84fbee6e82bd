"""Replays of captured whole-graph calls (needs an MI355X): a batch's own graph,
which reads the work lists kept before its capture, over graphs that have
centres and triangle nodes of every bin; and a graph that the caller captures,
which must not depend on what the handle builds or drops between replays."""
import numpy as np
import pytest

import oracle
from paper_2306_00606_amd import efgpu, gen

pytestmark = pytest.mark.gpu

REL = {"fp64": 1e-9, "fp32c": 1e-5}


@pytest.mark.parametrize("prec", ["fp32c", "fp64"])
@pytest.mark.parametrize("graphs", [
    [gen.rmat(12, 16, 3, perm_seed=1), gen.barabasi_albert(5000, 4, 2), gen.erdos_renyi(7, 0.5, 1)],
    [gen.erdos_renyi(400, 0.004, 5), gen.erdos_renyi(2, 0.9, 6)],  # no centre above the small bins
])
def test_batch_kept_lists(graphs, prec):
    torch = pytest.importorskip("torch")
    want = [np.concatenate(x) for x in zip(*(oracle.ef(rp, ci, threads=4) for rp, ci in graphs))]
    with efgpu.Batch(graphs) as b:
        out = (torch.empty(b.n, dtype=torch.float64, device="cuda"),
               *(torch.empty(b.n, dtype=torch.int64, device="cuda") for _ in range(2)))
        first = None
        for i in range(4):
            for t in out:
                t.zero_()
            b.compute(prec=prec, out=out, design="phased")
            torch.cuda.synchronize()
            ef, D, N = (t.cpu().numpy() for t in out)
            assert np.array_equal(N, want[0]) and np.array_equal(D, want[1]), i
            assert np.all(np.abs(ef - want[2]) <= REL[prec] * np.abs(want[2])), i
            first = ef if first is None else first
            assert np.array_equal(ef, first), i
            if i == 1:  # other work lists in between
                b.autotune(prec)
                first = None


@pytest.mark.parametrize("prec", ["fp32c", "fp64"])
def test_captured_by_the_caller(prec, monkeypatch):
    torch = pytest.importorskip("torch")
    rp, ci = gen.rmat(12, 12, 4, perm_seed=2)
    oN, oD, oE = oracle.ef(rp, ci, threads=4)
    seeds = np.arange(0, rp.size - 1, 7, dtype=np.int32)
    with efgpu.Graph(rp, ci) as g:
        out = (torch.empty(g.n, dtype=torch.float64, device="cuda"),
               *(torch.empty(g.n, dtype=torch.int64, device="cuda") for _ in range(2)))
        g.compute(prec="fp64", out=out)  # sizes the workspace, keeps lists and the score table
        torch.cuda.synchronize()
        graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        with torch.cuda.graph(graph, stream=stream):
            g.compute(prec=prec, out=out, stream=stream.cuda_stream)
        for i in range(3):
            for t in out:
                t.zero_()
            graph.replay()
            torch.cuda.synchronize()
            ef, D, N = (t.cpu().numpy() for t in out)
            assert np.array_equal(N, oN) and np.array_equal(D, oD), i
            assert np.all(np.abs(ef - oE) <= REL[prec] * np.abs(oE)), i
            # no memory for another slot of workspace: what is kept is dropped
            if i == 0:
                monkeypatch.setenv("EF_MAX_DEVICE_BYTES", "1")
                with pytest.raises(efgpu.EFError):
                    g.compute(prec="fp32c", j=3, out=out)
                monkeypatch.delenv("EF_MAX_DEVICE_BYTES")
            elif i == 1:
                g.compute(prec="fp32c", algo="per_seed", out=out)
                torch.cuda.synchronize()
