"""Calls of one handle on different streams (needs an MI355X): the FP64 score
table, filled on the stream of the first FP64 call, is read by calls on other
streams only behind its fill."""
import numpy as np
import pytest

import oracle
from paper_2306_00606_amd import efgpu, gen

pytestmark = pytest.mark.gpu


def _out(torch, n):
    return (torch.empty(n, dtype=torch.float64, device="cuda"),
            *(torch.empty(n, dtype=torch.int64, device="cuda") for _ in range(2)))


@pytest.mark.parametrize("prec", ["fp64", "fp32c"])  # FP32C recomputes some seeds in FP64
def test_score_table_on_two_streams(prec):
    torch = pytest.importorskip("torch")
    rp, ci = gen.barabasi_albert(3000, 3, 5)
    oN, oD, oE = oracle.ef(rp, ci, threads=4)
    with efgpu.Graph(rp, ci) as g:
        want = g.compute(prec=prec, j=3)
    busy = torch.randn(4096, 4096, device="cuda")
    for _ in range(3):
        with efgpu.Graph(rp, ci) as g:
            out, out3 = _out(torch, g.n), _out(torch, g.n)
            g.compute(prec="fp32c", j=3, out=out3)
            g.compute(prec="fp32c", out=out)
            a, b = torch.cuda.Stream(), torch.cuda.Stream()
            torch.cuda.synchronize()
            with torch.cuda.stream(a):  # the fill waits behind some milliseconds of work
                x = busy
                for _ in range(20):
                    x = busy @ x
            g.compute(prec="fp64", out=out, stream=a.cuda_stream)
            g.compute(prec=prec, j=3, out=out3, stream=b.cuda_stream)
            torch.cuda.synchronize()
            ef, D, N = (t.cpu().numpy() for t in out)
            assert np.array_equal(N, oN) and np.array_equal(D, oD)
            assert np.all(np.abs(ef - oE) <= 1e-9 * np.abs(oE))
            ef, D, N = (t.cpu().numpy() for t in out3)
            assert np.array_equal(N, want[2]) and np.array_equal(D, want[1])
            assert np.all(np.abs(ef - want[0]) <= 1e-12 * np.abs(want[0]))
