"""FP32C pass 2 (needs an MI355X): flagged positions found by the pass itself
(up to 2^18 positions) and listed first (above), at the edges of the scan's
grid and of that rule."""
import numpy as np
import pytest

import oracle
from paper_2306_00606_amd import efgpu, gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 255, 2047, 2048, 2049, 4097, 40_000])
def test_scan_sizes(n):
    rp, ci = gen.config_model(n, 2.2, 5) if n > 3 else gen.from_edges(3, np.array([0, 1]), np.array([1, 2]))
    oN, oD, oE = oracle.ef(rp, ci, threads=4)
    with efgpu.Graph(rp, ci) as g:
        ef, D, N = g.compute(prec="fp32c")
        whole = g.stats()["promoted"]
        seeds = np.arange(n, dtype=np.int32)[::-1].copy()
        es, Ds, Ns = g.compute(prec="fp32c", seeds=seeds)
    assert np.array_equal(N, oN) and np.array_equal(D, oD)
    assert np.array_equal(Ns, oN[seeds]) and np.array_equal(Ds, oD[seeds])
    assert np.all(np.abs(ef - oE) <= 1e-5 * oE) and np.all(np.abs(es - oE[seeds]) <= 1e-5 * oE[seeds])
    assert n < 2000 or whole > 0


def test_listed_and_found_agree():
    rp, ci = gen.config_model(40_000, 2.2, 6)
    got = []
    for n in (1 << 18, (1 << 18) + 1):  # the rest isolated
        pad = np.concatenate([rp, np.full(n - 40_000, rp[-1], rp.dtype)])
        with efgpu.Graph(pad, ci) as g:
            ef, D, N = g.compute(prec="fp32c")
            got.append((ef[:40_000], D[:40_000], N[:40_000], g.stats()["promoted"]))
            assert not ef[40_000:].any()
    assert got[0][3] == got[1][3] > 0
    for a, b in zip(got[0][:3], got[1][:3]):
        assert np.array_equal(a, b)
