"""The triangle pass's lane-bin records, written on the device (needs an
MI355X): one workgroup up to 4096 nodes, 48 beyond, with ranges that end
inside and at a round of 1024; sums of rows on both sides of 128 entries among
neighbouring hubs. N and D are exact only if every record is there once."""
import numpy as np
import pytest

import oracle
from paper_2306_00606_amd import efgpu, gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5, 1023, 1024, 1025, 4095, 4096, 4097, 49_152, 49_153, 60_001])
def test_every_record_once(n):
    rp, ci = gen.barabasi_albert(n, 4, n)
    oN, oD, oE = oracle.ef(rp, ci, threads=4)
    with efgpu.Graph(rp, ci) as g:
        ef, D, N = g.compute(prec="fp64")
    assert np.array_equal(N, oN) and np.array_equal(D, oD)
    assert np.all(np.abs(ef - oE) <= 1e-9 * oE)
    # the same graph in a batch, whose lists go by graph
    with efgpu.Batch([(rp, ci), gen.barabasi_albert(77, 3, 1)]) as b:
        for design in ("phased", "persistent"):
            _, D, N = b.compute(prec="fp64", design=design)
            assert np.array_equal(N[:n], oN) and np.array_equal(D[:n], oD), design
