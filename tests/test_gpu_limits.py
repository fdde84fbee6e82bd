"""EF_MAX_DEVICE_BYTES (needs an MI355X): under the smallest limit that a load
fits, calls whose own buffers are small run too. The block that the load leaves
for ef_compute gives way to them, before and after it has been used."""

import numpy as np
import pytest

from paper_2306_00606_amd import efgpu, gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graph", [gen.rmat(14, 10, 3), gen.barabasi_albert(20_000, 5, 2)])
def test_calls_fit_where_the_load_does(graph, monkeypatch):
    rp, ci = graph
    seeds = np.arange(0, rp.size - 1, 3, dtype=np.int32)
    with efgpu.Graph(rp, ci) as g:
        want = {s is None: g.compute(algo="per_seed", prec="fp64", seeds=s) for s in (None, seeds)}

    def load(limit):
        monkeypatch.setenv("EF_MAX_DEVICE_BYTES", str(limit))
        try:
            return efgpu.Graph(rp, ci)
        except efgpu.EFError as e:
            assert e.name == "EF_ERR_NOMEM"
            return None

    lo, hi = 0, 1 << 28
    while hi - lo > 1:
        mid = (lo + hi) // 2
        g = load(mid)
        if g is None:
            lo = mid
        else:
            g.close()
            hi = mid
    sur = efgpu.Surrogate(seed=1)
    for s in (None, seeds):
        with load(hi) as g:
            for _ in range(2):
                got = g.compute(algo="per_seed", prec="fp64", seeds=s)
                assert all(np.array_equal(a, b) for a, b in zip(got[1:], want[s is None][1:]))
                assert np.allclose(got[0], want[s is None][0], rtol=1e-12, atol=0)
                assert sur.predict(g).shape == (g.n,)
                g.sir(0.05, 1 / 3, 1, 5)
