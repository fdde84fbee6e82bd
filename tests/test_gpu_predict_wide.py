"""Features and predictions of graphs whose largest hub takes longer than all
the rest (needs an MI355X): they run on workgroups of twice the threads. The
rest of such a graph has the features it has alone; predictions are the network
on the features."""
import numpy as np
import pytest

from paper_2306_00606_amd import efgpu, gen
from tests.test_gpu_predict_tiers import tier_graph

pytestmark = pytest.mark.gpu


# leaves of the hub: on both sides of the rule, in one round and in eight
@pytest.mark.parametrize("leaves", [32768, 32769, 60320, 60321, 131_077])
def test_one_hub_over_the_rest(leaves):
    rp0, ci0 = gen.erdos_renyi(700, 0.01, 3) if leaves < 60000 else tier_graph(5215, 1)
    n0 = rp0.size - 1
    n = n0 + 1 + leaves
    rp = np.concatenate([rp0, rp0[-1] + leaves + np.arange(leaves + 1)]).astype(np.int32)
    ci = np.concatenate([ci0, n0 + 1 + np.arange(leaves), np.full(leaves, n0)]).astype(np.int32)
    s = efgpu.Surrogate(seed=7)
    with efgpu.Graph(rp0, ci0) as g:
        X0, L0 = g.features()
    flat = s.params()[0]
    s.set_params(np.random.default_rng(3).normal(0, 0.2, flat.size).astype(np.float32), X0.mean(0),
                 (1.0 / (X0.std(0) + 1e-3)).astype(np.float32))
    mean, inv = s.params()[1:]
    with efgpu.Graph(rp, ci) as g:
        X, L = g.features()
        ef = s.predict(g)
    # sums of at most 5000 terms in double, in another order, then one rounding
    # to float
    assert np.allclose(X[:n0], X0, rtol=2e-7, atol=1e-9) and np.array_equal(L[:n0], L0)
    k = np.float64(leaves)
    N = k * k - k  # all paths of two leaves around the hub
    D = k * (k - 1) * (k - 4) + 2 * (k - 1) * k
    want = [np.log1p(k), np.log1p(k), np.log1p(k), 0, 0, 0, np.log1p(N), np.log1p(D), np.log(D / N),
            0, 0, 0, 0, np.log1p(k * k), 1, 0]
    assert np.allclose(X[n0], want, rtol=1e-6, atol=1e-6)
    assert np.array_equal(X[n0 + 1:], np.broadcast_to(X[n - 1], (leaves, 16)))
    y = s.forward((X - mean) * inv)
    assert np.array_equal(ef, np.maximum(L - y, np.float32(0)).astype(np.float64))
