"""Features and predictions by degree tier (needs an MI355X): one launch takes
every tier, in one round per wavefront below 65536 nodes and eight from there,
and predictions run the network in the wavefronts that have the features. Both
are the same operations per node, so every comparison is for equal bits."""
import numpy as np
import pytest

from paper_2306_00606_amd import efgpu, gen

pytestmark = pytest.mark.gpu


def tier_graph(n, seed):
    """Hubs at the edges of the tiers (32, 512 and 4096 neighbours) over random
    nodes, with isolated ones at the end."""
    rs = np.random.default_rng(seed)
    hubs = [1, 8, 9, 31, 32, 33, 64, 511, 512, 513, 1000, 4095, 4096, 4097, 5000]
    pool = 5200
    src, dst = [rs.integers(0, pool, 3 * pool)], [rs.integers(0, pool, 3 * pool)]
    for i, k in enumerate(hubs):
        src.append(np.full(k, pool + i))
        dst.append(rs.choice(pool, k, replace=False))
    return gen.from_edges(n, np.concatenate(src), np.concatenate(dst))


@pytest.mark.parametrize("n", [5215, 5216, 5279, 65535, 65536, 65601])
def test_predict_is_the_network_on_the_features(n):
    s = efgpu.Surrogate(seed=7)
    flat, mean, inv = s.params()
    rs = np.random.default_rng(3)
    small = tier_graph(5215, 1)
    with efgpu.Graph(*small) as g:
        X0, L0 = g.features()
    s.set_params(rs.normal(0, 0.2, flat.size).astype(np.float32), X0.mean(0),
                 (1.0 / (X0.std(0) + 1e-3)).astype(np.float32))
    mean, inv = s.params()[1:]
    rp, ci = tier_graph(n, 1)
    with efgpu.Graph(rp, ci) as g:
        X, L = g.features()
        ef = s.predict(g)
    assert np.array_equal(X[:5215], X0) and np.array_equal(L[:5215], L0)
    assert np.array_equal(X[5215:], np.broadcast_to(X[n - 1], (n - 5215, 16)))
    y = s.forward((X - mean) * inv)
    assert np.array_equal(ef, np.maximum(L - y, np.float32(0)).astype(np.float64))
