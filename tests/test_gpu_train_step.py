"""The training kernels (needs an MI355X): a gradient over more tiles than
slots adds up from its parts, and one optimiser step is Adam's on that
gradient and leaves the packed weights of the new parameters."""
import numpy as np
import pytest

from paper_2306_00606_amd import efgpu

pytestmark = pytest.mark.gpu


def rows_of(n, seed):
    rs = np.random.default_rng(seed)
    return rs.normal(0, 1, (n, 16)).astype(np.float32), rs.normal(0, 1, n).astype(np.float32)


@pytest.mark.parametrize("n,cut", [(33, 32), (129, 64), (8192, 4096), (8193, 8192), (20011, 9984)])
def test_gradient_adds_up(n, cut):
    X, y = rows_of(n, n)
    s = efgpu.Surrogate(seed=1)
    g, loss = s.gradients(X, y)
    ga, la = s.gradients(X[:cut], y[:cut])
    gb, lb = s.gradients(X[cut:], y[cut:])
    want = (ga.astype(np.float64) * cut + gb.astype(np.float64) * (n - cut)) / n
    # the parts scale dz by another power of the row count, so their BF16
    # roundings differ: one step of 2^-8 per term, averaged over the rows
    assert np.abs(g - want).max() <= 2.0 ** -8 * np.abs(want).max() + 1e-6
    assert abs(loss - (la * cut + lb * (n - cut)) / n) <= 1e-4 * loss


@pytest.mark.parametrize("n", [64, 1000, 9000])
def test_one_step_is_adam_and_repacks(n):
    X, y = rows_of(n, n + 1)
    s = efgpu.Surrogate(seed=2)
    P0, _, _ = s.params()
    lr = 2e-3
    s.train(X, y, lr=lr, epochs=1, batch=n, val_fraction=0.0, lr_end=1.0)
    P1, mean, inv = s.params()
    assert np.allclose(mean, X.mean(0, dtype=np.float64), rtol=1e-5, atol=1e-6)
    assert np.allclose(inv, 1.0 / X.std(0, dtype=np.float64), rtol=1e-5)
    Xs = ((X - mean) * inv).astype(np.float32)
    ref = efgpu.Surrogate(seed=2)
    g, _ = ref.gradients(Xs, y)
    g = g.astype(np.float64)
    # rows come shuffled: FP32 sums in another order, so only gradients well
    # above their rounding have a certain first step of lr g / (|g| + eps)
    clear = np.abs(g) > 1e-3 * np.abs(g).max()
    assert clear.sum() > 1000
    step = (P0.astype(np.float64) - P1)[clear]
    assert np.abs(step - lr * g[clear] / (np.abs(g[clear]) + 1e-8)).max() <= 1e-3 * lr
    # the step's packed weights are those of its parameters
    ref.set_params(P1, mean, inv)
    assert np.array_equal(s.forward(Xs).view(np.int32), ref.forward(Xs).view(np.int32))
