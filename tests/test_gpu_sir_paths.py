"""SIR outbreaks at the sizes where the kernels' paths change (needs an
MI355X): one to 1024 simulations in a batch (one to four per thread of the
prefix), chunks of frontier nodes shared by a workgroup or one per wavefront,
step limits around the rounds that the host reads. Exact against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2306_00606_amd import efgpu, gen

pytestmark = pytest.mark.gpu

KEYS = ("index", "size", "t_end", "t_peak", "sp_sum", "inf_count")


def check(rp, ci, beta, mu, seed, sims, t_max=100000):
    with efgpu.Graph(rp, ci) as g:
        got = g.sir(beta, mu, seed, sims, t_max=t_max)
    want = oracle.sir(rp, ci, beta, mu, seed, sims, t_max=t_max)
    for k in KEYS:
        assert np.array_equal(got[k], want[k]), (k, sims, t_max)


@pytest.mark.parametrize("sims", [1, 2, 255, 256, 257, 513, 1024, 1030])
def test_simulations_per_batch(sims):
    rp, ci = gen.barabasi_albert(260, 3, 5)
    check(rp, ci, 0.1, 1.0 / 3.0, 11, sims)


@pytest.mark.parametrize("t_max", [0, 1, 7, 8, 9, 16, 17, 24])
def test_step_limits(t_max):
    rp, ci = gen.barabasi_albert(500, 4, 6)
    check(rp, ci, 0.08, 0.2, 3, 40, t_max=t_max)


@pytest.mark.parametrize("n,sims,beta", [(4000, 30, 0.5), (20000, 40, 0.4), (20000, 25, 1.0)])
def test_large_frontiers(n, sims, beta):
    # up to n sims / 64 chunks of frontier nodes: below and above 4096
    rp, ci = gen.barabasi_albert(n, 4, 7)
    check(rp, ci, beta, 0.5, 19, sims)


def test_hub_rows():
    rs = np.random.default_rng(2)
    src = np.concatenate([np.zeros(5000, np.int64), np.ones(3000, np.int64)])
    dst = np.concatenate([np.arange(2, 5002), rs.choice(np.arange(2, 6000), 3000, replace=False)])
    rp, ci = gen.from_edges(6000, src, dst)
    check(rp, ci, 0.3, 0.4, 5, 70)
