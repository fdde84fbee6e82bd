"""Top-k at the sizes where its paths change (needs an MI355X): one-launch
ranking up to 8192 values, selection above; one sorted tile up to 4096
winners, merged tiles up to 262144, radix sort above. Bit for bit against a
plain sort, with infinities, NaN, negative values and zeros among the input."""
import numpy as np
import pytest

from paper_2306_00606_amd import efgpu

pytestmark = pytest.mark.gpu


def values(n, seed, special):
    rs = np.random.default_rng(seed)
    v = rs.random(n) * 20.0
    pick = rs.random(n)
    v[pick < 0.4] = rs.choice([1.5, 2.0, 7.25, 0.0], size=int((pick < 0.4).sum()))
    if special:
        v[pick > 0.97] = rs.choice([np.inf, np.nan, -3.0, -0.0, 5e-324, 1.7e308],
                                   size=int((pick > 0.97).sum()))
    return v


def reference(v, k):
    key = np.where(v > 0, v, 0.0)
    order = np.lexsort((np.arange(v.size), -key))[:k]
    return order.astype(np.int32), key[order]


@pytest.mark.parametrize("special", [False, True])
@pytest.mark.parametrize("n", [64, 65, 8191, 8192, 8193, 12289, 70001, 1048577])
def test_path_edges(n, special):
    torch = pytest.importorskip("torch")
    v = values(n, n, special)
    dv = torch.from_numpy(v).cuda()
    ks = sorted({k for k in (1, 63, 64, 4096, 4097, 8193, 65536, 262144, 262145, n) if k <= min(n, 300000)})
    with efgpu.Graph(np.zeros(n + 1, np.int32), np.zeros(0, np.int32)) as g:
        for k in ks:
            nodes, ef = g.topk_values(dv, k)
            want_n, want_v = reference(v, k)
            assert np.array_equal(nodes, want_n), (n, k)
            assert np.array_equal(ef.view(np.int64), want_v.view(np.int64)), (n, k)


@pytest.mark.parametrize("n,k", [(5000, 5000), (5000, 17), (9000, 4000), (9000, 5000)])
def test_outputs_over_the_values(n, k):
    torch = pytest.importorskip("torch")
    v = values(n, 3, False)
    dv = torch.from_numpy(v).cuda()
    nodes = torch.empty(k, dtype=torch.int32, device="cuda")
    efgpu.topk_values_noalloc(dv, k, nodes, dv)
    torch.cuda.synchronize()
    want_n, want_v = reference(v, k)
    assert np.array_equal(nodes.cpu().numpy(), want_n)
    assert np.array_equal(dv[:k].cpu().numpy(), want_v)
