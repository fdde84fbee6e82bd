"""EF_VALIDATE on the device (needs an MI355X): a CSR broken in one place is
refused with the status that the host check gives it, from host and from
device arrays, and a sound one loads; without EF_VALIDATE an id out of range
is still refused."""
import ctypes

import numpy as np
import pytest

from paper_2306_00606_amd import efgpu, gen

pytestmark = pytest.mark.gpu


def load(rp, ci, flags, device):
    h = ctypes.c_void_p()
    if device:
        torch = pytest.importorskip("torch")
        drp, dci = torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda()
        st = efgpu.lib().ef_graph_load_csr(rp.size - 1, ci.size, drp.data_ptr(), dci.data_ptr(),
                                           flags | efgpu.EF_DEVICE_PTRS, None, ctypes.byref(h))
    else:
        st = efgpu.lib().ef_graph_load_csr(rp.size - 1, ci.size, rp.ctypes.data, ci.ctypes.data,
                                           flags, None, ctypes.byref(h))
    if st == 0:
        efgpu.lib().ef_graph_free(h)
    return st


def broken(kind, rs):
    rp, ci = gen.rmat(9, 6, int(rs.integers(1, 1000)), perm_seed=2)
    deg = np.diff(rp)
    v = int(rs.choice(np.flatnonzero(deg >= 3)))
    e = int(rp[v] + rs.integers(0, deg[v] - 1))
    if kind == "swapped":
        ci[[e, e + 1]] = ci[[e + 1, e]]
    elif kind == "duplicate":
        ci[e + 1] = ci[e]
    elif kind == "self_loop":
        row = ci[rp[v]:rp[v + 1]]
        row[0] = v
        row.sort()
    elif kind == "past_end":
        ci[e] = rp.size - 1
    elif kind == "negative":
        ci[e] = -1
    elif kind == "one_way":
        # an ascending row with one neighbour exchanged for a non-neighbour
        row = ci[rp[v]:rp[v + 1]]
        other = np.setdiff1d(np.arange(rp.size - 1), np.append(row, v))
        row[int(rs.integers(0, row.size))] = int(rs.choice(other))
        row.sort()
    elif kind == "odd":
        # one arc missing
        rp[v + 1:] -= 1
        ci = np.delete(ci, e)
    return rp, ci


@pytest.mark.parametrize("device", [False, True])
@pytest.mark.parametrize("kind", ["sound", "swapped", "duplicate", "self_loop", "past_end",
                                  "negative", "one_way", "odd"])
def test_status_matches_the_host_check(kind, device):
    rs = np.random.default_rng(7)
    for _ in range(4):
        rp, ci = broken(kind, rs)
        want = efgpu.lib().ef_validate_csr(rp.size - 1, ci.size, rp.ctypes.data, ci.ctypes.data)
        text = efgpu.last_error()
        assert (want == 0) == (kind == "sound")
        assert load(rp, ci, efgpu.EF_VALIDATE, device) == want, kind
        if want:
            assert efgpu.last_error() == text
        if kind in ("past_end", "negative"):
            assert efgpu.STATUS_NAMES[load(rp, ci, 0, device)] == "EF_ERR_RANGE"
        if kind == "odd":
            assert efgpu.STATUS_NAMES[load(rp, ci, 0, device)] == "EF_ERR_NOT_SYMMETRIC"
