"""Several results read back together: sizes around the slots' bounds, host and
device destinations mixed, some left out."""
import ctypes as C

import numpy as np
import pytest

from paper_2501_04456_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ld():
    import torch
    assert torch.cuda.is_available()
    from paper_2501_04456_amd import ldrop
    ldrop.lib()
    return ldrop


# 128 KiB slots to 512 KiB ones; one piece ending with a slot, inside one, beyond all
@pytest.mark.parametrize("n", [2, 1365, 5461, 5462, 10922, 10923, 16385, 21846, 43691, 150001])
def test_forces(ld, n):
    import torch
    w = W.config_large(n=n, seed=n)
    s = ld.System.from_workload(w)
    L = ld.lib()
    shape = {"F": (n, 3), "E": (n, 3), "S": (n,), "U": (2,)}

    def call(kinds):
        out = {}
        for k in shape:
            if kinds.get(k) == "host":
                out[k] = np.full(shape[k], np.nan)
            elif kinds.get(k) == "device":
                out[k] = torch.full(shape[k], float("nan"), dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        ptr = [None if k not in out else C.c_void_p(
            out[k].ctypes.data if kinds[k] == "host" else out[k].data_ptr()) for k in shape]
        assert L.ld_forces(s.h, *ptr) == 0
        return {k: v if kinds[k] == "host" else v.cpu().numpy() for k, v in out.items()}

    ref = call({k: "device" for k in shape})
    assert all(np.isfinite(v).all() for v in ref.values())
    for kinds in ({k: "host" for k in shape}, {"F": "host", "E": "device", "S": "host", "U": "host"},
                  {"F": "device", "S": "host", "U": "host"}, {"S": "host"}, {"U": "host"}):
        got = call(kinds)
        for k in got:
            if "S" in kinds or "U" in kinds:     # the diagnostic kernel's sums, as ref's
                assert np.array_equal(got[k], ref[k]), (kinds, k)
    assert L.ld_forces(s.h, None, None, None, None) == 0


@pytest.mark.parametrize("n", [2, 10922, 10923, 21846, 43691, 150001])
def test_positions(ld, n):
    import torch
    w = W.config_medium(n=n, seed=n)
    s = ld.System.from_workload(w)
    s.step(2, 1e-6)
    x = s.positions64()
    hi, lo = s.positions()
    assert np.array_equal(hi, x.astype(np.float32))
    assert np.array_equal(hi.astype(np.float64) + lo, x)
    L = ld.lib()
    d, h = torch.empty((n, 3), device="cuda"), np.empty((n, 3), np.float32)
    torch.cuda.synchronize()
    assert L.ld_get_positions(s.h, C.c_void_p(d.data_ptr()), C.c_void_p(h.ctypes.data)) == 0
    assert np.array_equal(d.cpu().numpy(), hi) and np.array_equal(h, lo)
    assert L.ld_get_positions(s.h, None, C.c_void_p(h.ctypes.data)) == 0
    assert np.array_equal(h, lo)
    assert L.ld_get_positions(s.h, None, None) == 0
    s.paper_enable(range_factor=4.0)
    v = np.random.default_rng(n).normal(size=(n, 3))
    s.set_velocities(v)
    assert np.array_equal(s.velocities(), v)
    a = s.aggregates(1.1, labels=True)
    assert len(np.unique(a["labels"])) == a["components"]
