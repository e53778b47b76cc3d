"""Read-back through the pinned slots: sizes on both sides of the direct write,
of one slot and of all slots, host and device destinations, and the batches of
a training pass against the same batch on the device."""
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


@pytest.mark.parametrize("n", [2, 5461, 5462, 21845, 87382, 100003])
def test_positions(ld, n):
    import torch
    w = W.config_large(n=n)
    s = ld.System.from_workload(w)
    s.step(2, 1e-6)
    hi, lo = s.positions()
    x = s.positions64()
    assert np.array_equal(x, hi.astype(np.float64) + lo.astype(np.float64))
    assert np.abs(x - w.pos).max() < 0.1          # the original order
    d = torch.empty((n, 3), dtype=torch.float64, device="cuda")
    assert ld.lib().ld_get_positions64(s.h, C.c_void_p(d.data_ptr())) == 0
    assert np.array_equal(d.cpu().numpy(), x)
    only = np.full((n, 3), -1.0, np.float32)
    s.positions_into(only)
    assert np.array_equal(only, hi)
    assert ld.lib().ld_get_positions64(s.h, None) != 0


def test_ensemble_positions(ld):
    drops = W.config_ensemble(n_drop=9, n_min=2, n_max=9000, seed=4).droplets
    e = ld.Ensemble(drops)
    e.step(2, 1e-6)
    hi, lo = e.positions()
    x = e.positions64()
    assert np.array_equal(x, hi.astype(np.float64) + lo.astype(np.float64))
    assert np.abs(x - np.concatenate([d.pos for d in drops])).max() < 0.1


@pytest.mark.parametrize("m", [1, 1042, 1043, 4500])
def test_training_batch(ld, m):
    import torch
    s = ld.System.from_workload(W.config_small(n=300))
    s.ff_enable(grid=32, block=5, hidden=128, near_mode=ld.NEAR_BLOCK)
    rng = np.random.default_rng(m)
    X = rng.standard_normal((m, 503)).astype(np.float32)
    T = rng.standard_normal((m, 3)).astype(np.float32)
    loss, g = s.ff_grads(X, T)
    Xd, Td = torch.as_tensor(X, device="cuda"), torch.as_tensor(T, device="cuda")
    torch.cuda.synchronize()
    g2, l2 = np.empty_like(g), C.c_double()
    ptr = lambda v: C.c_void_p(v.data_ptr() if hasattr(v, "data_ptr") else v.ctypes.data)  # noqa: E731
    assert ld.lib().ld_ff_grads(s.h, ptr(Xd), ptr(Td), m, ptr(g2), C.byref(l2)) == 0
    assert l2.value == loss and np.array_equal(g, g2)
