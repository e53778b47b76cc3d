"""Box counting and the moments of the fractal statistics against numpy: tiny
and ragged sizes, boxes that all hold one particle, all particles in one box,
box indices beyond 32 bits."""
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


@pytest.mark.parametrize("n,eps0", [(2, 0.0), (3, 1e-3), (257, 0.0), (4097, 1e-4), (65536, 0.0),
                                    (131073, 0.3), (20000, 1e-5)])
def test_boxes(ld, n, eps0):
    w = W.config_large(n=n, seed=n)
    x = w.pos.astype(np.float64)
    x[n // 2:] = x[:n - n // 2]                  # every box twice over
    w.pos = x.astype(np.float32)
    s = ld.System.from_workload(w)
    rg, df, dbox, K, boxes = s.fractal(eps0=eps0)
    sig = np.asarray(w.params.sigma)[w.type]
    ref = np.sqrt(((x - x.mean(0)) ** 2).sum(1).mean())
    assert rg == pytest.approx(ref, rel=1e-12)
    assert df == pytest.approx(np.log(n / 1.593) / np.log(2 * ref / sig.mean()), rel=1e-11)
    e0 = eps0 or sig.min()
    want = []
    for k in range(32):
        e = e0 * 2.0 ** k
        if e > ref:
            break
        want.append(len(np.unique(np.floor((x - x.min(0)) / e), axis=0)))
    assert K == len(want) and list(boxes) == want
