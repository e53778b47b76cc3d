"""The truncated scheme's steps split into calls, with other calls between them
that sort the cells or use their scratch: the same bits as in one call."""
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


def run(ld, n, calls, between=lambda s: None):
    w = W.config_medium(n=n, seed=5)
    s = ld.System.from_workload(w)
    s.paper_enable(range_factor=4.0, kick=0.5)
    for k in calls:
        s.step(k, 5e-3)
        between(s)
    assert s.state()[0] == 20
    return s.positions64(), s.velocities()


def same(a, b):
    return np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


# one lane a particle, eight, a single tile
@pytest.mark.parametrize("n", [63, 5000, 59999, 60000])
def test_split(ld, n):
    whole = run(ld, n, (20,))
    assert same(whole, run(ld, n, (1,) * 20))
    assert same(whole, run(ld, n, (7, 0, 1, 9, 3)))


@pytest.mark.parametrize("n", [5000, 60001])
@pytest.mark.parametrize("call", ["paper_forces", "forces", "diagnostics", "aggregates", "rdf",
                                  "fractal", "velocities"])
def test_calls_between(ld, n, call):
    args = {"rdf": (5.0, 50)}.get(call, ())
    whole = run(ld, n, (20,))
    assert same(whole, run(ld, n, (4, 1, 15), lambda s: getattr(s, call)(*args)))


def test_positions_written(ld):
    """New positions: cells of their own coordinates, far beyond the old ones'."""
    w = W.config_medium(n=3000, seed=5)
    far = (w.pos * np.float32(30.0)).astype(np.float32)
    a, b = ld.System.from_workload(w), ld.System.from_workload(w.replace(pos=far))
    a.paper_enable(range_factor=4.0)
    a.step(3, 1e-4)
    a.set_positions(far)
    b.paper_enable(range_factor=4.0)
    Fa, Fb = a.paper_forces(), b.paper_forces()
    assert np.abs(Fa - Fb).max() <= 1e-12 * np.abs(Fb).max()
