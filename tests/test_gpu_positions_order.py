"""Replaced positions leave the slots in no spatial order: forces and diagnostics
taken there, with re-sorts and without, and the steps that follow them."""
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


@pytest.fixture(scope="module")
def orc():
    import oracle
    oracle.build()
    return oracle


def shuffled(n):
    w = W.config_large(n=n, seed=n)
    return w, W.sample_positions(w.type, w.params.sigma, 0.5 * w.radius.R0, n + 1)


@pytest.mark.parametrize("n", [3000, 12500])
@pytest.mark.parametrize("tune", [{}, dict(sort_every=-1), dict(sort_every=4, graph_steps=1),
                                  dict(sort_every=-1, graph_steps=4), dict(cull=0)])
def test_forces_and_steps(ld, orc, n, tune):
    w, x = shuffled(n)
    Fo, So, _ = orc.pair_forces(x, w.type, w.charge, w.params)
    do = orc.State(w, pos=x).diagnostics()
    got = []
    for look in (True, False):
        s = ld.System.from_workload(w)
        s.set_tuning(**tune)
        s.set_positions(x)
        if look:
            F = s.forces(ext=False)["pair"].cpu().numpy()
            assert (np.linalg.norm(F - Fo, axis=1) <= 1e-5 * So).all()
            d = s.diagnostics()
            assert d[0] == pytest.approx(do[0], rel=1e-5)
            assert d[1] == pytest.approx(do[1], rel=1e-5)
        s.step(12, 1e-6)
        got.append(s.positions64())
    assert np.array_equal(got[0], got[1])        # looking changes nothing


@pytest.mark.parametrize("sort_every", [50, -1])
def test_sorting_turned_off_after(ld, orc, sort_every):
    w, x = shuffled(3000)
    s = ld.System.from_workload(w)
    s.set_positions(x)
    s.set_tuning(sort_every=sort_every)
    Fo, So, _ = orc.pair_forces(x, w.type, w.charge, w.params)
    F = s.forces(ext=False)["pair"].cpu().numpy()
    assert (np.linalg.norm(F - Fo, axis=1) <= 1e-5 * So).all()


@pytest.mark.parametrize("sort_every", [50, -1])
def test_truncated_scheme(ld, orc, sort_every):
    """Its velocities lie in slot order, which forces taken meanwhile leave."""
    w, x = shuffled(3000)
    v0 = np.random.default_rng(1).normal(size=(w.n, 3))
    got = []
    for look in (True, False):
        s = ld.System.from_workload(w)
        s.set_tuning(sort_every=sort_every)
        s.paper_enable(range_factor=4.0)
        s.set_velocities(v0)
        s.set_positions(x)
        if look:
            Fo, So, _ = orc.pair_forces(x, w.type, w.charge, w.params)
            F = s.forces(ext=False)["pair"].cpu().numpy()
            assert (np.linalg.norm(F - Fo, axis=1) <= 1e-5 * So).all()
            assert np.array_equal(s.velocities(), v0)
        s.step(5, 1e-5)
        got.append((s.positions64(), s.velocities()))
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
