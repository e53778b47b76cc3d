"""Lennard-Jones ranges beyond every distance, up to infinite: the padding of a
near group's slots is no partner, in any of the kernels that take the groups."""
import dataclasses

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


def lj_droplet(n, cut):
    """Lennard-Jones alone, at contact density (FP64 on both sides)."""
    w = W.config_large(n=n, seed=n)
    w.pos = W.sample_positions(w.type, w.params.sigma, 0.35 * w.radius.R0, n)
    w.charge = np.zeros(n)
    w.params.lj_cut = cut
    return w


# sizes that leave a last group of 1, 2, 3 and 63 slots, and none
@pytest.mark.parametrize("cut", [2.5, 1e15, 1e19, 1e30, np.inf])
@pytest.mark.parametrize("n,tune", [(65, {}), (130, {}), (1027, {}), (1024, {}), (1087, dict(cull=0)),
                                    (12353, {})])
def test_forces(ld, orc, n, tune, cut):
    w = lj_droplet(n, cut)
    s = ld.System.from_workload(w)
    if tune:
        s.set_tuning(**tune)
    F = s.forces(ext=False)["pair"].cpu().numpy()
    rows = np.unique(np.linspace(0, n - 1, 300).astype(int))
    Fo, So, _ = orc.pair_forces(w.pos, w.type, w.charge, w.params, rows=rows)
    # the same FP64 terms in another order: a few hundred ulp of their sum
    assert (np.linalg.norm(F[rows] - Fo, axis=1) <= 1e-12 * So).all()


@pytest.mark.parametrize("cut", [2.5, 1e30])
@pytest.mark.parametrize("drops", [2, 8193])
def test_ensemble(ld, orc, drops, cut):
    w = lj_droplet(131, cut)
    ens = ld.Ensemble([w.replace(seed=k) for k in range(drops)])
    F = ens.forces().cpu().numpy().reshape(drops, w.n, 3)
    Fo, So, _ = orc.pair_forces(w.pos, w.type, w.charge, w.params)
    assert (np.linalg.norm(F - Fo, axis=2) <= 1e-12 * So).all()



# partners on either side of the range, which only the low words tell apart
@pytest.mark.parametrize("far", [0.0, 300.0, 3e4, 1e6])
@pytest.mark.parametrize("n,tune", [(130, {}), (1087, dict(cull=0)), (12353, {})])
def test_far_from_the_origin(ld, orc, n, tune, far):
    w = lj_droplet(n, 2.5)
    rng = np.random.default_rng(n)
    w.type = rng.permutation(w.type)
    m = (n + 1) // 2
    side = int(np.ceil(m ** (1 / 3)))
    # pairs on a lattice wide enough that nobody else is in range
    site = np.stack(np.unravel_index(np.arange(m), (side,) * 3), 1) * 16.0 - 8.0 * side
    site += far * np.array([1.0, -0.7, 0.4])
    u = rng.normal(size=(m, 3))
    u /= np.linalg.norm(u, axis=1)[:, None]
    s = np.asarray(w.params.sigma)
    rc = 2.5 * 0.5 * (s[w.type[:m]] + s[np.resize(w.type[m:], m)])
    r = rc * (1.0 + rng.choice([-1.0, 1.0], m) * 10.0 ** rng.uniform(-7, -3, m))
    x = np.concatenate([site, site + u * r[:, None]])[:n]
    hi = x.astype(np.float32)
    lo = (x - hi).astype(np.float32)
    x = hi.astype(np.float64) + lo
    order = rng.permutation(n)
    w.type, hi, lo, x = w.type[order], hi[order], lo[order], x[order]
    d = ld.System.from_workload(w)
    if tune:
        d.set_tuning(**tune)
    d.set_positions(hi, lo)
    F = d.forces(ext=False)["pair"].cpu().numpy()
    Fo, So, _ = orc.pair_forces(x, w.type, w.charge, w.params)
    assert 0.2 < (So > 0).mean() < 0.8               # both sides occur
    assert (np.linalg.norm(F - Fo, axis=1) <= 1e-12 * So).all()


# ranges either side of the one from which dense windows are taken at once (a
# longest range of 20), and windows with few, some and all slots in range
@pytest.mark.parametrize("cut", [8.0, 11.0, 30.0])
@pytest.mark.parametrize("n,tune", [(65, {}), (1027, {}), (1087, dict(cull=0)), (9001, {}),
                                    (12353, {})])
def test_long_ranges(ld, orc, n, tune, cut):
    w = W.config_large(n=n, seed=n)
    hi = w.pos.astype(np.float32)
    w.pos = hi.astype(np.float64) + (w.pos - hi).astype(np.float32)     # as it is held
    w.charge = np.zeros(n)
    w.params.lj_cut = cut
    s = ld.System.from_workload(w)
    if tune:
        s.set_tuning(**tune)
    rows = np.unique(np.linspace(0, n - 1, 300).astype(int))
    Fo, So, _ = orc.pair_forces(w.pos, w.type, w.charge, w.params, rows=rows)
    F = s.forces(ext=False)["pair"].cpu().numpy()
    assert (np.linalg.norm(F[rows] - Fo, axis=1) <= 1e-12 * So).all()
    d = s.forces(ext=False, S=True)                  # the diagnostic instances
    assert (np.linalg.norm(d["pair"].cpu().numpy()[rows] - Fo, axis=1) <= 1e-12 * So).all()
    assert (np.abs(d["S"].cpu().numpy()[rows] - So) <= 1e-12 * So).all()


@pytest.mark.parametrize("cut", [11.0, 30.0])
@pytest.mark.parametrize("drops", [3, 150, 8193])
def test_long_ranges_of_ensembles(ld, orc, drops, cut):
    """150: the groups in a launch of their own; 8193: exact differences.  One
    droplet's range alone decides for all of them."""
    w = W.config_large(n=131 if drops > 150 else 4000, seed=5)
    hi = w.pos.astype(np.float32)
    w.pos = hi.astype(np.float64) + (w.pos - hi).astype(np.float32)
    w.charge = np.zeros(w.n)
    e = [w.replace(seed=k) for k in range(drops)]
    far = w.replace(seed=1)
    far.params = dataclasses.replace(w.params, lj_cut=cut)
    e[1] = far
    F = ld.Ensemble(e).forces().cpu().numpy().reshape(drops, w.n, 3)
    rows = np.unique(np.linspace(0, w.n - 1, 300).astype(int))
    for d in (0, 1, drops - 1):
        Fo, So, _ = orc.pair_forces(e[d].pos, e[d].type, e[d].charge, e[d].params, rows=rows)
        assert (np.linalg.norm(F[d, rows] - Fo, axis=1) <= 1e-12 * So).all()
