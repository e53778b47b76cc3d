"""The ensemble's pair tasks at the edges of their plan: droplets of one tile,
of a ragged last tile or block, of many blocks, and of more blocks than
super-blocks, against the oracle's force rows and single-droplet runs."""
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


def _droplets(sizes, neutral=0):
    out = []
    for k, n in enumerate(sizes):
        w = W.config_ensemble(n_drop=1, n_min=n, n_max=n, seed=20 + k).droplets[0]
        if neutral:
            w = w.replace(charge=np.where(np.arange(n) % neutral == 0, 0.0, w.charge))
        out.append(w)
    return out


@pytest.mark.parametrize("sizes,neutral", [((2, 64, 65, 255, 256, 257, 513), 0),
                                           ((2, 64, 65, 256, 1025), 3),
                                           ((33000, 5), 0), ((9001,), 1), ((2, 3), 1)])
def test_forces(ld, orc, sizes, neutral):
    drops = _droplets(sizes, neutral)
    ens = ld.Ensemble(drops)
    ens.step(1, 1e-12)                       # sorted slots and the update's own boxes
    x = ens.positions64()
    F = ens.forces().cpu().numpy()
    for d, w in enumerate(drops):
        o, e = ens.offsets[d], ens.offsets[d + 1]
        rows = np.unique(np.linspace(0, e - o - 1, 100).astype(int))
        Fo, So, _ = orc.pair_forces(x[o:e], w.type, w.charge, w.params, rows=rows)
        # FP32 pair terms in blocks of 32: 31 u sum|f| < 2e-6 of S per block
        assert (np.linalg.norm(F[o:e][rows] - Fo, axis=1) <= 1e-5 * So).all(), (d, w.n)


def test_clock_and_graph(ld):
    """Steps in one call, in several with reads between, and replayed from a
    graph see the same clock and noise."""
    drops = _droplets((70, 300, 2))
    a, b, c = (ld.Ensemble(drops) for _ in range(3))
    c.set_tuning(graph_steps=4)
    b.set_tuning(graph_steps=0)
    a.step(12, 5e-3)
    for k in (1, 3, 0, 8):
        b.step(k, 5e-3)
        b.forces()
    c.step(12, 5e-3)
    assert a.state() == b.state() and a.state()[0] == c.state()[0] == 12
    assert np.array_equal(a.positions64(), b.positions64())
    assert np.abs(c.positions64() - a.positions64()).max() <= 1e-4


def test_many_droplets(ld, orc):
    """More droplets than the sort key holds: unsorted slots."""
    w = _droplets((2,))[0]
    ens = ld.Ensemble([w.replace(seed=k) for k in range(8193)])
    F = ens.forces().cpu().numpy().reshape(8193, 2, 3)
    Fo, So, _ = orc.pair_forces(w.pos, w.type, w.charge, w.params)
    assert (np.linalg.norm(F - Fo, axis=2) <= 1e-5 * So).all()


@pytest.mark.parametrize("drops", [127, 128])
def test_groups_apart(ld, orc, drops):
    """The largest ensemble with the groups between the tasks and the smallest
    with a launch of their own (64 tiles each)."""
    w = _droplets((4096,), 5)[0]
    ens = ld.Ensemble([w.replace(seed=k) for k in range(drops)])
    F = ens.forces().cpu().numpy().reshape(drops, w.n, 3)
    rows = np.unique(np.linspace(0, w.n - 1, 100).astype(int))
    Fo, So, _ = orc.pair_forces(w.pos, w.type, w.charge, w.params, rows=rows)
    assert (np.linalg.norm(F[:, rows] - Fo, axis=2) <= 1e-5 * So).all()
    ens.kernel_timing(True)                 # the timed launches give the same steps
    ens.step(2, 1e-6)
    x = ens.positions64()
    other = ld.Ensemble([w.replace(seed=k) for k in range(drops)])
    other.step(2, 1e-6)
    assert np.array_equal(x, other.positions64())
