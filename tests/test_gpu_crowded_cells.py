"""Cells crowded by one particle far outside, where a lane takes a particle by
itself and candidates in full windows: forces of the truncated scheme and pair
counts, and the same bits however steps are split."""
import numpy as np
import pytest
from scipy.spatial import cKDTree

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
    oracle.lib()
    return oracle


def droplet(n, far):
    w = W.config_large(n=n, seed=n)
    w.pos = w.pos.copy()
    w.pos[17] = (far, -0.5 * far, 3.0)
    w.params.jump_max = 0.0
    w.params.k_wall = [0.0] * len(w.params.k_wall)
    return w


# cells of half a droplet, of a quarter, and not crowded; rows that end in every
# remainder of a window occur among the sampled particles
@pytest.mark.parametrize("far", [2e4, 1500.0, 0.0])
@pytest.mark.parametrize("n", [60000, 60007])
def test_forces(ld, orc, n, far):
    w = droplet(n, far)
    s = ld.System.from_workload(w)
    s.paper_enable(range_factor=6.0)
    c = np.sqrt(w.params.kT * w.params.bjerrum)
    q = (w.charge * c).astype(np.float32).astype(np.float64) / c     # as a context stores them
    rows = np.unique(np.concatenate([[0, 17, n - 1], np.linspace(0, n - 1, 300).astype(int)]))
    F = s.paper_forces()
    Fo, So = orc.paper_forces(w.pos, w.type, q, w.params, 6.0, rows=rows)
    assert (So > 0).mean() > 0.2
    # FP64 pair terms: a few ulp of each
    assert (np.linalg.norm(F[rows] - Fo, axis=1) <= 1e-12 * So).all()


@pytest.mark.parametrize("far", [2e4, 1500.0])
def test_pair_counts(ld, far):
    n, r_max, bins = 75003, 8.0, 160
    w = droplet(n, far)
    s = ld.System.from_workload(w)
    counts = s.rdf(r_max, bins, V=1.0)[0]
    x = w.pos.astype(np.float64)
    p = cKDTree(x).query_pairs(r_max * (1 + 1e-9), output_type="ndarray")
    d = x[p[:, 0]] - x[p[:, 1]]
    r = np.sqrt(d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1] + d[:, 2] * d[:, 2])
    b = np.floor(r[r < r_max] / (r_max / bins)).astype(int)
    assert np.array_equal(counts, np.bincount(b, minlength=bins)[:bins])


def test_split(ld):
    x = []
    for calls in ((6,), (1, 2, 3)):
        s = ld.System.from_workload(droplet(60007, 1500.0))
        s.paper_enable(range_factor=4.0, kick=0.05)
        for k in calls:
            s.step(k, 5e-4)
        x.append((s.positions64(), s.velocities()))
    assert np.array_equal(x[0][0], x[1][0]) and np.array_equal(x[0][1], x[1][1])
