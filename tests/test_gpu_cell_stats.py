"""Statistics over the counted cell lists at their edges: one cell, both lane
counts, no surface NP, a giant component, against trees on the CPU."""
import numpy as np
import pytest
from scipy.sparse import coo_matrix
from scipy.sparse.csgraph import connected_components
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


def _labels(x, sig, factor, on):
    """Smallest index of each particle's contact component, -1 where not on."""
    lab = np.full(len(x), -1, np.int64)
    idx = np.flatnonzero(on)
    if len(idx) == 0:
        return lab
    pairs = cKDTree(x[idx]).query_pairs(factor * sig.max() * 1.0001, output_type="ndarray")
    i, j = idx[pairs[:, 0]], idx[pairs[:, 1]]
    d = x[i] - x[j]
    hit = (d * d).sum(1) < (factor * 0.5 * (sig[i] + sig[j])) ** 2
    n = len(x)
    _, c = connected_components(coo_matrix((np.ones(hit.sum()), (i[hit], j[hit])), (n, n)), False)
    small = np.full(n, n, np.int64)
    np.minimum.at(small, c, np.arange(n))
    lab[idx] = small[c[idx]]
    return lab


@pytest.mark.parametrize("n,factor", [(2, 1.1), (300, 1e3), (4097, 4.0), (74999, 3.0),
                                      (75000, 3.0), (75000, 6.0)])
def test_components(ld, n, factor):
    w = W.config_medium(n=n, seed=3)
    s = ld.System.from_workload(w)
    x, sig = w.pos.astype(np.float64), np.asarray(w.params.sigma)[w.type]
    st = s.aggregates(factor, labels=True)
    lab = _labels(x, sig, factor, np.ones(n, bool))
    assert np.array_equal(st["labels"], lab)
    size = np.bincount(lab, minlength=n)
    assert [st[k] for k in ("components", "aggregates", "largest")] == \
        [np.count_nonzero(size), np.count_nonzero(size >= 2), size.max()]


@pytest.mark.parametrize("n,n_surf,factor", [(2000, 0, 1.5), (3000, 800, 1.1), (80000, 9000, 1.3),
                                             (500, 400, 1e3)])
def test_surface_components(ld, n, n_surf, factor):
    sigma, R0 = [1.0, 1.5], 60.0
    rng = np.random.default_rng(n)
    r = np.where(np.arange(n) < n_surf, R0 + 0.4 * (rng.random(n) - 0.5),
                 0.9 * R0 * rng.random(n) ** (1 / 3))
    u = rng.standard_normal((n, 3))
    x = (r[:, None] * u / np.linalg.norm(u, axis=1, keepdims=True)).astype(np.float32)
    typ = (rng.random(n) < 0.5).astype(np.int32)
    p = W.config_medium(n=100, with_positions=False).params
    w = W.Workload("s", n, typ, np.zeros(n), x, p, W.Radius(kind=W.RADIUS_CONST, R0=R0), 5e-4, 1, 1)
    s = ld.System.from_workload(w)
    x, sig = x.astype(np.float64), np.asarray(sigma)[typ]
    on = np.abs(np.linalg.norm(x, axis=1) - R0) < 0.5 * sig
    assert np.count_nonzero(on) == n_surf
    got = s.surface_fractal(contact_factor=factor, labels=True)
    lab = _labels(x, sig, factor, on)
    assert np.array_equal(got["labels"], lab)
    size = np.bincount(lab[on], minlength=1)
    assert got["components"] == np.count_nonzero(size)
    if n_surf:
        assert (got["largest"], got["label"]) == (size.max(), int(size.argmax()))


@pytest.mark.parametrize("n,r_max", [(3000, 12.0), (74999, 8.0), (75000, 8.0)])
def test_rdf_counts(ld, n, r_max):
    w = W.config_medium(n=n, seed=9)
    s = ld.System.from_workload(w)
    counts = s.rdf(r_max, 37)[0]
    t = cKDTree(w.pos.astype(np.float64))
    edges = np.arange(1, 38) * (r_max / 37)
    c = (t.count_neighbors(t, edges) - n) // 2           # pairs within the edge, inclusive
    assert np.array_equal(np.cumsum(counts.astype(np.int64)), c)
