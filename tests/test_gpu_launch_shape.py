"""The default launch shapes of the two one-sided kernels below the symmetric
kernel's range: each has its own, a shape set by the caller serves both."""
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


def pair_default(n):
    """Many workgroups, at least 256 columns to a split."""
    block = 256 if n > 8192 else 128
    tiles = (n + block - 1) // block
    return block, min((32768 + tiles - 1) // tiles, max(n // 256, 1), 32)


def direct_default(n):
    """Eight wavefronts and two groups each up to 8192, then 2048 workgroups."""
    groups = (n + 63) // 64
    return (512, (groups + 15) // 16) if n <= 8192 else (256, (2048 + groups - 1) // groups)


@pytest.mark.parametrize("n", [2, 255, 257, 1000, 5000, 8192, 8193, 12287, 12288, 16383, 16384])
def test_defaults(ld, n):
    w = W.config_medium(n=n, seed=n)
    s = ld.System.from_workload(w)
    t = s.tuning()
    assert (t["block"], t["j_split"]) == pair_default(n)
    # a captured step and an eager one take the same shape
    a, b = ld.System.from_workload(w), ld.System.from_workload(w)
    for x in (a, b):
        x.set_tuning(sort_every=3)
    b.set_tuning(graph_steps=3)
    a.step(6, 1e-6)
    b.step(6, 1e-6)
    assert np.array_equal(a.positions64(), b.positions64())


@pytest.mark.parametrize("n", [257, 1000, 5000, 8193, 12287])
def test_shapes_used(ld, n):
    """The same partials, bit for bit, as with the shape given."""
    w = W.config_medium(n=n, seed=n)
    s = ld.System.from_workload(w)

    def forces(**kw):
        s.set_tuning(**kw)
        return s.forces(ext=False)["pair"].cpu().numpy()

    (pb, ps), (db, ds) = pair_default(n), direct_default(n)
    own = forces(block=pb, j_split=ps)
    assert np.array_equal(own, forces(block=db, j_split=ds))
    plain = forces(block=pb, j_split=ps, cull=0)
    assert np.array_equal(plain, forces(block=pb, j_split=ps, cull=0))
    other = forces(block=256, j_split=max(ps - 1, 1), cull=1)
    nrm = np.linalg.norm(own, axis=1)
    assert np.median(np.linalg.norm(other - own, axis=1) / nrm) <= 1e-6
    assert np.median(np.linalg.norm(plain - own, axis=1) / nrm) <= 1e-6


# the Lennard-Jones groups in the tiles' launch (1 and 2 groups; more than 24
# to a part) and in one of their own
@pytest.mark.parametrize("n,parts", [(64, 1), (128, 4), (129, 1), (1536, 1), (1537, 1), (4999, 3),
                                     (4999, 8)])
@pytest.mark.parametrize("cut", [2.5, 30.0])
def test_blocks_of_one_wavefront(ld, n, parts, cut):
    w = W.config_large(n=n, seed=n)
    w.params.lj_cut = cut
    a, b = ld.System.from_workload(w), ld.System.from_workload(w)
    a.set_tuning(block=64, j_split=parts, sort_every=3)
    b.set_tuning(block=256, j_split=parts, sort_every=3)
    Fa, Fb = (s.forces(ext=False)["pair"].cpu().numpy() for s in (a, b))
    S = b.forces(ext=False, S=True)["S"].cpu().numpy()
    # FP32 terms of the same pairs, two roundings of 2^-24 each at most apart
    assert (np.linalg.norm(Fa - Fb, axis=1) <= 1e-6 * S).all()
    # the clock goes on once a step, eager and captured
    c = ld.System.from_workload(w)
    c.set_tuning(block=64, j_split=parts, sort_every=3, graph_steps=3)
    d = [s.step(6, 1e-6, diag=True) for s in (a, c)]
    assert np.array_equal(a.positions64(), c.positions64())
    assert all(x["step"] == 6 and x["t"] == pytest.approx(6e-6, rel=1e-12) for x in d)
