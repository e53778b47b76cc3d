"""The size from which the symmetric kernel takes over, and super-blocks of four
and more blocks, against the oracle."""
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


def check(orc, s, w, rows):
    F = s.forces(ext=False)["pair"].cpu().numpy()
    Fo, So, _ = orc.pair_forces(w.pos, w.type, w.charge, w.params, rows=rows)
    # FP32 pair terms, at most 36 roundings in a row: 36 u sum|f| < 2.2e-6 of S,
    # and as much for the terms themselves
    assert (np.linalg.norm(F[rows] - Fo, axis=1) <= 1e-5 * So).all()
    assert np.linalg.norm(F.sum(0)) <= 1e-6 * np.abs(F).sum()
    return F


# 12288 slots are the first that the symmetric kernel takes; the sizes below are
# the one-launch kernel's.  large: a fifth uncharged, behind the charged ones
@pytest.mark.parametrize("recipe", ["medium", "large"])
@pytest.mark.parametrize("n", [12287, 12288, 12289, 12351, 12353])
def test_threshold(ld, orc, recipe, n):
    w = {"medium": W.config_medium, "large": W.config_large}[recipe](n=n)
    s = ld.System.from_workload(w)
    rows = np.unique(np.concatenate([[0, n - 1], np.random.default_rng(n).choice(n, 300)]))
    F = check(orc, s, w, rows)
    # a launch shape of the one-sided kernels moves the bits of one side only
    s.set_tuning(block=64, j_split=7)
    G = check(orc, s, w, rows)
    assert np.array_equal(F, G) == (n >= 12288)
    # eager steps and replayed ones take the same kernel
    a, b = ld.System.from_workload(w), ld.System.from_workload(w)
    for x in (a, b):
        x.set_tuning(sort_every=3)
    b.set_tuning(graph_steps=3)
    st = orc.State(w)
    a.step(6, w.dt)
    b.step(6, w.dt)
    assert np.array_equal(a.positions64(), b.positions64())
    st.run(6)
    assert np.abs(a.positions64() - st.x).max() <= 1e-4


# all charged: super-blocks of 4, 8 and 16 blocks of 512 slots
@pytest.mark.parametrize("n", [270001, 350003, 500009])
def test_super_blocks(ld, orc, n):
    w = W.config_medium(n=n)
    s = ld.System.from_workload(w)
    rows = np.unique(np.concatenate([[0, n - 1], np.random.default_rng(n).choice(n, 60)]))
    check(orc, s, w, rows)
