"""The one-launch kernel of small droplets against the oracle: tile edges,
more splits than groups, both defaults, and the step clock that the next
step's force launch advances."""
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


@pytest.mark.parametrize("n,tune", [(2, {}), (64, {}), (129, dict(block=64, j_split=64)),
                                    (1025, dict(block=512, j_split=40)), (8192, {}), (8193, {}),
                                    (8193, dict(block=128, j_split=1, comp=0))])
def test_forces(ld, orc, n, tune):
    w = W.config_large(n=n)
    s = ld.System.from_workload(w)
    if tune:
        s.set_tuning(**tune)
    rows = np.unique(np.linspace(0, n - 1, 200).astype(int))
    F = s.forces(ext=False)["pair"].cpu().numpy()
    Fo, So, _ = orc.pair_forces(w.pos, w.type, w.charge, w.params, rows=rows)
    # FP32 pair terms in blocks of 32: 31 u sum|f| < 2e-6 of S per block
    assert (np.linalg.norm(F[rows] - Fo, axis=1) <= 1e-5 * So).all()


def test_clock(ld, orc, tmp_path):
    """Steps in one call, in several, with recorded frames and with other
    calls between them all see the same clock and noise."""
    w = W.config_medium(n=700)
    a, b, c = (ld.System.from_workload(w) for _ in range(3))
    a.step(9, w.dt)
    path = str(tmp_path / "x.trj")
    b.record_open(path, 2)
    for k in (1, 2, 0, 5, 1):
        b.step(k, w.dt)
        b.forces()
        c.step(k, w.dt, diag=True)
    b.record_close()
    for s in (b, c):
        assert s.state()[:2] == a.state()[:2]
        assert np.array_equal(s.positions64(), a.positions64())
    assert a.state()[0] == 9
    assert list(ld.read_trajectory(path)["step"]) == [2, 4, 6, 8]
    st = orc.State(w)
    st.run(9)
    assert np.abs(a.positions64() - st.x).max() <= 1e-4
