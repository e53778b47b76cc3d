"""The launch-shape search times the kernel whose shape it sets, and its cache
keeps the kernels apart: sizes of one bucket on either side of the symmetric
kernel's range, lines without a kernel, and the learned path's direct sums."""
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


def lines(path):
    return [x.split() for x in open(path).read().splitlines()]


def system(ld, n):
    return ld.System.from_workload(W.config_medium(n=n, seed=n))


@pytest.mark.parametrize("first,second", [(13000, 11800), (11800, 13000)])
def test_kernels_apart(ld, tmp_path, first, second):
    cache = str(tmp_path / "tune.txt")       # both in the bucket 2^13.5 .. 2^13.75
    system(ld, first).autotune(cache_path=cache)
    assert len(lines(cache)) == 1
    s = system(ld, second)
    t = s.autotune(cache_path=cache)
    got = lines(cache)
    assert len(got) == 2 and got[0][0] != got[1][0]
    assert (t["block"], t["j_split"]) == (int(got[1][1]), int(got[1][2]))
    # a hit takes the line of its own kernel
    hit = system(ld, second).autotune(cache_path=cache)
    assert (hit["block"], hit["j_split"]) == (t["block"], t["j_split"])
    assert len(lines(cache)) == 2


def test_unculled_and_learned(ld, tmp_path):
    cache = str(tmp_path / "tune.txt")
    s = system(ld, 3000)
    s.autotune(cache_path=cache)             # the one-launch kernel
    s = system(ld, 3000)
    s.ff_enable(grid=8, block=3, hidden=16, near_mode=ld.NEAR_BLOCK)
    s.ff_mode(2)
    s.autotune(cache_path=cache)             # the tiled kernel of the fallback
    s = system(ld, 3000)
    s.set_tuning(cull=0)
    s.autotune(cache_path=cache)
    assert len({x[0] for x in lines(cache)}) == 3


def test_line_without_kernel(ld, tmp_path):
    """A line of the key without a kernel, as an older library wrote it, is of
    another kernel's shape and not taken."""
    cache = str(tmp_path / "tune.txt")
    system(ld, 5000).autotune(cache_path=cache)
    (key, block, split, ms), = lines(cache)
    with open(cache, "w") as f:
        f.write(f"{key.rsplit('/', 1)[0]} 128 1 0.001\n")
    s = system(ld, 5000)
    s.autotune(cache_path=cache)
    assert len(lines(cache)) == 2


def test_symmetric_context(ld, tmp_path):
    """Searches the tiled kernel's shape (the symmetric one has none): the steps'
    forces stay as they are."""
    cache = str(tmp_path / "tune.txt")
    s = system(ld, 13000)
    F = s.forces(ext=False)["pair"].cpu().numpy()
    s.autotune(cache_path=cache)
    assert lines(cache)[0][0].endswith("/pair2")
    assert np.array_equal(F, s.forces(ext=False)["pair"].cpu().numpy())
