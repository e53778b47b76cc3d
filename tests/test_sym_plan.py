"""The symmetric kernel's launch plan on the CPU: every unordered pair of blocks
has one owner, whose task visits it, and every force partial that the update
reads is written."""
import ctypes as C

import numpy as np
import pytest

from paper_2501_04456_amd import ldrop

MAX_CHUNKS = 96


class SymPlan(C.Structure):
    _fields_ = [(k, C.c_int) for k in
                ("jb", "nbc", "mA", "nA", "nds", "nchunk", "slots", "n_full")]
    _fields_ += [("start", C.c_short * (MAX_CHUNKS + 1))]


def plan(n, charged):
    f = ldrop.lib()["_ZN2ld8sym_planEllPNS_7SymPlanE"]
    f.argtypes, f.restype = [C.c_long, C.c_long, C.POINTER(SymPlan)], C.c_bool
    p = SymPlan()
    return p if f(n, charged, C.byref(p)) else None


def owners(nbc):
    """owner[a, b]: block a takes the pair (a, b), a != b, as the kernel decides."""
    a, b = np.meshgrid(np.arange(nbc), np.arange(nbc), indexing="ij")
    d = (b - a) % nbc
    return (a != b) & ((2 * d < nbc) | ((2 * d == nbc) & (a < b)))


def check(n, charged):
    p = plan(n, charged)
    if p is None:
        # refused for its memory alone: more than 6 GiB with the fewest column
        # partials (super-blocks of 16 blocks of 512) and a row partial for each
        assert 24 * n * (1 + 2 * (charged // (2 * 16 * 512) + 3)) > 6 << 30, (n, charged)
        return None
    per = 64 * p.jb
    assert p.jb == (4 if n < 81920 else 8)
    assert p.nbc == -(-charged // per) and p.nA == -(-p.nbc // p.mA)
    assert p.n_full == min(p.nbc * per, n)
    start = list(p.start)[:p.nchunk + 1]
    if charged:
        # runs of column super-blocks, none empty, all of them
        assert start[0] == 0 and start[-1] == p.nds and (np.diff(start) > 0).all()
        assert p.nchunk <= MAX_CHUNKS
    else:
        assert p.nchunk == 0
    assert p.slots == 1 + p.nds + p.nchunk
    # distinct column super-blocks for each row super-block: one writer a partial,
    # and every row super-block reaches every column partial of the first nds
    assert p.nds <= p.nA
    if 1 < p.nbc <= 900:
        own = owners(p.nbc)
        assert (own ^ own.T | np.eye(p.nbc, dtype=bool)).all() and not (own & own.T).any()
        a, b = np.nonzero(own)
        assert ((b // p.mA - a // p.mA) % p.nA < p.nds).all(), (n, charged)
    return p


def test_small_block_counts():
    for charged in range(0, 60 * 256 + 1, 97):
        check(max(12288, charged), charged)


@pytest.mark.parametrize("n", [12288, 12289, 24577, 81919, 81920, 81921, 100001, 250000, 300001,
                               420007, 999999, 3000001])
def test_sizes(n):
    for charged in (0, 1, 2, 255, 256, 257, 513, n // 3, n - 1, n):
        check(n, charged)


def test_super_blocks():
    """Every super-block size occurs, and what takes too much memory is refused."""
    seen = {check(n, n).mA for n in (20000, 100000, 270000, 350000, 500000, 1500000)}
    assert {1, 2, 4, 8, 16} <= seen, seen
    assert plan(1 << 27, 1 << 27) is None
