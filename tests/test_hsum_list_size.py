"""Size of the harmonic sums' hit-row list (the library's own function, no GPU).

Phase 1 appends at most one entry per thread, a thread having four columns and a
segment of the rows: four segments for 85-row spectra of up to 2^18 bins, up to
eight for the other maps below 786,432 bins, and four for the highest-anchored map
from 2^18 to 2^20.  A plan's list has to hold them for
every spectrum that the plan takes, or the launch falls back to fewer segments
than its rule says, and a small plan's list stays small.
"""

import ctypes

import pytest

from paper_1806_01556_amd import fdas


def _entries(n_max, index):
    fn = ctypes.CDLL(fdas.LIB_PATH)._ZN4fdas19harmsum_hit_entriesEli  # fdas::harmsum_hit_entries(int64_t, int)
    fn.argtypes, fn.restype = [ctypes.c_int64, ctypes.c_int], ctypes.c_int64
    return fn(n_max, index)


@pytest.mark.parametrize("n_max", [1, 3361, 16_384, 98_305, 204_800, 204_801, 230_000, 1 << 18, (1 << 18) + 1, 300_000,
                                   786_432, 786_433, 1 << 20, 1 << 22, 1 << 24])
def test_list_holds_every_segment(n_max):
    lengths = (1, 3360, 16_384, 98_304, 200_003, 204_801, 1 << 18, (1 << 18) + 1, 393_216, 1 << 19, 786_432, 1 << 20, n_max)
    for n in sorted({n for n in lengths if n <= n_max}):
        have = _entries(n_max, fdas.HSUM_STRETCH)
        if n <= 1 << 18:
            assert have >= 4 * ((n + 3) // 4), n
        segs = max(1, min(8, 786_432 // n))
        stretch = (n + 3) // 4
        assert have >= segs * stretch, n
        assert _entries(n_max, fdas.HSUM_FUNDAMENTAL) >= segs * ((n + 1023) // 1024 * 256), n
        if 1 << 18 < n <= 1 << 20:
            segs = 4
        assert _entries(n_max, fdas.HSUM_HIGHEST) >= segs * (((n + 3359) // 3360 * 840 + 255) // 256 * 256), n


def test_small_plans_hold_small_lists():
    for index in (fdas.HSUM_STRETCH, fdas.HSUM_FUNDAMENTAL, fdas.HSUM_HIGHEST):
        assert 16 * _entries(16_384, index) <= 1 << 20
        assert _entries(1 << 22, index) <= (1 << 20) + 9000
