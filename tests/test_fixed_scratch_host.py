"""Plans of a forces call inside a fixed scratch region (host code, no GPU)."""
import ctypes
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2609_24722_amd", "libcoulombdisk.so")

pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="library not built")

OK, CAPACITY = 0, -5
FP64, MIXED = 0, 1


@pytest.fixture(scope="module")
def fits():
    f = ctypes.CDLL(LIB)._ZN2cd17forces_fixed_fitsElim  # cd::forces_fixed_fits(long, int, unsigned long)
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_size_t]
    return f


# one-sided by size (below 7000), symmetric above; mixed with one and with many super-blocks
@pytest.mark.parametrize("precision,n", [(FP64, 1), (FP64, 64), (FP64, 6999), (FP64, 7000), (FP64, 100000),
                                         (MIXED, 1), (MIXED, 128), (MIXED, 6999), (MIXED, 100000)])
def test_too_small_a_region_is_refused(fits, precision, n):
    assert fits(n, precision, 1 << 40) == OK
    for cap in (0, 1, 256, 1024):
        assert fits(n, precision, cap) == CAPACITY
    # a region that fits is found by halving, and every larger one fits too
    lo, hi = 0, 1 << 40
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if fits(n, precision, mid) == CAPACITY else (lo, mid)
    for cap in (hi, hi + 255, 2 * hi, 5 * hi):
        assert fits(n, precision, cap) == OK
