"""The batch scheduler over radii from 0 to the disk's, caps from 1 up and both
orders: exactly the oracle's batches, at a cost set by the number of zones and
not by how small they are (host code, no GPU)."""
import os
import time

import numpy as np
import pytest

from oracle import zones as Z

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2609_24722_amd", "libcoulombdisk.so")

pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="library not built")


def _zones(T, r_lo, r_hi, seed):
    rng = np.random.default_rng(seed)
    a, r = rng.uniform(0, 2 * np.pi, T), np.sqrt(rng.uniform(0, 1, T))
    return r * np.cos(a), r * np.sin(a), rng.uniform(r_lo, r_hi, T)


# up to 64 batches and beyond (T = 300 at radius 1: a batch per zone), one zone, one cell and many
@pytest.mark.parametrize("r_lo,r_hi", [(0.0, 0.0), (0.0, 0.002), (0.002, 0.002), (0.01, 0.05), (0.05, 0.3), (1.0, 1.0)])
@pytest.mark.parametrize("cap", [1, 3, 64, 300])
@pytest.mark.parametrize("keep_order", [False, True])
def test_equal_oracle(r_lo, r_hi, cap, keep_order):
    from paper_2609_24722_amd import zones
    for T, gap, seed in ((1, 0.0, 1), (2, 0.1, 2), (65, 0.0, 3), (300, 0.01, 4)):
        cx, cy, rz = _zones(T, r_lo, r_hi, seed)
        b, nb = zones.zone_batches(cx, cy, rz, gap, cap, keep_order)
        want = Z.zone_batches(cx, cy, rz, gap, cap, keep_order)
        assert np.array_equal(b, want) and nb == int(want.max()) + 1, (T, gap)


def test_elongated_and_repeated_centres():
    from paper_2609_24722_amd import zones
    for cx, cy in ((np.linspace(-1, 1, 200), np.zeros(200)), (np.zeros(200), np.linspace(-1, 1, 200)),
                   (np.repeat(np.linspace(-1, 1, 20), 10), np.tile(np.linspace(-1, 1, 4), 50))):
        for r in (0.0, 1e-4, 0.004, 0.3):
            for keep_order in (False, True):
                rz = np.full(cx.size, r)
                b, _ = zones.zone_batches(cx, cy, rz, 0.0, 100, keep_order)
                assert np.array_equal(b, Z.zone_batches(cx, cy, rz, 0.0, 100, keep_order)), (r, keep_order)


def test_small_zones_cost_no_more_than_large_ones():
    """The grid of cells is bounded by the number of zones: 50 zones of radius
    0.001 (a million cells of their size in the disk) take what 50 zones of
    radius 0.1 do."""
    from paper_2609_24722_amd import zones

    def best(r):
        cx, cy, rz = _zones(50, r, r, 5)
        t = []
        for _ in range(30):
            t0 = time.perf_counter()
            zones.zone_batches(cx, cy, rz, 0.0, 256)
            t.append(time.perf_counter() - t0)
        return min(t)

    # the two are within a factor of two; clearing a million cells takes hundreds of times longer
    assert best(0.001) < 20 * best(0.1)
