"""Voronoi cells with as many vertices as a polygon holds (48) and more: a
charge in the middle of a circle of k others has a cell of exactly k vertices,
each on the bisector of one of them, and no step on the way has more (every
bisector touches the same circle, and the square's corners are gone once the
others surround it).  Against the structure oracle (scipy)."""
import numpy as np
import pytest
import torch

from oracle import structure as S
from paper_2609_24722_amd import structure as ST, workloads as W

pytestmark = pytest.mark.gpu

LIMIT = 48


def wheel(k):
    rng = np.random.default_rng(k)
    a = 2 * np.pi * (np.arange(k) + rng.uniform(-0.1, 0.1, k)) / k
    x, y = W.uniform_disk(400, 20)
    far = np.hypot(x, y) > 0.65
    return np.concatenate([[0.0], 0.3 * np.cos(a), x[far]]), np.concatenate([[0.0], 0.3 * np.sin(a), y[far]])


@pytest.mark.parametrize("k", [5, 17, 40, 47, 48, 49, 64, 65, 120])
def test_wheel(dev, k):
    print(f"[case] wheel of {k}", flush=True)
    x, y = wheel(k)
    z, psi = ST.voronoi(torch.tensor(x, device=dev), torch.tensor(y, device=dev))
    z, psi = z.cpu().numpy(), psi.cpu().numpy()
    zo, po = S.voronoi_z(x, y), S.psi6(x, y)
    po[zo < 0] = 0  # on the hull
    assert zo[0] == k and np.max(zo[1:]) < 24
    if k > LIMIT:
        assert z[0] == -1 and psi[0].real == 0 and psi[0].imag == 0
    else:
        # k unit vectors to the sixth power: six times the angle's rounding, averaged
        assert z[0] == k and abs(psi[0] - po[0]) < 1e-13
    assert np.array_equal(z[1:], zo[1:])
    assert np.max(np.abs(psi[1:] - po[1:])) < 1e-12


def test_ring(dev):
    """9000 charges on the circle and 500 inside: the inner ones next to the
    circle have cells around and above the limit.  A cell is the oracle's, or
    -1: where it has more vertices than the polygon holds, and where it has so
    many (above 36) that a step on the way may have had."""
    a = np.sort(np.random.default_rng(4).uniform(0, 2 * np.pi, 9000))
    a = a[np.concatenate([[True], np.diff(a) > 1e-6])]
    x, y = W.uniform_disk(500, 18)
    x, y = np.concatenate([np.cos(a), 0.9 * x]), np.concatenate([np.sin(a), 0.9 * y])
    z, psi = ST.voronoi(torch.tensor(x, device=dev), torch.tensor(y, device=dev))
    z, psi = z.cpu().numpy(), psi.cpu().numpy()
    zo, po = S.voronoi_z(x, y), S.psi6(x, y)
    po[zo < 0] = 0  # on the hull
    assert np.all((z == zo) | ((z == -1) & (zo > 36))) and np.all(z[zo > LIMIT] == -1)
    bad = z == -1
    assert np.all(psi[bad] == 0) and np.max(np.abs(psi[~bad] - po[~bad])) < 1e-11
