"""The staging order of the pair passes at the sizes around the two sort
paths' line and their tiles, with thousands of charges in few Morton cells.

The mixed pass groups the charges in blocks of 64 in the order of (Morton
key, index), so its results depend on that order bit for bit: the same
charges handed over already in order, and shuffled (charges of one key kept
in their order), have to give the same forces."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2609_24722_amd import FP64, MIXED, ops, workloads as W

pytestmark = pytest.mark.gpu


def morton(x, y):
    def spread(v):
        v = np.clip((v + 1.0) * 2048.0, 0.0, 4095.0).astype(np.uint32)
        for s, m in ((8, 0x00ff00ff), (4, 0x0f0f0f0f), (2, 0x33333333), (1, 0x55555555)):
            v = (v | (v << np.uint32(s))) & np.uint32(m)
        return v
    return spread(x) | (spread(y) << np.uint32(1))


@pytest.mark.parametrize("n", [63, 64, 65, 1023, 2049, 12287, 12288, 12289, 14336, 14337, 262144, 262145, 264193])
def test_shuffled_charges_take_the_same_order(dev, n):
    print(f"[case] n={n}", flush=True)
    rng = np.random.default_rng(n)
    x, y = W.uniform_disk(n, n)
    few = rng.random(n) < 0.2
    x[few], y[few] = 0.01 * x[few] + 0.3, 0.01 * y[few] - 0.2
    o = np.argsort(morton(x, y), kind="stable")
    x, y = x[o], y[o]
    k = morton(x, y)
    # place[s]: where charge s of the order goes; the places of one key increase
    place = rng.permutation(n)
    place = place[np.lexsort((place, k))]
    sx, sy = np.empty(n), np.empty(n)
    sx[place], sy[place] = x, y
    a = ops.forces(torch.tensor(x, device=dev), torch.tensor(y, device=dev), MIXED)
    b = ops.forces(torch.tensor(sx, device=dev), torch.tensor(sy, device=dev), MIXED)
    p = torch.tensor(place, device=dev)
    assert torch.equal(a[0], b[0][p]) and torch.equal(a[1], b[1][p]) and torch.equal(a[2], b[2])


@pytest.mark.parametrize("n", [12288, 12289])
def test_forces_on_both_sides_of_the_line(dev, n):
    x, y = W.warped_lattice(n, 0.02, n)
    fx, fy, _ = ops.forces(torch.tensor(x, device=dev), torch.tensor(y, device=dev), FP64)
    rows = np.arange(0, n, 97, dtype=np.int32)
    ox, oy, _ = O.rows(x, y, rows)
    fx, fy = fx.cpu().numpy()[rows], fy.cpu().numpy()[rows]
    assert np.sqrt(np.sum((fx - ox) ** 2 + (fy - oy) ** 2)) <= 1e-11 * np.sqrt(np.sum(ox ** 2 + oy ** 2))
