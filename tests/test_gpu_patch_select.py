"""Patch construction where its histogram does not decide: clustered charges
(thousands in one bin), a centre far from all others (nothing in range), exact
ties, and sizes around the waves' shares; bit-exact against the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2609_24722_amd import relax as R, workloads as W

pytestmark = pytest.mark.gpu


def clustered(n, seed):
    rng = np.random.default_rng(seed)
    x, y = W.uniform_disk(n, seed)
    k = n // 2
    x[:k], y[:k] = 0.4 + 1e-7 * x[:k], -0.3 + 1e-7 * y[:k]
    p = rng.permutation(n)
    return x[p], y[p]


def far(n, seed):
    x, y = W.uniform_disk(n, seed)
    x, y = -0.8 + 0.05 * x, 0.05 * y
    x[n // 2], y[n // 2] = 0.99, 0.0
    return x, y


def equal_distances(n, seed):
    # every charge on one circle around charge 0, and 20 on another
    a = 2 * np.pi * np.arange(n) / n
    x, y = 0.5 * np.cos(a), 0.5 * np.sin(a)
    x[1:], y[1:] = np.where(np.arange(1, n) % 4 < 2, 0.25, -0.25), np.where(np.arange(1, n) % 2 == 0, 0.25, -0.25)
    x[0] = y[0] = 0.0
    x[1:21], y[1:21] = 0.125, 0.0
    return x, y


@pytest.mark.parametrize("make", [clustered, far, equal_distances], ids=lambda f: f.__name__)
@pytest.mark.parametrize("n", [64, 1023, 1025, 9000])
def test_patches_bit_exact(dev, make, n):
    print(f"[case] {make.__name__} n={n}", flush=True)
    x, y = make(n, n)
    rng = np.random.default_rng(n)
    centres = np.concatenate([[0, n // 2, n - 1], rng.integers(0, n, 9)]).astype(np.int32)
    sizes = np.array([1, 2, 20, 21, 22, n // 4, n // 2, n // 2 + 1, n - 1, n, 33, 40], dtype=np.int32)
    for shift in range(3):
        c = np.roll(centres, shift)
        ptr, idx = R.build_patches(torch.tensor(x, device=dev), torch.tensor(y, device=dev), c, sizes)
        assert np.array_equal(idx.cpu().numpy(), O.patches(x, y, c, sizes))


@pytest.mark.parametrize("n", [1, 2, 63, 65, 40003])
def test_ordinary_sizes(dev, n):
    x, y = W.uniform_disk(n, n)
    c = np.arange(0, n, max(1, n // 9)).astype(np.int32)
    for size in sorted({1, min(n, 64), max(1, n // 3), n}):
        s = np.full(c.size, size, dtype=np.int32)
        ptr, idx = R.build_patches(torch.tensor(x, device=dev), torch.tensor(y, device=dev), c, s)
        assert np.array_equal(idx.cpu().numpy(), O.patches(x, y, c, s))
