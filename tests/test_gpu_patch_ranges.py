"""Patches on both sides of the size from which the histogram of the distances
spans the whole disk (half of the charges), about centres at the rim and in
the middle, on uniform, lattice and clustered charges; bit-exact against the
oracle."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2609_24722_amd import relax as R, workloads as W

pytestmark = pytest.mark.gpu


def positions(layout, n):
    if layout == "lattice":
        return W.warped_lattice(n, 0.02, n)
    x, y = W.uniform_disk(n, n)
    if layout == "cluster":  # two clusters: one bin of the histogram or a few
        k = n // 3
        x[:k], y[:k] = 0.5 + 1e-3 * x[:k], 0.1 + 1e-3 * y[:k]
        x[k:2 * k], y[k:2 * k] = -0.9 + 1e-9 * x[k:2 * k], 0.2 + 1e-9 * y[k:2 * k]
    return x, y


@pytest.mark.parametrize("layout", ["uniform", "lattice", "cluster"])
@pytest.mark.parametrize("n", [65, 513, 3000, 12289])
def test_sizes_around_half(dev, layout, n):
    print(f"[case] {layout} n={n}", flush=True)
    x, y = positions(layout, n)
    n = x.size
    r = np.hypot(x, y)
    sizes = np.array([n // 3, n // 2 - 1, n // 2, n // 2 + 1, n // 2 + 2, 3 * n // 4, n - 1, n], dtype=np.int32)
    for c in (int(np.argmax(r)), int(np.argmin(r)), n // 7):
        centres = np.full(sizes.size, c, dtype=np.int32)
        _, idx = R.build_patches(torch.tensor(x, device=dev), torch.tensor(y, device=dev), centres, sizes)
        assert np.array_equal(idx.cpu().numpy(), O.patches(x, y, centres, sizes))
