"""Defect lists on both sides of the size up to which one workgroup writes the
list, and zone lists where the workgroups per zone change (128 and 256 zones),
at charge counts around the groups a wave loads; against their definitions in
numpy (bit-exact)."""
import numpy as np
import pytest
import torch

from paper_2609_24722_amd import workloads as W, zones as Z

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 1023, 2049, 8193, 10241, 16383, 16384, 16385, 20481])
def test_defect_lists(dev, n):
    print(f"[case] n={n}", flush=True)
    x, y = (torch.tensor(v, device=dev) for v in W.uniform_disk(n, n))
    rng = np.random.default_rng(n)
    none = torch.zeros(0, dtype=torch.float64, device=dev)
    # integers: their sums and the mean's rounding are the same in any order
    for e in (rng.integers(0, 2 ** 20, n).astype(np.float64), np.full(n, 3.0), np.arange(n, dtype=np.float64)):
        z = Z.defect_zones(x, y, torch.tensor(e, device=dev), none, 0.5)
        mu, sd, thr, cnt = z["stats"].cpu().tolist()
        assert mu == e.sum() / n and abs(sd - e.std()) <= 1e-12 * max(1.0, e.std())
        want = np.nonzero(e > thr)[0]
        assert int(cnt) == want.size and np.array_equal(z["defects"].cpu().numpy()[:want.size], want)


@pytest.mark.parametrize("zones", [128, 129, 256, 257])
@pytest.mark.parametrize("n", [100, 1025, 4097, 8193, 16385])
def test_zone_lists(dev, n, zones):
    print(f"[case] n={n} zones={zones}", flush=True)
    x, y = W.uniform_disk(n, n)
    rng = np.random.default_rng(zones)
    cx, cy, rz = rng.uniform(-0.7, 0.7, zones), rng.uniform(-0.7, 0.7, zones), rng.uniform(0.0, 0.3, zones)
    rz[0] = 3.0  # every charge
    f = dict(dtype=torch.float64, device=dev)
    ptr, idx = Z.zone_patches(torch.tensor(x, device=dev), torch.tensor(y, device=dev), torch.tensor(cx, **f),
                              torch.tensor(cy, **f), torch.tensor(rz, **f))
    idx = idx.cpu().numpy()
    for p in range(zones):
        dx, dy = x - cx[p], y - cy[p]
        assert np.array_equal(idx[ptr[p]:ptr[p + 1]], np.nonzero(dx * dx + dy * dy <= rz[p] * rz[p])[0])
