"""Zone lists and defect lists at charge counts around the waves' and
workgroups' shares, against their definitions in numpy (bit-exact)."""
import numpy as np
import pytest
import torch

from paper_2609_24722_amd import workloads as W, zones as Z

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 64, 65, 4095, 4096, 4097, 8193, 40003])
def test_zone_and_defect_lists(dev, n):
    print(f"[case] n={n}", flush=True)
    x, y = W.uniform_disk(n, n)
    rng = np.random.default_rng(n)
    xt, yt = torch.tensor(x, device=dev), torch.tensor(y, device=dev)
    cx = np.concatenate([[0.0, x[n // 2], 2.0], rng.uniform(-0.7, 0.7, 30)])
    cy = np.concatenate([[0.0, y[n // 2], 2.0], rng.uniform(-0.7, 0.7, 30)])
    rz = np.concatenate([[3.0, 0.0, 0.1], rng.uniform(0.0, 0.6, 30)])
    f = dict(dtype=torch.float64, device=dev)
    ptr, idx = Z.zone_patches(xt, yt, torch.tensor(cx, **f), torch.tensor(cy, **f), torch.tensor(rz, **f))
    idx = idx.cpu().numpy()
    for p in range(cx.size):
        dx, dy = x - cx[p], y - cy[p]
        want = np.nonzero(dx * dx + dy * dy <= rz[p] * rz[p])[0]
        assert np.array_equal(idx[ptr[p]:ptr[p + 1]], want)
    # integers: their sums and the mean's rounding are the same in any order
    e = rng.integers(0, 2 ** 20, n).astype(np.float64)
    z = Z.defect_zones(xt, yt, torch.tensor(e, device=dev), torch.zeros(0, **f), 0.5)
    mu, sd, thr, cnt = z["stats"].cpu().tolist()
    assert mu == e.sum() / n and abs(sd - e.std()) <= 1e-12 * max(1.0, e.std())
    want = np.nonzero(e > thr)[0]
    assert int(cnt) == want.size and np.array_equal(z["defects"].cpu().numpy()[:want.size], want)
