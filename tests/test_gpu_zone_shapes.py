"""Defect lists on both sides of the size up to which one workgroup writes the
list, and around the groups of loads; against their definition in numpy
(bit-exact)."""
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
