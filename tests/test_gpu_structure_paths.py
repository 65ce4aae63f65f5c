"""Structure analysis where its paths change: hull candidates in one copy and
in two, cells of the grid with hundreds of charges, polygons of many vertices,
radial counts in LDS and in memory; against the structure oracle (scipy)."""
import numpy as np
import pytest
import torch

from oracle import structure as S
from paper_2609_24722_amd import structure as ST, workloads as W

pytestmark = pytest.mark.gpu


def configuration(name):
    rng = np.random.default_rng(len(name))
    if name.startswith("uniform"):
        return W.uniform_disk(int(name[7:]), 17)
    if name == "ring":  # 9000 hull vertices: more candidates than the first copy holds
        a = np.sort(rng.uniform(0, 2 * np.pi, 9000))
        a = a[np.concatenate([[True], np.diff(a) > 1e-6])]
        x, y = W.uniform_disk(500, 18)
        return np.concatenate([np.cos(a), 0.9 * x]), np.concatenate([np.sin(a), 0.9 * y])
    if name == "cluster":  # hundreds of charges in one cell, and a few far from all others
        x, y = W.uniform_disk(3000, 19)
        x[:1500], y[:1500] = 0.2 + 0.004 * x[:1500], 0.1 + 0.004 * y[:1500]
        return x, y
    # one charge in the middle of a circle of 40: a cell of 40 vertices
    a = 2 * np.pi * (np.arange(40) + rng.uniform(-0.1, 0.1, 40)) / 40
    x, y = W.uniform_disk(400, 20)
    far = np.hypot(x, y) > 0.5
    return np.concatenate([[0.0], 0.3 * np.cos(a), x[far]]), np.concatenate([[0.0], 0.3 * np.sin(a), y[far]])


@pytest.mark.parametrize("name", ["uniform65", "uniform129", "uniform4097", "uniform8191", "uniform8193", "uniform20000",
                                  "ring", "cluster", "wheel"])
def test_coordination(dev, name):
    print(f"[case] {name}", flush=True)
    x, y = configuration(name)
    z, psi = ST.voronoi(torch.tensor(x, device=dev), torch.tensor(y, device=dev))
    zo = S.voronoi_z(x, y)
    po = S.psi6(x, y)
    # a cell of more than 48 vertices is reported as -1 (the charges next to the sparse side of the ring), one
    # that comes near it may outgrow the polygon on the way
    zg = z.cpu().numpy()
    assert np.all(zg[zo > 48] == -1) and np.all((zg == zo) | (zo > 36))
    zo = np.where(zo > 36, zg, zo)
    po[zo < 0] = 0
    assert np.max(np.abs(psi.cpu().numpy() - po)) < 1e-11  # coordinates 1e-3 apart in the cluster: 1e-13 in an angle
    st = ST.stats(z, psi)
    assert st["bounded_cells"] == int((zo >= 0).sum()) and st["hull"] == int((zo == -2).sum())


@pytest.mark.parametrize("nbins", [1, 50, 8192, 8193, 30000])
@pytest.mark.parametrize("n", [1, 1023, 300001])
def test_radial_counts(dev, n, nbins):
    x, y = W.uniform_disk(n, 21)
    c = ST.radial_histogram(torch.tensor(x, device=dev), torch.tensor(y, device=dev), nbins).cpu().numpy()
    assert np.array_equal(c, S.radial_counts(x, y, nbins))
