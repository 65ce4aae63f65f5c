"""The greedy commit with more candidates than one group of results holds, and
with overlapping, single-charge and whole-block candidates, against the same
greedy loop on the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2609_24722_amd import relax as R, workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,P,hi", [(60, 40, 1), (300, 50, 3), (2000, 300, 4), (1500, 20, 260)])
def test_greedy_order(dev, n, P, hi):
    print(f"[case] n={n} P={P} hi={hi}", flush=True)
    rng = np.random.default_rng(n + P)
    x, y = W.warped_lattice(n, 0.1, n)
    h = W.spacing(n)
    sizes = rng.integers(1, hi + 1, P).astype(np.int32)
    idx = O.patches(x, y, rng.integers(0, n, P).astype(np.int32), sizes)
    ptr = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    kx, ky = W.kicks(idx.size, 0.1 * h, 3)
    xr, yr = x[idx] + kx, y[idx] + ky
    rr = np.hypot(xr, yr)
    xr, yr = np.where(rr > 1, xr / rr, xr), np.where(rr > 1, yr / rr, yr)
    key = rng.uniform(-2.0, 0.3, P)  # a few are not tried
    X, Y = x.copy(), y.copy()
    taken = np.zeros(n, bool)
    ref_c, ref_d = np.zeros(P, np.int32), np.zeros(P)
    for p in np.argsort(key, kind="stable"):
        sl = slice(ptr[p], ptr[p + 1])
        if key[p] >= 0 or taken[idx[sl]].any():
            continue
        ref_d[p] = O.esub_delta(X, Y, idx[sl], xr[sl], yr[sl])
        if ref_d[p] < 0:
            X[idx[sl]], Y[idx[sl]] = xr[sl], yr[sl]
            taken[idx[sl]] = True
            ref_c[p] = 1
    xt, yt = torch.tensor(x, device=dev), torch.tensor(y, device=dev)
    c, d = R.commit_patches(xt, yt, ptr, torch.tensor(idx, device=dev), torch.tensor(xr, device=dev),
                            torch.tensor(yr, device=dev), key)
    torch.cuda.synchronize()
    assert np.array_equal(c, ref_c) and 0 < ref_c.sum() < P
    # 1e-13 of the energy of the pairs that change, n / r of them for each of the candidate's charges
    np.testing.assert_allclose(d, ref_d, rtol=1e-9, atol=1e-13 * O.energy(x, y))
    assert np.array_equal(xt.cpu().numpy(), X) and np.array_equal(yt.cpu().numpy(), Y)
