"""The exact FP64 passes of the relax as an evaluation (no iteration): E_sub,
its reduced gradient and the energy change of moved actives, at patch sizes
and charge counts around the 64-charge blocks and the shares of the waves."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2609_24722_amd import FP64, MIXED, relax as R, workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,sizes", [(70, (1, 63, 69)), (129, (64, 65)), (257, (1, 128, 257)), (1000, (3, 200, 999)),
                                     (4097, (17, 64, 700)), (20011, (5000, 1, 321))])
def test_evaluation_against_the_oracle(dev, n, sizes):
    print(f"[case] n={n} sizes={sizes}", flush=True)
    x, y = W.uniform_disk(n, 100 + n)
    xt, yt = torch.tensor(x, device=dev), torch.tensor(y, device=dev)
    rng = np.random.default_rng(n)
    ptr, idx = R.build_patches(xt, yt, rng.choice(n, len(sizes), replace=False).astype(np.int32),
                               np.array(sizes, dtype=np.int32))
    ia = idx.cpu().numpy()
    kx, ky = W.kicks(ia.size, 0.05 * W.spacing(n), 7)
    sx, sy = x[ia] + kx, y[ia] + ky
    r = np.maximum(1.0, np.hypot(sx, sy) * (1 + 1e-12))  # inside the disk: the relax projects nothing
    sx, sy = sx / r, sy / r
    for prec in (FP64, MIXED):
        res = R.relax_subdomains(xt, yt, ptr, idx, torch.tensor(sx, device=dev), torch.tensor(sy, device=dev),
                                 precision=prec, max_iter=0)
        torch.cuda.synchronize()
        for p in range(len(sizes)):
            s = slice(ptr[p], ptr[p + 1])
            E, gx, gy = O.esub(x, y, ia[s], sx[s], sy[s], grad=True)
            g = O.reduce_grad(sx[s], sy[s], gx, gy)[3]
            dE = O.esub_delta(x, y, ia[s], sx[s], sy[s])
            # every term of the change is right to about eight roundings; the sums are compensated per block
            ox, oy = x[ia[s]], y[ia[s]]
            F = np.ones(n, dtype=bool)
            F[ia[s]] = False
            v = np.abs(1 / np.hypot(sx[s][:, None] - x[F], sy[s][:, None] - y[F]) -
                       1 / np.hypot(ox[:, None] - x[F], oy[:, None] - y[F])).sum()
            with np.errstate(divide="ignore", invalid="ignore"):
                w = np.abs(1 / np.hypot(sx[s][:, None] - sx[s], sy[s][:, None] - sy[s]) -
                           1 / np.hypot(ox[:, None] - ox, oy[:, None] - oy))
            v += 0.5 * np.nansum(np.where(np.isfinite(w), w, 0.0))
            got = (res.e_sub[p].item(), res.dE[p].item(), res.gtan_inf[p].item())
            print(f"[err] n={n} size={sizes[p]} E={abs(got[0] - E) / E:.1e} dE={abs(got[1] - dE) / max(v, 1e-300):.1e}"
                  f" g={abs(got[2] - g) / g:.1e}")
            assert abs(got[0] - E) <= 1e-13 * E
            assert abs(got[1] - dE) <= 4e-15 * v
            assert abs(got[2] - g) <= 1e-11 * g
