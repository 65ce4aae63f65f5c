"""The relax's update at patch sizes around its waves' shares of the actives
(256 per wave, 320 in a call with a patch above 4096, more than its registers
hold above 5120): endpoints re-checked by the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2609_24722_amd import FP64, MIXED, relax as R, workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [FP64, MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("sizes", [(1, 63, 64, 65, 255, 256, 257), (511, 512, 513, 1024, 1025), (4096,), (4097, 320, 321, 1),
                                   (5120, 640, 641), (5121,)], ids=lambda s: "-".join(map(str, s)))
def test_endpoints(dev, sizes, prec):
    n = 20000
    print(f"[case] sizes={sizes} prec={prec}", flush=True)
    x, y = W.warped_lattice(n, 0.02, 91)
    h = W.spacing(n)
    xt, yt = torch.tensor(x, device=dev), torch.tensor(y, device=dev)
    # inside the disk, but for the largest, so that the small ones converge from a small kick
    inner = np.nonzero(np.hypot(x, y) < 0.3)[0]
    ptr, idx = R.build_patches(xt, yt, np.random.default_rng(5).choice(inner, len(sizes), replace=False).astype(np.int32),
                               np.array(sizes, dtype=np.int32))
    ia = idx.cpu().numpy()
    kx, ky = W.kicks(ia.size, 0.02 * h, 92)
    sx, sy = x[ia] + kx, y[ia] + ky
    large = max(sizes) > 1100  # a few iterations suffice to run every part of the update there
    kw = dict(gtol=1e-6, polish=R.POLISH_LBFGS)
    if large:
        kw.update(max_iter=40, max_outer=1)
    res = R.relax_subdomains(xt, yt, ptr, idx, torch.tensor(sx, device=dev), torch.tensor(sy, device=dev),
                             precision=prec, **kw)
    torch.cuda.synchronize()
    xo, yo = res.x.cpu().numpy(), res.y.cpu().numpy()
    for p in range(len(sizes)):
        s = slice(ptr[p], ptr[p + 1])
        E, gx, gy = O.esub(x, y, ia[s], xo[s], yo[s], grad=True)
        g = O.reduce_grad(xo[s], yo[s], gx, gy)[3]
        E0 = O.esub(x, y, ia[s], sx[s], sy[s])
        E0 = E0[0] if isinstance(E0, tuple) else E0
        print(f"[err] size={sizes[p]} E={abs(res.e_sub[p].item() - E) / E:.1e} g={g:.1e} drop={E0 - E:.3e}")
        assert abs(res.e_sub[p].item() - E) <= 1e-13 * E
        assert E < E0
        if large:
            assert abs(res.gtan_inf[p].item() - g) <= 1e-9 * g + 1e-8
        else:
            assert int(res.status[p].item()) == 0 and g <= 1.01e-6
