"""Newton polish where a round takes one, two or three CG iterations (mixed path
and fewer than 64 actives; fewer than eight patches or 8192 charges; the rest):
every endpoint re-checked by the oracle (E_sub to 1e-13, the reduced gradient
below the tolerance, the exact energy change), and the rounds replayed from HIP
graphs bit for bit as the launches made one by one."""
import numpy as np
import pytest
import torch

from paper_2609_24722_amd import FP64, MIXED, workloads as W
from paper_2609_24722_amd import relax as R
from test_gpu_relax import check_endpoints, t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,n,sizes", [(FP64, 6000, [1]), (FP64, 6000, [63]), (FP64, 6000, [64]), (FP64, 6000, [8] * 8),
                                          (FP64, 1024, [300]), (FP64, 1024, [64] * 5), (FP64, 8191, [40] * 8),
                                          (FP64, 8192, [40] * 7), (FP64, 8192, [40] * 8), (FP64, 9000, [511] + [512] * 7),
                                          (MIXED, 6000, [300]), (MIXED, 9000, [40] * 8)],
                         ids=lambda v: f"{len(v)}x{v[-1]}" if isinstance(v, list) else ("fp64", "mixed")[v] if v < 2 else str(v))
def test_endpoints_across_the_rule(dev, prec, n, sizes):
    print(f"[case] prec={prec} n={n} sizes={sizes}", flush=True)
    x, y = W.warped_lattice(n, 0.02, 31)
    inner = np.nonzero(np.hypot(x, y) < 0.6)[0]
    centres = np.random.default_rng(32).choice(inner, len(sizes), replace=False).astype(np.int32)
    xt, yt = t(x, dev), t(y, dev)
    ptr, idx = R.build_patches(xt, yt, centres, np.array(sizes, dtype=np.int32))
    ia = idx.cpu().numpy()
    kx, ky = W.kicks(ia.size, 0.02 * W.spacing(n), 33)
    out = []
    for launch in (R.LAUNCH_GRAPH, R.LAUNCH_PLAIN):
        res = R.relax_subdomains(xt, yt, ptr, idx, t(x[ia] + kx, dev), t(y[ia] + ky, dev), precision=prec, gtol=1e-6,
                                 polish=R.POLISH_NEWTON, launch=launch)
        torch.cuda.synchronize()
        out.append(res)
    check_endpoints(x, y, ptr, ia, out[0], 1e-6, f"cg-{prec}-{sum(sizes)}")
    assert sizes == [1] or (out[0].polish.cpu().numpy() > 0).all()
    for f in ("x", "y", "dE", "e_sub", "iters", "status", "polish"):
        assert torch.equal(getattr(out[0], f), getattr(out[1], f)), f
