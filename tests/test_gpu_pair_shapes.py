"""The pair passes at the sizes where their launch shape changes and around
whole super-blocks, against the CPU oracle's rows.  Tolerances as in
test_gpu_pairs: the shape moves only the order of FP64 sums."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2609_24722_amd import FP64, MIXED, ops, workloads as W

pytestmark = pytest.mark.gpu

TOL = {FP64: dict(E=1e-13, F=1e-11, H=1e-11, e=1e-12), MIXED: dict(E=1e-7, F=1e-5, H=1e-5, e=1e-6)}
# 128- and 256-charge super-blocks: one, one and a charge, two, an odd and an even number of them, and the
# numbers of offsets (40, 160, 320 of 128 charges) where the shape changes, on both sides
SIZES = (128, 129, 255, 256, 257, 385, 512, 513, 1023, 1025, 10367, 10369, 41087, 41216, 82176)


def rel_rms(ax, ay, bx, by):
    return np.sqrt(np.sum((ax - bx) ** 2 + (ay - by) ** 2) / np.sum(bx ** 2 + by ** 2))


@pytest.mark.parametrize("prec", [FP64, MIXED], ids=["fp64", "mixed"])
@pytest.mark.parametrize("n", SIZES)
def test_pair_passes_at_shape_edges(dev, n, prec):
    print(f"[case] n={n} prec={prec}", flush=True)
    x, y = W.uniform_disk(n, 7000 + n) if n < 2000 else W.warped_lattice(n, 0.02, 7000 + n)
    vx, vy = W.unit_vector(n, 7100 + n)
    xt, yt, vxt, vyt = (torch.tensor(a, device=dev) for a in (x, y, vx, vy))
    fx, fy, E = ops.forces(xt, yt, prec)
    E2, e = ops.energy(xt, yt, prec, local=True)
    E3 = ops.energy(xt, yt, prec)
    hx, hy = ops.hvp(xt, yt, vxt, vyt, prec)
    torch.cuda.synchronize()
    rows = np.sort(np.random.default_rng(n).choice(n, min(n, 256), replace=False)).astype(np.int32)
    ofx, ofy, oe = O.rows(x, y, rows)
    ohx, ohy, _ = O.rows(x, y, rows, vx, vy)
    fx, fy, e, hx, hy = (a.cpu().numpy() for a in (fx, fy, e, hx, hy))
    E0 = e.sum() if n > 20000 else O.energy(x, y)  # the rows pin e there
    tol = TOL[prec]
    errs = dict(F=rel_rms(fx[rows], fy[rows], ofx, ofy), H=rel_rms(hx[rows], hy[rows], ohx, ohy),
                e=np.max(np.abs(e[rows] - oe) / oe), E=max(abs(q.item() - E0) / E0 for q in (E, E2, E3)))
    print(f"[err] n={n} prec={prec} {errs}")
    assert all(errs[k] <= tol[k] for k in errs), errs
