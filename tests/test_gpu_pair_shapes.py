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
# FP64: the sizes where the symmetric pass begins (total energy, forces and products, local energies), and where
# its shape changes (one, two and four offsets, four i charges per lane)
SIZES += (4499, 4500, 4609, 6999, 7000, 7041, 8000, 8001, 11999, 12000, 14000, 14001, 59999, 60000, 60001, 60161)


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


@pytest.mark.parametrize("n", [150001, 700001])
def test_noalloc_fp64_batched_and_one_sided(dev, n):
    # the fixed scratch holds a few chunks of the symmetric pass at the smaller size (summed in the same order as
    # in one batch: identical results) and not one at the larger (one-sided pass)
    import ctypes
    x, y = W.warped_lattice(n, 0.02, 7200)
    xt, yt = torch.tensor(x, device=dev), torch.tensor(y, device=dev)
    fx, fy, E = (torch.full((k,), float("nan"), dtype=torch.float64, device=dev) for k in (n, n, 1))
    f = ops.lib().coulomb_forces_noalloc
    vp = ctypes.c_void_p
    f.restype, f.argtypes = ctypes.c_int, [vp, vp, ctypes.c_int64, ctypes.c_int, vp, vp, vp, vp]
    print(f"[case] noalloc n={n}", flush=True)
    assert f(xt.data_ptr(), yt.data_ptr(), n, FP64, fx.data_ptr(), fy.data_ptr(), E.data_ptr(), ops.stream_ptr(dev)) == 0
    gx, gy, gE = ops.forces(xt, yt, FP64)
    torch.cuda.synchronize()
    if n < 200000:
        assert torch.equal(fx, gx) and torch.equal(fy, gy) and torch.equal(E, gE)
    rows = np.sort(np.random.default_rng(1).choice(n, 64, replace=False)).astype(np.int32)
    ox, oy, _ = O.rows(x, y, rows)
    for ax, ay in ((fx, fy), (gx, gy)):
        assert rel_rms(ax.cpu().numpy()[rows], ay.cpu().numpy()[rows], ox, oy) <= 1e-11
    assert abs(E.item() - gE.item()) <= 1e-13 * gE.item()
