"""The certificate at sizes around its dot products' chunks and the FP64 pair
passes' line, against the same Lanczos steps in numpy with the oracle's
Hessian-vector product."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2609_24722_amd import ops, workloads as W

pytestmark = pytest.mark.gpu


def start_vector(n, seed):
    with np.errstate(over="ignore"):
        z = np.uint64(seed) ^ np.arange(2 * n, dtype=np.uint64)
        z = z + np.uint64(0x9e3779b97f4a7c15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xbf58476d1ce4e5b9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94d049bb133111eb)
        z = z ^ (z >> np.uint64(31))
    u = (z >> np.uint64(11)).astype(np.float64) * 2.0 ** -52 - 1.0
    return u[0::2], u[1::2]


def reference(x, y, k, mask, deflate, seed):
    n = x.size
    fx, fy = O.forces(x, y)
    r = np.hypot(x, y)
    ux, uy = x / r, y / r
    fr = fx * ux + fy * uy
    held = mask & (r >= 1.0 - 1e-14) & (fr > 0)
    w0 = np.where(held, fr, 0.0)

    def proj(vx, vy):
        vr = np.where(held, vx * ux + vy * uy, 0.0)
        return np.concatenate([np.where(mask, vx - vr * ux, 0.0), np.where(mask, vy - vr * uy, 0.0)])

    def apply(v):
        hx, hy = O.hvp(x, y, np.ascontiguousarray(v[:n]), np.ascontiguousarray(v[n:]))
        return proj(hx, hy) + np.concatenate([w0 * v[:n], w0 * v[n:]])

    B = []
    if deflate:
        q = np.concatenate([np.where(mask, -y, 0.0), np.where(mask, x, 0.0)])
        B.append(q / np.linalg.norm(q))
    v = proj(*start_vector(n, seed))
    for b in B:
        v = v - (b @ v) * b
    B.append(v / np.linalg.norm(v))
    al, be = [], []
    for j in range(k):
        w = apply(B[-1])
        A = np.array(B)
        a = 0.0
        for _ in range(2):
            c = A @ w
            a += c[-1]
            w = w - c @ A
        al.append(a)
        be.append(np.linalg.norm(w))
        B.append(w / be[-1])
    ev, ec = np.linalg.eigh(np.diag(al) + np.diag(be[:-1], 1) + np.diag(be[:-1], -1))
    u = ec[:, 0] @ np.array(B[-k - 1:-1])
    return ev[0], ev[-1], np.linalg.norm(apply(u) - ev[0] * u)


@pytest.mark.parametrize("n,deflate,masked", [(64, True, False), (65, False, True), (4096, True, False), (4097, True, True),
                                              (7001, True, False)])
def test_ritz_values_against_numpy(dev, n, deflate, masked):
    print(f"[case] n={n} deflate={deflate} masked={masked}", flush=True)
    x, y = W.warped_lattice(n, 0.02, 61)
    edge = np.hypot(x, y) > 1.0 - 0.8 * W.spacing(n)  # the outer ring onto the wall, where it is held
    r = np.hypot(x, y)
    x, y = np.where(edge, x / r, x), np.where(edge, y / r, y)
    mask = np.arange(n) % 3 != 0 if masked else np.ones(n, dtype=bool)
    k = 12
    m = torch.tensor(mask.astype(np.int32), device=dev) if masked else None
    got = ops.tangent_lanczos(torch.tensor(x, device=dev), torch.tensor(y, device=dev), k=k, mask=m,
                              deflate_rotation=deflate, seed=99)
    tmin, tmax, resid = reference(x, y, k, mask, deflate, 99)
    print(f"[err] n={n} {abs(got['theta_min'] - tmin) / tmax:.1e} {abs(got['theta_max'] - tmax) / tmax:.1e} "
          f"{abs(got['resid'] - resid) / tmax:.1e}")
    # the steps are the same up to rounding, 1e-16 of the largest eigenvalue each, grown over 12 of them
    assert got["steps"] == k
    assert abs(got["theta_min"] - tmin) <= 1e-11 * tmax
    assert abs(got["theta_max"] - tmax) <= 1e-11 * tmax
    assert abs(got["resid"] - resid) <= 1e-9 * tmax
