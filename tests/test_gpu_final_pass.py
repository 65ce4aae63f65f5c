"""The relax's final pass with the state and the energy change at once against
calls that ask for one of them, at patch sizes around its 64-active blocks.
Both sum the same terms in the same order; tolerances are a few ulps of the
energies and of the sum of the terms' magnitudes (within 1e3 of the change)."""
import numpy as np
import pytest
import torch

from paper_2609_24722_amd import FP64, ops, relax as R, workloads as W

pytestmark = pytest.mark.gpu
X_OUT, DE = (9, 10, 12, 13, 14, 15), (11,)  # positions in relax_subdomains' arguments


class Without:
    """The library with some output pointers of relax_subdomains left null."""

    def __init__(self, lib, drop):
        self._lib, self._drop = lib, drop

    def __getattr__(self, k):
        return getattr(self._lib, k)

    def relax_subdomains(self, *a):
        return self._lib.relax_subdomains(*(None if q in self._drop else v for q, v in enumerate(a)))


@pytest.mark.parametrize("n", [300, 5000])
def test_both_as_alone(dev, n, monkeypatch):
    print(f"[case] n={n}", flush=True)
    x, y = W.warped_lattice(n, 0.02, 97)
    h = W.spacing(n)
    xt, yt = torch.tensor(x, device=dev), torch.tensor(y, device=dev)
    sizes = np.array([1, 63, 64, 65, 130], dtype=np.int32)
    ptr, idx = R.build_patches(xt, yt, np.random.default_rng(7).choice(n, sizes.size, replace=False).astype(np.int32), sizes)
    ia = idx.cpu().numpy()
    kx, ky = W.kicks(ia.size, 0.05 * h, 98)
    sx, sy = torch.tensor(x[ia] + kx, device=dev), torch.tensor(y[ia] + ky, device=dev)

    def relax():
        r = R.relax_subdomains(xt, yt, ptr, idx, sx, sy, precision=FP64, max_iter=0)
        torch.cuda.synchronize()
        return r

    both, lib = relax(), ops.lib()
    monkeypatch.setattr(ops, "lib", lambda: Without(lib, DE))
    state = relax()
    monkeypatch.setattr(ops, "lib", lambda: Without(lib, X_OUT))
    change = relax()
    assert torch.equal(both.x, state.x) and torch.equal(both.y, state.y)
    assert torch.allclose(both.e_sub, state.e_sub, rtol=1e-14, atol=0)
    assert torch.allclose(both.gtan_inf, state.gtan_inf, rtol=1e-12, atol=1e-14 * both.e_sub.max().item())
    assert torch.allclose(both.dE, change.dE, rtol=1e-12, atol=1e-15 * both.e_sub.max().item())
