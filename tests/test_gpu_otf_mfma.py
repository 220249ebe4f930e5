"""On-the-fly RBF operators on the matrix cores (p <= 32) at the edges of their
tiles (16 columns), stages (64), tile-rows (128) and coordinate paddings."""
import numpy as np
import pytest
import torch

from paper_2510_07929_amd import kqr

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24
GAMMA = 0.05


def _entries(Xr, Xc):
    """FP64 entries and the FP32 kernels' bound on each one's error: the
    distance from norms and products of p terms, each rounded to FP32 (twice
    for the split operands), the argument's own rounding and the exponential."""
    Xr, Xc = Xr.double().cpu().numpy(), Xc.double().cpu().numpy()
    p = Xr.shape[1]
    q = (Xr ** 2).sum(1)[:, None] + (Xc ** 2).sum(1)[None, :]
    arg = GAMMA * ((Xr[:, None, :] - Xc[None, :, :]) ** 2).sum(2)
    K = np.exp(-arg)
    return K, K * (GAMMA * 2 * (p + 6) * EPS * 2 * q + 4 * EPS * (1 + arg))


@pytest.mark.parametrize("p", [1, 8, 9, 12, 16, 17, 30, 31, 32])
@pytest.mark.parametrize("m,n", [(1, 1), (33, 64), (127, 65), (129, 1), (128, 129), (31, 1025), (300, 700)])
def test_rectangular(m, n, p):
    g = torch.Generator(device="cuda").manual_seed(7 * p + n)
    X = torch.randn(n, p, device="cuda", generator=g)
    Z = torch.randn(m, p, device="cuda", generator=g)
    a = torch.randn(n, device="cuda", dtype=torch.float64, generator=g)
    f = kqr.kqr_predict(X, a, 0.25, 0.5, "rbf", GAMMA, Z).cpu().numpy()
    K, bound = _entries(Z, X)
    an = a.cpu().numpy()
    ref = 0.25 + 2.0 * (K @ an)
    tol = 2.0 * (bound @ np.abs(an)) + 1e-12 * (1 + np.abs(ref))
    assert (np.abs(f - ref) <= tol).all()


@pytest.mark.parametrize("mode", ["exact", "fast"])
@pytest.mark.parametrize("p", [3, 10, 16, 17, 30, 32])
@pytest.mark.parametrize("n", [1, 15, 64, 65, 128, 129, 193, 400])
def test_square(n, p, mode):
    g = torch.Generator(device="cuda").manual_seed(11 * p + n)
    X = torch.randn(n, p, device="cuda", generator=g)
    v = torch.randn(n, device="cuda", dtype=torch.float64, generator=g)
    m = kqr.KQR_APPLY_EXACT if mode == "exact" else kqr.KQR_APPLY_FAST
    u = kqr.kqr_kernel_apply(v, X=X, kernel="rbf", gamma=GAMMA, mode=m).cpu().numpy()
    K, bound = _entries(X, X)
    vn = np.abs(v.cpu().numpy())
    ref = K @ v.cpu().numpy()
    # fast: v rounded to FP32, products and sums of up to 128 terms in FP32
    tol = (bound + (131 * EPS * K if mode == "fast" else 0.0)) @ vn + 1e-12 * (1 + np.abs(ref))
    assert (np.abs(u - ref) <= tol).all()
