"""On-the-fly Laplacian apply for every count of coordinates per pair it is built for, at the edges of its tiles."""
import numpy as np
import pytest
import torch

from paper_2510_07929_amd import kqr

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24
GAMMA = 0.1


@pytest.mark.parametrize("mode", [kqr.KQR_APPLY_FAST, kqr.KQR_APPLY_EXACT])
@pytest.mark.parametrize("p", [1, 2, 4, 5, 8, 9, 11, 14, 17, 20, 21, 24, 26, 27, 30, 32, 33, 64])
@pytest.mark.parametrize("n", [1, 2, 33, 64, 127, 128, 129, 300])
def test_laplacian_square(n, p, mode):
    g = torch.Generator(device="cuda").manual_seed(13 * p + n)
    X = torch.randn(n, p, device="cuda", generator=g)
    v = torch.randn(n, device="cuda", dtype=torch.float64, generator=g)
    u = kqr.kqr_kernel_apply(v, X=X, kernel="laplacian", gamma=GAMMA, mode=mode).cpu().numpy()
    Xn, vn = X.double().cpu().numpy(), v.cpu().numpy()
    arg = GAMMA * np.abs(Xn[:, None, :] - Xn[None, :, :]).sum(2)
    K = np.exp(-arg)
    # both points' coordinates rounded to a grid of 2^-20 or finer, then the distance, its scale and the exponential
    bound = K * (GAMMA * p * 2.0 ** -20 + 4 * EPS * (1 + arg))
    if mode == kqr.KQR_APPLY_FAST:  # v rounded to FP32, products and sums of up to 128 terms in FP32
        bound = bound + 131 * EPS * K
    ref = K @ vn
    assert (np.abs(u - ref) <= bound @ np.abs(vn) + 1e-12 * (1 + np.abs(ref))).all()
