"""GPU check of PCG where its single-workgroup kernels change from vectors held in registers to vectors reread,
and to several workgroups."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2510_07929_amd import kqr

pytestmark = pytest.mark.gpu


def say(*a):
    print("[gpu-test]", *a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("n", [2, 63, 1024, 1025, 4096, 4097, 16384, 16385])
def test_pcg_with_a_rank_two_kernel(n):
    """Two distinct points make K a rank-two matrix: the system has a closed solution by Woodbury in FP64, and
    PCG with a factor of K as preconditioner reaches its residual target."""
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(n)
    side = rng.integers(0, 2, n)
    side[:2] = (0, 1)
    X = np.where(side[:, None] == 0, 0.0, 1.0).astype(np.float32) * np.ones((1, 2), dtype=np.float32)
    gamma, c = 0.5, 0.7
    k01 = float(np.float32(np.exp(-gamma * 2.0)))
    L = rng.uniform(0.5, 2.0, n)
    b = rng.standard_normal(n)
    U = np.zeros((n, 2))
    U[np.arange(n), side] = 1.0
    M = np.array([[1.0, k01], [k01, 1.0]]) + c  # K + c 1 1^T = U M U^T
    core = np.linalg.inv(M) + (U / L[:, None]).T @ U
    ref = b / L - (U @ np.linalg.solve(core, U.T @ (b / L))) / L
    low = np.linalg.cholesky(np.array([[1.0, k01], [k01, 1.0]]))
    F = np.zeros((n, 4), dtype=np.float32)
    F[:, :2] = U @ low
    say("pcg", n)
    Xt = torch.from_numpy(X).to(dev)
    K = kqr.kqr_kernel_build(Xt, "rbf", gamma)
    tol = 1e-7 * np.linalg.norm(b)
    x, it, res = kqr.kqr_pcg_solve(Xt, "rbf", gamma, c, torch.from_numpy(L).to(dev), torch.from_numpy(b).to(dev), tol,
                                   50, K=K, F=torch.from_numpy(F).to(dev), r=2)
    assert res <= tol and 1 <= it < 50
    # the operator rounds p to FP32 in each step, and K_01 of X is within two FP32 roundings of k01; the smallest
    # eigenvalue of the system is at least min(L) = 0.5
    err = np.linalg.norm(x.cpu().numpy() - ref)
    slack = 8 * 2.0 ** -24 * n * np.linalg.norm(ref)
    assert err <= (tol + slack) / 0.5
