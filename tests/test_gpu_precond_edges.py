"""GPU checks of the preconditioner kernels at the sizes where their tiles end."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2510_07929_amd import kqr

pytestmark = pytest.mark.gpu


def say(*a):
    print("[gpu-test]", *a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    kqr.lib()
    return torch.device("cuda:0")


@pytest.mark.parametrize("n,r", [(1, 0), (7, 0), (3, 2), (31, 1), (33, 15), (64, 16), (65, 63), (500, 64), (1000, 127),
                                 (1025, 128), (4097, 200), (9000, 447), (20001, 500)])
def test_woodbury_core_at_tile_edges(dev, n, r):
    """P^{-1} w against a dense FP64 solve of the core, at ranks around the 64-entry tiles of its weighted
    Gram matrix and row counts around the groups of its chunks."""
    rng = np.random.default_rng((n, r))
    F = np.zeros((n, max(4, (r + 3) // 4 * 4)), dtype=np.float32)
    F[:, :r] = rng.standard_normal((n, r)) / np.sqrt(max(r, 1))
    F[:, r:] = np.nan  # padding columns are not part of the factor
    L = rng.uniform(0.5, 2.0, n)
    w = rng.standard_normal(n)
    c = 0.75
    say("woodbury", n, r)
    out = kqr.kqr_woodbury_apply(torch.from_numpy(F).to(dev), r, c, torch.from_numpy(L).to(dev),
                                 torch.from_numpy(w).to(dev)).cpu().numpy()
    U = np.concatenate([F[:, :r].astype(np.float64), np.ones((n, 1))], 1)
    core = np.diag(np.r_[np.ones(r), 1.0 / c]) + U.T @ (U / L[:, None])
    ref = (w - U @ np.linalg.solve(core, U.T @ (w / L))) / L
    # forward error of an SPD solve: (terms of a sum) x unit roundoff x condition of the core
    tol = (n + r + 1) * 2.0 ** -53 * np.linalg.cond(core)
    assert np.linalg.norm(out - ref) <= tol * np.linalg.norm(w / L)


@pytest.mark.parametrize("r", [2, 3, 16, 17, 32, 33, 64, 65, 97, 223, 224, 225])
def test_rank_rule_at_register_block_edges(dev, r):
    """lambda_1 and the rank of F0^T F0 against LAPACK's eigenvalues, at orders around the 16- and 32-entry
    blocks of the tridiagonalisation and where its matrix leaves the registers."""
    rng = np.random.default_rng(r)
    n = 2 * r + 5
    q, _ = np.linalg.qr(rng.standard_normal((n, r)))
    p, _ = np.linalg.qr(rng.standard_normal((r, r)))
    F = np.zeros((n, (r + 3) // 4 * 4), dtype=np.float32)
    F[:, :r] = q @ np.diag(10.0 ** -np.linspace(0.0, 4.0, r)) @ p  # eigenvalues 1 .. 1e-8
    say("rank rule", r)
    xi = 1e-5
    rank, top = kqr.kqr_adaptive_rank(torch.from_numpy(F).to(dev), r, xi)
    F64 = F[:, :r].astype(np.float64)
    ev = np.linalg.eigvalsh(F64.T @ F64)[::-1]
    # backward error of forming and reducing the matrix: n r units of its norm
    tol = n * r * 2.0 ** -53
    assert abs(top - ev[0]) <= tol * ev[0]
    below = np.nonzero(ev <= xi * ev[0])[0]
    want = int(below[0]) + 1 if below.size else r
    if rank != want:  # an eigenvalue within rounding of the threshold may count either way
        assert np.min(np.abs(ev - xi * ev[0])) <= tol * ev[0], (rank, want)


@pytest.mark.parametrize("diag", [(1.0, 1.0, 1.0, 1.0), (2.0, 0.0, 0.0, 0.0), (0.0, 0.0, 0.0, 0.0)])
def test_rank_rule_of_diagonal_gram_matrices(dev, diag):
    """Zero reflections throughout: equal eigenvalues, a single one, and the zero matrix."""
    F = np.zeros((6, 4), dtype=np.float32)
    F[:4, :4] = np.diag(diag)
    rank, top = kqr.kqr_adaptive_rank(torch.from_numpy(F).to(dev), 4, 1e-3)
    assert top == max(diag) ** 2
    assert rank == (2 if diag[1] == 0.0 and diag[0] > 0.0 else 4)


@pytest.mark.parametrize("n,rank,stored", [(2, 2, False), (3, 3, True), (65, 18, False), (255, 67, True),
                                           (256, 68, False), (257, 131, True), (65535, 21, False),
                                           (65537, 66, False), (131073, 5, False)])
def test_rpcholesky_steps_at_chunk_edges(dev, n, rank, stored):
    """Pivots, factor columns and the zero residual at the pivots, against the steps in FP64 on the host, at row
    counts around the 256 chunks of rows (one and several passes of 256 rows each) and ranks around the
    16-byte pieces of a pivot row."""
    rng = np.random.default_rng((n, rank))
    X = rng.uniform(-1.0, 1.0, (n, 3)).astype(np.float32)
    gamma = 2.0
    u = rng.uniform(0.0, 1.0, rank)
    say("rpcholesky", n, rank, stored)
    Xt = torch.from_numpy(X).to(dev)
    K = kqr.kqr_kernel_build(Xt, "rbf", gamma) if stored else None
    F, piv, r = kqr.kqr_rpcholesky(rank, u, X=Xt, kernel="rbf", gamma=gamma, K=K)
    F = F.cpu().numpy().astype(np.float64)
    assert r == rank and len(set(piv.tolist())) == rank
    x = X.astype(np.float64)
    G = np.zeros((n, rank))
    d = np.ones(n)
    for i, s in enumerate(piv):
        # the draw: the running sum passes u_i sum(d) at the pivot, up to the FP32 entries' rounding
        run, target = np.cumsum(d), u[i] * d.sum()
        slack = 1e-5 * d.sum()
        assert run[s] > target - slack and run[s] - d[s] <= target + slack, (i, s)
        g = np.exp(-gamma * ((x - x[s]) ** 2).sum(1)) - G[:, :i] @ G[s, :i]
        G[:, i] = g / np.sqrt(g[s])
        # an entry carries FP32 roundings of K and F (a few 2^-24), magnified by 1 / sqrt(g_s) and the earlier columns
        tol = 64 * (i + 1) * 2.0 ** -24 / g[s]
        assert np.max(np.abs(F[:, i] - G[:, i])) <= tol, (i, np.max(np.abs(F[:, i] - G[:, i])), tol)
        G[:, i] = F[:, i]
        d = np.maximum(d - G[:, i] ** 2, 0.0)
        d[s] = 0.0
