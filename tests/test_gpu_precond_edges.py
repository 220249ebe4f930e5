"""GPU checks of the preconditioner kernels at the sizes where their tiles end."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2510_07929_amd import inputs, kqr

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


def _rpc_inputs(dev, X, gamma, form):
    """(kernel, K): entries from X, or a stored K."""
    Xt = torch.from_numpy(X).to(dev)
    if form in ("rbf", "laplacian"):
        return Xt, form, None
    return Xt, "rbf", kqr.kqr_kernel_build(Xt, "rbf", gamma, form)


@pytest.mark.parametrize("form", ["rbf", "laplacian", "fp32", "bf16"])
@pytest.mark.parametrize("n,rank", [(7, 7), (300, 12), (70001, 9)])
def test_rpcholesky_stops_at_the_rank_of_k(dev, n, rank, form):
    """Seven places whose kernel values underflow between them: K is a 0-1 block matrix, every step is exact, and
    the residual is zero after seven pivots, one per place; the columns from there on are zero."""
    places = np.zeros((7, 3), dtype=np.float32)
    for k in range(3):
        places[2 * k + 1, k], places[2 * k + 2, k] = 16.0, -16.0
    rng = np.random.default_rng((n, rank))
    at = rng.permutation(np.arange(n) % 7)
    gamma = 16.0  # exp(-16 * 16) and below: zero in FP32
    say("rpcholesky rank", n, rank, form)
    Xt, kernel, K = _rpc_inputs(dev, places[at], gamma, form)
    F, piv, r = kqr.kqr_rpcholesky(rank, rng.uniform(0.0, 1.0, rank), X=Xt, kernel=kernel, gamma=gamma, K=K)
    assert r == 7 and sorted(at[piv].tolist()) == list(range(7))
    want = np.zeros((n, F.shape[1]), dtype=np.float32)
    want[:, :7] = at[:, None] == at[piv][None, :]
    assert np.array_equal(F.cpu().numpy(), want)


@pytest.mark.parametrize("form", ["laplacian", "bf16"])
@pytest.mark.parametrize("n,rank", [(257, 70), (2049, 45)])
def test_rpcholesky_columns_of_other_kernels(dev, n, rank, form):
    """The columns at the pivots drawn, against the steps in FP64 on the host on the same entries."""
    rng = np.random.default_rng((n, rank, 1))
    X = rng.uniform(-1.0, 1.0, (n, 3)).astype(np.float32)
    gamma = 2.0
    say("rpcholesky columns", n, rank, form)
    Xt, kernel, K = _rpc_inputs(dev, X, gamma, form)
    F, piv, r = kqr.kqr_rpcholesky(rank, rng.uniform(0.0, 1.0, rank), X=Xt, kernel=kernel, gamma=gamma, K=K)
    F = F.cpu().numpy().astype(np.float64)
    assert r == rank and len(set(piv.tolist())) == rank
    x = X.astype(np.float64)
    for i, s in enumerate(piv):
        if K is None:
            col = np.exp(-gamma * np.abs(x - x[s]).sum(1))
        else:
            col = K[s, :n].double().cpu().numpy()
        g = col - F[:, :i] @ F[s, :i]
        # FP32 roundings of an entry from X and of F's column, magnified by 1 / sqrt(g_s) as g_s carries them too
        tol = 64 * (i + 1) * 2.0 ** -24 / g[s]
        assert np.max(np.abs(F[:, i] - g / np.sqrt(g[s]))) <= tol, i


@pytest.mark.parametrize("kd", ["fp32", "bf16"])
def test_preconditioner_from_a_packed_k(dev, kd):
    """A fit on the packed layout draws its pivots from the tiles: the same entries as the full layout's, so the rank
    rule keeps the same columns, and Phase I needs about as many iterations."""
    prob = inputs.workload("c0", n=1500)
    X, y = torch.from_numpy(prob.X).to(dev), torch.from_numpy(prob.y).to(dev)
    got = []
    for layout in (0, 1):
        say("packed preconditioner", kd, layout)
        _, _, info, st = kqr.kqr_fit(X, y, prob.tau, prob.lam, prob.kernel, prob.gamma, k_layout=layout,
                                     k_dtype=kqr.KDTYPES[kd], xi=1e-4, uniforms=inputs.pivot_uniforms(64, (1500, 1)))
        assert st == kqr.KQR_OK
        got.append((info["rank_used"], info["admm_pcg_iters"]))
    (r0, it0), (r1, it1) = got
    assert r0 == r1 == 39  # ceil(sqrt n): the rule keeps them all
    assert abs(it0 - it1) <= 0.2 * it0
