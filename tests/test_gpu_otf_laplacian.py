"""On-the-fly Laplacian apply for every count of coordinates per pair it is built for, at the edges of its tiles."""
import ctypes

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


class _PoolProps(ctypes.Structure):
    _fields_ = [("alloc_type", ctypes.c_int), ("handle_types", ctypes.c_int), ("location_type", ctypes.c_int),
                ("location_id", ctypes.c_int), ("security", ctypes.c_void_p), ("max_size", ctypes.c_size_t),
                ("reserved", ctypes.c_ubyte * 56)]


@pytest.fixture
def small_pool():
    """The device's stream-ordered memory limited to 64 MiB: yields a function that reads the bytes in use."""
    torch.zeros(1, device="cuda")
    hip = ctypes.CDLL("libamdhip64.so.7")
    props = _PoolProps(1, 0, 1, 0, None, 64 << 20)  # pinned device memory of device 0, no export
    old, pool = ctypes.c_void_p(), ctypes.c_void_p()
    assert hip.hipDeviceGetMemPool(ctypes.byref(old), 0) == 0
    assert hip.hipMemPoolCreate(ctypes.byref(pool), ctypes.byref(props)) == 0
    assert hip.hipDeviceSetMemPool(0, pool) == 0

    def used():
        torch.cuda.synchronize()
        out = ctypes.c_uint64(0)
        assert hip.hipMemPoolGetAttribute(pool, 7, ctypes.byref(out)) == 0  # bytes in use
        return out.value

    yield used
    torch.cuda.synchronize()
    assert hip.hipDeviceSetMemPool(0, old) == 0
    assert hip.hipMemPoolDestroy(pool) == 0


def _check_wide_ranges(X, v, gamma):
    n, p = X.shape
    u = kqr.kqr_kernel_apply(v, X=X, kernel="laplacian", gamma=gamma, mode=kqr.KQR_APPLY_EXACT)
    rows = torch.arange(0, n, 977, device="cuda")
    x = X.double()
    arg = gamma * sum((x[rows, k, None] - x[None, :, k]).abs() for k in range(p))
    # FP32 roundings of the differences and their sum, its scale and the exponential
    bound = torch.exp(-arg) * (p + 4) * EPS * (1 + arg)
    ref = torch.exp(-arg) @ v
    assert bool(((u[rows] - ref).abs() <= bound @ v.abs() + 1e-12 * (1 + ref.abs())).all())


def _wide_points(n, p):
    g = torch.Generator(device="cuda").manual_seed(n)
    X = 2000.0 * (2.0 * torch.rand(n, p, device="cuda", generator=g) - 1.0)  # p times the range is past 4096
    return X, torch.randn(n, device="cuda", dtype=torch.float64, generator=g)


@pytest.mark.parametrize("n", [1, 300, 60000])
def test_laplacian_square_of_wide_ranges(n):
    """Points whose ranges do not allow fixed point: the float form, with the sums of the other form in hand
    (n = 300) and given back (n = 60,000)."""
    X, v = _wide_points(n, 3)
    _check_wide_ranges(X, v, 1e-3)


def test_laplacian_square_where_memory_is_short(small_pool):
    """n = 60,000: the fixed-point form's partial sums (over 112 MB) do not fit the pool.  Points whose ranges do not
    allow fixed point need 17 MB and get their product; others fail for lack of memory, and give back what they held."""
    X, v = _wide_points(60000, 3)
    _check_wide_ranges(X, v, 1e-3)
    assert small_pool() == 0
    with pytest.raises(kqr.KqrError) as e:
        kqr.kqr_kernel_apply(v, X=1e-3 * X, kernel="laplacian", gamma=1.0)
    assert e.value.status == kqr.KQR_ENOMEM
    assert small_pool() == 0
