"""GPU checks of the materialised K-apply of one column at the sizes where its rows per wave change."""
import sys

import pytest

torch = pytest.importorskip("torch")

from paper_2510_07929_amd import kqr

pytestmark = pytest.mark.gpu


def say(*a):
    print("[gpu-test]", *a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("kd", ["fp32", "bf16"])
@pytest.mark.parametrize("n", [1, 9, 513, 6250, 6251, 8192, 8193, 12500, 12501, 16383, 16384])
def test_apply_of_one_column_at_rule_edges(n, kd):
    """K v of the stored entries against an FP64 product: fast rounds v and sums up to 16 products in FP32
    between FP64 additions, exact works in FP64; a vector off 16-byte alignment takes the copying path and
    gives the same bits."""
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(n)
    X = torch.randn((n, 4), generator=g, device=dev)
    K = kqr.kqr_kernel_build(X, "rbf", 0.5, kd)
    w = torch.randn(n + 1, generator=g, device=dev, dtype=torch.float64)
    v = w[:n].clone()
    say("apply rows", kd, n)
    ref = torch.zeros(n, device=dev, dtype=torch.float64)
    scale = torch.zeros(n, device=dev, dtype=torch.float64)
    for i in range(0, n, 2048):
        k = K[i:i + 2048, :n].double()
        ref[i:i + 2048] = k @ v
        scale[i:i + 2048] = k @ v.abs()
    for mode, rel in ((kqr.KQR_APPLY_FAST, 18 * 2.0 ** -24), (kqr.KQR_APPLY_EXACT, 2 * n * 2.0 ** -53)):
        u = kqr.kqr_kernel_apply(v, K=K, mode=mode)
        assert bool(((u - ref).abs() <= rel * scale).all()), (mode, float(((u - ref).abs() / scale).max()))
        w[1:] = v
        assert w[1:].data_ptr() % 16 == 8
        assert torch.equal(kqr.kqr_kernel_apply(w[1:], K=K, mode=mode), u)


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("mode", [kqr.KQR_APPLY_FAST, kqr.KQR_APPLY_EXACT])
@pytest.mark.parametrize("kd", ["fp32", "bf16"])
@pytest.mark.parametrize("n", [1, 130, 6251, 12501, 16384])
def test_apply_of_one_column_into_its_own_vector(n, kd, mode, static):
    """K v written over v, over part of v from either side, and beside v: the bits of a call with its own output."""
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(n)
    X = torch.randn((n, 4), generator=g, device=dev)
    K = kqr.kqr_kernel_build(X, "rbf", 0.5, kd)
    v = torch.randn(n, generator=g, device=dev, dtype=torch.float64)

    def apply(x, out=None):
        if static:
            return kqr.kqr_kernel_apply_static(x, K, mode, u=out)
        return kqr.kqr_kernel_apply(x, K=K, mode=mode, U=out)

    want = apply(v)
    say("apply in place", kd, n, mode, static)
    at = 2 * n  # (even: v is 16-byte aligned)
    for off in (0, 1, -1, 64, -64, n - 1, 1 - n, n, -n):
        if abs(off) > n:
            continue
        w = torch.full((5 * n,), float("nan"), device=dev, dtype=torch.float64)
        w[at:at + n] = v
        u = apply(w[at:at + n], w[at + off:at + off + n])
        assert torch.equal(u, want), off
        if abs(off) == n:
            assert torch.equal(w[at:at + n], v)
