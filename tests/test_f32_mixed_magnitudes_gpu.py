"""FP32 products of the split kernels (three BF16 pieces per operand) on rows and
columns of mixed magnitude: values below 2^-110, from which the pieces take bits,
beside ones of order 1, where the large ones meet zeros or cancel, so that the
output shows every bit of the small ones.

Bound per element, against FP64: (K + 2) 2^-24 sum_k |a_ik b_kj|, what K rounded
products and sums in FP32 may lose, plus K 2^-149 for subnormal sums."""
import math

import pytest

import synth

pytestmark = pytest.mark.gpu

SPLIT = [(64, 64, 8, 16), (64, 128, 8, 16), (128, 64, 8, 32), (128, 128, 8, 16), (128, 128, 8, 32)]


def _rows(torch, r, c):
    return torch.zeros((r, (c + 15) // 16 * 16), device="cuda")[:, :c]


def _check(h, torch, a, b, ta, tb):
    """a (M, K) and b (K, N) through every split configuration."""
    (M, K), N = a.shape, b.shape[1]
    A, B = _rows(torch, *((K, M) if ta else (M, K))), _rows(torch, *((N, K) if tb else (K, N)))
    A.copy_(a.t() if ta else a)
    B.copy_(b.t() if tb else b)
    ref = a.double() @ b.double()
    bound = (K + 2) * 2.0 ** -24 * (a.double().abs() @ b.double().abs()) + K * 2.0 ** -149
    h.set_full_rows(True)
    try:
        for cfg in SPLIT:
            C = torch.full((M, N), 7.0, device="cuda")
            h.gemm(A, B, C, ta, tb, config_id=h.configs().index(cfg))
            torch.cuda.synchronize()
            err = (C.double() - ref).abs()
            assert bool((err <= bound).all()), (cfg, float((err / bound.clamp(min=1e-300)).max()))
    finally:
        h.set_full_rows(False)


@pytest.mark.parametrize("ta,tb", synth.LAYOUTS)
@pytest.mark.parametrize("e", [109, 112, 118, 126, 134, 140, 147])
@pytest.mark.parametrize("side", ["a", "b"])
def test_small_values_beside_large_ones_that_meet_zero(gpu, ta, tb, e, side):
    h, torch = gpu
    g = torch.Generator(device="cuda").manual_seed(e)
    M, N, K = 130, 133, 48
    a = torch.randn(M, K, generator=g, device="cuda")
    b = torch.randn(K, N, generator=g, device="cuda")
    # the first half of K: values of order 1 that meet zeros, or (columns from
    # 100 on) that cancel in pairs; the second half: small values against large ones
    a[:, 1:24:2] = a[:, 0:24:2]
    b[:24] = 0
    b[0:24:2, 100:] = 1.0
    b[1:24:2, 100:] = -1.0
    a[:, 24:] *= 2.0 ** -100
    a[:, 24:] *= 2.0 ** (100 - e)
    b[24:] *= 2.0 ** min(e - 10, 120)
    if side == "b":
        a, b = b.t().contiguous(), a.t().contiguous()
    _check(h, torch, a, b, ta, tb)


@pytest.mark.parametrize("ta,tb", synth.LAYOUTS)
@pytest.mark.parametrize("K", [16, 33, 200])
def test_one_small_value(gpu, ta, tb, K):
    """Single values of 2^-121 in every 32 rows and columns, first, last and
    inside K; everything else of their rows meets zero."""
    h, torch = gpu
    g = torch.Generator(device="cuda").manual_seed(K)
    M, N = 128, 160
    a = torch.randn(M, K, generator=g, device="cuda")
    b = torch.randn(K, N, generator=g, device="cuda")
    for n, (i, k) in enumerate([(0, 0), (33, K - 1), (95, K // 2), (127, 1)]):
        j = [5, 37, 159, 64][n]
        a[i, k] = 1.2345678 * 2.0 ** -121
        b[:, j] = 0
        b[k, j] = 1.3 * 2.0 ** 60
    for n, (k, j) in enumerate([(0, 31), (K - 1, 100), (K // 3, 130)]):
        i = [70, 20, 100][n]
        b[k, j] = 1.7654321 * 2.0 ** -123
        a[i] = 0
        a[i, k] = 1.1 * 2.0 ** 60
    _check(h, torch, a, b, ta, tb)


def test_small_probabilities(gpu):
    """Rows of a softmax whose smallest values fall below 2^-110, against values
    of order 1."""
    h, torch = gpu
    g = torch.Generator(device="cuda").manual_seed(1)
    a = torch.softmax(20 * torch.randn(200, 160, generator=g, device="cuda"), dim=1)
    assert bool(((a > 0) & (a < 2.0 ** -110)).any())
    _check(h, torch, a, torch.randn(160, 150, generator=g, device="cuda"), 0, 0)
