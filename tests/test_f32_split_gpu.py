"""FP32 products on the BF16 matrix cores (three BF16 pieces per operand):
exactness against FP64 beside the FP32 MFMA kernels, and the operands that do
not split -- infinities, NaN, values that round to infinity in BF16, rows
below BF16's range -- which must come out as FP32 arithmetic gives them."""
import math

import pytest

import synth

pytestmark = pytest.mark.gpu

SPLIT = [(64, 64, 8, 16), (128, 128, 8, 32), (64, 128, 8, 64)]
PLAIN = (64, 64, 4, 32)


def _rows(torch, r, c, g):
    """Values (r, c) in rows padded to 16 elements."""
    buf = torch.zeros((r, (c + 15) // 16 * 16), device="cuda")
    v = buf[:, :c]
    v.copy_(torch.randn(r, c, generator=g, device="cuda"))
    return v


def _run(h, torch, A, B, ta, tb, cfg):
    M, N = A.shape[1] if ta else A.shape[0], B.shape[0] if tb else B.shape[1]
    C = torch.full((M, N), 7.0, device="cuda")
    h.set_full_rows(True)
    try:
        h.gemm(A, B, C, ta, tb, config_id=h.configs().index(cfg))
        torch.cuda.synchronize()
    finally:
        h.set_full_rows(False)
    return C


def _ref(A, B, ta, tb):
    a, b = A.double(), B.double()
    return (a.t().contiguous() if ta else a.contiguous()) @ (b.t().contiguous() if tb else b.contiguous())


@pytest.mark.parametrize("ta,tb", synth.LAYOUTS)
@pytest.mark.parametrize("K", [15, 16, 17, 48, 65, 200, 1000])
def test_no_further_from_fp64_than_fp32_mfma(gpu, kt, ta, tb, K):
    h, torch = gpu
    g = torch.Generator(device="cuda").manual_seed(K)
    M, N = 330, 205
    A = _rows(torch, K if ta else M, M if ta else K, g)
    B = _rows(torch, N if tb else K, K if tb else N, g)
    ref = _ref(A, B, ta, tb)
    rel = lambda C: float((C.double() - ref).norm() / ref.norm())   # noqa: E731
    plain = rel(_run(h, torch, A, B, ta, tb, PLAIN))
    for cfg in SPLIT:
        C = _run(h, torch, A, B, ta, tb, cfg)
        # 67650 sums: a few percent for the sample, K = 15 runs the same MFMAs
        assert rel(C) <= 1.03 * plain, (cfg, rel(C), plain)
        tol = 1e-5 * math.sqrt(K) * float(A.abs().max()) * float(B.abs().max())
        assert float((C.double() - ref).abs().max()) <= tol


@pytest.mark.parametrize("ta,tb", synth.LAYOUTS)
@pytest.mark.parametrize("cfg", SPLIT)
def test_values_that_do_not_split(gpu, kt, ta, tb, cfg):
    """Infinities, NaN and the largest finite floats in single elements: each
    output is non-finite exactly where the FP32 MFMA kernel's is, the same
    kind, and within the bound elsewhere."""
    h, torch = gpu
    g = torch.Generator(device="cuda").manual_seed(3)
    M, N, K = 150, 200, 130
    A = _rows(torch, K if ta else M, M if ta else K, g)
    B = _rows(torch, N if tb else K, K if tb else N, g)
    at = (lambda m, k: (k, m)) if ta else (lambda m, k: (m, k))
    bt = (lambda k, n: (n, k)) if tb else (lambda k, n: (k, n))
    A[at(3, 7)] = math.inf
    A[at(70, 129)] = -math.inf
    A[at(149, 0)] = math.nan
    B[bt(5, 199)] = math.inf
    B[bt(9, 80)] = math.nan
    A[at(20, 4)] = 3.4e38            # rounds to infinity in BF16
    B[bt(4, 10)] = 0.25
    B[bt(100, 33)] = 0.0
    plain, got = _run(h, torch, A, B, ta, tb, PLAIN), _run(h, torch, A, B, ta, tb, cfg)
    fin = torch.isfinite(plain)
    assert torch.equal(fin, torch.isfinite(got))
    assert torch.equal(torch.isnan(plain), torch.isnan(got))
    inf = torch.isinf(plain)
    assert torch.equal(plain[inf], got[inf])
    assert int(fin.sum()) > 0.9 * M * N
    # rows and columns bounded by their own largest finite operand
    z = lambda t: torch.where(torch.isfinite(t), t, torch.zeros_like(t)).abs()   # noqa: E731
    am = z(A).amax(0 if ta else 1)[:, None].double()
    bm = z(B).amax(1 if tb else 0)[None, :].double()
    tol = 1e-5 * math.sqrt(K) * am * bm
    assert bool(((plain.double() - got.double()).abs() <= 2 * tol)[fin].all())


@pytest.mark.parametrize("ta,tb", synth.LAYOUTS)
@pytest.mark.parametrize("ea,eb", [(-120, 100), (100, -126), (-60, -40), (-90, 60)])
def test_small_and_large_magnitudes(gpu, kt, ta, tb, ea, eb):
    """Operands scaled by powers of two, one of them below the range in which
    BF16 pieces keep their bits: the relative error stays the unscaled one."""
    h, torch = gpu
    g = torch.Generator(device="cuda").manual_seed(8)
    M, N, K = 100, 130, 96
    A = _rows(torch, K if ta else M, M if ta else K, g)
    B = _rows(torch, N if tb else K, K if tb else N, g)
    A.mul_(2.0 ** ea)
    B.mul_(2.0 ** (eb / 2)).mul_(2.0 ** (eb - eb / 2))
    A[(slice(None), 4) if ta else (4, slice(None))] = 0      # a zero row is no small row
    ref = _ref(A, B, ta, tb)
    rel = lambda C: float((C.double() - ref).norm() / ref.norm())   # noqa: E731
    plain = rel(_run(h, torch, A, B, ta, tb, PLAIN))
    for cfg in SPLIT:
        assert rel(_run(h, torch, A, B, ta, tb, cfg)) <= 1.05 * plain
