"""The second pass of the split kernels, through the same stages as the first:
products deep enough (32 stages) that the first stage is looked through, and
shallower ones, with infinities, NaN and values that overflow in the first stage,
in the middle and at the end of K, on padded rows and on dense rows of odd length
(whose last chunk is moved to its place in both passes), for work-groups of one,
two and four waves.

Every output has the kind (finite, +inf, -inf, NaN) that the FP32 MFMA kernel
gives it; finite ones lie within 1e-5 sqrt(K) max|a_i| max|b_j| of FP64, the bound
of the plain GEMM tests per row and column."""
import math

import pytest

import synth

pytestmark = pytest.mark.gpu

SPLIT = [(64, 64, 8, 16), (64, 128, 8, 16), (128, 64, 8, 32), (128, 128, 8, 16), (128, 128, 8, 32)]
PLAIN = (64, 64, 4, 32)


@pytest.mark.parametrize("ta,tb", synth.LAYOUTS)
@pytest.mark.parametrize("K", [99, 1021, 1056])
@pytest.mark.parametrize("where", ["first", "middle", "last", "nowhere"])
@pytest.mark.parametrize("padded", [True, False])
def test_second_pass(gpu, ta, tb, K, where, padded):
    h, torch = gpu
    g = torch.Generator(device="cuda").manual_seed(K)
    M, N = 201, 151
    a = torch.randn(M, K, generator=g, device="cuda")
    b = torch.randn(K, N, generator=g, device="cuda")
    if where != "nowhere":
        k = {"first": 3, "middle": K // 2, "last": K - 1}[where]
        a[3, k], a[70, k], a[140, k], a[200, k] = math.inf, math.nan, 3.4e38, 2.0 ** 70
        b[k, 150] = -math.inf
        b[k, 20] = 2.0 ** 61
        b[max(k - 1, 0), 100] = 2.0 ** 63

    def rows(x):
        buf = torch.zeros(x.shape[0], (x.shape[1] + 15) // 16 * 16 if padded else x.shape[1], device="cuda")
        buf[:, :x.shape[1]] = x
        return buf[:, :x.shape[1]]

    A, B = rows(a.t() if ta else a), rows(b.t() if tb else b)
    h.set_full_rows(padded)
    try:
        out = {}
        for cfg in SPLIT + [PLAIN]:
            out[cfg] = torch.full((M, N), 7.0, device="cuda")
            h.gemm(A, B, out[cfg], ta, tb, config_id=h.configs().index(cfg))
        torch.cuda.synchronize()
    finally:
        h.set_full_rows(False)
    ref = out[PLAIN]
    exact = a.double() @ b.double()
    z = lambda t: torch.where(torch.isfinite(t), t, torch.zeros_like(t)).abs().double()   # noqa: E731
    tol = 1e-5 * math.sqrt(K) * z(a).amax(1)[:, None] * z(b).amax(0)[None, :]
    for cfg in SPLIT:
        C = out[cfg]
        assert torch.equal(C.isnan(), ref.isnan()), cfg
        assert torch.equal(C.isposinf(), ref.isposinf()) and torch.equal(C.isneginf(), ref.isneginf()), cfg
        f = C.isfinite() & exact.isfinite()
        assert int(f.sum()) > 0.9 * M * N
        assert bool(((C.double() - exact).abs() <= tol)[f].all()), cfg
