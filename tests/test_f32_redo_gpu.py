"""FP32 products of the split kernels on data that has left the finite range, or
is about to: every output has the kind (finite, +inf, -inf, NaN) that the FP32
MFMA kernel gives it and lies within the bound where finite, whether the values
stand in the first stage (the split is left out), later in K (the tile is done
again) or nowhere near; K at the edges of the eights that the second pass takes
and of a stage."""
import math

import pytest

import synth

pytestmark = pytest.mark.gpu

SPLIT = [(128, 128, 8, 16), (128, 128, 8, 32), (64, 64, 8, 16)]
PLAIN = (64, 64, 4, 32)


@pytest.mark.parametrize("ta,tb", synth.LAYOUTS)
@pytest.mark.parametrize("K", [16, 23, 24, 33, 64, 129])
@pytest.mark.parametrize("where", ["first", "last", "all"])
def test_same_kinds_as_fp32(gpu, kt, ta, tb, K, where):
    h, torch = gpu
    g = torch.Generator(device="cuda").manual_seed(K)
    M, N = 200, 150
    a = torch.randn(M, K, generator=g, device="cuda")
    b = torch.randn(K, N, generator=g, device="cuda")
    k = {"first": 0, "last": K - 1}.get(where)
    if k is None:   # whole rows and columns
        a[3] = float("inf")
        a[70] = float("nan")
        a[140] = 2.0 ** 100   # overflows with column 90, whatever the order
        b[:, 5] = -float("inf")
        b[:, 90] = 2.0 ** 60
    else:
        a[3, k], a[70, k], a[140, k], a[199, k] = float("inf"), float("nan"), 3.4e38, 2.0 ** 49
        b[k, 149] = -float("inf")
    def rows(x):
        buf = torch.zeros(x.shape[0], (x.shape[1] + 15) // 16 * 16, device="cuda")
        buf[:, :x.shape[1]] = x
        return buf[:, :x.shape[1]]
    A, B = rows(a.t() if ta else a), rows(b.t() if tb else b)
    out = {}
    h.set_full_rows(True)
    try:
        for cfg in SPLIT + [PLAIN]:
            out[cfg] = torch.full((M, N), 7.0, device="cuda")
            h.gemm(A, B, out[cfg], ta, tb, config_id=h.configs().index(cfg))
        torch.cuda.synchronize()
    finally:
        h.set_full_rows(False)
    ref = out[PLAIN]
    exact = (a.double() @ b.double())
    scale = (a.abs().double().amax(1)[:, None] * b.abs().double().amax(0)[None, :])
    for cfg in SPLIT:
        C = out[cfg]
        assert torch.equal(C.isnan(), ref.isnan()), cfg
        assert torch.equal(C.isposinf(), ref.isposinf()) and torch.equal(C.isneginf(), ref.isneginf()), cfg
        f = C.isfinite() & exact.isfinite()
        err = (C.double() - exact).abs()[f]
        assert bool((err <= 1e-5 * math.sqrt(K) * scale[f]).all()), cfg
