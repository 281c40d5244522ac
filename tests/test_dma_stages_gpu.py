"""Stage counts of the DMA pipelines around the point where the K loop passes
from stages whose successors are all under way to the last few: one to seven
stages (two to four are in flight at once), whole, barely begun and nearly whole
last ones, padded rows and, in FP32, dense rows of odd length.

Operands are small whole numbers, exact in every type and sum, so the results
equal FP64's."""
import pytest

import synth

pytestmark = pytest.mark.gpu

CONFIGS = {"f32": [(64, 64, 2, 8), (32, 32, 2, 32), (128, 32, 2, 64), (128, 128, 4, 8), (64, 32, 4, 32)],
           "bf16": [(32, 128, 2, 32), (64, 64, 2, 64), (128, 128, 4, 64)],
           "fp8": [(32, 128, 2, 128), (64, 32, 2, 128), (64, 64, 4, 64)]}


@pytest.mark.parametrize("ta,tb", synth.LAYOUTS)
@pytest.mark.parametrize("dtype,padded", [("f32", True), ("f32", False), ("bf16", True), ("fp8", True)])
def test_stage_counts(gpu, kt, ta, tb, dtype, padded):
    h, torch = gpu
    dt = {"f32": kt.F32, "bf16": kt.BF16, "fp8": kt.FP8E4M3}[dtype]
    tt = {"f32": torch.float32, "bf16": torch.bfloat16, "fp8": torch.float8_e4m3fn}[dtype]
    M, N, batch = 133, 70, 2
    g = torch.Generator(device="cuda").manual_seed(5)
    one = torch.ones(1, device="cuda")

    def operand(r, c):
        ld = (c + 15) // 16 * 16 if padded else c
        x = torch.randint(-4, 5, (batch, r, ld), generator=g, device="cuda").float()
        return x[:, :, :c], x.to(tt), ld

    h.set_full_rows(padded)
    try:
        for cfg in CONFIGS[dtype]:
            bk = cfg[3]
            for K in sorted({bk * n + r for n in range(7) for r in (0, 1, bk - 1)} - {0}):
                a, A, lda = operand(*((K, M) if ta else (M, K)))
                b, B, ldb = operand(*((N, K) if tb else (K, N)))
                C = torch.full((batch, M, N), 7.0, device="cuda")
                h.gemm_raw(dt, kt.shape(M, N, K, batch, ta, tb), 1.0, A.data_ptr(), lda, A.stride(0), B.data_ptr(),
                           ldb, B.stride(0), 0.0, C.data_ptr(), N, M * N,
                           scaleA=one.data_ptr() if dtype == "fp8" else None,
                           scaleB=one.data_ptr() if dtype == "fp8" else None,
                           config_id=h.configs(dt).index(cfg))
                x = (a.transpose(1, 2) if ta else a).double().contiguous()
                y = (b.transpose(1, 2) if tb else b).double().contiguous()
                ref = torch.stack([x[i] @ y[i] for i in range(batch)])
                assert torch.equal(C.double(), ref), (cfg, K)
    finally:
        h.set_full_rows(False)
