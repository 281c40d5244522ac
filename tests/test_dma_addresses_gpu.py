"""Addresses of the LDS-DMA pipeline at the edges of its two forms: 32-bit
offsets from a scalar base while a tile spans less than 2^31 bytes, whole
addresses beyond.  The same values stored with a small and with a large
leading dimension give the same bits."""
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ta,tb", synth.LAYOUTS)
@pytest.mark.parametrize("dtype,cfg", [(0, (32, 32, 4, 16)), (0, (64, 128, 8, 16)), (1, (128, 64, 8, 64)),
                                       (1, (32, 32, 2, 64)), (2, (64, 64, 8, 64))])
@pytest.mark.parametrize("below", [True, False])
def test_large_leading_dimension(gpu, kt, dtype, cfg, ta, tb, below):
    """The last leading dimension with offsets and the first one without;
    several stages, a partial last stage and ragged rows."""
    h, torch = gpu
    cid = h.configs(dtype).index(cfg)
    bm, bn, _, bk = cfg
    eb = (4, 2, 1)[dtype]
    M, N, K = 19, 17, bk + 16         # the widest operand takes 3 GB
    ce = 16 // eb
    g = torch.Generator(device="cuda").manual_seed(11)

    def operand(r, c, tile_rows):
        c16 = (c + ce - 1) // ce * ce
        big = (1 << 31) // (tile_rows * eb) - (ce if below else 0)
        vals = torch.randint(-3, 4, (r, c16), generator=g, device="cuda").float()
        vals = vals if dtype == 0 else vals.bfloat16() if dtype == 1 else vals.to(torch.float8_e4m3fn).view(torch.uint8)
        far = torch.empty((r - 1) * big + c16, dtype=vals.dtype, device="cuda")
        view = torch.as_strided(far, (r, c16), (big, 1))
        view.copy_(vals)
        return vals, far, c16, big

    # stored K-contiguous operands have M or N rows, the others K rows
    A, Af, lda, ldA = operand(K if ta else M, M if ta else K, bk if ta else bm)
    B, Bf, ldb, ldB = operand(N if tb else K, K if tb else N, bn if tb else bk)
    one = torch.ones(1, device="cuda")
    sc = one if dtype == 2 else None
    shp = kt.shape(M, N, K, 1, ta, tb)
    h.set_full_rows(True)
    try:
        C0 = torch.zeros(M, N, device="cuda")
        C1 = torch.zeros(M, N, device="cuda")
        assert h.dma_pipeline(dtype, shp, A, lda, 0, B, ldb, 0)
        assert h.dma_pipeline(dtype, shp, Af, ldA, 0, Bf, ldB, 0)
        h.gemm_raw(dtype, shp, 1.0, A, lda, 0, B, ldb, 0, 0.0, C0, N, 0, sc, sc, cid)
        h.gemm_raw(dtype, shp, 1.0, Af, ldA, 0, Bf, ldB, 0, 0.0, C1, N, 0, sc, sc, cid)
        torch.cuda.synchronize()
    finally:
        h.set_full_rows(False)
    assert torch.equal(C0, C1)
    a, b = A.cpu(), B.cpu()
    if dtype == 2:
        a, b = a.view(torch.float8_e4m3fn), b.view(torch.float8_e4m3fn)
    a, b = a.double(), b.double()
    a = (a.t() if ta else a)[:M, :K]
    b = (b.t() if tb else b)[:K, :N]
    assert torch.equal(C0.cpu().double(), a @ b)     # small integers: exact in every type
