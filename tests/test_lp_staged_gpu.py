"""Register staging of BF16 / FP8 operands the DMA may not read (rows of any
alignment), against the LDS-DMA pipeline.

Both pipelines feed the same MFMAs with the same fragments in the same K order,
so the run on operands of odd leading dimensions at odd offsets equals, bit for
bit, the run on copies with rows padded to 16 bytes.  The odd operands lie in
buffers of NaN codes (before, after and between rows), so anything read beyond
them and multiplied shows.  Sizes at the edges of a 16-byte chunk (extents below
one, one more, one less than a tile), tails of K, and whole tiles."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = [(1, 1, 1), (5, 7, 9), (3, 300, 33), (33, 17, 3), (129, 131, 65), (64, 200, 127),
         (257, 15, 130), (128, 256, 512), (255, 129, 257)]
TILES = {1: [(32, 32, 4, 64), (64, 64, 2, 64), (128, 128, 8, 64), (256, 256, 8, 32)],
         2: [(32, 32, 4, 64), (64, 64, 2, 128), (128, 128, 8, 128), (256, 256, 8, 64)]}


def _place(torch, codes, ld, off, nan):
    """codes (batch, rows, ext) with leading dimension ld, off elements into a
    buffer of NaN codes."""
    bt, r, e = codes.shape
    buf = torch.full((off + bt * r * ld + 64,), nan, dtype=codes.dtype, device="cuda")
    buf[off:off + bt * r * ld].view(bt, r, ld)[:, :, :e] = codes
    return buf, buf.data_ptr() + off * codes.element_size()


@pytest.mark.parametrize("dtype", [1, 2])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_odd_rows_equal_padded_rows(gpu, kt, dtype, ta, tb):
    _, torch = gpu
    h = kt.Handle(0)
    try:
        h.set_full_rows(True)
        ids = [i for i, c in enumerate(h.configs(dtype)) if c in TILES[dtype]]
        assert ids
        g = torch.Generator(device="cuda").manual_seed(100 * dtype + 2 * ta + tb)
        one = torch.ones(1, device="cuda")
        ct, nan, ce = (torch.int16, 0x7FC0, 8) if dtype == 1 else (torch.uint8, 0x7F, 16)
        for M, N, K in SIZES:
            bt = 2
            ops = []
            for r, e in [(K, M) if ta else (M, K), (N, K) if tb else (K, N)]:
                x = torch.randn((bt, r, e), generator=g, device="cuda")
                ops.append(x.to(torch.bfloat16).view(torch.int16) if dtype == 1
                           else x.to(torch.float8_e4m3fn).view(torch.uint8))
            shp = kt.shape(M, N, K, bt, ta, tb)
            for off, pad in [(1, 0), (3, 2 if dtype == 1 else 3), (2, 1)]:
                odd, even = [], []
                for c in ops:
                    ld = c.shape[2] + pad
                    ld += (ld + 1) % 2                       # odd
                    odd.append((*_place(torch, c, ld, off, nan), ld))
                    ld = -(-c.shape[2] // ce) * ce
                    even.append((*_place(torch, c, ld, 0, 0), ld))
                assert not h.dma_pipeline(dtype, shp, odd[0][1], odd[0][2], ops[0].shape[1] * odd[0][2],
                                          odd[1][1], odd[1][2], ops[1].shape[1] * odd[1][2])
                for cfg in ids:
                    out = []
                    for (_, pa, lda), (_, pb, ldb) in (odd, even):
                        C = torch.full((bt, M, N), float("nan"), device="cuda")
                        h.gemm_raw(dtype, shp, 1.0, pa, lda, ops[0].shape[1] * lda, pb, ldb,
                                   ops[1].shape[1] * ldb, 0.0, C, N, M * N, scaleA=one.data_ptr(),
                                   scaleB=one.data_ptr(), config_id=cfg)
                        out.append(C)
                    torch.cuda.synchronize()
                    a, b = (o.cpu().numpy().view(np.uint32) for o in out)
                    assert np.array_equal(a, b), (M, N, K, off, pad, h.get_config(cfg, dtype))
    finally:
        h.close()
