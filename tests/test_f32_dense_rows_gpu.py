"""FP32 operands whose rows start on 4-byte boundaries only through the DMA
pipeline: the same values stored dense, off 16-byte boundaries and at odd
leading dimensions give the bits of the 16-byte aligned layout, at the edges
of chunks, tiles and stages.  Where K is too shallow for that pipeline (256 for
T = 2, three stages otherwise) they run register-staged, within the bound."""
import pytest

import synth

pytestmark = pytest.mark.gpu

CFGS = [(16, 16, 2, 16), (32, 64, 2, 64), (32, 32, 4, 8), (64, 64, 4, 16), (128, 128, 4, 32), (128, 128, 8, 32),
        (64, 128, 8, 64)]
# (M, N, K): single chunks, one beyond, one short; tiles and stages likewise
SIZES = [(4, 4, 4), (5, 7, 6), (64, 64, 64), (65, 63, 65), (127, 129, 35), (130, 70, 97), (33, 200, 128), (4, 129, 255),
         (65, 127, 256), (130, 70, 257), (33, 201, 323)]


def _place(torch, vals, ld, off, gap):
    """Batch of matrices with leading dimension ld, `off` floats after a
    256-byte boundary, `gap` floats between items, nothing after the last."""
    b, r, c = vals.shape
    stride = r * ld + gap
    buf = torch.empty(off + (b - 1) * stride + (r - 1) * ld + c, device="cuda")
    view = torch.as_strided(buf, (b, r, c), (stride, ld, 1), off)
    view.copy_(vals)
    return view


@pytest.mark.parametrize("ta,tb", synth.LAYOUTS)
@pytest.mark.parametrize("M,N,K", SIZES)
def test_same_bits_as_aligned_rows(gpu, kt, ta, tb, M, N, K):
    h, torch = gpu
    g = torch.Generator(device="cuda").manual_seed(M * 7 + K)
    bt = 2
    a = torch.randn(bt, *((K, M) if ta else (M, K)), generator=g, device="cuda")
    b = torch.randn(bt, *((N, K) if tb else (K, N)), generator=g, device="cuda")
    r16 = lambda v: (v + 15) // 16 * 16   # noqa: E731
    pa, pb = (torch.zeros(bt, t.shape[1], r16(t.shape[2]), device="cuda")[:, :, :t.shape[2]] for t in (a, b))
    pa.copy_(a)
    pb.copy_(b)
    ref = (a.transpose(1, 2) if ta else a).double().contiguous() @ (b.transpose(1, 2) if tb else b).double().contiguous()
    for cfg in CFGS:
        cid = h.configs().index(cfg)
        C0 = torch.full((bt, M, N), 5.0, device="cuda")
        h.set_full_rows(True)
        try:
            h.gemm(pa, pb, C0, ta, tb, config_id=cid)
        finally:
            h.set_full_rows(False)
        assert float((C0.double() - ref).norm() / ref.norm()) < 1e-5
        for lda, offa, ldb, offb, gap in ((0, 0, 0, 0, 0), (1, 1, 3, 2, 1), (2, 3, 0, 1, 3), (4, 2, 5, 3, 0)):
            A = _place(torch, a, a.shape[2] + lda, offa, gap)
            B = _place(torch, b, b.shape[2] + ldb, offb, gap)
            C1 = torch.full((bt, M, N), 5.0, device="cuda")
            h.gemm(A, B, C1, ta, tb, config_id=cid)
            torch.cuda.synchronize()
            if K < (256 if cfg[2] == 2 else 3 * cfg[3]) or (K < 16 and cfg[2] == 8):
                # shallow products run register-staged (below 16 the split kernels' in both layouts)
                assert float((C1.double() - ref).norm() / ref.norm()) < 1e-5
            else:
                assert torch.equal(C0, C1), (cfg, lda, offa, ldb, offb, gap)
