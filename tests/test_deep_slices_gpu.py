"""Deep products of a plain configuration picked by the selector: kt_gemm(-1)
runs them in slices of K where the rule in splitk.hip says so, and unsplit
elsewhere.

Parity: the sliced run equals kt_gemm_splitk with the same configuration and
slice count bit for bit, the unsplit one the forced configuration, and both lie
within the FP32 bound of the plain GEMM tests against the FP64 oracle,
1e-5 * sqrt(K) * |alpha| * max|A_b| * max|B_b| + 2^-23 * |beta * C0|.  Sizes on
both sides of each line of the rule (K = 1536; 64 and 128 tiles of 32 x 32;
batch 1; a workspace that holds the planes), all layouts and offset operands."""
import math

import numpy as np
import pytest

import synth
from oracle import gemm as og

pytestmark = pytest.mark.gpu

CONFIG = (32, 32, 2, 64)


def _ops(M, N, K, bt, seed):
    return [synth.uniform_operand(synth.operand_seed(seed, i), bt * n).reshape(bt, *d)
            for i, (n, d) in enumerate([(M * K, (M, K)), (K * N, (K, N)), (M * N, (M, N))])]


@pytest.fixture(scope="module")
def plain(gpu, kt):
    """A handle whose selector always picks one configuration without slices."""
    hs = kt.Handle(0)
    cfg = hs.configs().index(CONFIG)
    problems = synth.sweep_problems(20, 515)
    T = np.full((len(problems), hs.num_kernels()), 9000, dtype=np.int64)
    T[:, cfg] = 1000
    hs.fit_selector(kt.SEL_DT_A, problems, T, [cfg])
    hs.set_fallback(0)
    yield hs, cfg, gpu[1]
    hs.close()


@pytest.mark.parametrize("M,N,K,bt,ws_planes,slices", [
    (33, 70, 1535, 1, 8, 1),          # too shallow
    (33, 70, 1536, 1, 8, 8),
    (1, 1, 1793, 1, 8, 8),            # one element; a last slice one deep
    (256, 256, 1999, 1, 8, 8),        # 64 tiles
    (256, 257, 1999, 1, 8, 4),        # 72 tiles
    (512, 255, 2048, 1, 8, 4),        # 128 tiles
    (513, 256, 2048, 1, 8, 1),        # 136 tiles
    (40, 40, 2048, 2, 8, 1),          # batched
    (40, 40, 2048, 1, 7, 1),          # planes do not fit
    (40, 40, 2048, 1, 0, 1),          # no workspace
])
def test_deep_products_run_in_slices(plain, kt, M, N, K, bt, ws_planes, slices):
    hs, cfg, torch = plain
    a, b, c0 = _ops(M, N, K, bt, 600 + M + K)
    alpha, beta = 1.25, -0.5
    ref = og.gemm(M, N, K, bt, 0, 0, alpha, beta, a, K, M * K, b, N, K * N, c0, N, M * N)
    amax = np.abs(a).reshape(bt, -1).max(axis=1)[:, None, None]
    bmax = np.abs(b).reshape(bt, -1).max(axis=1)[:, None, None]
    tol = 1e-5 * math.sqrt(K) * alpha * amax * bmax + 2.0 ** -23 * np.abs(beta * c0)
    ws = torch.empty(ws_planes * M * N * bt + 64, dtype=torch.float32, device="cuda")
    own = torch.empty(slices * M * N * bt + 64, dtype=torch.float32, device="cuda")
    try:
        hs.set_workspace(ws if ws_planes else None)
        for ta, tb in synth.LAYOUTS:
            for off in (0, 1):    # rows on and off 16 bytes
                dA = torch.zeros(a.size + 1, device="cuda")[off:off + a.size].view(
                    (bt, K, M) if ta else (bt, M, K))
                dB = torch.zeros(b.size + 1, device="cuda")[off:off + b.size].view(
                    (bt, N, K) if tb else (bt, K, N))
                dA.copy_(torch.from_numpy(a.swapaxes(1, 2).copy() if ta else a))
                dB.copy_(torch.from_numpy(b.swapaxes(1, 2).copy() if tb else b))
                dC = torch.from_numpy(c0).cuda()
                dF = dC.clone()
                hs.gemm(dA, dB, dC, ta, tb, alpha=alpha, beta=beta)
                if slices > 1:
                    used = hs.gemm_splitk(dA, dB, dF, slices, own, own.numel() * 4, ta, tb,
                                          alpha=alpha, beta=beta, config_id=cfg)
                    assert used == slices
                else:
                    hs.gemm(dA, dB, dF, ta, tb, alpha=alpha, beta=beta, config_id=cfg)
                torch.cuda.synchronize()
                C, F = dC.cpu().numpy(), dF.cpu().numpy()
                assert np.array_equal(C.view(np.uint32), F.view(np.uint32)), (ta, tb, off)
                assert np.all(np.abs(C - ref) <= tol), (ta, tb, off)
    finally:
        hs.set_workspace(None)


def test_convolution_in_slices_applies_bias_and_relu(plain, kt):
    """A 1 x 1 convolution is the plain product: 64 pixels, K = 1792, 48 channels."""
    hs, cfg, torch = plain
    x, w, y0 = _ops(64, 48, 1792, 1, 77)
    bias = np.linspace(-3, 3, 48, dtype=np.float32)
    ref = np.maximum(og.gemm(64, 48, 1792, 1, 0, 0, 1.0, 0.0, x, 1792, 0, w, 48, 0, None, 48, 0)
                     + bias, 0)
    tol = 1e-5 * math.sqrt(1792) * np.abs(x).max() * np.abs(w).max() + 2.0 ** -23 * 3
    ws = torch.empty(8 * 64 * 48 + 64, device="cuda")
    dx = torch.from_numpy(x).cuda().view(1, 8, 8, 1792)
    dw = torch.from_numpy(w).cuda().view(1, 1, 1792, 48)
    try:
        hs.set_workspace(ws)
        cs = kt.conv_shape(1, 8, 8, 1792, 48, 1, 1, 1, 0)
        y = torch.full((64, 48), float("nan"), device="cuda")
        n = kt.Handle.conv_workspace_bytes(cs, kt.CONV_IM2COL)
        cws = torch.empty(max(n, 256), dtype=torch.uint8, device="cuda")
        hs.conv2d(kt.CONV_IM2COL, cs, dx, dw, torch.from_numpy(bias).cuda(), True, y, cws, n)
        torch.cuda.synchronize()
        assert np.all(np.abs(y.cpu().numpy() - ref[0]) <= tol)
    finally:
        hs.set_workspace(None)
