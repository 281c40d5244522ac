"""FP8 quantization in one work-group (up to 65536 elements on 16-byte
boundaries): the codes and the scale of the oracle, bit for bit, at the edges of
a chunk, of the threads' strides and of the rule, and off 16-byte boundaries
(the general kernels); zeros, infinities and NaN as the general kernels have
them."""
import numpy as np
import pytest

import synth
from oracle import convert as cv

pytestmark = pytest.mark.gpu


def _run(h, torch, x, off):
    n = x.size
    dx = torch.zeros(n + off, device="cuda")
    dx[off:] = torch.from_numpy(x).cuda()
    y = torch.full((n + 16,), 0x55, dtype=torch.uint8, device="cuda")
    sc = torch.zeros(1, device="cuda")
    ws = torch.full((4,), -1, dtype=torch.int32, device="cuda")
    h.quantize_fp8(dx[off:], n, y, sc, ws, 16)
    torch.cuda.synchronize()
    assert (y[n:] == 0x55).all()
    return y[:n].cpu().numpy(), sc.cpu().numpy()


@pytest.mark.parametrize("n", [1, 3, 4, 5, 63, 4095, 4096, 4099, 48000, 65533, 65535, 65536, 65537, 65540])
def test_codes_and_scale(gpu, kt, n):
    h, torch = gpu
    x = (synth.uniform_operand(n, n) * 37.0).astype(np.float32)
    codes, s = cv.quantize_fp8(x)
    for off in (0, 1):
        got, sc = _run(h, torch, x, off)
        assert np.array_equal(got, codes) and np.float32(s) == sc[0], off


@pytest.mark.parametrize("special", [[0.0], [np.inf, 1.0], [-np.inf, 0.0, 2.0], [np.nan, 1.0], [1e-38, 3e-39]])
@pytest.mark.parametrize("at", [0, 4096, 9997])
def test_special_values_as_the_general_kernels(gpu, kt, special, at):
    h, torch = gpu
    x = np.zeros(10000, np.float32) if special == [0.0] else synth.uniform_operand(3, 10000).copy()
    x[at:at + len(special)] = special
    a, sa = _run(h, torch, x, 0)
    b, sb = _run(h, torch, x, 1)
    assert np.array_equal(a, b) and sa.view(np.uint32)[0] == sb.view(np.uint32)[0]
