"""Winograd layers on images without rows or columns: with a padding of two or
more the output is not empty, every position of it lies in the padding, and the
layer gives act(bias), as the lowering by patches does.  x points into the
middle of a buffer of NaN, of which nothing is read."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,pad", [(0, 5, 2), (6, 0, 2), (0, 0, 3), (0, 1, 2)])
@pytest.mark.parametrize("C,O", [(8, 12), (3, 5)])
def test_empty_image(gpu, kt, H, W, pad, C, O):
    h, torch = gpu
    cs = kt.conv_shape(2, H, W, C, O, 3, 3, 1, pad)
    Ho, Wo = H + 2 * pad - 2, W + 2 * pad - 2
    assert Ho > 0 and Wo > 0
    x = torch.full((4096,), float("nan"), device="cuda")[2048:]
    w = torch.ones(9 * C * O, device="cuda")
    b = torch.linspace(-1, 1, O, device="cuda")
    for algo in (kt.CONV_WINOGRAD, kt.CONV_IM2COL):
        n = kt.Handle.conv_workspace_bytes(cs, algo)
        ws = torch.empty(n, dtype=torch.uint8, device="cuda")
        for relu in (False, True):
            y = torch.full((2, Ho, Wo, O), float("nan"), device="cuda")
            h.conv2d(algo, cs, x, w, b, relu, y, ws, n, config_id=h.configs().index((32, 32, 2, 32)))
            torch.cuda.synchronize()
            assert torch.equal(y, (b.clamp(min=0) if relu else b).expand_as(y)), (algo, relu)
