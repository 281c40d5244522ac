"""Several workspaces of one handle: where split-K kernels have been stays theirs
when the program goes to another buffer and back (their work may still be queued
there), also over more buffers than the handle remembers one by one."""
import pytest

from test_deep_streams_gpu import K, M, N, PLANES, _ops, _refs, deep  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("others", [1, 40])
def test_a_workspace_set_again(deep, others):   # noqa: F811
    hs, cfg, torch = deep
    a, b, c = _ops(torch, 11)
    sliced, plain = _refs(hs, cfg, torch, a, b)
    variant = next(v for v in range(hs.num_configs(), hs.num_kernels()) if hs.get_kernel(v)[0][4] == 4)
    need = hs.kernel_workspace_bytes(M, N, K, id=variant)
    size = need + PLANES - 256   # not for both
    pool = torch.empty((others + 1) * size, dtype=torch.uint8, device="cuda")
    spaces = [pool[i * size:(i + 1) * size] for i in range(others + 1)]
    cv = torch.zeros_like(c)
    for ws in spaces:
        hs.set_workspace(ws)
        hs.gemm(a, b, cv, config_id=variant)
    for ws in spaces:
        hs.set_workspace(ws)
        hs.gemm(a, b, c)
        torch.cuda.synchronize()
        assert torch.equal(c, plain)
    # a buffer that none has been in
    fresh = torch.empty(size, dtype=torch.uint8, device="cuda")
    hs.set_workspace(fresh)
    hs.gemm(a, b, c)
    torch.cuda.synchronize()
    assert torch.equal(c, sliced)
