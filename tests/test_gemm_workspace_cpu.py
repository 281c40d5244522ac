"""kt_gemm_workspace_bytes: the planes of what kt_gemm(-1) runs, on a host-only
handle whose selector always picks one kernel."""
import numpy as np
import pytest

import synth


def _fitted(kt, pick):
    h = kt.Handle(-1)
    problems = synth.sweep_problems(20, 515)
    T = np.full((len(problems), h.num_kernels()), 9000, dtype=np.int64)
    T[:, pick(h)] = 1000
    h.fit_selector(kt.SEL_DT_A, problems, T, [pick(h)])
    return h


@pytest.mark.parametrize("M,N,K,bt,planes", [
    (33, 70, 1535, 1, 0),           # too shallow
    (33, 70, 1536, 1, 8),
    (33, 70, 2100, 1, 7),           # slices of 320
    (256, 257, 2048, 1, 4),         # 72 tiles
    (513, 256, 2048, 1, 0),         # 136 tiles
    (40, 40, 2048, 2, 0),           # batched
    (0, 40, 2048, 1, 0),
])
def test_plain_pick(kt, M, N, K, bt, planes):
    h = _fitted(kt, lambda h: h.configs().index((32, 32, 2, 64)))
    try:
        assert h.gemm_workspace_bytes(M, N, K, bt) == (planes * M * N * 4 + 255) // 256 * 256
        assert h.kernel_workspace_bytes(M, N, K, bt, id=h.configs().index((32, 32, 2, 64))) == 0
    finally:
        h.close()


def test_split_k_pick_and_errors(kt):
    h = _fitted(kt, lambda h: h.num_configs() + 2)
    try:
        for s in ((100, 70, 3000), (100, 70, 60), (40, 30, 900, 3)):
            assert h.gemm_workspace_bytes(*s) == h.kernel_workspace_bytes(*s, id=h.num_configs() + 2)
        with pytest.raises(kt.KtError) as e:
            h.gemm_workspace_bytes(-1, 2, 3)
        assert e.value.status == -1
    finally:
        h.close()
    h = kt.Handle(-1)
    with pytest.raises(kt.KtError):
        h.gemm_workspace_bytes(40, 40, 2048)   # nothing fitted
    h.close()
