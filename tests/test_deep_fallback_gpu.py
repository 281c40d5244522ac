"""The timed fallback ranks what kt_gemm(-1) runs: of two plain kernels on a deep
product, one with too many tiles to be sliced (about 215 us whatever the
workspace) and one with few (about 460 us unsplit, 70 in slices), the first wins
without a workspace for the planes and the second with one."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

UNSLICED, SLICED = (32, 16, 2, 64), (16, 128, 2, 32)
SHAPE = (1, 4096, 25088, 1, 0, 0)


@pytest.mark.parametrize("workspace,best", [(None, UNSLICED), (1 << 10, UNSLICED), (1 << 20, SLICED)])
def test_fallback_times_plain_kernels_as_they_run(gpu, kt, workspace, best):
    torch = gpu[1]
    hs = kt.Handle(0)
    try:
        chosen = [hs.configs().index(c) for c in (UNSLICED, SLICED)]
        assert not any(hs.get_kernel(v)[1] in chosen for v in range(hs.num_configs(), hs.num_kernels()))
        problems = synth.sweep_problems(20, 515)
        T = np.full((len(problems), hs.num_kernels()), 9000, dtype=np.int64)
        T[:, chosen] = 1000
        hs.fit_selector(kt.SEL_DT_A, problems, T, chosen)
        ws = torch.empty(workspace, dtype=torch.uint8, device="cuda") if workspace else None
        hs.set_workspace(ws)
        assert hs.get_config(hs.select(*SHAPE)) == best
    finally:
        hs.close()
