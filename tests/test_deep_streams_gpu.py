"""Deep products of a plain pick on several streams of one handle: their
partial planes share the handle's workspace, so each waits for the one before
it, keeps clear of what split-K kernels have taken, and runs unsplit under
stream capture or where the planes would touch memory in use.

Parity is bit for bit: in slices with kt_gemm_splitk of the same configuration
and slice count, unsplit with the forced configuration."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

CONFIG = (32, 32, 2, 64)
# slices of 320: seven of the eight; their ends are no ends of the unsplit sum's
# blocks of 256, so the two forms differ in bits
M, N, K, SLICES = 40, 70, 2100, 8
PLANES = (7 * M * N * 4 + 255) // 256 * 256


@pytest.fixture
def deep(gpu, kt):
    """A handle whose selector always picks CONFIG for shallow and deep shapes."""
    hs = kt.Handle(0)
    cfg = hs.configs().index(CONFIG)
    problems = synth.sweep_problems(20, 515)
    T = np.full((len(problems), hs.num_kernels()), 9000, dtype=np.int64)
    T[:, cfg] = 1000
    hs.fit_selector(kt.SEL_DT_A, problems, T, [cfg])
    hs.set_fallback(0)
    yield hs, cfg, gpu[1]
    gpu[1].cuda.synchronize()
    hs.close()


def _ops(torch, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return (torch.randn(1, M, K, generator=g, device="cuda"), torch.randn(1, K, N, generator=g, device="cuda"),
            torch.zeros(1, M, N, device="cuda"))


def _refs(hs, cfg, torch, a, b):
    own = torch.empty(PLANES // 4, device="cuda")
    sliced, plain = torch.zeros(1, M, N, device="cuda"), torch.zeros(1, M, N, device="cuda")
    hs.gemm_splitk(a, b, sliced, SLICES, own, PLANES, config_id=cfg)
    hs.gemm(a, b, plain, config_id=cfg)
    torch.cuda.synchronize()
    assert not torch.equal(sliced, plain)   # else the tests below tell nothing
    return sliced, plain


def test_products_on_two_streams_are_ordered(deep):
    hs, cfg, torch = deep
    ws = torch.empty(PLANES, dtype=torch.uint8, device="cuda")
    hs.set_workspace(ws)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    big = torch.randn(4096, 4096, device="cuda")
    ops = [_ops(torch, i) for i in range(2)]
    refs = [_refs(hs, cfg, torch, a, b)[0] for a, b, _ in ops]
    for (a, b, c) in ops:   # first launches load code: not under the timing below
        hs.gemm(a, b, c, stream=s1)
    torch.cuda.synchronize()
    for _ in range(3):
        for _, _, c in ops:
            c.zero_()
        torch.cuda.synchronize()
        before = torch.cuda.Event()
        with torch.cuda.stream(s1):
            for _ in range(8):   # some milliseconds
                big = torch.mm(big, big).clamp_(-1, 1)
            before.record(s1)
        hs.gemm(*ops[0], stream=s1)
        hs.gemm(*ops[1], stream=s2)
        s2.synchronize()
        assert before.query()   # the second product came after the first
        torch.cuda.synchronize()
        for (_, _, c), ref in zip(ops, refs):
            assert torch.equal(c, ref)


def test_planes_keep_clear_of_split_kernels(deep, kt):
    hs, cfg, torch = deep
    a, b, c = _ops(torch, 7)
    sliced, plain = _refs(hs, cfg, torch, a, b)
    variant = next(v for v in range(hs.num_configs(), hs.num_kernels()) if hs.get_kernel(v)[0][4] == 4)
    need = hs.kernel_workspace_bytes(M, N, K, id=variant)
    assert 0 < need < PLANES
    # room for both: the planes lie at the end, the start is left alone
    ws = torch.full((need + PLANES,), 7, dtype=torch.uint8, device="cuda")
    hs.set_workspace(ws)
    hs.gemm(a, b, c)
    torch.cuda.synchronize()
    assert torch.equal(c, sliced) and bool((ws[:need] == 7).all()) and not bool((ws[need:] == 7).all())
    tail = ws[need:].clone()
    hs.gemm(a, b, c, config_id=variant)
    torch.cuda.synchronize()
    assert torch.equal(ws[need:], tail) and not bool((ws[:need] == 7).all())
    hs.gemm(a, b, c)
    torch.cuda.synchronize()
    assert torch.equal(c, sliced)
    # a byte less: the variant has been where the planes would lie
    hs.set_workspace(ws[:need + PLANES - 1])
    for _ in range(2):
        hs.gemm(a, b, c)
        torch.cuda.synchronize()
        assert torch.equal(c, plain)
        hs.set_workspace(None)   # its place is remembered
        hs.set_workspace(ws[:need + PLANES - 1])
    # another buffer holds them
    other = torch.empty(PLANES, dtype=torch.uint8, device="cuda")
    hs.set_workspace(other)
    hs.gemm(a, b, c)
    torch.cuda.synchronize()
    assert torch.equal(c, sliced)
    # a variant that reaches into the planes' part waits for them
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    big = torch.randn(4096, 4096, device="cuda")
    c2, cv = torch.zeros_like(c), torch.zeros_like(c)
    torch.cuda.synchronize()
    before = torch.cuda.Event()
    with torch.cuda.stream(s1):
        for _ in range(8):
            big = torch.mm(big, big).clamp_(-1, 1)
        before.record(s1)
    hs.gemm(a, b, c2, stream=s1)
    hs.gemm(a, b, cv, config_id=variant, stream=s2)
    s2.synchronize()
    assert before.query()
    torch.cuda.synchronize()
    assert torch.equal(c2, sliced)


def test_unsplit_under_capture(deep):
    hs, cfg, torch = deep
    ws = torch.full((4 * PLANES,), 7, dtype=torch.uint8, device="cuda")
    a, b, c = _ops(torch, 9)
    sliced, plain = _refs(hs, cfg, torch, a, b)
    hs.set_workspace(ws)
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        hs.gemm(a, b, c, stream=s)
    for _ in range(3):
        c.fill_(3.0)
        g.replay()
        eager = torch.zeros_like(c)
        torch.cuda.synchronize()
        assert torch.equal(c, plain) and bool((ws == 7).all())
        hs.gemm(a, b, eager)
        torch.cuda.synchronize()
        assert torch.equal(eager, sliced)
        ws.fill_(7)


def test_convolution_whose_workspace_is_the_handles(deep, kt):
    """A 3 x 3 layer, K = 9 x 240 = 2160: the patch matrix and the planes may
    not meet when a program passes the one buffer for both."""
    hs, cfg, torch = deep
    g = torch.Generator(device="cuda").manual_seed(3)
    C, O, H = 240, 48, 6
    cs = kt.conv_shape(1, H, H, C, O, 3, 3, 1, 1)
    x = torch.randn(1, H, H, C, generator=g, device="cuda")
    w = torch.randn(3, 3, C, O, generator=g, device="cuda")
    n = kt.Handle.conv_workspace_bytes(cs, kt.CONV_IM2COL)
    planes = (7 * H * H * O * 4 + 255) // 256 * 256
    w1 = torch.empty(n + planes, dtype=torch.uint8, device="cuda")
    w2 = torch.empty(planes, dtype=torch.uint8, device="cuda")
    out = {}
    for name, mine, cid in (("apart", w2, -1), ("behind", w1, -1), ("inside", w1[:n], -1), ("plain", None, cfg)):
        hs.set_workspace(mine)
        out[name] = torch.zeros(H * H, O, device="cuda")
        hs.conv2d(kt.CONV_IM2COL, cs, x, w, None, False, out[name], w1, n, config_id=cid)
        torch.cuda.synchronize()
    assert torch.equal(out["apart"], out["behind"])      # in slices
    assert torch.equal(out["inside"], out["plain"])      # the patch matrix fills the buffer
    assert not torch.equal(out["apart"], out["plain"])
