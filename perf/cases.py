"""The library's work as a program has it do, as timed cases.

A case is a dict of plain values; its "kind" names the entry points it goes
through:

  gemm     one batched product through the deployed selector (config_id -1),
           FP32 / BF16 / FP8 operands already in device memory, rows dense or
           padded to 16 elements (with the whole-rows promise)
  linear   a fully connected layer from FP32 activations: conversion to BF16
           or per-tensor quantization to FP8, then the product with weights
           converted when they were loaded
  grouped  one launch of a planned group of uneven BF16 products
  conv     one NHWC FP32 convolution layer with bias and ReLU, filters laid
           out when they were loaded
  vgg16    single-image VGG16 inference, 224x224x3 to 1000 logits
  prune    k-means pruning of a benchmark table (host table in, choice out)
  mlp      training the learned selector on a benchmark table

Sizes follow the sweep set (M, N, K 16..4096, batch 1..64), the grouped set
(32..2048) and the VGG16 layers of this repository.
"""
import functools
import math

import numpy as np
import torch

import paper_2008_13145_amd as kt
import synth
from paper_2008_13145_amd import tune

DTYPES = {"f32": kt.F32, "bf16": kt.BF16, "fp8": kt.FP8E4M3}
ELEM = {"f32": 4, "bf16": 2, "fp8": 1}
VGG_CONV = (64, 64, 0, 128, 128, 0, 256, 256, 256, 0, 512, 512, 512, 0, 512, 512, 512, 0)   # 0: pool
VGG_FC = ((25088, 4096), (4096, 4096), (4096, 1000))
N_KERNELS = 8          # deployed kernels per data type


def _gemm(name, dtype, M, N, K, batch, ta, tb, padded):
    c = {"name": name} if name else {}
    return {**c, "kind": "gemm", "dtype": dtype, "M": M, "N": N, "K": K, "batch": batch,
            "ta": ta, "tb": tb, "padded": padded}


def listed():
    return [
        # a single small product in a larger program: launch and latency bound
        _gemm("f32_small", "f32", 150, 97, 70, 2, 1, 0, False),
        # dense tensors of odd sizes, as a caller's slices have them
        _gemm("f32_ragged", "f32", 1021, 515, 997, 3, 0, 1, False),
        # a batched product of the sweep set's upper half (weight gradients are TN)
        _gemm("f32_batched", "f32", 2048, 1024, 1536, 16, 1, 0, True),
        # the largest sweep-set sizes in one product
        _gemm("f32_square", "f32", 4096, 4096, 4096, 1, 0, 0, True),
        # low precision on dense odd-sized tensors
        _gemm("bf16_ragged", "bf16", 1021, 771, 515, 8, 0, 0, False),
        # projection layers of a batch of tokens, converted on the way in
        {"name": "bf16_linear", "kind": "linear", "dtype": "bf16", "M": 4096, "N": 4096, "K": 4096},
        {"name": "fp8_linear", "kind": "linear", "dtype": "fp8", "M": 4096, "N": 4096, "K": 4096},
        # many uneven products at once
        {"name": "grouped", "kind": "grouped", "members": 512, "shape_seed": 4, "padded": True},
        # a batch of images through one 3x3 layer, filters transformed at load
        {"name": "conv_batch", "kind": "conv", "n": 16, "H": 56, "Cin": 256, "Cout": 256, "R": 3,
         "stride": 1, "winograd": True},
        # one image through the whole network: small launches, weight streaming
        {"name": "vgg16", "kind": "vgg16"},
        # tuning: prune a measured table to the kernels that ship, fit the selector
        {"name": "prune", "kind": "prune", "rows": 960, "kernels": 188, "k": N_KERNELS, "norm": 0},
        {"name": "mlp_fit", "kind": "mlp", "rows": 960, "kernels": 188, "k": N_KERNELS, "steps": 3000},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["gemm"] * 6 + ["linear"] * 2 + ["grouped", "conv", "conv", "prune", "mlp"])
    if kind == "gemm":
        dtype = rng.choice(["f32", "f32", "bf16", "fp8"])
        while True:
            M, N, K = (_log_int(rng, 17, 4095) for _ in range(3))
            batch = _log_int(rng, 1, 63)
            if 2 * M * N * K * batch <= 1.2e11 and batch * max(M * K, K * N, M * N) <= 1 << 26:
                break
        return _gemm(None, dtype, M, N, K, batch, rng.randrange(2), rng.randrange(2),
                     rng.random() < 0.5)
    if kind == "linear":
        return {"kind": "linear", "dtype": rng.choice(["bf16", "fp8"]), "M": _log_int(rng, 32, 4096),
                "N": 16 * _log_int(rng, 8, 256), "K": 16 * _log_int(rng, 8, 256)}
    if kind == "grouped":
        return {"kind": "grouped", "members": _log_int(rng, 24, 400),
                "shape_seed": rng.randrange(1 << 20), "padded": rng.random() < 0.5}
    if kind == "conv":
        while True:
            n, H = _log_int(rng, 1, 16), rng.choice([7, 14, 27, 28, 35, 56, 61, 112])
            cin, cout = _log_int(rng, 16, 512), 8 * _log_int(rng, 4, 64)
            wino = rng.random() < 0.6
            R = 3 if wino else rng.choice([1, 3, 5])
            if 2 * n * H * H * cin * cout * R * R <= 5e10 and n * H * H * cin * R * R <= 1 << 26:
                break
        return {"kind": "conv", "n": n, "H": H, "Cin": cin, "Cout": cout, "R": R,
                "stride": 1 if wino else rng.choice([1, 1, 2]), "winograd": wino}
    if kind == "prune":
        return {"kind": "prune", "rows": rng.randrange(200, 961), "kernels": rng.randrange(60, 189),
                "k": rng.randrange(4, 9), "norm": rng.randrange(4)}
    return {"kind": "mlp", "rows": rng.randrange(200, 961), "kernels": rng.randrange(60, 189),
            "k": rng.randrange(4, 9), "steps": rng.randrange(400, 3001)}


# ------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 13)


def _randn(shape, g, scale=1.0):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).mul_(scale)


@functools.lru_cache(maxsize=None)
def _deployed(dtype, padded):
    """A handle with the data type's measured table pruned and its learned
    selector fitted, as a program makes once when it starts."""
    dt = DTYPES[dtype]
    h = kt.Handle(0)
    h.set_full_rows(padded)
    ws = torch.empty(kt.SPLIT_PLANE_CAP, dtype=torch.uint8, device="cuda")
    h.set_workspace(ws)
    T, P, _, _ = tune.load_table(tune.table_path(dtype))
    rows = synth.rows_of_shapes(synth.train_test_split()[0])
    nb = max(kt.Handle.prune_workspace_bytes(len(rows), T.shape[1], N_KERNELS, 10),
             kt.Handle.mlp_workspace_bytes(len(rows), T.shape[1], N_KERNELS))
    tmp = torch.empty(nb, dtype=torch.uint8, device="cuda")
    stream = torch.cuda.current_stream()
    chosen = tune.select_pruning(h, T[rows], N_KERNELS, synth.SEED, workspace=tmp, ws_bytes=nb,
                                 stream=stream)["chosen"]
    h.fit_selector(kt.SEL_MLP, P[rows].tolist(), T[rows], chosen, workspace=tmp, ws_bytes=nb,
                   stream=stream, dtype=dt)
    torch.cuda.synchronize()
    return h, ws


def _rows(batch, r, c, padded):
    """Row-major storage of a batch of r x c matrices and its (padded) view."""
    ld = (c + 15) // 16 * 16 if padded else c
    return ld, (batch, r, ld)


def _fp8_codes(h, x):
    q = torch.empty(x.numel(), dtype=torch.uint8, device="cuda")
    s = torch.empty(1, dtype=torch.float32, device="cuda")
    ws = torch.empty(16, dtype=torch.uint8, device="cuda")
    h.quantize_fp8(x, x.numel(), q, s, ws, stream=torch.cuda.current_stream())
    return q, s


def _operand(case, seed, role):
    """FP32 source values of GEMM operand A (role 0) or B (role 1), as stored."""
    M, N, K = case["M"], case["N"], case["K"]
    r, c = ((K, M) if case["ta"] else (M, K)) if role == 0 else ((N, K) if case["tb"] else (K, N))
    ld, shp = _rows(case["batch"], r, c, case["padded"])
    return _randn(shp, _gen(2 * seed + role)), c


def _vgg_layers():
    layers, H, C = [], 224, 3
    for v in VGG_CONV:
        if v == 0:
            layers.append(("pool", (H, C)))
            H //= 2
        else:
            layers.append(("conv", kt.conv_shape(1, H, H, C, v)))
            C = v
    for fi, fo in VGG_FC:
        layers.append(("fc", kt.conv_shape(1, 1, 1, fi, fo, 1, 1, 1, 0)))
    return layers


def _vgg_values(seed):
    g = _gen(seed)
    x = _randn((224, 224, 3), g)
    wb = []
    for kind, cs in _vgg_layers():
        if kind != "pool":
            fan = cs.R * cs.S * cs.Cin
            wb.append((_randn((cs.R * cs.S, cs.Cin, cs.Cout), g, math.sqrt(2.0 / fan)),
                       _randn((cs.Cout,), g, 0.05)))
    return x, wb


def _conv_values(case, seed):
    g = _gen(seed)
    n, H, ci, co, R = (case[k] for k in ("n", "H", "Cin", "Cout", "R"))
    x = _randn((n, H, H, ci), g).relu_()
    return x, _randn((R * R, ci, co), g, math.sqrt(2.0 / (R * R * ci))), _randn((co,), g, 0.1)


def _conv_shape(case):
    return kt.conv_shape(case["n"], case["H"], case["H"], case["Cin"], case["Cout"], case["R"],
                         case["R"], case["stride"], case["R"] // 2)


def _group_shapes(case):
    return synth.grouped_shapes(case["members"], synth.SEED + case["shape_seed"])


def _group_layout(case):
    rnd = (lambda v: (v + 7) // 8 * 8) if case["padded"] else (lambda v: v)
    a128 = lambda v: (v + 127) // 128 * 128   # noqa: E731
    oa, ob, oc, ld, na, nb, nc = [], [], [], [], 0, 0, 0
    for M, N, K in _group_shapes(case):
        ld.append((rnd(K), rnd(N), N))
        oa.append(na); ob.append(nb); oc.append(nc)
        na += a128(M * rnd(K)); nb += a128(K * rnd(N)); nc += a128(M * N)
    return oa, ob, oc, ld, na, nb, nc


def _group_values(case, seed):
    _, _, _, _, na, nb, _ = _group_layout(case)
    g = _gen(seed)
    return _randn((na,), g).bfloat16(), _randn((nb,), g).bfloat16()


def _table(case, seed):
    """A benchmark table: problems, and times whose ratios come from a few
    hidden traits of problem and kernel plus measurement noise."""
    r = np.random.RandomState(int(seed) + 17)
    n, d = case["rows"], case["kernels"]
    size = np.exp(r.uniform(math.log(16), math.log(4096), (n, 3)))
    shapes = [(int(m), int(nn), int(k), int(r.randint(1, 65)), int(r.randint(2)), int(r.randint(2)))
              for m, nn, k in size]
    base = np.array([2.0 * m * nn * k * b / 6e4 + 4000.0 for m, nn, k, b, _, _ in shapes])
    traits = np.concatenate([np.log(size) / 4.0 - 1.4, r.randn(n, 1) * 0.3], axis=1)
    off = traits @ (r.randn(4, d) * 0.25) + np.abs(r.randn(1, d)) * 0.25
    off = off - off.min(axis=1, keepdims=True)
    T = base[:, None] * np.exp(off) * (1.0 + 0.02 * r.randn(n, d))
    return shapes, np.maximum(T, 1.0).astype(np.int64)


def prepare(case, seed):
    kind = case["kind"]
    stream = torch.cuda.current_stream()
    if kind == "gemm":
        dtype = case["dtype"]
        h, _ = _deployed(dtype, case["padded"])
        ops, scales = [], []
        for role in (0, 1):
            x, cols = _operand(case, seed, role)
            if dtype == "bf16":
                x = x.bfloat16()
            elif dtype == "fp8":
                q, s = _fp8_codes(h, x)
                x = q.reshape(x.shape)
                scales.append(s)
            ops.append(x[:, :, :cols])
        C = torch.zeros((case["batch"], case["M"], case["N"]), dtype=torch.float32, device="cuda")
        return {"case": case, "h": h, "A": ops[0], "B": ops[1], "C": C, "scales": scales or (None, None),
                "stream": stream}
    if kind == "linear":
        dtype = case["dtype"]
        h, _ = _deployed(dtype, False)
        M, N, K = case["M"], case["N"], case["K"]
        x, w = _randn((M, K), _gen(2 * seed)), _randn((N, K), _gen(2 * seed + 1), 1.0 / math.sqrt(K))
        y = torch.zeros((M, N), dtype=torch.float32, device="cuda")
        st = {"case": case, "h": h, "x": x, "y": y, "stream": stream}
        if dtype == "bf16":
            st.update(w=w.bfloat16(), xl=torch.zeros((M, K), dtype=torch.int16, device="cuda"))
        else:
            q, s = _fp8_codes(h, w)
            st.update(w=q.reshape(N, K), sw=s, xl=torch.zeros((M, K), dtype=torch.uint8, device="cuda"),
                      sx=torch.zeros(1, dtype=torch.float32, device="cuda"),
                      ws=torch.empty(16, dtype=torch.uint8, device="cuda"))
        return st
    if kind == "grouped":
        h = kt.Handle(0)
        oa, ob, oc, ld, _, _, nc = _group_layout(case)
        A, B = _group_values(case, seed)
        C = torch.zeros(nc, dtype=torch.float32, device="cuda")
        shapes = _group_shapes(case)
        nb = kt.Handle.grouped_workspace_bytes([(m, n, k, 1, 0, 0) for m, n, k in shapes])
        ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
        plan = h.grouped_plan(shapes, [A.data_ptr() + 2 * o for o in oa],
                              [B.data_ptr() + 2 * o for o in ob], [C.data_ptr() + 4 * o for o in oc],
                              workspace=ws, ws_bytes=nb, stream=stream, ld=ld)
        return {"case": case, "h": h, "A": A, "B": B, "C": C, "ws": ws, "plan": plan, "stream": stream}
    if kind == "conv":
        h, _ = _deployed("f32", False)
        cs = _conv_shape(case)
        x, w, b = _conv_values(case, seed)
        algo = kt.CONV_IM2COL
        if case["winograd"]:
            algo = kt.CONV_WINOGRAD_PRETRANSFORMED
            U = torch.empty(16 * cs.Cin * cs.Cout, dtype=torch.float32, device="cuda")
            h.winograd_filter(w, cs.Cin, cs.Cout, U, stream=stream)
            w = U
        nb = kt.Handle.conv_workspace_bytes(cs, algo)
        Ho = (case["H"] + 2 * (case["R"] // 2) - case["R"]) // case["stride"] + 1
        y = torch.zeros((case["n"], Ho, Ho, case["Cout"]), dtype=torch.float32, device="cuda")
        return {"case": case, "h": h, "cs": cs, "algo": algo, "x": x, "w": w, "b": b, "y": y, "nb": nb,
                "ws": torch.empty(max(nb, 1), dtype=torch.uint8, device="cuda"), "stream": stream}
    if kind == "vgg16":
        h, _ = _deployed("f32", False)
        x, wb = _vgg_values(seed)
        layers, li, net, nb = _vgg_layers(), 0, [], 1
        for lk, cs in layers:
            if lk == "pool":
                net.append((lk, cs, None, None, None))
                continue
            w, b = wb[li]
            algo = kt.CONV_IM2COL
            if lk == "conv":
                algo = kt.CONV_WINOGRAD_PRETRANSFORMED
                U = torch.empty(16 * cs.Cin * cs.Cout, dtype=torch.float32, device="cuda")
                h.winograd_filter(w, cs.Cin, cs.Cout, U, stream=stream)
                w = U
            nb = max(nb, kt.Handle.conv_workspace_bytes(cs, algo))
            net.append((algo, cs, w, b, li < len(wb) - 1))
            li += 1
        return {"case": case, "h": h, "x": x, "net": net, "nb": nb, "stream": stream,
                "ws": torch.empty(nb, dtype=torch.uint8, device="cuda"),
                "buf": [torch.empty(224 * 224 * 64, dtype=torch.float32, device="cuda") for _ in range(2)]}
    h = kt.Handle(0)
    shapes, T = _table(case, seed)
    n, d, k = case["rows"], case["kernels"], case["k"]
    if kind == "prune":
        nb = kt.Handle.prune_workspace_bytes(n, d, k, 10)
    else:
        nb = kt.Handle.mlp_workspace_bytes(n, d, k)
    return {"case": case, "h": h, "shapes": shapes, "T": T, "nb": nb, "stream": stream,
            "chosen": [int(c) for c in np.random.RandomState(int(seed)).permutation(d)[:k]],
            "ws": torch.empty(nb, dtype=torch.uint8, device="cuda")}


# --------------------------------------------------------------------- run
def run(st):
    case, h, stream = st["case"], st["h"], st["stream"]
    kind = case["kind"]
    if kind == "gemm":
        h.gemm(st["A"], st["B"], st["C"], case["ta"], case["tb"], dtype=DTYPES[case["dtype"]],
               scaleA=st["scales"][0], scaleB=st["scales"][1], stream=stream)
        return st["C"]
    if kind == "linear":
        x = st["x"]
        if case["dtype"] == "bf16":
            h.convert_bf16(x, x.numel(), st["xl"], stream=stream)
            h.gemm(st["xl"], st["w"], st["y"], 0, 1, dtype=kt.BF16, stream=stream)
            return {"y": st["y"], "x": st["xl"]}
        h.quantize_fp8(x, x.numel(), st["xl"], st["sx"], st["ws"], stream=stream)
        h.gemm(st["xl"], st["w"], st["y"], 0, 1, dtype=kt.FP8E4M3, scaleA=st["sx"], scaleB=st["sw"],
               stream=stream)
        return {"y": st["y"], "x": st["xl"], "scale": st["sx"]}
    if kind == "grouped":
        h.grouped_launch(st["plan"], stream=stream)
        return st["C"]
    if kind == "conv":
        h.conv2d(st["algo"], st["cs"], st["x"], st["w"], st["b"], True, st["y"], st["ws"], st["nb"],
                 stream=stream)
        return st["y"]
    if kind == "vgg16":
        src = st["x"]
        for algo, cs, w, b, relu in st["net"]:
            dst = st["buf"][0] if src is not st["buf"][0] else st["buf"][1]
            if algo == "pool":
                h.maxpool2x2(src, 1, cs[0], cs[0], cs[1], dst, stream=stream)
            else:
                h.conv2d(algo, cs, src, w, b, relu, dst, st["ws"], st["nb"], stream=stream)
            src = dst
        return src[:1000]
    if kind == "prune":
        r = h.prune(st["T"], case["k"], norm=case["norm"], workspace=st["ws"], ws_bytes=st["nb"],
                    stream=stream)
        return {"chosen": np.array(r["chosen"], np.int64), "labels": r["labels"],
                "centroids": r["centroids"], "inertia": int(r["inertia"])}
    h.fit_selector(kt.SEL_MLP, st["shapes"], st["T"], st["chosen"], mlp_steps=case["steps"],
                   workspace=st["ws"], ws_bytes=st["nb"], stream=stream)
    return h.get_mlp()


# -------------------------------------------------------------------- work
def work(case):
    kind = case["kind"]
    if kind == "gemm":
        M, N, K, b, e = case["M"], case["N"], case["K"], case["batch"], ELEM[case["dtype"]]
        return {"bytes": b * (e * (M * K + K * N) + 4 * M * N), "flops": 2.0 * b * M * N * K}
    if kind == "linear":
        M, N, K, e = case["M"], case["N"], case["K"], ELEM[case["dtype"]]
        return {"bytes": 4 * M * K + e * (M * K + N * K) + 4 * M * N, "flops": 2.0 * M * N * K}
    if kind == "grouped":
        s = _group_shapes(case)
        return {"bytes": sum(2 * (m * k + k * n) + 4 * m * n for m, n, k in s),
                "flops": sum(2.0 * m * n * k for m, n, k in s)}
    if kind == "conv":
        n, H, ci, co, R = (case[k] for k in ("n", "H", "Cin", "Cout", "R"))
        Ho = (H + 2 * (R // 2) - R) // case["stride"] + 1
        g = kt.Handle.conv_gemm_shape(_conv_shape(case), kt.CONV_WINOGRAD if case["winograd"] else kt.CONV_IM2COL)
        return {"bytes": 4 * (n * H * H * ci + (16 if case["winograd"] else R * R) * ci * co + n * Ho * Ho * co),
                "flops": 2.0 * g[0] * g[1] * g[2] * g[3]}
    if kind == "vgg16":
        bts = fl = 0
        for lk, cs in _vgg_layers():
            if lk == "pool":
                continue
            g = kt.Handle.conv_gemm_shape(cs, kt.CONV_WINOGRAD if lk == "conv" else kt.CONV_IM2COL)
            bts += 4 * (16 if lk == "conv" else 1) * cs.Cin * cs.Cout
            fl += 2.0 * g[0] * g[1] * g[2] * g[3]
        return {"bytes": bts + 4 * 224 * 224 * 3, "flops": fl}
    n, d, k = case["rows"], case["kernels"], case["k"]
    if kind == "prune":   # k-means++ and at least two assignments of each of the 10 restarts
        return {"bytes": 8 * n * d, "flops": 10 * 3 * 3.0 * n * d * k}
    return {"bytes": 8 * n * d, "flops": case["steps"] * 6.0 * n * (6 * 64 + 64 * 64 + 64 * k)}


# ------------------------------------------------------------------- exact
def _exact_conv(x, w, b, R, stride, relu):
    """NHWC convolution in 64 bits: x (n, H, W, C), w (R*R, C, O)."""
    n, H, W, C = x.shape
    p = R // 2
    xp = torch.zeros((n, H + 2 * p, W + 2 * p, C), dtype=torch.float64, device=x.device)
    xp[:, p:p + H, p:p + W] = x.double()
    Ho, Wo = (H + 2 * p - R) // stride + 1, (W + 2 * p - R) // stride + 1
    y = b.double().expand(n * Ho * Wo, -1).clone()
    for r in range(R):
        for s in range(R):
            v = xp[:, r:r + (Ho - 1) * stride + 1:stride, s:s + (Wo - 1) * stride + 1:stride]
            y.addmm_(v.reshape(-1, C).contiguous(), w[r * R + s].double().contiguous())
    y = y.reshape(n, Ho, Wo, -1)
    return y.clamp_(min=0) if relu else y


def _exact_fp8(x):
    """FP8 e4m3 values of a tensor under its per-tensor scale, and the scale."""
    a = x.abs().max()
    s = torch.tensor(448.0, device=x.device) / a
    return (x * s).clamp(-448.0, 448.0).to(torch.float8_e4m3fn), s


def exact(case, seed):
    kind = case["kind"]
    if kind == "gemm":
        vals = []
        for role in (0, 1):
            x, cols = _operand(case, seed, role)
            s = None
            if case["dtype"] == "bf16":
                x = x.bfloat16()
            elif case["dtype"] == "fp8":
                x, s = _exact_fp8(x)
            vals.append((x[:, :, :cols], s))
        (A, sa), (B, sb) = vals
        out = []
        for b in range(case["batch"]):
            a, w = A[b].double(), B[b].double()
            y = (a.t().contiguous() if case["ta"] else a.contiguous()) @ \
                (w.t().contiguous() if case["tb"] else w.contiguous())
            out.append(y / (sa.double() * sb.double()) if sa is not None else y)
        return torch.stack(out)
    if kind == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        x, w = _randn((M, K), _gen(2 * seed)), _randn((N, K), _gen(2 * seed + 1), 1.0 / math.sqrt(K))
        if case["dtype"] == "bf16":
            return {"y": x.bfloat16().double() @ w.bfloat16().double().t().contiguous(), "x": None}
        (xq, sx), (wq, sw) = _exact_fp8(x), _exact_fp8(w)
        y = xq.double() @ wq.double().t().contiguous()
        return {"y": y / (sx.double() * sw.double()), "x": None, "scale": 448.0 / x.double().abs().max().reshape(1)}
    if kind == "grouped":
        oa, ob, oc, ld, _, _, nc = _group_layout(case)
        A, B = _group_values(case, seed)
        C = torch.zeros(nc, dtype=torch.float64, device="cuda")
        for i, (M, N, K) in enumerate(_group_shapes(case)):
            a = A[oa[i]:oa[i] + M * ld[i][0]].reshape(M, -1)[:, :K].double().contiguous()
            b = B[ob[i]:ob[i] + K * ld[i][1]].reshape(K, -1)[:, :N].double().contiguous()
            C[oc[i]:oc[i] + M * N] = (a @ b).reshape(-1)
        return C
    if kind == "conv":
        x, w, b = _conv_values(case, seed)
        return _exact_conv(x, w, b, case["R"], case["stride"], True)
    if kind == "vgg16":
        x, wb = _vgg_values(seed)
        x, li = x.double()[None], 0
        for lk, cs in _vgg_layers():
            if lk == "pool":
                n, H, W, C = x.shape
                x = x.reshape(n, H // 2, 2, W // 2, 2, C).amax(dim=(2, 4))
                continue
            w, b = wb[li]
            li += 1
            x = _exact_conv(x.reshape(1, cs.H, cs.W, cs.Cin), w, b, cs.R, 1, li < len(wb))
        return x.reshape(-1)
    return None   # whole numbers; or weights after thousands of Adam steps, which diverge by rounding alone
