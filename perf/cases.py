"""What a user of this library has it do, as cases that can be timed: layers of the pruned networks
that the workload configurations are made of, from one image to a full batch, in every data type,
through the C ABI (binding.Plan).

A case is one convolution layer (or the 13-layer quantised VGG-16-shaped stack as one chain of
calls).  prepare() makes what a program holds before the call: the plan, made from seeded weights,
with a launch shape that the library's own search chose for this layer (a program searches once per
layer and installs the result for every plan of that layer, which is what _SHAPES is), the input and
the output buffer on the GPU.  run() is the forward pass.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2112_15445_amd import binding as B
from paper_2112_15445_amd import workloads as W

_X = {"f32": torch.float32, "f16": torch.float16, "cb4h": torch.float16, "i8": torch.int8, "cb4": torch.int8}


def _layer_case(name, C, D, H, W_, R, S, stride, pad, N, sparsity, dtype, ragged=False, search=True, relu=False, pool=0):
    c = dict(kind="layer", C=C, D=D, H=H, W=W_, R=R, S=S, stride=stride, pad_h=pad if R > 1 else 0, pad_w=pad if S > 1 else 0,
             N=N, sparsity=sparsity, dtype=dtype, ragged=ragged, search=search, relu=relu, pool=pool)
    if name:
        c["name"] = name
    return c


def listed():
    L = _layer_case
    return [
        # one image through one layer: an interactive request, bound by launches and latency
        L("f32 3x3 64-64 @32 b1", 64, 64, 32, 32, 3, 3, 1, 1, 1, 0.90, "f32"),
        # ResNet-50 stage 1, the layer with the most traffic: fp32 pointwise, a full batch
        L("f32 1x1 256-64 @56 b32", 256, 64, 56, 56, 1, 1, 1, 0, 32, 0.90, "f32"),
        # ResNet-50 stage 2, the 3x3 of the block at moderate sparsity: most arithmetic in fp32
        L("f32 3x3 128-128 @28 b32", 128, 128, 28, 28, 3, 3, 1, 1, 32, 0.80, "f32"),
        # ResNet-50 stage 4, first block: strided, deep, few positions
        L("f32 3x3s2 512-512 @14 b32", 512, 512, 14, 14, 3, 3, 2, 1, 32, 0.90, "f32"),
        # ResNet-50 stage 4, deep pointwise on 7x7 planes (rows of 49 values: nothing is aligned)
        L("f32 1x1 2048-512 @7 b32", 2048, 512, 7, 7, 1, 1, 1, 0, 32, 0.80, "f32"),
        # the 1-D convolution of text models: 300 channels along a sequence of 64
        L("f32 1d k3 300-64 @64 b128", 300, 64, 1, 64, 1, 3, 1, 0, 128, 0.83, "f32"),
        # a layer of no round size, rows of unequal length, an odd batch
        L("f32 3x3 100-90 @27x31 b7", 100, 90, 27, 31, 3, 3, 1, 1, 7, 0.85, "f32", ragged=True),
        # ResNet-50 in half precision: the stage 1 3x3 and the stage 2 expand layer
        L("f16 3x3 64-64 @56 b32", 64, 64, 56, 56, 3, 3, 1, 1, 32, 0.80, "f16"),
        L("f16 1x1 128-512 @28 b32", 128, 512, 28, 28, 1, 1, 1, 0, 32, 0.70, "f16"),
        # a program that makes its plans on the fly and does not pay for a search
        L("f16 3x3 256-256 @14 b32 def", 256, 256, 14, 14, 3, 3, 1, 1, 32, 0.80, "f16", search=False),
        # the 4b/16b quantisation on a deep VGG-16 layer: 4x4 planes
        L("cb4h 3x3 512-512 @4 b64", 512, 512, 4, 4, 3, 3, 1, 1, 64, 0.90, "cb4h"),
        # a whole quantised network: the 13 int8 VGG-16 layers, each with ReLU, pooling at the end of a
        # stage and requantisation to the codes that the next layer reads
        dict(name="i8 vgg16 stack b64", kind="stack", N=64, sparsity=0.90, dtype="i8"),
    ]


def _dims(c):
    P = (c["H"] + 2 * c["pad_h"] - c["R"]) // c["stride"] + 1
    Q = (c["W"] + 2 * c["pad_w"] - c["S"]) // (c["stride"] if c["S"] > 1 else 1) + 1
    return P, Q


def draw(rng):
    """One more layer of the same ranges: channels, planes, batches, sparsities and types of the workload
    configurations, with odd sizes between them; at most the work of the largest listed layer."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        shape = rng.choice(["3x3", "3x3", "3x3s2", "1x1", "1x1", "1d"])
        dtype = rng.choice(["f32", "f32", "f32", "f16", "f16", "i8", "cb4", "cb4h"])
        even = rng.random() < 0.5                       # half of them channel counts and planes of round size
        ch = (lambda lo, hi: 8 * max(1, log_int(lo, hi) // 8)) if even else log_int
        C, D = ch(16, 2048 if shape == "1x1" else 512), ch(16, 1024 if shape == "1x1" else 512)
        N = log_int(1, 64)
        sp = round(rng.uniform(0.70 if dtype == "f32" else 0.50, 0.95), 3)
        if shape == "1d":
            k = rng.choice([2, 3, 5])
            H, W_, R, S, stride, pad = 1, log_int(16, 128), 1, k, 1, 0
        else:
            hw = log_int(4, 56)
            H, W_ = hw, hw if rng.random() < 0.7 else max(3, hw + rng.randint(-3, 3))
            R = S = 1 if shape == "1x1" else 3
            stride, pad = (2 if shape == "3x3s2" else 1), (0 if shape == "1x1" else 1)
        epi = dtype != "f32" and shape == "3x3" and rng.random() < 0.25
        c = _layer_case(None, C, D, H, W_, R, S, stride, pad, N, sp, dtype, ragged=rng.random() < 0.2, relu=epi, pool=2 if epi else 0)
        P, Q = _dims(c)
        macs = N * D * P * Q * C * R * S
        if c["pool"] and (P < 4 or Q < 4):
            continue
        w = work(c)
        if 2e7 <= 2 * macs <= 7.4e9 and w["bytes"] <= 1.2e8 and w["flops"] <= 1.5e9:
            return c


# ---------------------------------------------------------------------------------------------
# weights and inputs from the seed
# ---------------------------------------------------------------------------------------------

def _wl(c):
    """The workload description of a layer case (its sizes, stored entries and byte counts)."""
    return W.Layer("case", c["C"], c["D"], c["H"], c["W"], c["R"], c["S"], c["stride"] if c["R"] > 1 else 1,
                   c["stride"] if c["S"] > 1 else 1, c["pad_h"], c["pad_w"], c["N"], c["sparsity"], c["dtype"])


def _stack(c):
    """The layers of the stack, and for each whether 2x2 max-pooling follows it."""
    ls = [W.Layer(f"vgg{i + 1}", ci, co, hw, hw, N=c["N"], sparsity=c["sparsity"], dtype=c["dtype"])
          for i, ((ci, co), hw) in enumerate(zip(W.VGG_WIDTHS, W.VGG_SPATIAL))]
    return [(l, 2 if i + 1 < len(ls) and 2 * ls[i + 1].H == l.H else 0) for i, l in enumerate(ls)]


def _draw_rows(l, rng, ragged):
    """CSR of seeded weights: n (ragged: 0.6 n .. n) random positions per output channel, N(0, 0.05)."""
    n, K, D = l.n, l.K, l.D
    lens = rng.integers(max(1, int(0.6 * n)), n + 1, size=D) if ragged else np.full(D, n)
    rank = np.argpartition(rng.random((D, K), dtype=np.float32), n - 1, axis=1)[:, :n]
    rowptr = np.zeros(D + 1, np.int32)
    rowptr[1:] = np.cumsum(lens)
    colidx = np.concatenate([np.sort(rank[d, :lens[d]]) for d in range(D)]).astype(np.int32)
    return rowptr, colidx, rng.normal(0.0, 0.05, size=colidx.size).astype(np.float32)


def _weights(l, rng, ragged=False):
    """(rowptr, colidx, values as the plan takes them, scales, codebook, values as numbers)"""
    rowptr, colidx, w = _draw_rows(l, rng, ragged)
    if l.dtype == "f32":
        return rowptr, colidx, w, None, None, w
    if l.dtype == "f16":
        h = w.astype(np.float16)
        return rowptr, colidx, h, None, None, h
    if l.dtype == "i8":
        q, sc = W.quantise_weights_int8(rowptr, w)
        return rowptr, colidx, q, sc, None, q
    cent, cb, sc = W.codebook16()
    idx = W.assign_codebook(w, cent)
    if l.dtype == "cb4":
        return rowptr, colidx, idx, np.full(l.D, sc, np.float32), cb, cb[idx]
    cbh = cent.astype(np.float16)
    return rowptr, colidx, idx, None, cbh, cbh[idx]


def _input(l, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 7 + 1)
    shape = (l.N, l.C, l.H, l.W)
    if l.dtype in ("i8", "cb4"):
        return torch.randint(-127, 128, shape, generator=g, device="cuda", dtype=torch.int8)
    return (torch.rand(shape, generator=g, device="cuda") * 2 - 1).to(_X[l.dtype])


def _requant_scale(k, l, values):
    """Multipliers that bring the accumulators of stack layer k to codes: a channel's standard deviation
    (uniform inputs for the first layer, the codes of the one before for the others) becomes 32."""
    rms_x = 73.0 if k == 0 else 27.0
    q = values.reshape(l.D, l.n).astype(np.float64)
    return (32.0 / (np.sqrt((q * q).sum(axis=1)) * rms_x)).astype(np.float32)


# ---------------------------------------------------------------------------------------------
# plans
# ---------------------------------------------------------------------------------------------

_SHAPES = {}      # launch shape found by the search, per layer: a program searches a layer once


def _plan(l, weights, N, x, relu=False, pool=0, requant=None, search=True, ragged=False):
    """(plan, output buffer, workspace)"""
    rowptr, colidx, values, scales, codebook, _ = weights
    layer = B.make_layer(l.C, l.D, l.H, l.W, l.R, l.S, (l.stride_h, l.stride_w), (l.pad_h, l.pad_w))
    plan = B.Plan.create_csr(layer, B.DTYPES[l.dtype], rowptr, colidx, values, scales, codebook)
    if relu or pool or requant is not None:
        plan.set_epilogue(relu=relu, pool=pool, requant_scale=requant)
    inf = plan.info()
    out = torch.int8 if requant is not None else B.torch_out_dtype(plan.dtype)
    y = torch.empty((N, l.D, inf.out_P, inf.out_Q), dtype=out, device="cuda")
    if search:
        key = (l, N, relu, pool, requant is not None, ragged)
        if key not in _SHAPES:
            ws = torch.empty(max(plan.workspace_size_max(N), 1), dtype=torch.uint8, device="cuda")
            st = torch.cuda.current_stream().cuda_stream
            plan.autotune(x.data_ptr(), y.data_ptr(), N, ws.data_ptr(), ws.numel(), st)
            _SHAPES[key] = plan.get_tuning()
        else:
            plan.set_tuning(_SHAPES[key])
    ws = torch.empty(max(plan.workspace_size(N), 1), dtype=torch.uint8, device="cuda")
    return plan, y, ws


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    if case["kind"] == "stack":
        steps = []
        x = _input(_stack(case)[0][0], seed)
        cur = x
        for k, (l, pool) in enumerate(_stack(case)):
            w = _weights(l, rng)
            plan, y, ws = _plan(l, w, l.N, cur, True, pool, _requant_scale(k, l, w[5]))
            steps.append((plan, cur, y, ws))
            cur = y
        return {"steps": steps}
    l = _wl(case)
    w = _weights(l, rng, case["ragged"])
    x = _input(l, seed)
    plan, y, ws = _plan(l, w, l.N, x, case["relu"], case["pool"], None, case["search"], case["ragged"])
    return {"steps": [(plan, x, y, ws)]}


def run(state):
    stream = torch.cuda.current_stream().cuda_stream
    for plan, x, y, ws in state["steps"]:
        plan.forward(x.data_ptr(), y.data_ptr(), x.shape[0], ws.data_ptr(), ws.numel(), stream)
    return y


# ---------------------------------------------------------------------------------------------
# what a pass cannot do without, how close two correct passes are, and the result in 64 bits
# ---------------------------------------------------------------------------------------------

def work(case):
    if case["kind"] == "stack":
        b = f = 0.0
        for l, pool in _stack(case):
            per = l.P * l.Q // (4 if pool else 1)
            b += l.N * (l.C * l.H * l.W + l.D * per) + l.D * (l.n * 5 + 8)
            f += 2.0 * l.useful_macs
        return {"bytes": b, "flops": f}
    l = _wl(case)
    ex, ey, ew = l.elem_sizes()
    out = (l.P // 2) * (l.Q // 2) if case["pool"] else l.P * l.Q
    b = l.N * (l.C * l.H * l.W * ex + l.D * out * ey) + l.D * l.n * (ew + 4)
    return {"bytes": float(b), "flops": 2.0 * l.useful_macs * (0.8 if case["ragged"] else 1.0)}


def tolerance(case):
    if case["dtype"] in ("i8", "cb4"):
        return "exact"                                   # int32 sums, and codes formed from them
    if case["dtype"] == "f32":
        return {"rel": 1e-6, "max": 1e-5}                # 32-bit sums in another order
    return {"rel": 1e-4, "max": 2e-3}                    # fp32 sums in another order, then one rounding to fp16


def _conv64(x, l, rowptr, colidx, numbers):
    """The layer as the dense convolution of its weights, in 64 bits, one filter tap at a time."""
    dense = np.zeros((l.D, l.K))
    dense[np.repeat(np.arange(l.D), np.diff(rowptr)), colidx] = numbers.astype(np.float64)
    wt = torch.from_numpy(dense).cuda().view(l.D, l.C, l.R, l.S)
    xp = torch.nn.functional.pad(x.double(), (l.pad_w, l.pad_w, l.pad_h, l.pad_h))
    y = torch.zeros(l.N, l.D, l.P * l.Q, dtype=torch.float64, device="cuda")
    for r in range(l.R):
        for s in range(l.S):
            tap = xp[:, :, r:r + (l.P - 1) * l.stride_h + 1:l.stride_h, s:s + (l.Q - 1) * l.stride_w + 1:l.stride_w]
            y += torch.matmul(wt[:, :, r, s].contiguous(), tap.reshape(l.N, l.C, -1).contiguous())
    return y.view(l.N, l.D, l.P, l.Q)


def _pool64(y, relu, pool):
    if relu:
        y = y.clamp_min(0)
    if pool:
        P, Q = y.shape[2] // 2, y.shape[3] // 2
        y = y[:, :, :2 * P, :2 * Q].reshape(y.shape[0], y.shape[1], P, 2, Q, 2).amax(dim=(3, 5))
    return y


def exact(case, seed):
    rng = np.random.default_rng(seed)
    if case["kind"] == "stack":
        x = _input(_stack(case)[0][0], seed)
        for k, (l, pool) in enumerate(_stack(case)):
            rowptr, colidx, _, _, _, numbers = _weights(l, rng)
            y = _pool64(_conv64(x, l, rowptr, colidx, numbers), True, pool)
            # the code of an integer sum: three single-precision steps (convert, multiply, round)
            scale = torch.from_numpy(_requant_scale(k, l, numbers)).cuda().view(1, -1, 1, 1)
            x = (y.to(torch.int32).float() * scale).round().clamp(-127, 127).to(torch.int8)
        return x
    l = _wl(case)
    rowptr, colidx, _, _, _, numbers = _weights(l, rng, case["ragged"])
    y = _pool64(_conv64(_input(l, seed), l, rowptr, colidx, numbers), case["relu"], case["pool"])
    return y.round().to(torch.int32) if case["dtype"] in ("i8", "cb4") else y
