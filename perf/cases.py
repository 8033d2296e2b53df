"""The calls whose speed matters to a user of this library, as measurable cases.

A case is one pass through the public entry points of ``paper_2304_09049_amd.binding`` on operands that the caller holds
on the GPU: packed weights, the table, the run-time activations (float32 values, codes one per byte, or packed codes) and
buffers for the result.  The kinds:

  conv    one quantised convolution                   gemm    one quantised matrix product
  block   a residual block's three convolutions: quantise + pack, two layers that hand packed codes on, a last one to
          float32 (the encoding, the layers and the decoding of one network block)

Sizes are those of ResNet-18 / ResNet-50 / VGG-16 layers, of the benchmark GEMMs, and generic ones around them.
"""
from __future__ import annotations

import random

import numpy as np
import torch

from paper_2304_09049_amd import binding as dg
from paper_2304_09049_amd import workloads as wl

MAX_OPS = 1.1e12          # the largest listed case, in operations (two per product)


def _conv(name, B, H, W, Cin, Cout, k, stride=1, **kw):
    """A convolution with a k x k window, padded to keep the image's size at stride 1."""
    case = dict(name=name, kind="conv", B=B, H=H, W=W, Cin=Cin, Cout=Cout, k=k, stride=stride, bits=2, levels="fixed",
                input="codes", scale=False, skew=False)
    case.update(kw)
    return case


def _gemm(name, M, N, K, **kw):
    case = dict(name=name, kind="gemm", M=M, N=N, K=K, bits=2, levels="fixed", input="codes", scale=False, skew=False)
    case.update(kw)
    return case


def listed():
    return [
        # the smallest call: one small matrix product from codes, where launches and the host count
        _gemm("gemm_small", 64, 196, 576),
        # a ResNet-18 layer for one image, with the per-channel scale (latency of a single-image inference)
        _conv("conv3x3_b1", 1, 56, 56, 64, 64, 3, scale=True),
        # a ResNet-50 bottleneck's reducing layer for a batch, codes skewed as after a ReLU: bound by memory
        _conv("conv1x1_b32", 32, 56, 56, 256, 64, 1, skew=True),
        # a VGG-16 layer for a batch: bound by arithmetic
        _conv("conv3x3_b16", 16, 56, 56, 256, 256, 3),
        # a linear layer for one token, from float32 activations to float32 results (decode): the weights stream once
        _gemm("linear_decode", 8192, 1, 8192, levels="random_int8", input="float", scale=True),
        # the same layer for a chunk of a prompt (prefill)
        _gemm("linear_prefill", 8192, 256, 8192, levels="random_int8", input="float", scale=True),
        # the largest: a square matrix product on packed operands, int32 sums
        _gemm("gemm_square", 8192, 8192, 8192, levels="random_int8", input="packed"),
        # a ResNet-50 bottleneck block, packed codes between its layers
        dict(name="block_b8", kind="block", B=8, H=28, W=28, C=512, mid=128, dequant=False),
        # 4-bit codes (a 256-entry table)
        _conv("conv3x3_4bit", 8, 28, 28, 128, 128, 3, bits=4, scale=True),
        # non-uniform 8-bit levels, whose products need 16-bit table entries
        _conv("conv3x3_wide", 8, 28, 28, 256, 256, 3, levels="wide", scale=True),
        # channel counts that are no multiple of 32, as in networks with many narrow branches, and an odd image
        _conv("conv5x5_ragged", 8, 29, 27, 48, 120, 5, scale=True),
        # floating-point levels (non-uniform quantisation): a table of binary32 products
        _conv("conv3x3_f32", 4, 28, 28, 128, 128, 3, levels="f32", scale=True),
    ]


def _log(rng, lo, hi):
    """An integer from lo to hi, spread over the logarithm."""
    return int(round(np.exp(rng.uniform(np.log(lo), np.log(hi)))))


def _multiple(rng, lo, hi, of):
    return max(1, round(_log(rng, lo, hi) / of)) * of


def _draw_conv(rng, B, most, **kw):
    """A convolution of the networks' range: the image shrinks as the channels grow; every fourth one has an odd image."""
    while True:
        side = rng.choice((7, 14, 28, 56, 56, 112))
        H, W = (side, side) if rng.random() < 0.75 else (side + rng.randint(-2, 9), side + rng.randint(-2, 9))
        case = _conv("", _log(rng, *B), H, W, _multiple(rng, 64, min(2048, 14336 // side), 64),
                     _multiple(rng, 32, min(2048, 14336 // side), 8), rng.choice((1, 1, 3, 3)), rng.choice((1, 1, 1, 2)),
                     scale=rng.random() < 0.5, **kw)
        if 1e6 < work(case)["flops"] <= most and work(case)["bytes"] < 1.5e9:
            return case


def draw(rng: random.Random):
    family = rng.choice(("small", "conv_few", "conv_many", "linear", "square", "block", "bits", "wide", "ragged", "f32"))
    if family == "small":
        case = _gemm("", _log(rng, 16, 512), _log(rng, 8, 1024), _multiple(rng, 64, 1536, rng.choice((32, 32, 16, 64))),
                     scale=rng.random() < 0.3)
    elif family == "conv_few":
        case = _draw_conv(rng, (1, 4), 1e10)
    elif family == "conv_many":
        case = _draw_conv(rng, (8, 32), 2e11, skew=rng.random() < 0.5)
    elif family == "linear":
        case = _gemm("", _multiple(rng, 512, 8192, 8), _log(rng, 1, 512), _multiple(rng, 512, 8192, 128), levels="random_int8",
                     input="float", scale=True)
    elif family == "square":
        case = _gemm("", _log(rng, 256, 8192), _log(rng, 256, 8192), _multiple(rng, 256, 8192, 64), levels="random_int8",
                     input="packed", scale=rng.random() < 0.3)
    elif family == "block":
        side = rng.choice((7, 14, 28, 56))
        mid = rng.choice((32, 64, 96, 128)) * max(1, 28 // side)
        case = dict(kind="block", B=_log(rng, 1, 32), H=side, W=side + rng.randint(0, 3), C=4 * mid, mid=mid,
                    dequant=rng.random() < 0.5)
    elif family == "bits":
        case = _draw_conv(rng, (1, 16), 3e10, bits=rng.choice((3, 4)))
    elif family == "wide":
        case = _draw_conv(rng, (1, 16), 6e10, levels="wide")
    elif family == "ragged":
        while True:
            side = rng.choice((7, 14, 28, 56))
            case = _conv("", _log(rng, 1, 16), side + rng.randint(0, 3), side + rng.randint(0, 3),
                         _multiple(rng, 16, 528, rng.choice((4, 8, 16, 16))), _multiple(rng, 16, 384, 4), rng.choice((1, 3, 5)),
                         rng.choice((1, 1, 2)), scale=rng.random() < 0.5)
            if case["Cin"] % 32 and 1e6 < work(case)["flops"] <= 4e9:
                break
    else:
        while True:
            case = _draw_conv(rng, (1, 8), 3e9, levels="f32")
            case["Cin"] = _multiple(rng, 16, case["Cin"], 4)
            if work(case)["flops"] > 1e6:
                break
    case.pop("name", None)
    return case


def _convs(case):
    """The convolutions of a case as (H, W, Cin, Cout, k, stride)."""
    if case["kind"] == "block":
        H, W, C, mid = case["H"], case["W"], case["C"], case["mid"]
        return [(H, W, C, mid, 1, 1), (H, W, mid, mid, 3, 1), (H, W, mid, C, 1, 1)]
    return [(case["H"], case["W"], case["Cin"], case["Cout"], case["k"], case["stride"])]


def _out(size, k, stride):
    return (size + 2 * (k // 2) - k) // stride + 1


def work(case):
    """Every input read once in the form in which the caller has it, every output written once; two operations a product."""
    if case["kind"] == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        per_weight = 0.25 if case["bits"] == 2 else 0.5
        per_input = {"codes": 1.0, "packed": per_weight, "float": 4.0}[case["input"]]
        return {"bytes": M * K * per_weight + N * K * per_input + 4.0 * M * N + (4.0 * M if case["scale"] else 0.0),
                "flops": 2.0 * M * N * K}
    B, nbytes, flops = case["B"], 0.0, 0.0
    convs = _convs(case)
    for H, W, Cin, Cout, k, stride in convs:
        pixels = B * _out(H, k, stride) * _out(W, k, stride)
        nbytes += Cout * k * k * Cin * (0.25 if case.get("bits", 2) == 2 else 0.5) + 4.0 * Cout
        flops += 2.0 * Cout * pixels * k * k * Cin
    H, W, Cin = convs[0][:3]
    nbytes += B * H * W * Cin * (4.0 if case["kind"] == "block" else 1.0) + 4.0 * pixels * Cout
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Sums are whole numbers, and the float32 ones are defined operation by operation (one conversion and one multiply for
    the scale; a table of binary32 products is summed one addition at a time in ascending k): nothing may differ."""
    return "exact"


def _table(case, rng):
    bits, levels = case.get("bits", 2), case.get("levels", "symmetric")
    if levels == "symmetric":    # weights without a mean, so that codes handed from layer to layer keep their spread
        return dg.dg_build_lut((-3, -1, 1, 3), wl.LEVELS_A_UNSIGNED)
    if levels == "f32":          # the centres of a normal distribution's quarters, and those of a positive one
        lw = [float(np.float32(v * rng.uniform(0.9, 1.1))) for v in (-1.27, -0.32, 0.32, 1.27)]
        la = [float(np.float32(v * rng.uniform(0.9, 1.1))) for v in (0.05, 0.45, 0.98, 1.78)]
        return dg.dg_build_lut_f32(lw, la)
    if levels == "wide":         # levels spread as powers of two
        lw = [-rng.randint(32, 64), -rng.randint(4, 12), rng.randint(4, 12), rng.randint(32, 64)]
        la = [0, rng.randint(4, 12), rng.randint(16, 40), rng.randint(64, 127)]
        return dg.dg_build_lut(lw, la, dg.DG_LUT_I16)
    if levels == "random_int8":  # the benchmark's large products: 4 + 4 levels in -8 ... 7, a table of 16-bit entries
        return dg.dg_build_lut([rng.randint(-8, 7) for _ in range(4)], [rng.randint(-8, 7) for _ in range(4)], dg.DG_LUT_I16)
    if bits == 2:
        return dg.dg_build_lut(wl.LEVELS_W_SIGNED, wl.LEVELS_A_UNSIGNED)
    n = 1 << bits
    return dg.dg_build_lut_bits(bits, list(range(-n // 2, n // 2)), list(range(n)))


def _codes(gen, count, bits=2, skew=False):
    if skew:                     # code 0 with probability 1/2, the others with 1/6 each
        r = torch.randint(0, 6, (count,), dtype=torch.uint8, device="cuda", generator=gen)
        return torch.where(r < 3, torch.zeros_like(r), r - 2)
    return torch.randint(0, 1 << bits, (count,), dtype=torch.uint8, device="cuda", generator=gen)


def _pack(codes, rows, K, bits):
    return dg.dg_pack_activations(codes, rows, K) if bits == 2 else dg.dg_pack_codes_bits(codes, rows, K, bits)


def _scales(gen, count, reach):
    """Per-channel scales that take sums of `reach` positions to the order of one."""
    return (0.01 + 0.09 * torch.rand(count, device="cuda", generator=gen)) * (24.0 / reach) ** 0.5


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rng = random.Random(seed)
    state = {"kind": case["kind"], "lut": _table(case, rng)}
    bits = case.get("bits", 2)
    if case["kind"] == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        state.update(input=case["input"], M=M, N=N, K=K, Wp=_pack(_codes(gen, M * K, bits), M, K, bits),
                     scale=_scales(gen, M, K) if case["scale"] else None)
        dtype = torch.float32 if case["scale"] else torch.int32
        if case["input"] == "float":       # a linear layer: [N][K] in, [N][M] out
            state.update(x=torch.randn(N, K, device="cuda", generator=gen), strides=(1, M),
                         out=torch.empty(N, M, dtype=dtype, device="cuda"))
        else:
            state.update(x=_codes(gen, N * K, bits, case["skew"]), strides=None, out=torch.empty(M, N, dtype=dtype, device="cuda"))
            if case["input"] == "packed":
                state["x"] = _pack(state["x"], N, K, bits)
        state["work"] = torch.empty(dg.dg_packed_bytes_bits(N, K, bits), dtype=torch.uint8, device="cuda")
        return state
    B, layers = case["B"], []
    for H, W, Cin, Cout, k, stride in _convs(case):
        OH, OW, K = _out(H, k, stride), _out(W, k, stride), k * k * Cin
        layers.append(dict(desc=dg.conv_desc(B, H, W, Cin, Cout, k, k, (stride, stride), (k // 2, k // 2)), shape=(B, OH, OW, Cout),
                           Wp=_pack(_codes(gen, Cout * K, bits), Cout, K, bits), scale=_scales(gen, Cout, K),
                           packed=torch.empty(dg.dg_packed_bytes_bits(B * H * W, Cin, bits), dtype=torch.uint8, device="cuda")))
    state["layers"] = layers
    last = layers[-1]
    if case["kind"] == "block":
        state.update(x=torch.randn(B, case["H"], case["W"], case["C"], device="cuda", generator=gen), dequant=case["dequant"],
                     sums=torch.empty(last["shape"], dtype=torch.int32, device="cuda") if case["dequant"] else None,
                     out=torch.empty(last["shape"], dtype=torch.float32, device="cuda"))
    else:
        as_float = case["scale"] or case["levels"] == "f32"
        state.update(x=_codes(gen, B * case["H"] * case["W"] * case["Cin"], bits, case["skew"]),
                     out=torch.empty(last["shape"], dtype=torch.float32 if as_float else torch.int32, device="cuda"))
        if not case["scale"]:
            last["scale"] = None
    return state


def run(state):
    lut = state["lut"]
    if state["kind"] == "conv":
        layer = state["layers"][0]
        return dg.dg_conv2d_lut_codes(lut, layer["Wp"], state["x"], layer["desc"], work=layer["packed"], out=state["out"],
                                      scale=layer["scale"])
    if state["kind"] == "gemm":
        M, N, K = state["M"], state["N"], state["K"]
        if state["input"] == "codes":
            return dg.dg_gemm_lut_codes(lut, state["Wp"], state["x"], M, N, K, work=state["work"], out=state["out"],
                                        scale=state["scale"])
        packed = state["x"]
        if state["input"] == "float":
            packed = dg.dg_quantize_pack_activations(state["x"], N, K, 1.5, 1.5, 0, out=state["work"])
        return dg.dg_gemm_lut(lut, state["Wp"], packed, M, N, K, out=state["out"], scale=state["scale"], strides=state["strides"])
    first, second, third = state["layers"]
    d = first["desc"]
    dg.dg_quantize_pack_activations(state["x"], d.B * d.H * d.W, d.Cin, 1.5, 1.5, 0, out=first["packed"])
    dg.dg_conv2d_lut_requant(lut, first["Wp"], first["packed"], d, first["scale"], 1.5, 1.5, 0, out=second["packed"])
    dg.dg_conv2d_lut_requant(lut, second["Wp"], second["packed"], second["desc"], second["scale"], 1.5, 1.5, 0,
                             out=third["packed"])
    if not state["dequant"]:
        dg.dg_conv2d_lut(lut, third["Wp"], third["packed"], third["desc"], out=state["out"], scale=third["scale"])
    else:                        # the sums themselves are wanted too
        dg.dg_conv2d_lut(lut, third["Wp"], third["packed"], third["desc"], out=state["sums"])
        dg.dg_dequantize(state["sums"], d.B * d.H * d.W, third["desc"].Cout, third["scale"], out=state["out"])
    return [second["packed"], third["packed"], state["out"]]
