"""The calls this library is used for, as a fixed list of timed cases.

A case is one pass of the kind of work a program that serves low-bit LLMs hands to the library, at the layer shapes of
the benchmark models (a 7B and a 3.8B decoder, a 2B ternary model), through the Python binding:

  call          what one pass does
  x             one GEMV for one token, ``tman_mpgemv_x``
  x_batch       one token through ``layers`` decoder layers, one ``tman_mpgemv_x_batch_run`` launch per layer
  lut_batch     ``N`` tokens through ``layers`` layers: ``tman_build_lut_batch`` + ``tman_mpgemv_batch_run`` per layer
  i16_batch     the same with integer activations: ``tman_build_lut_i16_batch`` + ``tman_mpgemv_i16_batch_run``
  small_batch   ``N`` tokens (2..32) through ``layers`` layers, one ``tman_mpgemm_batch_run`` launch per layer
  gemm          one linear layer over a prompt of ``N`` tokens, ``tman_mpgemm``
  i8            the same for one (scale, zero) per row: ``tman_quantize_act_i8`` + ``tman_mpgemm_i8``
  pack          one linear layer's weights into the packed form at load time, ``tman_pack_weights``

The layered calls take a decoder layer's five GEMVs (QKV fused, O, gate, up, down) of model width ``hidden`` and MLP
width ``inter``; the others one M x K matrix.
"""
from __future__ import annotations

import math

import torch

import paper_2511_11248_amd as tman

LAYERED = ("x_batch", "lut_batch", "i16_batch", "small_batch")


def listed():
    return [
        # the smallest call: one token through one small projection (latency of the call and of the launch)
        dict(name="x_256x512_w4g64", call="x", bits=4, group=64, zero=True, N=1, M=256, K=512, outliers=False),
        # decode of one token, the whole linear stack of a 7B decoder with 2-bit weights (the headline benchmark)
        dict(name="decode1_7b_w2g64", call="x_batch", bits=2, group=64, zero=True, N=1, hidden=4096, inter=11008, layers=32,
             outliers=False),
        # the same with 4-bit weights and activations that have outlier channels; the largest decode stream
        dict(name="decode1_7b_w4g128", call="x_batch", bits=4, group=128, zero=True, N=1, hidden=4096, inter=11008,
             layers=32, outliers=True),
        # decode of one token of a 3.8B model with 1-bit sign weights
        dict(name="decode1_3p8b_w1g64", call="x_batch", bits=1, group=64, zero=False, N=1, hidden=3072, inter=8192,
             layers=32, outliers=False),
        # four sequences decoded together, through the shared lookup tables
        dict(name="decode4_7b_w4g128", call="lut_batch", bits=4, group=128, zero=True, N=4, hidden=4096, inter=11008,
             layers=8, outliers=True),
        # integer activations and integer tables, one token
        dict(name="decode1_7b_w4g128_i16", call="i16_batch", bits=4, group=128, zero=True, N=1, hidden=4096,
             inter=11008, layers=8, outliers=True),
        # eight sequences (or eight speculated tokens) decoded together on the matrix cores
        dict(name="decode8_7b_w4g128", call="small_batch", bits=4, group=128, zero=True, N=8, hidden=4096, inter=11008,
             layers=8, outliers=True),
        # prefill of a 1024-token prompt, the MLP up projection
        dict(name="prefill1024_11008x4096_w4g64", call="gemm", bits=4, group=64, zero=True, N=1024, M=11008, K=4096,
             outliers=False),
        # a long prompt, 2-bit weights, the fused QKV projection
        dict(name="prefill2048_12288x4096_w2g64", call="gemm", bits=2, group=64, zero=True, N=2048, M=12288, K=4096,
             outliers=False),
        # a short prompt of odd length through the down projection
        dict(name="prefill173_4096x11008_w4g128", call="gemm", bits=4, group=128, zero=True, N=173, M=4096, K=11008,
             outliers=False),
        # ternary weights with one scale, int8 activations: prefill of a 2B ternary model's up projection
        dict(name="i8_prefill1024_6912x2560_w2", call="i8", bits=2, group=128, zero=True, N=1024, M=6912, K=2560,
             outliers=False),
        # loading a model: one linear layer's codes, scales and zeros into the packed form
        dict(name="pack_11008x4096_w4g64", call="pack", bits=4, group=64, zero=True, N=1, M=11008, K=4096,
             outliers=False),
    ]


def _spread(rng, lo, hi, step=1):
    """A multiple of ``step`` in [lo, hi], spread over its logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(max(int(round(v / step)), -(-lo // step)), hi // step) * step


def draw(rng):
    call = rng.choice(["x", "x_batch", "lut_batch", "i16_batch", "small_batch", "gemm", "gemm", "i8", "pack"])
    bits = rng.choice([1, 2, 2, 4, 4, 4])
    group = rng.choice([32, 64, 64, 128, 128])
    case = dict(call=call, bits=bits, group=group, zero=bits > 1 or rng.random() < 0.5, outliers=rng.random() < 0.5)
    if call in LAYERED:
        hidden = _spread(rng, 1024, 4096, group)
        case.update(hidden=hidden, inter=_spread(rng, 2 * hidden, min(11008, 4 * hidden), group),
                    layers=rng.randint(8, 32) if call == "x_batch" else rng.randint(4, 8),
                    N={"x_batch": 1, "lut_batch": rng.randint(1, 8), "i16_batch": rng.randint(1, 8),
                       "small_batch": rng.randint(2, 32)}[call])
        return case
    K = _spread(rng, 512, 11008, group)
    M = _spread(rng, 256, 12288) if rng.random() < 0.5 else _spread(rng, 256, 12288, 64)
    if call in ("gemm", "i8"):
        case.update(N=_spread(rng, 33, 2048))
        if call == "i8":
            case.update(outliers=False)
        while case["N"] * M * K > 2048 * 12288 * 4096:
            M //= 2
    else:
        case.update(N=1)
    case.update(M=M, K=K)
    return case


def _matrices(case):
    """(M, K, which activation) of each matrix of a layer."""
    if case["call"] in LAYERED:
        h, i = case["hidden"], case["inter"]
        return [(3 * h, h, 0), (h, h, 1), (i, h, 2), (i, h, 2), (h, i, 3)]
    return [(case["M"], case["K"], 0)]


def _inputs(case, seed):
    """Codes, scales and zeros of every matrix and the activations, layer by layer, made from the seed on the GPU:
    uniform codes, scales U(0.005, 0.02), zeros in the middle of the code range, standard normal activations (with
    ``outliers`` 1 % of the channels 20 times as large).  ``i8``: ternary codes with zero 1 and one scale for 2 bits,
    otherwise one scale and zero per row."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    bits, group, N = case["bits"], case["group"], case["N"]
    zero_range = {1: (0.0, 1.0), 2: (1.0, 2.0), 4: (6.0, 9.0)}[bits]

    def uniform(shape, lo, hi):
        return (torch.rand(shape, generator=gen, device=dev) * (hi - lo) + lo).half()

    for _ in range(case.get("layers", 1)):
        weights, acts = [], {}
        for M, K, a in _matrices(case):
            G = K // group
            levels = 3 if case["call"] == "i8" and bits == 2 else 1 << bits
            codes = torch.randint(0, levels, (M, K), generator=gen, device=dev, dtype=torch.uint8)
            if case["call"] == "i8":
                scales = uniform((1, 1) if bits == 2 else (M, 1), 0.005, 0.02).expand(M, G).contiguous()
                zeros = torch.ones((M, G), device=dev, dtype=torch.float16) if bits == 2 else uniform(
                    (M, 1), *zero_range).expand(M, G).contiguous()
            else:
                scales, zeros = uniform((M, G), 0.005, 0.02), uniform((M, G), *zero_range)
            weights.append((codes, scales, zeros if case["zero"] else None))
            if a not in acts:
                x = torch.randn((N, K), generator=gen, device=dev)
                if case["outliers"]:
                    channels = torch.randperm(K, generator=gen, device=dev)[:math.ceil(0.01 * K)]
                    x[:, channels] *= 20.0
                acts[a] = x.half()
        yield weights, acts


def _buffer(n, zeroed=False):
    return (torch.zeros if zeroed else torch.empty)(max(1, n), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    call, N, group = case["call"], case["N"], case["group"]
    mats = _matrices(case)
    shapes = [tman.Shape(M, K, case["bits"], group, case["zero"]) for M, K, _ in mats]
    if call == "pack":
        (codes, scales, zeros), = next(_inputs(case, seed))[0]
        return dict(case=case, shape=shapes[0], codes=codes, scales=scales, zeros=zeros,
                    packed=_buffer(tman.tman_packed_bytes(shapes[0])))
    steps, outputs, keep = [], [], []
    for weights, acts in _inputs(case, seed):
        packed = []
        for shape, (codes, scales, zeros) in zip(shapes, weights):
            blob = _buffer(tman.tman_packed_bytes(shape))
            tman.tman_pack_weights(shape, codes, scales, zeros, blob)
            packed.append(blob)
        flat = torch.empty(N * sum(M for M, _, _ in mats), dtype=torch.float16, device="cuda")
        y = [part.view(N, -1) for part in flat.split([N * M for M, _, _ in mats])]
        query = tman.tman_mpgemm_workspace_bytes if call in ("gemm", "small_batch") else tman.tman_mpgemv_workspace_bytes
        ws = [_buffer(query(s, N), zeroed=True) for s in shapes] if call != "i8" else [None]
        xs = [acts[a] for _, _, a in mats]
        outputs.append(flat)
        keep.append((packed, ws, acts))
        if call not in LAYERED:
            state = dict(case=case, shape=shapes[0], packed=packed[0], x=xs[0], y=y[0], ws=ws[0])
            if call == "i8":
                state["xq"] = _buffer(tman.tman_act_i8_bytes(N, case["K"]))
            return state
        desc = _buffer(tman.tman_mpgemv_batch_desc_bytes(len(shapes)))
        keep.append(desc)
        if call == "x_batch":
            tman.tman_mpgemv_x_batch_prepare(shapes, packed, xs, y, ws, desc)
            steps.append(tman.bound_mpgemv_x_batch_run(shapes, desc))
        elif call == "small_batch":
            tman.tman_mpgemm_batch_prepare(shapes, packed, xs, N, y, ws, desc)
            steps.append(tman.bound_mpgemm_batch_run(shapes, N, desc))
        else:
            integer = call == "i16_batch"
            lut_bytes = tman.tman_lut_i16_bytes if integer else tman.tman_lut_bytes
            order = sorted(acts)
            Ks = [acts[a].shape[1] for a in order]
            luts = {a: _buffer(lut_bytes(N, K, group)) for a, K in zip(order, Ks)}
            keep.append(luts)
            tman.tman_mpgemv_batch_prepare(shapes, packed, [luts[a] for _, _, a in mats], N, y, ws, desc)
            build = tman.bound_build_lut_i16_batch if integer else tman.bound_build_lut_batch
            steps.append(build([acts[a] for a in order], N, Ks, group, [luts[a] for a in order]))
            steps.append((tman.bound_mpgemv_i16_batch_run if integer else tman.bound_mpgemv_batch_run)(shapes, N, desc))
    return dict(case=case, steps=steps, outputs=outputs, keep=keep)


def run(state):
    call, N = state["case"]["call"], state["case"]["N"]
    if call in LAYERED:
        stream = torch.cuda.current_stream().cuda_stream
        for step in state["steps"]:
            step(stream)
        return state["outputs"]
    if call == "pack":
        tman.tman_pack_weights(state["shape"], state["codes"], state["scales"], state["zeros"], state["packed"])
        return state["packed"]
    if call == "x":
        tman.tman_mpgemv_x(state["shape"], state["packed"], state["x"], state["y"], state["ws"])
    elif call == "gemm":
        tman.tman_mpgemm(state["shape"], state["packed"], state["x"], N, state["y"], state["ws"])
    else:
        tman.tman_quantize_act_i8(state["x"], N, state["shape"].K, state["xq"])
        tman.tman_mpgemm_i8(state["shape"], state["packed"], state["xq"], N, state["y"])
    return state["y"]


def work(case):
    """Packed weights and activations read once, results written once; two operations per weight and token."""
    nbytes = flops = 0
    seen = set()
    for M, K, a in _matrices(case):
        weights = M * K * case["bits"] / 8 + M * (K // case["group"]) * (4 if case["zero"] else 2)
        if case["call"] == "pack":
            nbytes += 2 * weights + M * K * (1 - case["bits"] / 8)  # one byte per code in, the packed form out
            continue
        nbytes += weights + 2 * case["N"] * M
        if a not in seen:
            nbytes += 2 * case["N"] * K
            seen.add(a)
        flops += 2 * case["N"] * M * K
    layers = case.get("layers", 1)
    return {"bytes": nbytes * layers, "flops": flops * layers}


def tolerance(case):
    """Four times the distance to the 64-bit result.  fp16 results alone give a relative error of 2.1e-4; 16-bit table
    entries or fp16 weights add 2e-4 to 3e-4 (independent of the sizes); the integer paths round nothing else, their
    activations' quantization being part of what they compute.  "max" is the largest of up to 2e7 such errors, about
    five and a half standard deviations."""
    if case["call"] == "pack":
        return "exact"
    if case["call"] in ("i16_batch", "i8"):
        return {"rel": 8.5e-4, "max": 2e-3}
    return {"rel": 1.6e-3, "max": 8e-3}


def exact(case, seed):
    if case["call"] == "pack":
        return None
    out = []
    for weights, acts in _inputs(case, seed):
        ys = []
        for (codes, scales, zeros), (M, K, a) in zip(weights, _matrices(case)):
            w = codes.double()
            blocks = w.view(M, K // case["group"], case["group"])
            if zeros is None:
                blocks.mul_(2.0).sub_(1.0)
            else:
                blocks.sub_(zeros.double().unsqueeze(-1))
            blocks.mul_(scales.double().unsqueeze(-1))
            x = acts[a]
            top = x.abs().amax(dim=1, keepdim=True)
            if case["call"] == "i16_batch":  # the power-of-two step that keeps the token's integers within 8191
                step = torch.pow(2.0, torch.frexp(top.float()).exponent.double() - 13.0)
                xd = torch.round(x.double() / step) * step
            elif case["call"] == "i8":  # absmax to 127, the rounding decided in binary32
                xd = torch.round(x.float() * torch.div(torch.full_like(top, 127.0).float(), top.float())).double() * (top.double() / 127.0)
            else:
                xd = x.double()
            ys.append(xd @ w.t())
        out.append(torch.cat([y.flatten() for y in ys]) if case["call"] in LAYERED else ys[0])
    return out if case["call"] in LAYERED else out[0]
