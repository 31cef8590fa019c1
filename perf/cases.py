"""The work a user of this library has it do, as cases that can be timed and compared.

A case is a dict of plain values.  `kind` says which calls make up a pass:

  "layer"      qlinear: the whole quantized linear layer (rotate, quantize, GEMM, dequantize)
  "shared"     rotate_quant once, then w4ax_gemm against several weights: projections of the same tokens (Q, K, V)
  "blockwise"  rotate_quant_blockwise, then w4ax_gemm: the layer with block-wise scaled activations
  "bgr"        bgr_quantize: the offline weight quantizer, once per layer of a model
  "gbs"        the bit-switching controller over a few denoising steps of one sampling run

Sizes come from the workloads of `dvdq_inputs` (video-DiT layers over 21x30x52 and 33x45x80 latent patches,
channel widths 1536, 3072, 4608, 5120, 8960 and 13824) and from what surrounds such layers in a transformer:
the conditioning vector, the text tokens, clips of few frames (a frame of the smaller grid is 1560 tokens).
"""
import math

import torch

import paper_2505_18663_amd as dvdq

DEV = "cuda"

# The largest listed work: a drawn case stays below it.
_MAX_FLOPS = 2 * 32760 * 13824 * 5120
_MAX_X = 32760 * 13824          # elements of X
_MAX_Y = 32760 * 8960           # elements of Y
_MAX_BGR = 1536 * 8960          # weights of one offline-quantized layer
_MAX_GBS = 118800 * 64          # elements of a model output


def _layer(name, M, K, N, had, bits, codes, weights, bias, zero, x="gauss"):
    return {"name": name, "kind": "layer", "M": M, "K": K, "N": N, "had_block": had, "act_bits": bits, "codes": codes,
            "weights": weights, "bias": bias, "zero": zero, "x": x}


def listed():
    return [
        # the smallest whole layer: launches and latency (the tiny workload of dvdq_inputs)
        _layer("tiny_layer_w4a4", 128, 256, 256, 256, 4, "fp6", "fp6", False, False),
        # the conditioning vector's modulation layer, both guidance branches at once: two tokens, six outputs per channel
        _layer("modulation_w4a8", 2, 1536, 9216, 256, 8, "int8", "native", True, False),
        # text tokens of the large model: keys and values of one cross-attention from the same codes, weights with
        # zero-points as the offline quantizer makes them
        {"name": "text_kv_w4a8", "kind": "shared", "M": 512, "K": 3072, "N": 3072, "had_block": 256, "act_bits": 8,
         "codes": "int8", "weights": "native", "bias": True, "zero": True, "count": 2, "x": "gauss"},
        # a two-frame clip and one token, channel counts that no tile divides, packed codes on the INT8 path
        _layer("ragged_clip_w4a4", 3121, 1152, 1160, 128, 4, "packed4", "native", True, True),
        # weights as the offline quantizer hands them over, K not a multiple of 128 (no native layout): five frames
        _layer("canonical_w4a8", 7800, 1440, 1440, 32, 8, "int8", "canonical", True, False),
        # block-wise scaled activations, ten frames, a square projection of the small model
        {"name": "blockwise_w4a4", "kind": "blockwise", "M": 15600, "K": 1536, "N": 1536, "had_block": 256, "act_bits": 4,
         "group": 128, "bias": True, "zero": True, "x": "gauss"},
        # the video-DiT layers at full length; the W4A6 one with the bias and the zero-points a quantized model has
        _layer("small_dit_qkv_w4a4", 32760, 1536, 4608, 256, 4, "fp6", "fp6", False, False),
        _layer("small_dit_ffn_up_w4a6", 32760, 1536, 8960, 256, 6, "int8", "native", True, True),
        _layer("large_dit_proj_w4a4", 118800, 3072, 3072, 256, 4, "fp6", "fp6", False, False),
        _layer("large_dit_ffn_down_w4a4", 32760, 13824, 5120, 512, 4, "fp6", "fp6", False, False, "postgelu"),
        # quantizing one FFN layer of the small model offline
        {"name": "bgr_ffn_down", "kind": "bgr", "N": 1536, "K": 8960, "n_steps": 100, "max_refine": 10, "search": "listing"},
        # three steps of the controller over outputs of the large model (118800 patches of 1x2x2 over 16 channels)
        {"name": "gbs_large", "kind": "gbs", "n": 118800 * 64, "steps": 3},
    ]


# ------------------------------------------------------------------ drawn cases
def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _fit_tokens(M, K, N):
    return max(1, min(M, _MAX_FLOPS // (2 * K * N), _MAX_X // K, _MAX_Y // N))


def _had(rng, K):
    sizes = [b for b in (32, 64, 128, 256, 512) if K % b == 0]
    return sizes[-1] if rng.random() < 0.6 else rng.choice(sizes)


def draw(rng):
    """One more case of the ranges the listed ones stand for."""
    kind = rng.choices(["layer", "shared", "blockwise", "bgr", "gbs"], [10, 2, 2, 2, 1])[0]
    if kind == "gbs":
        return {"kind": "gbs", "n": _log_int(rng, 4096, _MAX_GBS), "steps": rng.randint(1, 3)}
    if kind == "bgr":
        K = 2 * _log_int(rng, 64, 13824 // 2)
        return {"kind": "bgr", "N": _log_int(rng, 32, min(13824, _MAX_BGR // K)), "K": K, "n_steps": rng.choice([50, 100]),
                "max_refine": rng.choice([5, 10]), "search": rng.choice(["listing", "best_of_all"])}
    M = _log_int(rng, 1, 118800)
    N = _log_int(rng, 64, 13824)
    if rng.random() < 0.7:
        N = max(8, N // 8 * 8)      # channel counts are mostly multiples of 8, not always
    K = 128 * _log_int(rng, 1, 108)
    bits = rng.choice([4, 4, 6, 8])
    c = {"kind": kind, "M": M, "K": K, "N": N, "act_bits": bits, "bias": rng.random() < 0.5, "zero": rng.random() < 0.5,
         "x": rng.choice(["gauss", "postgelu"])}
    if kind == "blockwise":
        c["act_bits"] = rng.choice([4, 6])
        c["group"] = rng.choice([g for g in (128, 256, 512) if K % g == 0])
    else:
        c["codes"] = rng.choice(["fp6", "fp6", "packed4"]) if bits == 4 else "int8"
        c["weights"] = "fp6" if c["codes"] == "fp6" else "native"
        if kind == "shared":
            c["count"] = rng.choice([2, 3])
        elif rng.random() < 0.15:   # weights in the canonical layout
            K = 32 * _log_int(rng, 8, 432)
            c.update(K=K, codes="int8", weights="canonical", zero=False)
    c["had_block"] = _had(rng, K)
    c["M"] = _fit_tokens(M, K, N * c.get("count", 1))
    return c


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _activations(g, M, K, kind):
    """Tokens of varying magnitude with a few massive outlier channels, or what follows a GELU (one-sided)."""
    x = torch.randn((M, K), generator=g, device=DEV, dtype=torch.float32)
    if kind == "postgelu":
        x.abs_().sub_(0.2).clamp_(min=-0.17)
        n_out, gain = round(0.005 * K), 80.0
    else:
        x.mul_(torch.exp(0.5 * torch.randn((M, 1), generator=g, device=DEV)))
        n_out, gain = round(0.01 * K), 50.0
    if n_out:
        x[:, torch.randperm(K, generator=g, device=DEV)[:n_out]] *= gain
    return x.to(torch.bfloat16)


def _weights(g, N, K, zero):
    """(packed canonical codes, step sizes, zero-points or None) of Gaussian weights, per output channel:
    symmetric codes -7 .. 7 with a clipped range, or the 16 levels of an asymmetric grid."""
    w = 0.02 * torch.randn((N, K), generator=g, device=DEV)
    clip = 0.8 + 0.2 * torch.rand((N, 1), generator=g, device=DEV)
    if zero:
        lo, hi = clip * w.amin(1, keepdim=True), clip * w.amax(1, keepdim=True)
        step = (hi - lo) / 15
        z = torch.round(-lo / step).clamp_(0, 15)
        codes = (torch.round(w / step) + z).clamp_(0, 15) - 8
        z = (z - 8).to(torch.int8).flatten().contiguous()
    else:
        step = clip * w.abs().amax(1, keepdim=True) / 7
        codes, z = torch.round(w / step).clamp_(-7, 7), None
    c = codes.to(torch.int16) & 15
    packed = (c[:, 0::2] | (c[:, 1::2] << 4)).to(torch.uint8).contiguous()
    return packed, step.flatten().float().contiguous(), z


_CODES = {"int8": dvdq.CODES_INT8, "packed4": dvdq.CODES_PACKED4, "fp6": dvdq.CODES_FP6}
_LAYOUT = {"canonical": dvdq.W_CANONICAL, "native": dvdq.W_NATIVE, "fp6": dvdq.W_NATIVE_FP6}


def _layer_weights(g, case, weights):
    packed, scale, zero = _weights(g, case["N"], case["K"], case["zero"])
    if weights == "native":
        packed = dvdq.w4_prepack(packed)
    elif weights == "fp6":
        packed = dvdq.w4_prepack_fp6(packed)
    bias = (0.1 * torch.randn((case["N"],), generator=g, device=DEV)).to(torch.bfloat16) if case["bias"] else None
    return {"w": packed, "w_scale": scale, "w_zero": zero, "bias": bias}


def prepare(case, seed):
    """What the caller's program holds before the call: activations of this step, the laid-out weights and, for the
    whole layer, the workspace it keeps."""
    g = _gen(seed)
    s = {"case": case}
    if case["kind"] == "gbs":
        n = case["n"]
        f = torch.randn((n,), generator=g, device=DEV)
        s["outputs"] = [f.to(torch.bfloat16)]
        for _ in range(case["steps"]):   # successive outputs of a sampling run change by a few percent
            f = f + 0.05 * torch.randn((n,), generator=g, device=DEV)
            s["outputs"].append(f.to(torch.bfloat16))
        s["controller"] = dvdq.GbsController(0.07)
        return s
    if case["kind"] == "bgr":
        w = torch.randn((case["N"], case["K"]), generator=g, device=DEV)
        # heavier tails than a Gaussian, rows of varying magnitude and offset, as trained weights have
        w = w * torch.rsqrt(0.6 + 0.4 * torch.rand((case["N"], case["K"]), generator=g, device=DEV))
        s["w"] = (0.02 * torch.exp(0.3 * torch.randn((case["N"], 1), generator=g, device=DEV)) *
                  (w + 0.1 * torch.randn((case["N"], 1), generator=g, device=DEV))).contiguous()
        return s
    s["x"] = _activations(g, case["M"], case["K"], case["x"])
    if case["kind"] == "blockwise":
        s["layers"] = [_layer_weights(g, case, "native")]
    else:
        s["layers"] = [_layer_weights(g, case, case["weights"]) for _ in range(case.get("count", 1))]
    if case["kind"] == "layer":
        s["workspace"] = torch.empty((dvdq.qlinear_workspace_bytes(case["M"], case["K"], _CODES[case["codes"]]),),
                                     dtype=torch.uint8, device=DEV)
    return s


# ------------------------------------------------------------------ one pass
def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "layer":
        p = s["layers"][0]
        y, _ = dvdq.qlinear(s["x"], p["w"], p["w_scale"], c["had_block"], c["act_bits"], _LAYOUT[c["weights"]], bias=p["bias"],
                            workspace=s["workspace"], codes_format=_CODES[c["codes"]], w_zero=p["w_zero"])
        return y
    if kind == "shared":
        fmt = _CODES[c["codes"]]
        codes, scale, *rest = dvdq.rotate_quant(s["x"], c["had_block"], c["act_bits"], codes_format=fmt, want_rowsum=c["zero"])
        return [dvdq.w4ax_gemm(codes, scale, p["w"], p["w_scale"], c["act_bits"], _LAYOUT[c["weights"]], bias=p["bias"],
                               codes_format=fmt, w_zero=p["w_zero"], code_rowsum=rest[0] if rest else None, K=c["K"])
                for p in s["layers"]]
    if kind == "blockwise":
        p = s["layers"][0]
        values, scale, *rest = dvdq.rotate_quant_blockwise(s["x"], c["had_block"], c["act_bits"], c["group"],
                                                           want_rowsum=c["zero"])
        return dvdq.w4ax_gemm(values, scale, p["w"], p["w_scale"], 8, dvdq.W_NATIVE, bias=p["bias"], w_zero=p["w_zero"],
                              code_rowsum=rest[0] if rest else None)
    if kind == "bgr":
        search = dvdq.BGR_LISTING if c["search"] == "listing" else dvdq.BGR_BEST_OF_ALL
        return dvdq.bgr_quantize(s["w"], n_steps=c["n_steps"], max_refine=c["max_refine"], eps=0.0, want_error=True,
                                 search=search)
    ctl = s["controller"]
    ctl.reset()
    for prev, cur in zip(s["outputs"], s["outputs"][1:]):
        ctl.step(cur, prev)
    st = ctl.state
    return {"sum": st[:8].view(torch.float64), "l1": st[8:12].view(torch.float32), "bits": st[12:16].view(torch.int32)}


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    kind = case["kind"]
    if kind == "gbs":   # every output read once per step that uses it, three operations and two sums per element
        return {"bytes": 4 * case["n"] * case["steps"], "flops": 5 * case["n"] * case["steps"]}
    if kind == "bgr":   # the weights in, codes, steps, zero-points and errors out; one rounding and one error term per weight
        n, k = case["N"], case["K"]
        return {"bytes": 4 * n * k + n * k // 2 + 13 * n, "flops": 8 * n * k}
    M, K, N, count = case["M"], case["K"], case["N"], case.get("count", 1)
    per_n = 4 + (2 if case["bias"] else 0) + (1 if case["zero"] else 0)
    # activations in, packed weights and channel vectors in, outputs out; the codes need not leave the chip
    return {"bytes": 2 * M * K + count * (N * K // 2 + per_n * N + 2 * M * N), "flops": 2 * M * K * N * count}


def tolerance(case):
    """Measured against a plain fp64 evaluation of the same layer rounded to bf16, times about four.

    Layers: 1e-5 to 2.4e-4 in the 2-norm (fp32 products next to a bf16 rounding boundary, and the few 4-bit codes that
    sit on a rounding boundary in fp32); one element of up to 0.043 of the row's root mean square, where a token with a
    massive outlier channel has a code off by one.
    bgr: fp64 sums in another order; a row whose best two grids tie to rounding may take the other one.
    gbs: fp32 sums of a few hundred terms per thread, the rest in fp64."""
    if case["kind"] == "gbs":
        return {"rel": 1e-5, "differ": 0.0}
    if case["kind"] == "bgr":
        return {"rel": 1e-5, "max": 1e-2, "differ": 1e-3}
    return {"rel": 1e-3, "max": 0.16}
