"""The two-wave kernels with 128 x 128 tiles, three workgroups per compute unit (variant 6): the bits and accumulators of the same with
128 x 256, the oracle's accumulators, nothing written outside; the rule that takes them; and that they are what is launched."""
import re

import numpy as np
import pytest
import torch

import oracle
import paper_2505_18663_amd as dvdq

FORMATS = {"int8": (dvdq.CODES_INT8, 8, dvdq.W_NATIVE), "packed4": (dvdq.CODES_PACKED4, 4, dvdq.W_NATIVE),
           "fp6": (dvdq.CODES_FP6, 4, dvdq.W_NATIVE_FP6), "canonical": (dvdq.CODES_INT8, 8, dvdq.W_CANONICAL)}
LARGE = {"int8": 2, "packed4": 2, "fp6": 1, "canonical": 16}   # the variants with 128 x 256 tiles
GUARD = 4096


# less than a tile, one, edges in both directions, zero-points and biases across a tile's 128 channels, one slice, several tiles a workgroup
@pytest.mark.gpu
@pytest.mark.parametrize("fmt", list(FORMATS))
@pytest.mark.parametrize("M,K,N", [(1, 128, 8), (127, 128, 64), (128, 256, 128), (129, 384, 136), (300, 128, 385), (33, 640, 129), (1031, 1152, 1160),
                                   (70000, 256, 304), (140001, 128, 130), (513, 4096, 255)])
def test_narrow_tiles(fmt, M, K, N):
    codes_format, bits, layout = FORMATS[fmt]
    if fmt == "canonical" and K < 4096:
        K -= 32   # a last slice of 96 channels
    g = torch.Generator(device="cuda").manual_seed(M + 7 * K + 31 * N)
    x = torch.randn((M, K), generator=g, device="cuda").to(torch.bfloat16)
    packed = torch.randint(0, 256, (N, K // 2), generator=g, device="cuda", dtype=torch.uint8)
    w = packed if fmt == "canonical" else dvdq.w4_prepack_fp6(packed) if fmt == "fp6" else dvdq.w4_prepack(packed)
    ws = torch.rand((N,), generator=g, device="cuda") + 0.5
    z = torch.randint(-8, 8, (N,), generator=g, device="cuda", dtype=torch.int8)
    b = torch.randn((N,), generator=g, device="cuda").to(torch.bfloat16)
    try:
        for zero, bias in ((False, False), (False, True)) + (((True, False), (True, True)) if fmt != "canonical" else ()):
            print(f"narrow tiles {fmt} {M} {K} {N} zero={zero} bias={bias}", flush=True)
            codes, scale, *rest = dvdq.rotate_quant(x, 32, bits, codes_format=codes_format, want_rowsum=zero)
            kw = dict(bias=b if bias else None, codes_format=codes_format, w_zero=z if zero else None, code_rowsum=rest[0] if rest else None, K=K)
            dvdq.bench_set_gemm_variant(LARGE[fmt])
            ref, acc = dvdq.w4ax_gemm(codes, scale, w, ws, bits, layout, want_acc=True, **kw)
            dvdq.bench_set_gemm_variant(6)
            ref6, acc6 = dvdq.w4ax_gemm(codes, scale, w, ws, bits, layout, want_acc=True, **kw)
            assert torch.equal(acc6, acc) and torch.equal(ref6.view(torch.int16), ref.view(torch.int16))
            guarded = torch.full((M * N + 2 * GUARD,), 7.0, device="cuda", dtype=torch.bfloat16)
            y = guarded[GUARD:GUARD + M * N].view(M, N)
            for _ in range(2):   # (a second launch: tiles drawn from the counters too)
                y.fill_(3.0)
                dvdq.w4ax_gemm(codes, scale, w, ws, bits, layout, y=y, **kw)
                assert torch.equal(y.view(torch.int16), ref.view(torch.int16))
                assert bool((guarded[:GUARD] == 7).all()) and bool((guarded[GUARD + M * N:] == 7).all())
            if M * K * N < 1 << 31:
                int8, _, *rs = dvdq.rotate_quant(x, 32, bits, want_rowsum=True)
                lo, hi = (packed & 15).cpu().numpy().astype(np.int8), (packed >> 4).cpu().numpy().astype(np.int8)
                wc = np.stack([lo, hi], axis=2).reshape(N, K)
                wc = np.where(wc > 7, wc - 16, wc).astype(np.int8)
                want = oracle.int_gemm(int8.cpu().numpy(), wc)
                if zero:
                    want = want - rs[0].cpu().numpy().astype(np.int64)[:, None] * z.cpu().numpy().astype(np.int64)[None, :]
                assert np.array_equal(acc.cpu().numpy().astype(np.int64), want)
    finally:
        dvdq.bench_set_gemm_variant(-1)


@pytest.mark.parametrize("M,N,K,narrow", [(7800, 1440, 1440, True), (15600, 1536, 1536, True), (32760, 1536, 1536, False), (128 * 64, 1536, 1536, True),
                                          (128 * 64 + 1, 1536, 1536, False), (128 * 86, 1536, 1536, True), (128 * 128, 1536, 1536, True),
                                          (128 * 128 + 1, 1536, 1536, False), (128 * 86, 1536, 2560, True), (128 * 107, 1536, 2560, False),
                                          (128 * 107, 1536, 2432, True), (20912, 1664, 13568, False), (20912, 1664, 128 * 47, True), (90678, 640, 896, True), (118800, 640, 1536, False)])   # (the last: 7 rounds for 6)
def test_where_they_are_taken(M, N, K, narrow):
    """A round of 768 small tiles for one of 512 large ones; a last round of up to half large and over two thirds small ones below 20 slices
    in the second, below 48 later."""
    assert dvdq.bench_narrow_tiles(M, N, K) == narrow


def _launched(call):
    """The tile of the two-wave kernel, or the name of the kernel, that a call launches."""
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    names = [e.name for e in p.events() if "gemm" in e.name and "kernel" in e.name]
    assert len(names) == 1, names
    tile = re.search(r"(?:native|fp6_gemm)_kernel<(\d+), (\d+), ", names[0])
    return f"{tile[1]} x {tile[2]}" if tile else names[0]


@pytest.mark.gpu
@pytest.mark.parametrize("fmt", list(FORMATS))
def test_what_is_launched(fmt):
    """Forced, and by the library's choice: where the rules say 128 x 128, where they say 128 x 256 (few columns and deep products with
    canonical weights, a round more with the others), and as fixed shares where that makes a difference."""
    codes_format, bits, layout = FORMATS[fmt]
    narrow, large = "128 x 128", "128 x 256"
    # (2226 small tiles for 1113 large ones of 30 slices, canonical weights: large unless in fixed shares)
    cases = [(7800, 1440, 256, -1, narrow), (7800, 1440, 256, 0, narrow)]
    cases += [(40000, 256, 3072, -1, large), (53 * 128, 42 * 128, 3840, -1, large), (53 * 128, 42 * 128, 3840, 0, narrow)] if fmt == "canonical" else [
        (128 * 86, 1024, 256, -1, narrow), (128 * 98, 1280, 256, -1, large)]
    try:
        for M, N, K, schedule, want in cases:
            print(f"launched {fmt} {M} {N} {K} schedule {schedule}", flush=True)
            x = torch.randn((M, K), device="cuda").to(torch.bfloat16)
            packed = torch.randint(0, 256, (N, K // 2), device="cuda", dtype=torch.uint8)
            w = packed if fmt == "canonical" else dvdq.w4_prepack_fp6(packed) if fmt == "fp6" else dvdq.w4_prepack(packed)
            ws = torch.rand((N,), device="cuda") + 0.5
            codes, scale = dvdq.rotate_quant(x, 32, bits, codes_format=codes_format)[:2]
            gemm = lambda: dvdq.w4ax_gemm(codes, scale, w, ws, bits, layout, codes_format=codes_format, K=K)
            dvdq.bench_set_gemm_schedule(schedule)
            for variant, tile in ((-1, want), (6, narrow), (LARGE[fmt], large)):
                dvdq.bench_set_gemm_variant(variant)
                gemm()
                assert _launched(gemm) == tile, (M, N, K, schedule, variant)
    finally:
        dvdq.bench_set_gemm_variant(-1)
        dvdq.bench_set_gemm_schedule(-1)
