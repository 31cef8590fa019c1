"""Outputs whose rows begin at any even address (channel counts that are no multiple of 8): the kernels that store them in
16-byte pieces against the per-element stores of the accumulator hook's path, bit for bit, and nothing written outside."""
import pytest
import torch

import paper_2505_18663_amd as dvdq

pytestmark = pytest.mark.gpu

FORMATS = {"int8": (dvdq.CODES_INT8, 8, dvdq.W_NATIVE), "packed4": (dvdq.CODES_PACKED4, 4, dvdq.W_NATIVE),
           "fp6": (dvdq.CODES_FP6, 4, dvdq.W_NATIVE_FP6)}
GUARD = 4096   # elements in front of and behind the output


def _check(fmt, M, K, N, zero, bias, variant):
    codes_format, bits, layout = FORMATS[fmt]
    g = torch.Generator(device="cuda").manual_seed(M + 7 * K + 31 * N)
    x = torch.randn((M, K), generator=g, device="cuda").to(torch.bfloat16)
    packed = torch.randint(0, 256, (N, K // 2), generator=g, device="cuda", dtype=torch.uint8)
    w = dvdq.w4_prepack_fp6(packed) if fmt == "fp6" else dvdq.w4_prepack(packed)
    ws = torch.rand((N,), generator=g, device="cuda") + 0.5
    z = torch.randint(-8, 8, (N,), generator=g, device="cuda", dtype=torch.int8) if zero else None
    b = torch.randn((N,), generator=g, device="cuda").to(torch.bfloat16) if bias else None
    codes, scale, *rest = dvdq.rotate_quant(x, 128, bits, codes_format=codes_format, want_rowsum=zero)
    kw = dict(bias=b, codes_format=codes_format, w_zero=z, code_rowsum=rest[0] if rest else None, K=K)
    dvdq.bench_set_gemm_variant(variant)
    try:
        ref, _ = dvdq.w4ax_gemm(codes, scale, w, ws, bits, layout, want_acc=True, **kw)
        guarded = torch.full((M * N + 2 * GUARD,), 7.0, device="cuda", dtype=torch.bfloat16)
        y = guarded[GUARD:GUARD + M * N].view(M, N)
        for _ in range(2):   # (a second launch: tiles drawn from the counters too)
            y.fill_(3.0)
            dvdq.w4ax_gemm(codes, scale, w, ws, bits, layout, y=y, **kw)
            assert torch.equal(y.view(torch.int16), ref.view(torch.int16))
            assert bool((guarded[:GUARD] == 7).all()) and bool((guarded[GUARD + M * N:] == 7).all())
    finally:
        dvdq.bench_set_gemm_variant(-1)


# one tile and less, edges of tiles in both directions, one channel past a tile, several tiles a workgroup
@pytest.mark.parametrize("fmt", list(FORMATS))
@pytest.mark.parametrize("M,K,N", [(1, 128, 9), (127, 256, 63), (129, 128, 255), (300, 384, 257), (33, 640, 513), (1031, 128, 1028), (70000, 384, 300),
                                   (70001, 128, 12), (140000, 256, 130)])
def test_large_kernels(fmt, M, K, N):
    for zero, bias in ((False, False), (True, True), (False, True)):
        for variant in ((1, 3) if fmt == "fp6" else (2,)):   # 3: the wide kernel
            _check(fmt, M, K, N, zero, bias, variant)


@pytest.mark.parametrize("fmt", list(FORMATS))
@pytest.mark.parametrize("M,K,N", [(1, 128, 1), (2, 256, 7), (33, 128, 9), (65, 384, 129), (130, 256, 1001)])
def test_small_kernel(fmt, M, K, N):
    _check(fmt, M, K, N, True, True, -1)
