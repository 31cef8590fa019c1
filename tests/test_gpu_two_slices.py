"""The small-output kernel with 64 x 96 tiles and two slices in flight per wave (variant 17): the bits of the shape with 64 x 64 tiles
(13), for every number of slices a wave can be left with, at the edges of its tiles; and where it is taken."""
import pytest
import torch

import paper_2505_18663_amd as dvdq

FORMATS = {"int8": (dvdq.CODES_INT8, 8, dvdq.W_NATIVE), "packed4": (dvdq.CODES_PACKED4, 4, dvdq.W_NATIVE),
           "fp6": (dvdq.CODES_FP6, 4, dvdq.W_NATIVE_FP6)}
GUARD = 4096


# 1 to 3, 5, 8, 9, 12 and 24 slices for four waves; a tile and less, 95 to 97 channels, rows that begin at any even address, the weights' padded end
@pytest.mark.gpu
@pytest.mark.parametrize("fmt", list(FORMATS))
@pytest.mark.parametrize("M,K,N", [(1, 128, 8), (63, 256, 95), (64, 384, 96), (65, 640, 97), (130, 1024, 200), (33, 1152, 513), (100, 1536, 1160), (512, 3072, 768)])
def test_two_slices_in_flight(fmt, M, K, N):
    codes_format, bits, layout = FORMATS[fmt]
    g = torch.Generator(device="cuda").manual_seed(M + 7 * K + 31 * N)
    x = torch.randn((M, K), generator=g, device="cuda").to(torch.bfloat16)
    packed = torch.randint(0, 256, (N, K // 2), generator=g, device="cuda", dtype=torch.uint8)
    w = dvdq.w4_prepack_fp6(packed) if fmt == "fp6" else dvdq.w4_prepack(packed)
    ws = torch.rand((N,), generator=g, device="cuda") + 0.5
    z = torch.randint(-8, 8, (N,), generator=g, device="cuda", dtype=torch.int8)
    b = torch.randn((N,), generator=g, device="cuda").to(torch.bfloat16)
    try:
        for zero, bias in ((False, False), (False, True), (True, False), (True, True)):
            codes, scale, *rest = dvdq.rotate_quant(x, 128, bits, codes_format=codes_format, want_rowsum=zero)
            kw = dict(bias=b if bias else None, codes_format=codes_format, w_zero=z if zero else None, code_rowsum=rest[0] if rest else None, K=K)
            dvdq.bench_set_gemm_variant(13)
            ref, acc = dvdq.w4ax_gemm(codes, scale, w, ws, bits, layout, want_acc=True, **kw)
            dvdq.bench_set_gemm_variant(17)
            _, acc2 = dvdq.w4ax_gemm(codes, scale, w, ws, bits, layout, want_acc=True, **kw)
            assert torch.equal(acc, acc2)
            guarded = torch.full((M * N + 2 * GUARD,), 7.0, device="cuda", dtype=torch.bfloat16)
            y = guarded[GUARD:GUARD + M * N].view(M, N)
            dvdq.w4ax_gemm(codes, scale, w, ws, bits, layout, y=y, **kw)
            assert torch.equal(y.view(torch.int16), ref.view(torch.int16))
            assert bool((guarded[:GUARD] == 7).all()) and bool((guarded[GUARD + M * N:] == 7).all())
    finally:
        dvdq.bench_set_gemm_variant(-1)


@pytest.mark.parametrize("M,N,slices,variant", [(512, 3072, 24, 17), (512, 3072, 18, 17), (512, 3072, 17, 13), (512, 3073, 24, 13), (512, 2048, 24, 13),
                                                (256, 4160, 24, 17), (1024, 1536, 24, 17)])
def test_where_it_is_taken(M, N, slices, variant):
    """One round of 64 x 96 tiles for more than one of 64 x 64, from 18 slices on; canonical weights keep the 64 x 64 tiles."""
    for fmt, layout in ((dvdq.CODES_INT8, dvdq.W_NATIVE), (dvdq.CODES_PACKED4, dvdq.W_NATIVE), (dvdq.CODES_FP6, dvdq.W_NATIVE_FP6)):
        assert dvdq.bench_gemm_choice(M, N, 128 * slices, fmt, layout) == variant
    assert dvdq.bench_gemm_choice(M, N, 128 * slices, dvdq.CODES_INT8, dvdq.W_CANONICAL) == 13


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N", [(512, 2304, 3072), (256, 2336, 4160)])
def test_canonical_weights_where_others_take_it(M, K, N):
    """The library's choice against the shape with 64 x 64 tiles and the shape with 64 x 128, which 17 stands for with canonical weights."""
    assert dvdq.bench_gemm_choice(M, N, 2304, dvdq.CODES_INT8, dvdq.W_NATIVE) == 17
    g = torch.Generator(device="cuda").manual_seed(N)
    x = torch.randn((M, K), generator=g, device="cuda").to(torch.bfloat16)
    packed = torch.randint(0, 256, (N, K // 2), generator=g, device="cuda", dtype=torch.uint8)
    ws = torch.rand((N,), generator=g, device="cuda") + 0.5
    codes, scale = dvdq.rotate_quant(x, 32, 8)[:2]
    out = []
    try:
        for variant in (-1, 13, 17):
            dvdq.bench_set_gemm_variant(variant)
            out.append(dvdq.w4ax_gemm(codes, scale, packed, ws, 8, dvdq.W_CANONICAL, want_acc=True, K=K))
    finally:
        dvdq.bench_set_gemm_variant(-1)
    for y, acc in out[1:]:
        assert torch.equal(acc, out[0][1]) and torch.equal(y.view(torch.int16), out[0][0].view(torch.int16))
