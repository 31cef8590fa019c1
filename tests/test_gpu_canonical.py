"""Canonical weights on the large tiles (16), and a wave per 64 x 128 tile (17): the bits of the small-output kernel, for every length of the last K slice, at the edges of
tiles, with rows that begin at any even address, and with several tiles per workgroup."""
import pytest
import torch

import paper_2505_18663_amd as dvdq

pytestmark = pytest.mark.gpu
GUARD = 4096


@pytest.mark.parametrize("M,K,N", [(1, 32, 8), (5, 64, 1), (128, 96, 256), (129, 128, 257), (300, 160, 300), (257, 224, 1000), (64, 1440, 520),
                                   (1000, 352, 1031), (70000, 96, 264), (140000, 32, 20), (4097, 4128, 72)])
@pytest.mark.parametrize("variant", [16, 17])
def test_large_tiles_equal_the_small_kernel(M, K, N, variant):
    g = torch.Generator(device="cuda").manual_seed(M + 7 * K + 31 * N)
    codes = torch.randint(-127, 128, (M, K), generator=g, device="cuda", dtype=torch.int8)
    w = torch.randint(0, 256, (N, K // 2), generator=g, device="cuda", dtype=torch.uint8)
    xs, ws = torch.rand((M,), generator=g, device="cuda") + 0.1, torch.rand((N,), generator=g, device="cuda") + 0.1
    b = torch.randn((N,), generator=g, device="cuda").to(torch.bfloat16)
    for bias in (None, b):
        try:
            dvdq.bench_set_gemm_variant(13)
            ref, acc = dvdq.w4ax_gemm(codes, xs, w, ws, 8, dvdq.W_CANONICAL, bias=bias, want_acc=True)
            dvdq.bench_set_gemm_variant(variant)
            _, acc2 = dvdq.w4ax_gemm(codes, xs, w, ws, 8, dvdq.W_CANONICAL, bias=bias, want_acc=True)
            assert torch.equal(acc, acc2)
            guarded = torch.full((M * N + 2 * GUARD,), 7.0, device="cuda", dtype=torch.bfloat16)
            y = guarded[GUARD:GUARD + M * N].view(M, N)
            dvdq.w4ax_gemm(codes, xs, w, ws, 8, dvdq.W_CANONICAL, bias=bias, y=y)
            assert torch.equal(y.view(torch.int16), ref.view(torch.int16))
            assert bool((guarded[:GUARD] == 7).all()) and bool((guarded[GUARD + M * N:] == 7).all())
        finally:
            dvdq.bench_set_gemm_variant(-1)
