"""The layer of few tokens in one launch: outputs, and what it leaves in the workspace, are the bits of the quantizer and the GEMM
as two calls."""
import pytest
import torch

import paper_2505_18663_amd as dvdq

pytestmark = pytest.mark.gpu

FORMATS = {"int8": (dvdq.CODES_INT8, dvdq.W_NATIVE), "packed4": (dvdq.CODES_PACKED4, dvdq.W_NATIVE),
           "fp6": (dvdq.CODES_FP6, dvdq.W_NATIVE_FP6), "canonical": (dvdq.CODES_INT8, dvdq.W_CANONICAL)}


def _check(fmt, M, K, N, had_block, bits, zero, bias, x=None):
    codes_format, layout = FORMATS[fmt]
    g = torch.Generator(device="cuda").manual_seed(M + 7 * K + 31 * N)
    if x is None:
        x = torch.randn((M, K), generator=g, device="cuda") * torch.exp(torch.randn((M, 1), generator=g, device="cuda"))
        x = x.to(torch.bfloat16)
    packed = torch.randint(0, 256, (N, K // 2), generator=g, device="cuda", dtype=torch.uint8)
    w = packed if fmt == "canonical" else dvdq.w4_prepack_fp6(packed) if fmt == "fp6" else dvdq.w4_prepack(packed)
    ws = torch.rand((N,), generator=g, device="cuda") + 0.5
    z = torch.randint(-8, 8, (N,), generator=g, device="cuda", dtype=torch.int8) if zero else None
    b = torch.randn((N,), generator=g, device="cuda").to(torch.bfloat16) if bias else None
    codes, scale, *rest = dvdq.rotate_quant(x, had_block, bits, codes_format=codes_format, want_rowsum=zero)
    ref = dvdq.w4ax_gemm(codes, scale, w, ws, bits, layout, bias=b, codes_format=codes_format, w_zero=z,
                         code_rowsum=rest[0] if rest else None, K=K)
    workspace = torch.full((dvdq.qlinear_workspace_bytes(M, K, codes_format) + 256,), 0x5A, device="cuda", dtype=torch.uint8)
    y, _ = dvdq.qlinear(x, w, ws, had_block, bits, layout, bias=b, workspace=workspace, codes_format=codes_format, w_zero=z)
    assert torch.equal(y.view(torch.int16), ref.view(torch.int16))
    got_codes, got_scale = dvdq.workspace_views(workspace, M, K, codes_format)
    assert torch.equal(got_scale.view(torch.int32), scale.view(torch.int32))
    if fmt == "fp6":   # blocks of 32 rows x 128 channels: [block][slice][16-byte chunk][row][16]; rows past M are not written
        blocks = lambda t: t.view(-1, K // 128, 6, 32, 16).permute(0, 3, 1, 2, 4).reshape(-1, K // 128 * 96)
        assert torch.equal(blocks(got_codes)[:M], blocks(codes)[:M])
        assert bool((blocks(got_codes)[M:] == 0x5A).all())
    else:
        assert torch.equal(got_codes, codes)
    if zero:
        assert torch.equal(dvdq.workspace_rowsum(workspace, M, K, codes_format), rest[0])
    assert bool((workspace[-256:] == 0x5A).all())


# one token, a full and a part tile of 32 tokens, rows of one unit to many, units that do not divide among the waves, odd channel
# counts; tiles of 32 and 64 channels (width 1 and 2) with 1, 2, 4 and 8 units a wave each
@pytest.mark.parametrize("fmt", list(FORMATS))
@pytest.mark.parametrize("M,K,N,had_block,width,units", [
    (1, 128, 8, 128, 1, 1), (12, 512, 264, 256, 1, 2), (9, 896, 1161, 128, 1, 4), (128, 256, 256, 256, 1, 4), (300, 512, 96, 512, 1, 4),
    (8000, 384, 32, 1, 1, 4), (1, 32768, 33, 512, 1, 8), (5, 6144, 1161, 32, 1, 8),
    (2, 1536, 9216, 256, 2, 1), (12, 512, 9216, 64, 2, 2), (3, 2432, 9001, 128, 2, 2), (32, 512, 9216, 512, 2, 4), (41, 384, 6000, 8, 2, 4),
    (8, 4096, 9216, 256, 2, 8), (12, 2176, 8200, 2, 2, 8)])
def test_equals_two_calls(fmt, M, K, N, had_block, width, units):
    assert dvdq.bench_qlinear_choice(M, N, K) == width
    per_wave = -(-min(M, 32) * -(-K // 512) // 8)   # of the workgroup with most of them; the kernel has forms for 1, 2, 4 and 8
    assert min(u for u in (1, 2, 4, 8) if u >= per_wave) == units
    for zero, bias in ((False, False), (True, True)):
        if not (zero and fmt == "canonical"):   # (canonical weights carry no zero-points)
            _check(fmt, M, K, N, had_block, 4 if fmt in ("packed4", "fp6") else 6, zero, bias)


@pytest.mark.parametrize("fmt", list(FORMATS))
@pytest.mark.parametrize("M,K,N,had_block", [(32, 1024, 64, 64), (33, 640, 255, 128), (21, 1408, 5000, 8), (64, 512, 9216, 256)])
def test_just_past_the_line(fmt, M, K, N, had_block):
    """Two launches: more units than a workgroup takes, or more tiles than run at once."""
    assert dvdq.bench_qlinear_choice(M, N, K) == 0
    _check(fmt, M, K, N, had_block, 4 if fmt in ("packed4", "fp6") else 6, fmt != "canonical", True)


@pytest.mark.parametrize("M,K,N,had_block", [(3, 32, 40, 32), (15, 672, 70, 16), (1, 1440, 1440, 32), (9, 3104, 513, 2), (20, 480, 8300, 32), (2, 2080, 9001, 16)])
def test_canonical_part_slices(M, K, N, had_block):
    assert dvdq.bench_qlinear_choice(M, N, K) > 0
    _check("canonical", M, K, N, had_block, 8, False, True)


def test_rows_of_zeros_infinities_and_nan():
    x = torch.randn((7, 512), device="cuda").to(torch.bfloat16)
    x[1] = 0
    x[2, 5] = float("inf")
    x[3, 100] = float("nan")
    x[4] = 3e38
    for had_block in (1, 32, 256):
        _check("int8", 7, 512, 96, had_block, 8, True, True, x)
        _check("fp6", 7, 512, 96, had_block, 4, True, True, x)
