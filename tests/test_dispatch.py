"""Which GEMM kernel the library takes by itself, on both sides of its lines (host code only; that the kernels agree bit
for bit is tested on the GPU).  Variants: 2 and 5 on the INT8 path (two waves per SIMD, wide), 1 and 3 on the FP6 path,
10 + shape the small-output kernel."""
import pytest

import paper_2505_18663_amd as dvdq

INT8, PACKED4, FP6 = dvdq.CODES_INT8, dvdq.CODES_PACKED4, dvdq.CODES_FP6
NATIVE, NATIVE_FP6, CANONICAL = dvdq.W_NATIVE, dvdq.W_NATIVE_FP6, dvdq.W_CANONICAL


def int8(M, N, K, vectors=0):
    return dvdq.bench_gemm_choice(M, N, K, INT8, NATIVE, vectors)


def fp6(M, N, K, vectors=0):
    return dvdq.bench_gemm_choice(M, N, K, FP6, NATIVE_FP6, vectors)


@pytest.mark.parametrize("vectors", [0, 1, 2])
@pytest.mark.parametrize("M,N,K", [(15601, 1161, 1280), (5000, 4609, 3072), (8192, 3074, 6144), (32760, 4612, 13824)])
def test_channel_counts_that_are_no_multiple_of_8(M, N, K, vectors):
    """INT8: the two-wave kernel.  FP6: the wide one from depths that are from when such tiles were stored per element."""
    assert int8(M, N, K, vectors) == 2
    assert fp6(M, N, K, vectors) == (3 if K >= (6144, 12288, 1 << 30)[vectors] else 1)


def test_depth_of_k():
    assert [int8(32760, 8960, 128 * s, 2) for s in (11, 12)] == [2, 5]
    assert [fp6(32760, 4608, 128 * s, 2) for s in (5, 6)] == [1, 3]
    assert dvdq.bench_gemm_choice(32760, 4608, 1536, PACKED4, NATIVE) == 2


@pytest.mark.parametrize("tiles,variant", [(192, 5), (256, 5), (257, 2), (358, 2), (359, 5), (512, 5), (513, 2), (614, 2), (615, 5),
                                           (768, 5), (870, 2), (871, 5), (1024, 5), (1025, 5), (4480, 5)])
def test_a_nearly_empty_last_round_of_int8_tiles(tiles, variant):
    assert int8(256 * tiles, 256, 3072) == variant   # one column of 256 x 256 tiles


def test_small_outputs_and_canonical_weights():
    assert int8(2, 9216, 1536) >= 10 and fp6(128, 256, 256) >= 10
    assert dvdq.bench_gemm_choice(32760, 4608, 1440, INT8, CANONICAL) == 16
    assert dvdq.bench_gemm_choice(1, 64, 32, INT8, CANONICAL) == 10
    assert dvdq.bench_gemm_choice(0, 64, 128, INT8, NATIVE) == -2


@pytest.mark.parametrize("codes,M,N,slices,tiles", [
    # up to 768 tiles of 64 x 128 (shape 5): by depth and by N; 263 x 13568: 318 of 128 x 128, 530 of 64 x 128
    ("int8", 263, 13568, 9, 128), ("int8", 263, 13568, 10, 64), ("int8", 263, 13568, 18, 64), ("int8", 263, 13569, 1, 64), ("int8", 263, 13569, 5, 64),
    ("packed4", 263, 13568, 5, 128), ("packed4", 263, 13568, 6, 64), ("packed4", 263, 13569, 2, 64), ("packed4", 385, 10240, 7, 64), ("packed4", 385, 10368, 7, 128),
    ("packed4", 385, 10368, 8, 64), ("fp6", 615, 6560, 5, 128), ("fp6", 615, 6560, 6, 64), ("fp6", 615, 6561, 3, 128), ("fp6", 615, 6561, 4, 64),
    # beyond; 768 and 770 of 64 x 128
    ("int8", 768, 8192, 9, 128), ("int8", 768, 8192, 40, 64), ("int8", 5 * 128, 77 * 128, 40, 128), ("int8", 5 * 128, 77 * 128 - 1, 40, 128),
    ("int8", 5 * 128, 77 * 128 - 1, 1, 64), ("int8", 768, 8191, 5, 64), ("packed4", 5 * 128, 77 * 128, 9, 128), ("packed4", 5 * 128, 77 * 128, 10, 64),
    ("packed4", 5 * 128, 77 * 128 - 1, 5, 128), ("packed4", 5 * 128, 77 * 128 - 1, 6, 64),
    # more than 512 of 128 x 128, and the largest FP6 takes (95 of 256 x 256)
    ("int8", 65 * 64, 15 * 128, 3, 128), ("int8", 63 * 64 + 1, 16 * 128, 3, 128), ("int8", 1, 128 * 1024, 3, 64), ("int8", 1, 128 * 512, 3, 32), ("fp6", 5 * 256, 19 * 256, 3, 128)])
def test_128_x_128_tiles_for_small_outputs(codes, M, N, slices, tiles):
    """The two-wave kernel with these tiles against the largest shape of the small-output kernel."""
    fmt, layout, two_wave = {"int8": (INT8, NATIVE, 2), "packed4": (PACKED4, NATIVE, 2), "fp6": (FP6, NATIVE_FP6, 1)}[codes]
    K = 128 * slices
    choice = dvdq.bench_gemm_choice(M, N, K, fmt, layout)
    assert choice == two_wave if tiles == 128 else choice >= 10
    assert tiles != 64 or choice == 15
    assert tiles != 128 or dvdq.bench_narrow_tiles(M, N, K)
    if codes == "int8" and tiles < 128:
        assert dvdq.bench_gemm_choice(M, N, K, INT8, CANONICAL) == choice


@pytest.mark.parametrize("M,N", [(263, 13568), (768, 8192), (5 * 128, 77 * 128)])
def test_canonical_weights_stay_with_64_x_128_tiles(M, N):
    for slices in (1, 9, 40):
        assert dvdq.bench_gemm_choice(M, N, 128 * slices, INT8, CANONICAL) == 15


# units of 512 channels a wave: 1 in rows of up to 512, 2 up to 1024, 3 up to 1536 or, in four waves, 6144 (12 units), 4 up to 2048
@pytest.mark.parametrize("K,waves_per_row,first,last", [(128, 1, 9216, None), (512, 1, 9216, None), (544, 1, 6656, None), (1024, 1, 6656, None), (1536, 1, 6144, 32768),
                                                       (6144, 4, 6144, 32768), (2048, 1, None, None), (5120, 4, 6144, 32768), (4096, 2, None, None)])
@pytest.mark.parametrize("codes_format", [INT8, PACKED4, FP6])
def test_resident_waves_of_the_quantizer(K, waves_per_row, first, last, codes_format):
    """24 from a number of rows per slot on, up to 8 rows a slot of 16 with three units; FP6 codes 16."""
    waves = lambda rows: dvdq.bench_quantizer_waves(rows, K, codes_format)
    if first is None or codes_format == FP6:
        assert {waves(m) for m in (1, 1600, 6144, 9216, 118800)} == {16}
        return
    assert [waves(first // waves_per_row - 1), waves(first // waves_per_row)] == [16, 24]
    assert waves(118800) == (24 if last is None else 16)
    assert last is None or [waves(last // waves_per_row), waves(last // waves_per_row + 1)] == [24, 16]
