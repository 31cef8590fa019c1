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
