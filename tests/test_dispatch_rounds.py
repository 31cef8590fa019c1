"""Which GEMM kernel the library takes where the last round of 256 x 256 tiles (256 at a time) is at most half full, and where it is
not (host code only; that the kernels agree bit for bit is tested on the GPU)."""
import pytest

import paper_2505_18663_amd as dvdq


def choice(tiles, slices, fp6, vectors=0):
    """of an output of `tiles` tiles in two columns (or four, for an odd half)"""
    cols = 2
    fmt, layout = (dvdq.CODES_FP6, dvdq.W_NATIVE_FP6) if fp6 else (dvdq.CODES_INT8, dvdq.W_NATIVE)
    return dvdq.bench_gemm_choice(256 * (tiles // cols), 256 * cols, 128 * slices, fmt, layout, vectors)


@pytest.mark.parametrize("tiles,variant", [(256, 5), (258, 2), (384, 2), (386, 5), (512, 5), (514, 2), (640, 2), (642, 5), (1024, 5), (1026, 2),
                                           (4094, 5), (4098, 5)])
def test_int8(tiles, variant):
    assert choice(tiles, 12, False) == choice(tiles, 108, False) == variant


def test_int8_of_few_slices():
    """Eight to eleven: the wide kernel with bias and zero-points only, in one or two rounds that end more than half full."""
    assert [choice(400, s, False, 2) for s in (7, 8, 11)] == [2, 5, 5]
    assert [choice(t, 8, False, 2) for t in (256, 384, 386, 510, 512, 770)] == [2, 2, 5, 5, 2, 2]
    assert [choice(400, s, False, v) for s in (8, 11) for v in (0, 1)] == [2] * 4


@pytest.mark.parametrize("tiles,slices", [(100, (10, 12, 12)), (128, (10, 12, 12)), (130, (6, 6, 6)), (256, (6, 6, 6)), (258, (8, 10, 12)),
                                          (384, (8, 10, 12)), (386, (6, 6, 6)), (514, (8, 10, 12)), (1408, (8, 10, 12)), (1538, (6, 6, 6)), (3968, (6, 6, 6))])
def test_fp6(tiles, slices):
    """The first depth, in slices, at which the wide kernel is taken, by the number of vectors (bias, zero-points)."""
    for vectors, s in enumerate(slices):
        assert choice(tiles, s, True, vectors) == 3 and choice(tiles, s - 1, True, vectors) == 1


def test_fp6_with_cached_stores():
    """N no multiple of 32, more than two rounds of tiles: 12 slices whatever the vectors."""
    fp6 = lambda m, slices, v: dvdq.bench_gemm_choice(256 * m, 264, 128 * slices, dvdq.CODES_FP6, dvdq.W_NATIVE_FP6, v)
    assert [[fp6(260, s, v) for s in (11, 12)] for v in range(3)] == [[1, 3]] * 3
    assert [[fp6(130, s, v) for s in (7, 8, 9, 10)] for v in range(2)] == [[1, 3, 3, 3], [1, 1, 1, 3]]


@pytest.fixture
def fixed_shares():
    """as under stream capture, where the tiles of a launch are fixed shares"""
    dvdq.bench_set_gemm_schedule(0)
    yield
    dvdq.bench_set_gemm_schedule(-1)


@pytest.mark.parametrize("tiles,variant", [(256, 5), (258, 2), (384, 2), (386, 5), (512, 5), (514, 2), (528, 2), (530, 5), (640, 5), (1026, 2),
                                           (1296, 2), (1538, 5), (4098, 5)])
def test_int8_with_fixed_shares(fixed_shares, tiles, variant):
    """The rest of a later round is not spread over the chip: half a round is gained below two rounds, then for 16 tiles at most."""
    assert choice(tiles, 12, False) == choice(tiles, 108, False) == variant


def test_fp6_with_fixed_shares(fixed_shares):
    assert [choice(t, 6, True) for t in (128, 258, 384, 514, 640, 1026, 3968)] == [1, 1, 1, 3, 3, 3, 3]


@pytest.mark.parametrize("M,N,variant", [(22528, 592, 17), (32768, 520, 16), (65536, 256, 16), (65600, 128, 17), (130944, 128, 17), (131200, 128, 16),
                                         (33024, 512, 16), (21760, 640, 16), (21888, 640, 17), (26112, 640, 17), (26240, 640, 16), (23080, 528, 17)])
def test_canonical_weights_beyond_the_small_outputs(M, N, variant):
    """17: more than 512 tiles of 128 x 256, at most 2048 of 64 x 128."""
    for K in (32, 1440):
        assert dvdq.bench_gemm_choice(M, N, K, dvdq.CODES_INT8, dvdq.W_CANONICAL) == variant


def narrow(M, N, slices, canonical=True, drawn=True):
    return dvdq.bench_narrow_tiles(M, N, 128 * slices, dvdq.CODES_INT8, dvdq.W_CANONICAL if canonical else dvdq.W_NATIVE, drawn)


# one round (288 rows of 128: 576 small tiles in two columns), two, three
@pytest.mark.parametrize("rows,N,first", [(300, 256, 24), (150, 500, 48), (144, 500, None), (200, 384, 48), (130, 640, None),
                                          (600, 250, 12), (400, 384, 36), (300, 512, None), (600, 320, 26), (514, 384, None), (580, 384, 26)])
@pytest.mark.parametrize("drawn", [True, False])
def test_canonical_weights_keep_128_x_256_tiles_from(rows, N, first, drawn):
    """The first depth, in slices, from which few columns keep the larger tiles; none up to 100 where tiles are few or columns many."""
    taken = [narrow(128 * rows, N, s, drawn=drawn) for s in range(1, 101)]
    assert taken == [first is None or s < first for s in range(1, 101)]


@pytest.mark.parametrize("M,N,canonical,drawn,first", [
    (128 * 115, 2304, True, True, 24), (128 * 58, 4992, True, True, 20), (128 * 58, 4992, True, False, 48), (128 * 52, 5000, True, True, 24), (128 * 52, 5000, True, False, 24),
    (128 * 60, 4800, True, True, 20), (128 * 79, 3352, False, True, 36), (128 * 79, 3352, False, False, 48), (128 * 84, 3352, False, True, 48)])
def test_a_nearly_empty_third_round_of_128_x_256_tiles(M, N, canonical, drawn, first):
    """The first depth from which it is preferred to a third round of 128 x 128 tiles that is half or three quarters full."""
    taken = [narrow(M, N, s, canonical, drawn) for s in range(1, 101)]
    assert taken == [s < first for s in range(1, 101)]


@pytest.mark.parametrize("K,n_steps,max_refine,threads", [(256, 50, 10, 512), (256, 80, 0, 256), (2048, 80, 0, 256), (2050, 80, 10, 512), (2050, 100, 3, 256),
                                                          (2050, 100, 2, 512), (4608, 100, 10, 256), (4610, 100, 10, 512), (4096, 20, 10, 512)])
def test_offline_quantizer_with_at_most_two_rows_per_compute_unit(K, n_steps, max_refine, threads):
    """The time is one row's own: workgroups of 256 threads only with starts enough to outweigh their sorting."""
    assert dvdq.bench_bgr_choice(257, K, n_steps, max_refine) == dvdq.bench_bgr_choice(512, K, n_steps, max_refine) == threads


def test_offline_quantizer_with_more_rows():
    assert [dvdq.bench_bgr_choice(513, K, s, 0) for K, s in ((5376, 3), (5378, 99), (5378, 100), (6144, 100), (6146, 100), (14336, 100), (14338, 100))] == [
        256, 512, 256, 256, 512, 512, 1024]
    assert dvdq.bench_bgr_choice(256, 256, 100, 10) == 1024
