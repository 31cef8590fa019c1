"""Where a whole layer goes as one launch, and where as two (host code only; that both leave the same bits is tested on the GPU)."""
import pytest

import paper_2505_18663_amd as dvdq

X, Y, WS = 1 << 40, 1 << 41, 1 << 42


@pytest.mark.parametrize("M,N,K", [(2, 1536, 1536), (128, 256, 256), (1, 4096, 4096), (32, 64, 512)])
def test_one_launch_only_where_nothing_it_stores_lies_over_x(M, N, K):
    """One workgroup stores while others still read x; y = x used to be read before it was written."""
    width = dvdq.bench_qlinear_choice(M, N, K, X, Y, WS, 4096)
    assert width in (1, 2)
    end = X + 2 * M * K
    for y in (X, X + 16, end - 16, X - 2 * M * N + 16):
        assert dvdq.bench_qlinear_choice(M, N, K, X, y, WS, 4096) == 0, hex(y)
    for y in (end, X - 2 * M * N):
        assert dvdq.bench_qlinear_choice(M, N, K, X, y, WS, 4096) == width, hex(y)
    for ws, over in ((X, True), (end - 256, True), (X - 4096 + 256, True), (end, False), (X - 4096, False)):
        assert (dvdq.bench_qlinear_choice(M, N, K, X, Y, ws, 4096) == 0) == over, hex(ws)


@pytest.mark.parametrize("M,N,K,width", [(1, 64, 32768, 1), (1, 64, 65536, 0), (32, 64, 512, 1), (33, 64, 512, 1), (32, 64, 520, 0), (16, 64, 1024, 1), (17, 64, 1024, 0),
                                         (10, 64, 1536, 1), (11, 64, 1536, 0), (16, 64, 2048, 1), (17, 64, 2048, 0), (1, 8192, 512, 1), (1, 8193, 512, 2),
                                         (1, 16384, 512, 2), (1, 16385, 512, 0), (8192, 32, 512, 1), (8193, 32, 512, 0)])
def test_lines(M, N, K, width):
    """32 units of 512 channels per 32 tokens, 64 for rows of four units and more; as long as all workgroups run at once."""
    assert dvdq.bench_qlinear_choice(M, N, K) == width
