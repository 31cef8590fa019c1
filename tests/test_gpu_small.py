"""Small-output GEMM kernel (K slices dealt to the waves of a workgroup): every tile shape and every container of
codes, at the edges of tiles, with fewer K slices than waves and with remainders, against exact integer sums and
bit for bit against the large-tile kernels."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_18663_amd as dvdq
from parity import check_y

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

FORMATS = {"int8": dvdq.CODES_INT8, "packed4": dvdq.CODES_PACKED4, "fp6": dvdq.CODES_FP6}
SIZES = [
    # M, K, N
    (1, 128, 1),          # one token, one channel, one slice: seven of eight waves have nothing to do
    (31, 128, 33),        # both sides of a 32 x 32 tile
    (33, 640, 70),        # slices do not divide over the waves; N not a multiple of 8
    (64, 1152, 128),      # whole tiles of every shape
    (65, 1024, 264),      # one row and one piece over
    (130, 2176, 1160),    # 17 slices
    (700, 256, 520),
]


@pytest.fixture(autouse=True)
def _restore():
    yield
    dvdq.bench_set_gemm_variant(-1)


@pytest.mark.parametrize("fmt", list(FORMATS))
@pytest.mark.parametrize("M,K,N", SIZES)
def test_every_shape_is_exact_and_equal_to_the_large_tiles(M, K, N, fmt):
    rng = np.random.default_rng(M * 7919 + K + N)
    bits = 8 if fmt == "int8" else 4
    q = 2 ** (bits - 1) - 1
    codes = rng.integers(-q, q + 1, (M, K)).astype(np.int8)
    wc = rng.integers(-8, 8, (N, K)).astype(np.int8)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    pack = {"int8": lambda c: c, "packed4": oracle.pack_a4, "fp6": oracle.pack_fp6}[fmt]
    w = (dvdq.w4_prepack_fp6 if fmt == "fp6" else dvdq.w4_prepack)(d(oracle.pack_w4(wc)))
    lay = dvdq.W_NATIVE_FP6 if fmt == "fp6" else dvdq.W_NATIVE
    xs, ws = d((rng.random(M) + 0.01).astype(np.float32)), d((rng.random(N) * 0.01 + 1e-3).astype(np.float32))
    bias = d(rng.standard_normal(N).astype(np.float32)).to(torch.bfloat16)
    wz = rng.integers(-8, 8, N).astype(np.int8)
    rowsum = codes.astype(np.int64).sum(axis=1)
    plain = codes.astype(np.int64) @ wc.astype(np.int64).T
    c_dev = d(pack(codes))
    for zero in (False, True):
        kw = dict(bias=bias if zero or N % 3 else None, codes_format=FORMATS[fmt], K=K)
        if zero:
            kw.update(w_zero=d(wz), code_rowsum=d(rowsum.astype(np.int32)))
        acc_ref = plain - rowsum[:, None] * wz[None, :].astype(np.int64) if zero else plain

        def run(variant):
            print(f"small M{M} K{K} N{N} {fmt} zero={zero} variant {variant}", flush=True)
            dvdq.bench_set_gemm_variant(variant)
            y, acc = dvdq.w4ax_gemm(c_dev, xs, w, ws, bits, lay, want_acc=True, **kw)
            y2 = dvdq.w4ax_gemm(c_dev, xs, w, ws, bits, lay, **kw)
            torch.cuda.synchronize()
            assert torch.equal(y.view(torch.int16), y2.view(torch.int16))
            return y, acc

        y_large, _ = run(1 if fmt == "fp6" else 2)
        for variant in (-1, 10, 11, 12, 13, 14, 15, 16):
            y, acc = run(variant)
            assert np.array_equal(acc.cpu().numpy().astype(np.int64), acc_ref), f"variant {variant} zero {zero}"
            assert torch.equal(y.view(torch.int16), y_large.view(torch.int16)), f"variant {variant} zero {zero}"


@pytest.mark.parametrize("M,K,N", [(1, 32, 1), (33, 96, 40), (65, 1440, 331), (64, 128, 128), (130, 2080, 264), (1100, 224, 2056)])
def test_canonical_weights_every_shape_exact(M, K, N):
    """K a multiple of 32: last slices of 32, 64 and 96 channels, a single part of a slice"""
    rng = np.random.default_rng(M + K + N)
    codes = rng.integers(-127, 128, (M, K)).astype(np.int8)
    wc = rng.integers(-8, 8, (N, K)).astype(np.int8)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    xs, ws = (rng.random(M) + 0.01).astype(np.float32), (rng.random(N) * 0.01 + 1e-3).astype(np.float32)
    bias = d(rng.standard_normal(N).astype(np.float32)).to(torch.bfloat16)
    bias_bits = bias.cpu().view(torch.int16).numpy().view(np.uint16)
    y_ref, acc_ref = oracle.w4ax_gemm(codes, xs, oracle.pack_w4(wc), ws, bias_bits, return_acc=True)
    for variant in (-1, 10, 11, 12, 13, 14, 15, 16):
        print(f"canonical M{M} K{K} N{N} variant {variant}", flush=True)
        dvdq.bench_set_gemm_variant(variant)
        y, acc = dvdq.w4ax_gemm(d(codes), d(xs), d(oracle.pack_w4(wc)), d(ws), 8, dvdq.W_CANONICAL, bias=bias, want_acc=True)
        torch.cuda.synchronize()
        assert np.array_equal(acc.cpu().numpy().astype(np.int64), acc_ref), f"variant {variant}"
        check_y(y.cpu().view(torch.int16).numpy().view(np.uint16), y_ref, f"canonical variant {variant}", bias_bits)
