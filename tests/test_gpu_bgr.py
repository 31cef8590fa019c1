"""GPU parity of the offline weight quantizer (Bounded-init Grid Refinement, Sec. 3.1 / Alg. 1)
against the oracle.  Both sides compute in fp64 and differ only in summation order, so grids
and codes are expected to be identical; a row may differ only if the two searches tie to
within rounding, in which case its error must still equal the oracle's (budget below)."""
import numpy as np
import pytest
import torch

import dvdq_inputs as di
import oracle
import paper_2505_18663_amd as dvdq
from parity import check_y

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def gpu_bgr(w, **kw):
    wp, ws, wz, err = dvdq.bgr_quantize(dev(w), want_error=True, **kw)
    torch.cuda.synchronize()
    q = oracle.unpack_w4(wp.cpu().numpy()).astype(np.int16) + 8          # back to the unsigned codes 0..15
    return q.astype(np.uint8), ws.cpu().numpy(), wz.cpu().numpy().astype(np.int32) + 8, err.cpu().numpy()


def compare(w, label, **kw):
    q_g, d_g, z_g, e_g = gpu_bgr(w, **kw)
    q_r, d_r, z_r, e_r = oracle.bgr(w, **kw)
    same = (z_g == z_r) & (d_g == d_r.astype(np.float32)) & np.all(q_g == q_r, axis=1)
    # errors agree to fp64 summation-order noise on every row, identical grid or not
    assert np.all(np.abs(e_g - e_r) <= 1e-9 * np.maximum(e_r, 1e-300)), f"{label}: row errors differ"
    budget = int(np.ceil(0.005 * w.shape[0]))
    assert (~same).sum() <= budget, f"{label}: {(~same).sum()} rows with a different grid (budget {budget})"
    # whatever grid the GPU returned, its codes are the Quant equation on that grid (checked in fp64 here)
    q_expect = np.clip(np.rint(w.astype(np.float64) / d_r[:, None]) + z_g[:, None], 0, 15).astype(np.uint8)
    assert np.array_equal(q_g[same], q_expect[same])
    return dict(rows=w.shape[0], differing=int((~same).sum()), max_rel_err_diff=float(np.max(np.abs(e_g - e_r) / np.maximum(e_r, 1e-300))))


@pytest.mark.parametrize("N,K,kw", [
    (96, 64, {}), (96, 256, {}), (256, 1536, {}), (64, 3072, {}), (24, 13824, {}), (5, 32768, dict(n_steps=20)),
    (96, 1536, dict(n_steps=16, max_refine=0)), (96, 1536, dict(n_steps=40, max_refine=3)),
    (96, 1536, dict(eps=1e-4)), (7, 130, dict(n_steps=7, max_refine=2)),
    (96, 256, dict(search=1)), (128, 1536, dict(search=1)), (96, 1536, dict(search=1, n_steps=16, max_refine=0)),
    (96, 1536, dict(search=1, eps=1e-4)), (24, 13824, dict(search=1)),
])
def test_bgr_matches_the_oracle_on_gaussian_rows(N, K, kw):
    rng = np.random.default_rng(N * 7 + K)
    w = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    w[0] += 0.05                                   # not zero-mean
    w[1, :4] = [0.4, -0.5, 0.45, -0.38]            # outliers
    print(compare(w, f"N{N} K{K} {kw}", **kw))


def test_bgr_special_rows():
    rng = np.random.default_rng(1)
    K = 256
    rows = [np.zeros(K), np.full(K, 0.37), np.full(K, -2.5),                      # constant rows: exact
            0.125 * (rng.integers(0, 16, K) - 3.0),                              # already on a grid: exact
            rng.standard_normal(K) * 0.1 + 5.0,                                  # all positive: zero-point pinned at 0
            np.concatenate([[1.0], np.zeros(K - 1)]),                            # one spike
            rng.standard_t(3, K) * 0.02]                                         # heavy tails
    rows[3][:16] = 0.125 * (np.arange(16) - 3.0)
    w = np.stack(rows).astype(np.float32)
    # exact: constant rows in either search; the on-grid row where plain MinMax (i = 0) is a candidate
    for search, exact in ((dvdq.BGR_BEST_OF_ALL, 4), (dvdq.BGR_LISTING, 3)):
        q_g, d_g, z_g, e_g = gpu_bgr(w, search=search)
        q_r, d_r, z_r, e_r = oracle.bgr(w, search=search)
        assert np.array_equal(z_g, z_r) and np.array_equal(d_g, d_r.astype(np.float32)) and np.array_equal(q_g, q_r)
        assert np.allclose(e_g, e_r, rtol=1e-9, atol=0)
        assert np.all(e_g[:exact] == 0)
        deq = d_g[:exact, None].astype(np.float64) * (q_g[:exact].astype(np.float64) - z_g[:exact, None])
        assert np.array_equal(deq, w[:exact].astype(np.float64))


def test_bgr_weights_through_the_layer():
    """fp32 weights -> BGR on the GPU -> pre-pack -> the whole layer with zero-points; the outputs
    match the oracle's zero-point GEMM on the GPU's own codes, and the layer is closer to the
    float layer than with plain MinMax weights (what the quantizer is for)."""
    wl = di.WORKLOADS[0]
    M, K, N, B = wl.M, wl.K, wl.N, wl.had_block
    rng = np.random.default_rng(11)
    w = (rng.standard_t(5, (N, K)) * 0.02).astype(np.float32)
    xb = di.make_x(wl)
    x_dev = torch.from_numpy(xb.view(np.int16)).view(torch.bfloat16).to(DEV)
    wp, ws, wz = dvdq.bgr_quantize(dev(w))
    y, wsp = dvdq.qlinear(x_dev, dvdq.w4_prepack(wp), ws, B, 8, dvdq.W_NATIVE, w_zero=wz)
    torch.cuda.synchronize()
    codes, scale = dvdq.workspace_views(wsp, M, K)
    y_ref = oracle.w4ax_gemm_zp(codes.cpu().numpy(), scale.cpu().numpy(), wp.cpu().numpy(), ws.cpu().numpy(),
                                wz.cpu().numpy())
    check_y(y.cpu().contiguous().view(torch.int16).numpy().view(np.uint16), y_ref, "bgr layer")
    # against the float layer  (X H)(W)^T  with W taken as already rotated
    xr = oracle.rotate(xb, B)
    y_float = xr @ w.astype(np.float64).T
    q_mm, d_mm, z_mm, _ = oracle.minmax_quant(w)
    w_mm = d_mm[:, None] * (q_mm.astype(np.float64) - z_mm[:, None])
    err_bgr = np.linalg.norm(y.float().cpu().numpy().astype(np.float64) - y_float)
    err_mm = np.linalg.norm(xr @ w_mm.T - y_float)
    assert err_bgr < err_mm


# One row length on each side of every change of the kernel's launch shape (rows in registers, prefix-sum spacing, number of
# value cells) and the shortest and longest rows; more rows than compute units where that decides as well.
@pytest.mark.parametrize("N,K", [(3, 2), (5, 30), (9, 1026), (300, 2048), (300, 2050), (9, 4098), (260, 10240), (258, 10242),
                                 (257, 14336), (257, 14338), (4, 16384), (4, 16386)])
@pytest.mark.parametrize("search", [dvdq.BGR_LISTING, dvdq.BGR_BEST_OF_ALL])
def test_bgr_row_lengths_around_the_launch_shapes(N, K, search):
    rng = np.random.default_rng(N + K)
    w = (rng.standard_normal((N, K)) * 0.02).astype(np.float32)
    print(compare(w, f"N{N} K{K} search{search}", n_steps=9, max_refine=3, search=search))


@pytest.mark.parametrize("K", [512, 4096, 20000])
@pytest.mark.parametrize("search", [dvdq.BGR_LISTING, dvdq.BGR_BEST_OF_ALL])
def test_bgr_crowded_rows(K, search):
    """Rows whose weights crowd into few value cells (the sorted row then comes from another network), weights that sit
    exactly on thresholds, and rows that a grid fits almost exactly (the expanded squared error would cancel)."""
    rng = np.random.default_rng(K)
    g = rng.standard_normal(K)
    rows = [np.where(rng.random(K) < 0.9, 0.0, g), g * 0.02 + np.eye(1, K, 7)[0] * 1e6, 5.0 + 1e-3 * g, -3.0 + 1e-6 * g,
            np.round(g * 4) / 8, 0.25 * (rng.integers(0, 16, K) - 6) + 1e-7 * g, np.sign(g) * np.abs(g) ** 5,
            np.where(np.arange(K) < 2, [[-1.0], [1.0]][0] + 2.0 * (np.arange(K) == 1), 1e-4 * g), g * 1e-30, np.exp(3 * g)]
    print(compare(np.stack(rows).astype(np.float32), f"K{K} search{search}", n_steps=30, max_refine=6, search=search))


def _exact_listing_error(w, n_steps, refine):
    """The error of the listing's best grid for one row with every sum in 80-bit arithmetic: starts i = 1, 2, ..., at
    most one refinement round each.  Grids are computed as the definition says, in fp64, from the sums rounded once."""
    L = np.longdouble
    wl, K = w.astype(L), len(w)
    w = w.astype(np.float64)
    lo0, hi0 = w.min(), w.max()
    step, mean, best = (hi0 - lo0) / n_steps, float(wl.sum()) / K, np.inf

    def sums(delta, z):
        c = np.clip(np.rint(w / delta) + z, 0, 15)
        d = (c - z).astype(L)
        r = wl - L(delta) * d
        return np.sqrt((r * r).sum()), float((d * wl).sum()), float((d * d).sum()), c.sum()

    for i in range(1, n_steps + 1):
        lo, hi = lo0 + i * step, hi0 - i * step
        if not lo < hi:
            break
        delta = (hi - lo) / 15
        e, num, den, sq = sums(delta, np.clip(np.rint(-(lo / delta)), 0, 15))
        if refine and den > 0 and num / den > 0:
            delta = num / den
            e = sums(delta, np.clip(np.rint(sq / K - mean / delta), 0, 15))[0]
        best = min(best, e)
    return best


@pytest.mark.parametrize("refine", [0, 1])
@pytest.mark.parametrize("K", [6, 1536, 8960, 20000])
def test_bgr_row_error_is_rounded_once(K, refine):
    """row_error is sqrt of a squared error whose sums are not rounded on the way (2^-53), then rounded itself (2^-53):
    1.5 * 2^-53 = 1.7e-16 together, and the yardstick's own K additions of 2^-64 (sqrt(K) of them: 1e-17)."""
    rng = np.random.default_rng(K + refine)
    g = rng.standard_normal(K)
    rows = [g * 0.02, 3.0 + 0.1 * g, -1.0 + g, np.sign(g) * np.abs(g) ** 3, np.exp(2 * g), g * 1e-30, g * 1e30,
            0.25 * (rng.integers(0, 16, K) - 6) + 5e-3 * g, 0.25 * (rng.integers(0, 16, K) - 6) + 2e-2 * g,
            np.where(np.arange(K) < 3, 200.0 * g, 0.01 * g)]
    w = np.stack(rows).astype(np.float32)
    _, _, _, err = dvdq.bgr_quantize(torch.from_numpy(w).to(DEV), n_steps=20, max_refine=refine, eps=0.0, want_error=True,
                                     search=dvdq.BGR_LISTING)
    torch.cuda.synchronize()
    err = err.cpu().numpy()
    rel = [abs(float((np.longdouble(e) - x) / x)) for e, x in zip(err, (_exact_listing_error(r, 20, refine) for r in w))]
    print(f"K{K} refine{refine}:", " ".join(f"{r:.1e}" for r in rel))
    assert max(rel) <= 2e-16, rel


def test_bgr_more_rows_than_one_launch_takes():
    """2^23 + 5 rows of two weights: at 512 threads a row, a launch of 2^32 threads, the grid limit, is full before that.
    Constant rows, whose grid is known, and one that has to be searched at the end."""
    N = 2 ** 23 + 5
    w = torch.randint(-3, 4, (N, 1), device=DEV).float().expand(N, 2).contiguous()
    w[-1] = torch.tensor([-0.3, 0.7], device=DEV)
    wp, ws, wz, err = dvdq.bgr_quantize(w, n_steps=5, max_refine=2, want_error=True)
    torch.cuda.synchronize()
    c = w[:-1, 0]
    assert torch.equal(ws[:-1], torch.where(c == 0, torch.ones_like(c), c.abs()))
    assert torch.equal(wz[:-1], (c < 0).to(torch.int8) - 8) and not err[:-1].any()
    q = (c > 0).to(torch.uint8)
    assert torch.equal(wp[:-1, 0], ((q + 8) & 15) * 17)
    q_r, d_r, z_r, e_r = oracle.bgr(w[-1:].cpu().numpy(), n_steps=5, max_refine=2)
    assert float(ws[-1]) == np.float32(d_r[0]) and int(wz[-1]) + 8 == z_r[0] and abs(float(err[-1]) - e_r[0]) <= 1e-15
    assert (int(wp[-1, 0]) ^ 0x88) == int(q_r[0, 0]) | int(q_r[0, 1]) << 4
