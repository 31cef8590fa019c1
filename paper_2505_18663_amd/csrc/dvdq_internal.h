// Internal declarations shared by the translation units of libdvdq (not installed).
#pragma once
#include <hip/hip_runtime.h>
#include <atomic>
#include <stddef.h>
#include <stdint.h>

#include "../../include/dvdq.h"

namespace dvdq {

constexpr size_t kLdsPerCu = 160 * 1024;
constexpr int kCusPerXcd = 32;

// Launchers: arguments are already validated by the C-ABI layer in api.hip.
// Each returns DVDQ_OK or DVDQ_ERR_HIP.
int launch_rotate_quant(const uint16_t *x, int64_t M, int64_t K, int log2_block, int act_bits, int codes_format,
                        int group_log2, int8_t *codes, float *x_scale, int32_t *code_rowsum, hipStream_t stream);


int launch_w4ax_gemm(const int8_t *codes, const float *x_scale, const uint8_t *w, const float *w_scale,
                     const int8_t *w_zero, const int32_t *code_rowsum, const uint16_t *bias, int64_t M, int64_t N,
                     int64_t K, int codes_format, int w_layout, uint16_t *y, int32_t *acc_out, hipStream_t stream);

// W4A4 on the FP6 matrix path (w4a4_fp6_gemm.hip): codes and weights in the FP6 block-slice layouts
int launch_w4a4_fp6_gemm(const uint8_t *codes, const float *x_scale, const uint8_t *w, const float *w_scale,
                         const int8_t *w_zero, const int32_t *code_rowsum, const uint16_t *bias, int64_t M, int64_t N,
                         int64_t K, uint16_t *y, int32_t *acc_out, hipStream_t stream);
// One 4-wave workgroup per compute unit, 128 x 128 wave tiles, accumulators in AGPRs (w4ax_gemm_wide.hip):
// int8 codes x native weights (fp6 = false) or FP6 codes x FP6 native weights (fp6 = true)
int launch_w4ax_gemm_wide(const uint8_t *codes, const float *x_scale, const uint8_t *w, const float *w_scale,
                          const int8_t *w_zero, const int32_t *code_rowsum, const uint16_t *bias, int64_t M, int64_t N,
                          int64_t K, bool fp6, uint16_t *y, int32_t *acc_out, hipStream_t stream);
// Small outputs, any container of codes with its native weight layout, and int8 codes with canonical weights
// (w4ax_gemm_small.hip).  small_gemm_shape: the shape of tile and waves for a size, or -1 (not a small output)
int small_gemm_shape(int64_t M, int64_t N, int64_t K, bool fp6);
constexpr int kSmallVariants = 8, kFirstSmallVariant = 10;   // tile variant 10 + shape stands for a shape
// canonical weights beyond the small outputs (w4ax_gemm.hip): the two-wave kernel; the small kernel's shape 6
constexpr int kCanonicalVariant = 16, kCanonicalShape6Variant = 17;
// the tile variants that the launchers take by themselves, where tiles are drawn from counters and where they are fixed shares
int w4ax_gemm_choice(int64_t M, int64_t N, int64_t K, int codes_format, int w_layout, int vectors, bool drawn);
int w4a4_fp6_gemm_choice(int64_t M, int64_t N, int64_t K, int vectors, bool drawn);
bool tiles_drawn(hipStream_t stream);   // false: the stream is being captured
bool drawing_enabled();                 // the benchmark hook
// waves of the row quantizer that are resident on a compute unit (rotate_quant.hip)
int quantizer_waves(int64_t M, int64_t K, int codes_format);
// The tiles of the two-wave kernels: 128 x 128, three workgroups per compute unit (true), or 128 x 256, two (false).  The larger tile
// moves a third fewer operand bytes per product with int8 codes, a quarter fewer with packed and FP6 ones, and has a round of 512 tiles done in some 26 us where 768 small ones take 21 (12 slices,
// bias and zero-points): 7 % less per output.  What decides is the last round, in which compute units hold one large tile or two, one
// small tile, two or three, at 14, 26 and 9, 14.5, 21 us.  So: small tiles unless they take a round more.  Over 5450 outputs of 100 to
// 2500 large tiles that these kernels take (int8, packed and FP6 codes, 2 to 48 slices, drawn and captured) small tiles have 0.84 to 0.87 of the
// time there in the mean, at most 1.10: below one round 0.67 to 0.88 (7800 x 1536 x 1440 int8 23.8 -> 21.9 us, packed 23.1 -> 20.0, 90678 x 896
// x 640 75.1 -> 63.0, FP6 2048 x 768 x 3072 10.6 -> 8.9, canonical 6200 x 1440 x 1440 24.2 -> 22.4), from 1.02 rounds on 0.75 to 0.96.  Where they
// take a round more: 0.86 to 1.13 there, two for one 1.04 to 1.2 (FP6 1.06 to 1.4), three for two 0.98 to 1.05 (FP6 1.05 to 1.17), from four for three on
// below six slices 0.91 to 0.95, six to eleven 0.94 to 1.00, beyond 0.97 to 1.07 (drawn; the GEMM alone); the line does not follow these.  Not in a last round that is at most half full of large tiles and more than two thirds full of
// small ones, from 20 slices on in the second round (1.01 to 1.04 there, int8 to canonical, up to 1.10; 0.90 to 0.99 with fewer slices) and
// from 48 on later (20912 x 13568 x 1664 int8 571 and 583 us; 0.88 to 1.00 with fewer).
// Canonical weights, half a cache line of a weight row per slice, have less to gain and lose more by code rows that are read again for each
// column of tiles.  Whole layers, small over large, 4700 outputs, the cases that keep large tiles: one round, up to 256 channels from 24
// slices on 1.03 (1.10 at most), up to 512 in 577 small tiles and more from 48 on 1.02 (1.06); two rounds, up to 256 channels from 12 on 1.02
// (1.10), up to 384 from 36 on 1.01 (1.08); three and more, up to 384 channels from 26 on 1.02 (1.08) unless less than a quarter of the
// last small round is there, else a last large round that is nearly empty, next to half a small one from 24 on 1.01 (1.10) or, drawn, next to one
// three quarters full 1.03 (1.11; 0.94 with fixed shares, which deal a nearly empty round of large tiles to one XCD).  The rest 0.95 in the mean, 88 of 3500
// above 1.03 (96274 x 4704 x 320 472 us with small, 436 with large tiles, 54984 x 7584 x 301 479 and 445).  int8 codes have the last of these from 36 slices on, 1.02
// (1.04: 10020 x 4992 x 3352 194 and 187).
inline bool narrow_tiles(int64_t M, int64_t N, int64_t K, int codes_format, int w_layout, bool drawn) {
    const int64_t rows = (M + 127) / 128, columns = (N + 127) / 128, large = rows * ((N + 255) / 256), small = rows * columns, slices = K / 128;
    if ((small + 767) / 768 > (large + 511) / 512) return false;
    const int64_t last_large = (large - 1) % 512, last_small = (small - 1) % 768;
    if (w_layout == DVDQ_W_CANONICAL) {
        if (large <= 512) {
            if (slices >= (columns <= 2 ? 24 : 48) && columns <= (small > 576 ? 4 : 2)) return false;
        } else if (large <= 1024) {
            if (columns <= 3 && slices >= (columns <= 2 ? 12 : 36)) return false;
        } else {
            if (columns <= 3 && slices >= 26 && last_small >= 192) return false;
            if (last_small >= 576 ? drawn && last_large < 192 && slices >= 20 : last_small >= 384 && last_large < 64 && slices >= 24) return false;
        }
    } else if (codes_format == DVDQ_CODES_INT8) {
        if (drawn && large > 1024 && last_large < 128 && last_small >= 576 && slices >= 36) return false;
    }
    return !(large > 512 && last_large < 256 && last_small >= 512 && slices >= (large <= 1024 ? 20 : 48));
}
// (asked of the stream only where the answer depends on it)
inline bool narrow_tiles(int64_t M, int64_t N, int64_t K, int codes_format, int w_layout, hipStream_t stream) {
    const bool if_drawn = narrow_tiles(M, N, K, codes_format, w_layout, true), if_fixed = narrow_tiles(M, N, K, codes_format, w_layout, false);
    return if_drawn == if_fixed || tiles_drawn(stream) ? if_drawn : if_fixed;
}
// 128 x 128 tiles (narrow_tiles takes them for all of these) for outputs of the largest of the small shapes, a wave or two per 64 x 128 tile.
// Both run in one round, so what counts is the fullest compute unit: two large tiles against three small ones, 256 rows to 192, up to 768 small
// tiles, against four beyond, and there are fewer bytes to read with the large ones.  Whole layers, large over small by the number of
// slices, in the mean (worst), N a multiple of 8 / any other N (tiles that are stored unaligned):
//   up to 768   int8    below 10: 0.95 to 0.98 (1.07), from 10 on 0.99 to 1.08 (1.13)  /  0.98 to 1.07 (1.14)
//               packed  below 6: 0.96 to 0.97 (1.06), 6 and 7 from 321 large tiles on 0.98, from 8 on 0.99 to 1.01 (1.07)  /  0.98 to 1.03 (1.07)
//               FP6     below 6: 0.93 to 0.96 (1.06), from 6 on 0.99 to 1.03 (1.10)  /  below 4: 0.95 to 0.98 (1.05), from 4 on 0.99 to 1.04 (1.12)
//   beyond      int8    0.90 to 0.98 (1.06)                                       /  one slice 0.99 (1.05), then 0.94 to 0.99 (1.07)
//               packed  below 10: 0.92 to 0.97 (1.05), 10 and 11 0.99 (1.05)      /  below 6: 0.95 to 0.98 (1.04), from 6 on 0.99 to 1.01 (1.07)
// 3000 outputs of int8 codes, 2600 packed, 3500 FP6 (5000 x 1536 x 1536 int8 19.4 -> 16.8 us the GEMM alone; with small tiles as before: 263 x
// 2304 x 13637 int8 23.6 us the layer, 25.2 with large ones, 615 x 1024 x 6561 FP6, two GEMMs, 24.3 and 27.2, 676 x 5376 x 8696 int8 45.3 and 51.0).
inline bool narrow_for_small_outputs(int64_t M, int64_t N, int64_t K, int codes_format) {
    const int64_t columns = (N + 127) / 128, large = ((M + 127) / 128) * columns, slices = K / 128;
    const bool beyond = ((M + 63) / 64) * columns > 768, aligned = (N & 7) == 0;
    if (large > 512) return false;   // (more than two on a compute unit)
    switch (codes_format) {
        case DVDQ_CODES_INT8: return beyond ? aligned || slices > 1 : aligned && slices < 10;
        case DVDQ_CODES_PACKED4: return slices < (beyond ? (aligned ? 10 : 6) : aligned ? (large > 320 ? 8 : 6) : 0);
        default: return slices < (aligned ? 6 : 4);
    }
}
// whether the large kernels store their tiles as whole lines, with 32-bit offsets
constexpr int64_t kMaxTileN = (int64_t)1 << 22;
inline bool whole_line_tiles(int64_t N) { return (N & 7) == 0 && N < kMaxTileN; }
// whether the two-wave kernels store them as 16-byte pieces at even addresses
inline bool unaligned_tiles(int64_t N) { return (N & 7) != 0 && N >= 8 && N < kMaxTileN; }
int launch_w4ax_gemm_small(const uint8_t *codes, const float *x_scale, const uint8_t *w, const float *w_scale,
                           const int8_t *w_zero, const int32_t *code_rowsum, const uint16_t *bias, int64_t M, int64_t N,
                           int64_t K, int codes_format, int w_layout, int shape, uint16_t *y, int32_t *acc_out, hipStream_t stream);
// A whole layer of few tokens in one launch (w4ax_gemm_small.hip).  qlinear_choice: 0 (two launches), or the tile width to take
int qlinear_choice(const void *x, const void *y, const void *workspace, size_t workspace_bytes, int64_t M, int64_t N, int64_t K);
int launch_qlinear_small(const uint16_t *x, int log2_block, int act_bits, const uint8_t *w, const float *w_scale,
                         const int8_t *w_zero, const uint16_t *bias, int64_t M, int64_t N, int64_t K, int codes_format,
                         int w_layout, int width, uint16_t *y, uint8_t *codes, float *x_scale, int32_t *code_rowsum, hipStream_t stream);
size_t w4_native_fp6_bytes(int64_t N, int64_t K);
size_t codes_fp6_bytes(int64_t M, int64_t K);
int launch_w4_prepack_fp6(const uint8_t *w_canonical, int64_t N, int64_t K, uint8_t *w_native, hipStream_t stream);

size_t w4_native_bytes(int64_t N, int64_t K);
int gemm_variant();            // the benchmark hook's tile variant (-1: the kernels' own choice)
void set_gemm_variant(int v);  // benchmark sweeps only; -1 = choose by shape
void set_gemm_schedule(int v); // benchmark only; 0 = fixed tile shares, -1 = drawn from counters where possible
void set_gemm_grid_limit(int v); // benchmark only; 0 = persistent grids fill the chip, else at most v workgroups
int limited_grid(int grid);
// A slot of tile counters: a word per XCD, each in a 64-byte line of its own.  Atomics on one line are served one after the other,
// whatever words they name: with the eight in one line the 256 workgroups that start together waited 3200 clocks (median; at
// most 6000 to 8000) for their first reply, apart 1200 (2100), and 1650 against 760 later on.  Time apart over time in one line, launches that
// draw, K 128 to 6000: two-wave kernels 0.96 in the mean with packed codes, 0.93 with int8, 0.89 with FP6, at most 1.04.
// The wide kernels keep their eight in one line (words 0 to 7 of the slot).  Replies that come one after the other keep the epilogues of
// their lone workgroups apart; a line each, they fall into step, and how dear that is differs from card to card: FP6 0.99 in the mean
// (0.95 to 1.01) on two, on a third up to 1.19 (35129 x 1280 x 2648 102 -> 119 us, 32760 x 1536 x 4608 152 -> 163, 18973 x 1024 x 3216
// 61.8 -> 69.8, its layer 75.1 -> 85.4).
constexpr int kSchedStride = 16, kSchedWords = 8 * kSchedStride;
// the stream's tile-counter slot (nullptr: fixed tile shares): for a GEMM, with whether the kernel enqueued last
// on the stream zeroes it; for a quantizer, the words to zero, noted as zeroed unless taken back (w4ax_gemm.hip)
unsigned *sched_slot(hipStream_t stream, bool *is_clear);
unsigned *idle_slot(hipStream_t stream);   // words for launches that have nothing to draw (nullptr: fixed tile shares)
unsigned *sched_slot_to_clear(hipStream_t stream);
void sched_slot_not_cleared(hipStream_t stream);
void release_sched_slot(hipStream_t stream);               // forget a stream's tile-counter slot (host bookkeeping only)
int fill_sched_slots(uint32_t value, hipStream_t stream);  // robustness tests only: overwrite every tile counter

int launch_w4_prepack(const uint8_t *w_canonical, int64_t N, int64_t K, uint8_t *w_native, hipStream_t stream);

size_t gbs_workspace_bytes();
void set_gbs_wait(int64_t ticks);   // tests only
int launch_gbs_reset(void *state, int bits, hipStream_t stream);
int launch_gbs_step(const uint16_t *ft, const uint16_t *fp, int64_t n, double delta, int b_low, int b_high,
                    void *state, void *workspace, hipStream_t stream);

int bgr_choice(int64_t N, int64_t K, int n_steps, int max_refine);   // threads per workgroup
int launch_bgr(const float *w, int64_t N, int64_t K, int n_steps, int max_refine, double eps, int search,
               uint8_t *w_packed, float *w_scale, int8_t *w_zero, double *row_error, hipStream_t stream);

// Raise a kernel's dynamic-LDS limit to `bytes` once per kernel and device (`done` is the call
// site's own bit mask of devices already configured).  Not a stream operation: after the first
// launch on a device nothing but the launch itself is issued, also under stream capture.
inline void allow_dynamic_lds(const void *kernel, size_t bytes, std::atomic<uint64_t> &done) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return;
    const uint64_t bit = dev >= 0 && dev < 64 ? (uint64_t)1 << dev : 0;
    if (bit && (done.load(std::memory_order_acquire) & bit)) return;
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) == hipSuccess && bit)
        done.fetch_or(bit, std::memory_order_release);
}

inline int check_launch() { return hipGetLastError() == hipSuccess ? DVDQ_OK : DVDQ_ERR_HIP; }

}  // namespace dvdq
