// Rotate + auto-scale + quantize for gfx950 (Sec. 3.2: X~ = XH by fast Hadamard
// transform; s = ||x~||_inf / qmax per token row; codes = round-half-even(x~ / s)).
//
// One pass over HBM: a token row is read once (bf16), kept in registers while the
// transform, the row abs-max and the quantizer run, and written once (int8 codes,
// 4-bit codes packed two per byte, or 4-bit codes as 6-bit E2M3 patterns for the FP6 matrix
// path; one fp32 scale; optionally the row's code sum for weights with zero-points).  A block-wise scaled mode gives every channel group its own
// power-of-two fraction of the token's step and folds it into the int8 value (see the
// quantizer section of the kernel).  The kernel is bound by HBM only if the transform is
// cheap in VALU instructions, so the 9 butterfly stages of a 512-channel unit are split:
//
//   * channel-index bits 0..4 (strides 1..16) go through the matrix cores: the lane's
//     8 raw bf16 values are the B operand of two 16x16x32 bf16 MFMAs whose A operand
//     is a constant +-1 / 0 matrix (H_32, or I (x) H_2^b for smaller blocks).  The
//     products are exact and the sums are accumulated in fp32.  No bf16 -> fp32
//     unpacking is needed and the result lands in the same lane, same order.
//   * bits 5..8 (strides 32..256) are butterflies between lanes, on fp32 values, with
//     DPP row operations: one fused multiply-add with a DPP operand per value and stage.  A 16-lane row
//     has single-operation pairings l ^ 1, l ^ 2 (quad permutes), l ^ 8 (row rotate) and l ^ 7 (half-row
//     mirror), but none for l ^ 4; 1, 2, 8, 7 is a basis of the row's 16 lane numbers all the same, and a
//     transform whose stages pair along a basis is the Hadamard transform in the coordinates over that
//     basis.  So the 16-byte chunks of a unit are dealt to lanes by those coordinates: the lane whose
//     number is u5 * 1 ^ u6 * 2 ^ u7 * 8 ^ u8 * 7 takes the chunk whose channel-index bits 5..8 are
//     u5 .. u8, and the result lands in place.
//
// Chunk c (16 bytes = 8 channels) of a unit belongs to lane
//   l = (c & 3) << 4 | ((c >> 2 & 1) * 1 ^ (c >> 3 & 1) * 2 ^ (c >> 4 & 1) * 8 ^ (c >> 5 & 1) * 7),
// i.e. lanes l, l+16, l+32, l+48 hold 64 contiguous bytes and a wave instruction still
// covers one contiguous kilobyte.  Rows longer than a few units are spread over the
// waves of a workgroup and the abs-max is combined through LDS.  Workgroups stay
// resident and stride over the rows, prefetching the next row while one is processed.
// The 1/sqrt(B) normalization is never applied to the data: it is folded into the
// scale and into the reciprocal the codes are taken with.
#include <type_traits>

#include "rotate.h"
#include "wave_reduce.h"

namespace dvdq {
namespace {


// CPW = units per wave.  waves_per_row (W) waves share a row; unit u of the row
// belongs to wave (u % W) as its (u / W)-th unit.
// FMT: container of the codes: 0 int8, 1 two 4-bit codes per byte, 2 FP6 (E2M3 patterns, block layout).
template <int LOG2B, int CPW, int FMT>
__global__ __launch_bounds__(1024) void rotate_quant_kernel(
    const uint16_t *__restrict__ x, int64_t M, int K, int waves_per_row, int rows_per_wg,
    double scale_mul,  // 1 / (sqrt(B) * qmax); fp64 so the fp32 scale is rounded once
    float recip_num,   // 1 / sqrt(B)
    int via_lds,       // FMT 1: gather the packed codes through LDS into 16-byte stores (K % 32 == 0);
                       // FMT 2: consecutive rows a wave takes in turn before it strides on (8, 4, 2 or 1)
    int group_log2,    // int8 container only: 0, or log2 of the channel group (7, 8, 9) of block-wise scaling
    int emax,          // block-wise scaling: largest power-of-two refinement of a group's step (8 - act_bits)
    int8_t *__restrict__ codes, float *__restrict__ x_scale,
    int32_t *__restrict__ code_rowsum,    // NULL, or [M]: sum of the row's codes (for weight zero-points)
    unsigned *__restrict__ clear_words) { // NULL, or the slot of tile counters to zero, for the GEMM that follows on the stream
    // (the counters as they lie a line apart, and in one line)
    if (clear_words && blockIdx.x == 0 && threadIdx.x < 16) clear_words[threadIdx.x < 8 ? threadIdx.x * kSchedStride : threadIdx.x - 8] = 0u;
    extern __shared__ float s_amax[];  // [2][rows_per_wg * waves_per_row], slots alternate per iteration
    // then [2][rows_per_wg * waves_per_row] per-wave code sums, then, 16-byte aligned,
    // [waves][CPW][64] dwords for gathering packed codes (via_lds), or [waves][rows in turn][CPW * 384 + 16] bytes for FP6
    int32_t *s_sum = reinterpret_cast<int32_t *>(s_amax) + 2 * rows_per_wg * waves_per_row;
    uint32_t *s_pack = reinterpret_cast<uint32_t *>(s_amax) + (4 * rows_per_wg * waves_per_row + 3) / 4 * 4;
    constexpr bool PACK4 = FMT == 1;
    constexpr int MASK5 = LOG2B >= 5 ? 31 : ((1 << LOG2B) - 1);
    const int lane = threadIdx.x & (kWave - 1);
    // (provably wave-uniform, so that row numbers and row base addresses live in scalar registers)
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int row_in_wg = wave / waves_per_row;
    const int wsub = wave - row_in_wg * waves_per_row;
    const HadamardLane had(lane, MASK5);
    const int chunk = had.chunk;
    const float flip = had.flip(LOG2B);

    // channel offsets of this lane's chunks; chunks at or past K are padding (zero in, nothing out)
    int k0[CPW];
#pragma unroll
    for (int c = 0; c < CPW; ++c) k0[c] = (wsub + c * waves_per_row) * kUnit + chunk * 8;

    // Unit c of this wave is unit wsub + c * waves_per_row of the row; only the last one can lie past the row's
    // end (the launcher gives every wave ceil(units / waves) slots).  Wave-uniform: such a wave branches around
    // the slot's work, which keeps the vector work of the SIMDs of a workgroup even when units do not divide.
    const bool last_unit_present = (wsub + (CPW - 1) * waves_per_row) * kUnit < K;
    auto present = [&] __device__(int c) { return c < CPW - 1 || last_unit_present; };

    // A row is read through a buffer descriptor of its own (base = the row, extent = its K bf16 values, or
    // nothing for rows past M): chunks past the end come back as zeros with no branch around the loads, so the
    // compiler can count the loads in flight and wait only for the row it needs while the next one is on its way.
    // X is read exactly once: streaming loads keep it from displacing the codes this kernel writes (and the
    // weights) from the caches the GEMM is about to read them from.
    auto load_row = [&] __device__(uint4 (&raw)[CPW], int64_t row) {
        const bool ok = row < M;
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t *>(x) + (ok ? row : 0) * K, 0, ok ? K * 2 : 0, 0x00020000);
#pragma unroll
        for (int c = 0; c < CPW; ++c) {
            typedef uint32_t v4u __attribute__((ext_vector_type(4)));
            const v4u t = __builtin_amdgcn_raw_buffer_load_b128(rsrc, k0[c] * 2, 0, 2 /* nt */);
            raw[c] = make_uint4(t[0], t[1], t[2], t[3]);
        }
    };

    // Workgroups stride over groups of rows; the next row's loads are in flight while this one is
    // processed.  A group is rows_per_wg rows handled at once, except for the FP6 container: there the
    // waves of a row take `run` consecutive rows in turn (a group is rows_per_wg runs), because the
    // 16-byte chunks of 8 neighbouring rows make up one 128-byte line of that layout; a wave collects
    // its chunks of a run in LDS and writes them as whole lines (16-byte stores scattered over 64 lines
    // per instruction make the whole kernel take twice as long).
    const int run = FMT == 2 ? via_lds : 1;
    // FP6 write-back of a unit's 24 chunks x run rows: item t * 64 + lane is row (lane % run) of the run and
    // chunk part = (t * 64 + lane) / run of the unit, i.e. slice part / 6, piece part % 6; parts >= 24 are idle
    int wb_in[3], wb_out[3], wb_slice[3];
    const int wb_rr = lane & (run - 1);
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        const int part = (t * kWave + lane) >> __builtin_ctz(run);
        wb_slice[t] = part < 24 ? part / 6 : (1 << 30);   // idle: past every row's slices
        wb_in[t] = wb_rr * (CPW * 384 + 16) + part * 16;
        wb_out[t] = (part / 6) * 3072 + (part % 6) * 512 + wb_rr * 16;
    }
    // The workgroup's iterations are numbered (g, turn): turn counts 0 .. run - 1 within group g, and wave row 0
    // takes row (blockIdx.x + g * gridDim.x) * run * rows_per_wg + turn; wave row r is r * run rows further on.
    // (Counted up by hand: a 64-bit division per iteration costs more than a hundred scalar instructions.)
    const int64_t group_stride = (int64_t)gridDim.x * (run * rows_per_wg);
    int64_t group_row = (int64_t)blockIdx.x * (run * rows_per_wg);   // first row of the current group
    int turn = 0;                                                    // turn of the row being processed
    int64_t row = group_row + row_in_wg * run;
    uint4 raw[CPW];
    load_row(raw, row);
    int slot = 0;
    for (int64_t base = group_row; base < M; slot ^= 1) {
        const bool last_turn = turn == run - 1;
        const int64_t next_group_row = last_turn ? group_row + group_stride : group_row;
        const int next_turn = last_turn ? 0 : turn + 1;
        const int64_t next_base = next_group_row + next_turn;
        uint4 nxt[CPW];
        load_row(nxt, next_base + row_in_wg * run);
        const bool row_ok = row < M;

        float v[CPW][8];
        float amax = 0.f;
#pragma unroll
        for (int c = 0; c < CPW; ++c) {
            if (!present(c)) continue;   // (its values are never read)
            had.low_bits(v[c], raw[c], LOG2B);
        }
#pragma unroll
        for (int c = 0; c < CPW; ++c) {
            if (!present(c)) continue;
            had.high_bits(v[c], LOG2B);
#pragma unroll
            for (int i = 0; i < 8; ++i) amax = fmaxf(amax, fabsf(v[c][i]));
        }
        amax = wave_max(amax);
        if (waves_per_row > 1) {
            float *slots = s_amax + slot * (rows_per_wg * waves_per_row);
            if (lane == 0) slots[wave] = amax;
            __syncthreads();
            amax = 0.f;
            for (int i = 0; i < waves_per_row; ++i) amax = fmaxf(amax, slots[row_in_wg * waves_per_row + i]);
        }
        // scale handed on = amax / (sqrt(B) * qmax); codes = rne(v * (1/sqrt(B)) / scale)
        const float scale = (float)((double)amax * scale_mul);
        const float r = scale > 0.f ? flip * (recip_num / scale) : 0.f;
        // (block-wise scaling stores values that carry a factor 2^emax, see below)
        if (row_ok && wsub == 0 && lane == 0) x_scale[row] = group_log2 ? ldexpf(scale, -emax) : scale;

        const float magic = kRoundMagic;
        int csum = 0;                    // this lane's share of the row's code sum (padding chunks hold zeros)
        if (FMT == 2) {
            // FP6 container (see pack_codes_fp6): the bytes of the group's rows are put together in LDS in channel order.
            constexpr int TURN_BYTES = CPW * 384 + 16;   // + 16: the 8 turns a quarter-wave reads back sit in different banks
            uint8_t *stage = reinterpret_cast<uint8_t *>(s_pack) + wave * (run * TURN_BYTES);
            uint8_t *sp = stage + turn * TURN_BYTES;
            uint8_t *d = sp + chunk * 6;
            uint32_t *d_word = reinterpret_cast<uint32_t *>(d + ((chunk & 1) ? 2 : 0));
            uint16_t *d_half = reinterpret_cast<uint16_t *>(d + ((chunk & 1) ? 0 : 4));
            const bool odd = chunk & 1;
            float fsum = 0.f;   // code sums stay exact in fp32: at most 8 * CPW values of magnitude <= 127
#pragma unroll
            for (int c0 = 0; c0 < CPW; c0 += 4) {
                // q_i = rne(v_i * r) as a float, by the same single-rounding fused multiply-add as the other containers (so that
                // all containers carry identical codes); elements past the lane's last chunk are don't-cares
                fp6_source qa = fp6_undefined(), qb = qa;
#pragma unroll
                for (int g = 0; g < 4 && c0 + g < CPW; ++g) {
                    if (!present(c0 + g)) continue;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        qa[4 * g + i] = fmaf(v[c0 + g][2 * i], r, magic) - magic;
                        qb[4 * g + i] = fmaf(v[c0 + g][2 * i + 1], r, magic) - magic;
                    }
                }
                if (code_rowsum) {
                    // (the empty volatile statement keeps the additions inside this branch: without it the
                    // compiler adds in every launch and selects afterwards, a tenth of the loop's vector work)
                    asm volatile("" : "+v"(fsum));
#pragma unroll
                    for (int g = 0; g < 4 && c0 + g < CPW; ++g) {
                        if (!present(c0 + g)) continue;
#pragma unroll
                        for (int i = 0; i < 4; ++i) fsum += qa[4 * g + i] + qb[4 * g + i];
                    }
                }
                const fp6_fields pk = pack_codes_fp6(qa, qb);
                auto put = [&] __device__(auto g_c) __attribute__((always_inline)) {
                    constexpr int G = decltype(g_c)::value;
                    if (c0 + G < CPW && present(c0 + G)) store_chunk_fp6<G>(pk, odd, d_word + (c0 + G) * 96, d_half + (c0 + G) * 192);
                };
                put(std::integral_constant<int, 0>{});
                put(std::integral_constant<int, 1>{});
                put(std::integral_constant<int, 2>{});
                put(std::integral_constant<int, 3>{});
            }
            if (code_rowsum) csum = (int)fsum;
            if (turn == run - 1 || next_base >= M) {
                // the run is complete (or the rows are): chunk j of slice s of rows row0 .. row0 + run - 1 is the
                // line [row / 32][s][j][row % 32][16 B]; neighbouring lanes take neighbouring rows.  Wave-private
                // LDS, in order: no workgroup barrier.
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                // (row0 is a multiple of `run`, a power of two <= 8: the run lies inside one 32-row block, so a
                // unit's address splits into a wave-uniform 64-bit base and the lane's fixed offsets wb_out[])
                const int64_t row0 = row - turn;
                const int slices = K >> 7;
                uint8_t *run_base = reinterpret_cast<uint8_t *>(codes) + ((row0 >> 5) * slices) * 3072 + (row0 & 31) * 16;
                const int rows_left = (int)min((int64_t)turn, M - 1 - row0);   // rows row0 .. row0 + rows_left exist
                const bool rr_ok = wb_rr <= rows_left;
#pragma unroll
                for (int c = 0; c < CPW; ++c) {
                    if (!present(c)) continue;
                    const int unit = wsub + c * waves_per_row;
                    uint8_t *unit_base = run_base + (int64_t)unit * (4 * 3072);
                    const int slices_here = slices - 4 * unit;   // a row's last unit may hold fewer than 4 slices
#pragma unroll
                    for (int t = 0; t < 3; ++t) {
                        if (t * kWave >= 24 * run) break;
                        if (rr_ok && wb_slice[t] < slices_here)
                            *reinterpret_cast<uint4 *>(unit_base + wb_out[t]) =
                                *reinterpret_cast<const uint4 *>(stage + wb_in[t] + c * 384);
                    }
                }
                __builtin_amdgcn_wave_barrier();   // the next run's LDS writes stay behind these reads
            }
        } else if (PACK4) {
            uint32_t p[CPW];
#pragma unroll
            for (int c = 0; c < CPW; ++c) {
                p[c] = 0;
                if (!present(c)) continue;
                uint32_t b[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) b[i] = __float_as_uint(fmaf(v[c][i], r, magic));
                p[c] = pack_codes_nibbles(b);
                if (code_rowsum) csum = __builtin_amdgcn_sdot8((int)p[c], 0x11111111, csum, false);  // 8 signed nibbles
            }
            if (via_lds) {
                // K % 32 == 0: a unit's 64 dwords (one per lane, in chunk order) are gathered through
                // LDS so that 16 lanes store the unit as 16-byte pieces; wave-private LDS, in-order
                uint32_t *sp = s_pack + wave * (CPW * 64);
#pragma unroll
                for (int c = 0; c < CPW; ++c) sp[c * 64 + chunk] = p[c];
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
                for (int idx0 = 0; idx0 < CPW * 16; idx0 += kWave) {
                    const int idx = idx0 + lane, c = idx >> 4, part = idx & 15;
                    const int k = (wsub + c * waves_per_row) * kUnit + part * 32;  // first channel of the piece
                    if (idx < CPW * 16 && row_ok && k < K)
                        *reinterpret_cast<uint4 *>(codes + (row * K + k) / 2) =
                            *reinterpret_cast<const uint4 *>(sp + c * 64 + part * 4);
                }
                __builtin_amdgcn_wave_barrier();   // the next row's LDS writes stay behind these reads
            } else {
#pragma unroll
                for (int c = 0; c < CPW; ++c)
                    if (row_ok && k0[c] < K) *reinterpret_cast<uint32_t *>(codes + (row * K + k0[c]) / 2) = p[c];
            }
        } else {
#pragma unroll
            for (int c = 0; c < CPW; ++c) {
                if (!present(c)) continue;
                uint32_t b[8];
                if (group_log2) {
                    // Block-wise scaling (a reading of the block-wise variant of Sec. 3.2): a channel group
                    // whose maximum a satisfies a * 2^e <= row maximum is quantized with the step scale / 2^e
                    // (e <= emax, the largest such e) and stored as code * 2^(emax - e), so that one token
                    // scale, scale / 2^emax, dequantizes every group and the GEMM is unchanged.  The lanes of
                    // a group are those that agree in lane bits 2, 3 (128 channels), bit 2 (256), none (512).
                    float a = 0.f;
#pragma unroll
                    for (int i = 0; i < 8; ++i) a = fmaxf(a, fabsf(v[c][i]));
                    // (All in registers, and the exponent without a loop: with LDS shuffles and a loop of ldexp and compares this
                    // mode took 19.5 us for 15600 x 1536, 5 more than without block-wise scaling; now 16.8.  The half-row mirror pairs lanes as l ^ 7, which is l ^ 4 once a quad agrees.)
                    auto max2 = [](float p, float q) { return fmaxf(p, q); };
                    a = fmaxf(a, dpp<DPP_XOR1>(a));
                    a = fmaxf(a, dpp<DPP_XOR2>(a));
                    if (group_log2 >= 9) a = fmaxf(a, dpp<DPP_HALF_MIRROR>(a));
                    if (group_log2 >= 8) a = fmaxf(a, dpp<DPP_ROR8>(a));
                    a = swap_rows<true>(swap_rows<false>(a, max2), max2);
                    // the largest e <= emax with a * 2^e <= amax, from the exponents: a = fa 2^ea, amax = fm 2^em with
                    // fractions in [0.5, 1), so it is em - ea, less one where fa > fm; any e for a = 0 (and, as a
                    // comparison says of them, for an infinite amax)
                    int e = __builtin_amdgcn_frexp_expf(amax) - __builtin_amdgcn_frexp_expf(a) -
                            (__builtin_amdgcn_frexp_mantf(a) > __builtin_amdgcn_frexp_mantf(amax) ? 1 : 0);
                    e = a == 0.f || amax == INFINITY ? emax : min(e, emax);
                    const float rg = ldexpf(r, e);
                    const int sh = emax - e;
#pragma unroll
                    for (int i = 0; i < 8; ++i) b[i] = __float_as_uint(fmaf(v[c][i], rg, magic)) << sh;
                } else {
#pragma unroll
                    for (int i = 0; i < 8; ++i) b[i] = __float_as_uint(fmaf(v[c][i], r, magic));
                }
                const uint2 out = pack_codes_int8(b);
                if (row_ok && k0[c] < K) *reinterpret_cast<uint2 *>(codes + row * K + k0[c]) = out;
                if (code_rowsum) {
                    csum = __builtin_amdgcn_sdot4((int)out.x, 0x01010101, csum, false);  // 4 signed bytes
                    csum = __builtin_amdgcn_sdot4((int)out.y, 0x01010101, csum, false);
                }
            }
        }
        if (code_rowsum) {   // (kernel argument: the whole workgroup takes the same path)
            csum = wave_sum(csum);
            if (waves_per_row > 1) {
                int32_t *slots = s_sum + slot * (rows_per_wg * waves_per_row);
                if (lane == 0) slots[wave] = csum;
                __syncthreads();
                csum = 0;
                for (int i = 0; i < waves_per_row; ++i) csum += slots[row_in_wg * waves_per_row + i];
            }
            if (row_ok && wsub == 0 && lane == 0) code_rowsum[row] = csum;
        }
#pragma unroll
        for (int c = 0; c < CPW; ++c) raw[c] = nxt[c];
        base = next_base;
        row = next_base + row_in_wg * run;
        group_row = next_group_row;
        turn = next_turn;
    }
}

template <int LOG2B>
int launch_cpw(int cpw, dim3 grid, dim3 block, size_t smem, hipStream_t stream, const uint16_t *x, int64_t M,
               int K, int W, int rpw, double scale_mul, float recip_num, int pack4, int group_log2, int emax,
               int8_t *codes, float *x_scale, int32_t *code_rowsum, unsigned *clear_words) {
#define DVDQ_RQ_CASE(C)                                                                                   \
    case C:                                                                                               \
        if (pack4 == 3) {                                                                                 \
            static std::atomic<uint64_t> lds_allowed{0};                                                  \
            allow_dynamic_lds(reinterpret_cast<const void *>(&rotate_quant_kernel<LOG2B, C, 2>),          \
                              kLdsPerCu, lds_allowed);                                                    \
            hipLaunchKernelGGL((rotate_quant_kernel<LOG2B, C, 2>), grid, block, smem, stream, x, M, K, W, \
                               rpw, scale_mul, recip_num, group_log2, 0, 0, codes, x_scale, code_rowsum, clear_words); \
        } else if (pack4)                                                                                   \
            hipLaunchKernelGGL((rotate_quant_kernel<LOG2B, C, 1>), grid, block, smem, stream, x, M, K, W, \
                               rpw, scale_mul, recip_num, pack4 == 2, 0, 0, codes, x_scale, code_rowsum, clear_words); \
        else                                                                                              \
            hipLaunchKernelGGL((rotate_quant_kernel<LOG2B, C, 0>), grid, block, smem, stream, x, M, K, W, \
                               rpw, scale_mul, recip_num, 0, group_log2, emax, codes, x_scale,            \
                               code_rowsum, clear_words);                                                 \
        break;
    switch (cpw) {
        DVDQ_RQ_CASE(1) DVDQ_RQ_CASE(2) DVDQ_RQ_CASE(3) DVDQ_RQ_CASE(4)
        DVDQ_RQ_CASE(5) DVDQ_RQ_CASE(6) DVDQ_RQ_CASE(7) DVDQ_RQ_CASE(8)
        default: return DVDQ_ERR_UNSUPPORTED;
    }
#undef DVDQ_RQ_CASE
    return check_launch();
}

// Waves of a row and units of 512 channels of a wave (the reasons: launch_rotate_quant)
struct RowWaves {
    int waves, units;
    explicit RowWaves(int64_t K) {
        const int all = (int)((K + kUnit - 1) / kUnit);
        waves = (all + 3) / 4;
        if (waves == 3) waves = 4;
        if (waves > 4) waves = (waves + 3) / 4 * 4;   // whole waves per SIMD
        if (waves > 16) waves = 16;
        units = (all + waves - 1) / waves;
    }
};

}  // namespace

// 24 waves for int8 and packed codes where a wave has few units or few rows: with one row loading while one is worked on, a slot's
// rows are as many round trips to memory (16 -> 24 waves, us: 15600 x 1536 int8 15.2 -> 15.0, block-wise 18.2 -> 16.9, 2000 x 5120 9.6 -> 8.6,
// 4096 x 3072 10.2 -> 9.6, 20000 x 1152 packed 14.5 -> 13.5, 100000 x 512 33.5 -> 29.5, 100000 x 256 int8 25.3 -> 21.6).  With three units and
// more than 8 rows a slot it is level, up to 5 % slower (118800 x 3072 201 -> 213); four units or more leave no registers for 24
// (8000 x 3584 block-wise 21.1 -> 23.2); 32 are behind 24 nearly everywhere, and behind 16 for most.
// Where some of the 24 waves' slots have one row and some two, the second row that some of 16 waves take costs less than the additional workgroups:
// layers of 1 unit 1.01 times the time with 24 up to one and a half rows a slot, up to 1.05 (6172 x 384 x 118 9.3 and 9.7 us), of 2 units up to
// a twelfth more than one (6192 x 896 x 112 11.7 and 12.2), 0.98 of 3 units from one on; below one row a slot 5000 x 512 4.5 and 4.9, 6000 x 640 packed 4.9 and 5.2.
int quantizer_waves(int64_t M, int64_t K, int codes_format) {
    const RowWaves row(K);
    const int64_t rows = M * row.waves;
    const bool many = row.units <= 2 || (row.units == 3 && rows <= 8 * 256 * 16);
    return codes_format != DVDQ_CODES_FP6 && many && rows >= 256 * (row.units == 1 ? 36 : row.units == 2 ? 26 : 24) ? 24 : 16;
}

int launch_rotate_quant(const uint16_t *x, int64_t M, int64_t K, int log2_block, int act_bits, int codes_format,
                        int group_log2, int8_t *codes, float *x_scale, int32_t *code_rowsum, hipStream_t stream) {
    const int emax = group_log2 ? 8 - act_bits : 0;
    // 0: int8; 1 / 2: packed nibbles stored per lane / gathered through LDS; 3: FP6 container
    const int pack4 = codes_format == DVDQ_CODES_FP6 ? 3 : (codes_format != DVDQ_CODES_PACKED4 ? 0 : ((K % 32) == 0 ? 2 : 1));
    // Waves per row (RowWaves): at most 4 units (32 fp32 values per lane) in registers per wave, never 3 waves, whole waves
    // per SIMD beyond 4, at most 16.  Workgroups of 8 waves, of 16 once a row takes 8 (two such rows then share a
    // workgroup and its barrier), 16 or 24 waves resident per compute unit (256 of them), every workgroup striding over
    // the rows.  Swept with the kernel timed where the layer runs it, between two GEMMs, over units per wave
    // (3 .. 8) and workgroups of 8 and 16 waves, rows of 2048 .. 16384 channels, both containers: rows of 4, 8 and
    // 16 units are 6-17 % faster as one, two and four waves of 4 units than in waves of 3 or fewer; 12 units are
    // 4 % slower as three waves of 4 than as four of 3; a 13824-channel row (27 units) takes 225 us per launch as
    // eight waves of 3-4 units in 16-wave workgroups, 238 in 8-wave workgroups, 252 as twelve waves of 2-3 units
    // (an earlier state of this rule, chosen from launches timed back to back).  Smaller workgroups stay within 2 % of
    // this on the video-DiT shapes.
    const RowWaves row(K);
    const int W = row.waves, cpw = row.units;
    if (cpw > 8) return DVDQ_ERR_UNSUPPORTED;
    const int wg_waves = W >= 8 ? 16 : 8;
    const int rows_per_wg = W >= wg_waves ? 1 : wg_waves / W;
    const dim3 block(kWave * W * rows_per_wg);
    const int resident = quantizer_waves(M, K, codes_format);
    int wgs_per_cu = resident / (W * rows_per_wg);
    if (wgs_per_cu < 1) wgs_per_cu = 1;
    // FP6: consecutive rows a wave takes in turn (see the kernel): 1, 2, 4 or 8, the largest run that the LDS for collecting
    // them allows and of which there are enough for 13/16 of the resident slots (a row each).  (Whole 128-byte
    // lines need 8 rows, but a wave takes them one after the other: with a run of 8 at any M, 128 rows of 1536 channels took
    // 11.6 us on two workgroups, with runs of one row 4.0.  Swept over the four runs, M = 1024 .. 32760 and 256 .. 13824
    // channels: the best run changes between 1.5 and 1.75, 3 and 3.5, 6 and 6.5 rows per slot.  1536 channels (4096 slots) as
    // runs of 1 / 2 / 4 / 8: 6144 rows 7.0 / 7.9 / 8.5 / 13.0 us, 7168: 8.6 / 8.1 / 8.7 / 13.2, 12288: 13.0 / 10.5 / 12.4 / 14.4,
    // 14336: 15.3 / 13.3 / 12.7 / 14.7, 24576: 29.5 / 21.4 / 19.1 / 21.8, 26624: 32.0 / 23.6 / 23.3 / 22.6, 32760: 39.1 / 28.0 /
    // 25.8 / 25.0.)
    const int64_t wgs_resident = 256 * (int64_t)wgs_per_cu;
    int run = 1;
    if (pack4 == 3) {
        const size_t budget = (kLdsPerCu - 8192) / wgs_per_cu;
        for (run = 8; run > 1 && ((size_t)W * rows_per_wg * run * (cpw * 384 + 16) > budget ||
                                  13 * wgs_resident * rows_per_wg * run > 16 * M);)
            run /= 2;
    }
    const int group_rows = rows_per_wg * run;
    const int64_t wgs_needed = (M + group_rows - 1) / group_rows;
    const dim3 grid((unsigned)(wgs_needed < wgs_resident ? wgs_needed : wgs_resident));
    size_t smem = 4 * sizeof(float) * W * rows_per_wg;   // abs-max slots, then code-sum slots
    if (pack4 == 2) smem = (smem + 15) / 16 * 16 + (size_t)W * rows_per_wg * cpw * 256;
    if (pack4 == 3) smem = (smem + 15) / 16 * 16 + (size_t)W * rows_per_wg * run * (cpw * 384 + 16);
    const double qmax = (double)((1 << (act_bits - 1)) - 1);
    const double norm = 1.0 / sqrt((double)(1 << log2_block));
    const double scale_mul = norm / qmax;
    const float recip_num = (float)norm;
    // the kernel also zeroes the tile counters of the stream: a GEMM enqueued next needs no clearing kernel of its own
    unsigned *clear_words = sched_slot_to_clear(stream);
    int rc = DVDQ_ERR_UNSUPPORTED;
#define DVDQ_RQ_B(L)                                                                                        \
    case L:                                                                                                 \
        rc = launch_cpw<L>(cpw, grid, block, smem, stream, x, M, (int)K, W, rows_per_wg, scale_mul,       \
                             recip_num, pack4, pack4 == 3 ? run : group_log2, emax, codes, x_scale, code_rowsum, clear_words); \
        break;
    switch (log2_block) {
        DVDQ_RQ_B(0) DVDQ_RQ_B(1) DVDQ_RQ_B(2) DVDQ_RQ_B(3) DVDQ_RQ_B(4)
        DVDQ_RQ_B(5) DVDQ_RQ_B(6) DVDQ_RQ_B(7) DVDQ_RQ_B(8) DVDQ_RQ_B(9)
    }
#undef DVDQ_RQ_B
    if (rc != DVDQ_OK && clear_words) sched_slot_not_cleared(stream);
    return rc;
}

}  // namespace dvdq
