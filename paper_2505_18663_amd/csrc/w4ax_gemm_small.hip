// W4Ax GEMM for outputs too small to fill the chip with the tiles of w4ax_gemm.hip and w4a4_fp6_gemm.hip
// (Sec. 3.2: Y = X^ Lambda W^^T; Sec. 3.1 DeQuant, optional zero-points): few tokens, or few output channels.
//
// What bounds such a product is neither the matrix cores nor HBM but the chain of K slices a workgroup walks: with
// one 128 x 256 tile per workgroup and 12 to 108 slices in series, each slice costs a round trip to the L2 or to
// memory while most compute units have no tile at all.  So here the tile is small (32 x 32 to 64 x 128), the K
// slices are dealt to the waves of the workgroup, each wave accumulates the WHOLE tile over its share, and the
// shares are added up through LDS at the end (integers, or fp32 sums that are exact integers: any order gives the
// same bits).  The waves run independently: no barrier before the reduction.
//
//   weights: straight from the native layouts into registers; a fragment load is one contiguous run per wave.
//   codes:   FP6 likewise.  The row-major containers are loaded as whole lines (rows of a slice: 128 or 64 bytes) and
//            turned into fragments through the wave's own LDS; fetched as fragments directly, a load instruction
//            would touch 32 lines.
//            Canonical weights ([N, K/2] as an offline quantizer hands them over, K any multiple of 32) take the same way.
//   K tails, rows past M: loads past the end of a buffer descriptor return zeros (zero codes add nothing).
//
// A layer of very few tokens (CPW > 0) is one launch: the workgroup also quantizes its own tokens, into LDS, before it
// multiplies, while its first weights are on their way.  Two launches in a row cost such a layer a launch's start and end, and a
// round trip of the codes through memory, more than quantizing the same tokens in every workgroup does (qlinear_choice).
// It is bound by the chain load - transform - maximum - codes - slices - sum, a few waits each.
//
// Measured (back-to-back launches, int8 codes, before -> now): 2 x 1536 x 9216 (tokens x K x channels): 22.6 -> 4.4 us;
// 512 x 3072 x 3072: 28.0 -> 10.7; 1 x 13824 x 5120: 104 -> 10.5; 3121 x 1152 x 1160: 27.7 -> 9.8.  Towards the upper
// end of the range the operand traffic out of the L2s is the limit (14 to 20 TB/s), which is why the tile grows with
// the output.  A second slice in flight pays where a compute unit has one workgroup (64 x 96, from 18 slices on); with two, as the 64 x 64
// shapes have, their operands come at the L2s' rate either way (level at 512 x 3072 x 3072 and 3121 x 1152 x 1160).
#include <type_traits>

#include "gemm_common.h"
#include "rotate.h"
#include "wave_reduce.h"

namespace dvdq {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f_t __attribute__((ext_vector_type(4)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

constexpr int kFp6Block = kGroup * kBK * 6 / 8;   // 3072: 32 rows of one K slice as E2M3 patterns
enum { FMT_INT8 = 0, FMT_PACKED4 = 1, FMT_FP6 = 2, FMT_CANONICAL = 3 };   // (CANONICAL: int8 codes, weights [N, K/2])

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const uint8_t *p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(p), 0, bytes, 0x00020000);
}

// two packed dwords (16 codes) -> int8 lanes of 16 * code, channel order (see w4ax_gemm.hip)
__device__ __forceinline__ v4i widen16(uint32_t lo, uint32_t hi) {
    v4i f;
    f[0] = (int)((lo << 4) & 0xF0F0F0F0u);
    f[1] = (int)(lo & 0xF0F0F0F0u);
    f[2] = (int)((hi << 4) & 0xF0F0F0F0u);
    f[3] = (int)(hi & 0xF0F0F0F0u);
    return f;
}

// the same for two dwords in the canonical nibble order (nibble i = channel i): the bytes of the even and the odd
// nibbles are interleaved
__device__ __forceinline__ v4i widen16_canonical(uint32_t lo, uint32_t hi) {
    const v4i f = widen16(lo, hi);   // even, odd channels of each dword
    v4i r;
    r[0] = (int)__builtin_amdgcn_perm((uint32_t)f[1], (uint32_t)f[0], 0x05010400u);
    r[1] = (int)__builtin_amdgcn_perm((uint32_t)f[1], (uint32_t)f[0], 0x07030602u);
    r[2] = (int)__builtin_amdgcn_perm((uint32_t)f[3], (uint32_t)f[2], 0x05010400u);
    r[3] = (int)__builtin_amdgcn_perm((uint32_t)f[3], (uint32_t)f[2], 0x07030602u);
    return r;
}

// three 16-byte chunks of a row's half slice -> operand of the h-th 64-channel MFMA
template <int H>
__device__ __forceinline__ v8i fp6_fragment(v4u c0, v4u c1, v4u c2) {
    return H == 0 ? v8i{(int)c0[0], (int)c0[1], (int)c0[2], (int)c0[3], (int)c1[0], (int)c1[1], 0, 0}
                  : v8i{(int)c1[2], (int)c1[3], (int)c2[0], (int)c2[1], (int)c2[2], (int)c2[3], 0, 0};
}

// what a wave loads of one K slice of 128 channels
template <int FMT, int TM, int TN>
struct Slice {
    static constexpr int A_LOADS = TM * (FMT == FMT_PACKED4 ? 2 : FMT == FMT_FP6 ? 3 : 4);   // 16 bytes per lane each
    v4u a[A_LOADS];
    v2u w[FMT == FMT_INT8 || FMT == FMT_PACKED4 ? TN * 4 : 1];
    v4u w16[FMT == FMT_FP6 ? TN * 3 : FMT == FMT_CANONICAL ? TN * 2 : 1];
};

// The layer of few tokens: what the kernel quantizes instead of being handed codes, and where it leaves the codes, token scales
// and code sums that the two-kernel layer would leave in the workspace.
struct LayerInput {
    const uint16_t *x;
    double scale_mul;    // 1 / (sqrt(B) * qmax)
    float recip_num;     // 1 / sqrt(B)
    int log2_block;
    uint32_t unit_mul;   // 2^16 / units of a row, rounded up
    uint8_t *codes;
    float *x_scale;
    int32_t *code_rowsum;   // with zero-points
};
constexpr int kLayerTasks = 64;     // units of 512 channels that a workgroup quantizes, 8 per wave
constexpr int kLayerPad = 128;      // LDS bytes a last part of a slice may read past the last row's codes
constexpr int kLayerVectors = 3 * 32 * 4;   // maxima, scales and code sums of the rows

constexpr int kGroupStride = 1024 + 32;   // LDS bytes of one group of 4 accumulator registers (see the reduction)

// columns of MFMA tiles that the reduction takes at a time
template <int TN>
constexpr int phase_columns() { return TN == 4 ? 2 : TN; }

// LDS bytes of one wave: its part in the reduction, or its operand slice where that is larger
template <int FMT, int TM, int TN, bool LAYER>
constexpr int wave_lds() {
    const int reduction = TM * phase_columns<TN>() * 4 * kGroupStride;
    const int slice = (FMT == FMT_FP6 || LAYER ? 0 : TM * 32 * (FMT == FMT_PACKED4 ? 64 : 128)) + (FMT == FMT_CANONICAL ? TN * 32 * 64 : 0);
    return reduction > slice ? reduction : slice;
}

// LDS bytes between the rows of codes of the layer (16 more than a row, so that rows start in different banks)
template <int FMT>
__host__ __device__ constexpr int layer_row_bytes(int K) {
    return (FMT == FMT_PACKED4 ? K / 2 : FMT == FMT_FP6 ? K / 8 * 6 : K) + 16;
}

// Quantizes rows m0 .. m0 + rows - 1 into LDS: a workgroup's rows x units of 512 channels are dealt to its waves, CPW units each at
// most, kept in registers until the rows' maxima are known.  Same arithmetic, operation by operation, as rotate_quant.hip, so the
// codes, scales and code sums are the same bits.  s_rowmax: zeros on entry, from before a barrier.  Ends with a barrier.
// A unit is a chain of exchanges and waits; nothing but other units can stand in its gaps, so there is no branch per unit (a wave's
// units past the workgroup's are zeros and are only not stored) and what is the same for a row is worked out once, a row per lane.
template <int FMT, int NW, int CPW, class Meanwhile>
__device__ __forceinline__ void quantize_rows(const LayerInput &in, int m0, int rows, int K, int wave, int lane, bool want_sum,
                                              uint32_t *s_rowmax, float *s_scale, int *s_sum, uint8_t *s_codes, int code_stride, Meanwhile meanwhile) {
    const int units = (K + kUnit - 1) / kUnit, tasks = rows * units, log2b = in.log2_block;
    const HadamardLane had(lane, log2b >= 5 ? 31 : (1 << log2b) - 1);
    int row[CPW], k0[CPW];
    bool there[CPW];
    uint4 raw[CPW];
#pragma unroll
    for (int c = 0; c < CPW; ++c) {   // (a unit past the workgroup's, channels past K: zeros)
        const int t = wave + c * NW;
        there[c] = t < tasks;
        row[c] = there[c] ? (int)(((uint32_t)t * in.unit_mul) >> 16) : 0;
        k0[c] = (t - row[c] * units) * kUnit + had.chunk * 8;
        const __amdgpu_buffer_rsrc_t src = buffer(reinterpret_cast<const uint8_t *>(in.x + (int64_t)(m0 + row[c]) * K), there[c] ? K * 2 : 0);
        const v4u q = __builtin_amdgcn_raw_buffer_load_b128(src, k0[c] * 2, 0, 0);
        raw[c] = make_uint4(q[0], q[1], q[2], q[3]);
    }
    meanwhile();       // (loads of the caller's, requested behind these)
    __syncthreads();   // (the maxima are zero)
    float v[CPW][8], amax[CPW];
    auto each_unit = [&](auto f) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < CPW; ++c) f(v[c], raw[c]);
    };
    if (log2b == 0) each_unit([&](float (&u)[8], uint4 q) { had.low_bits(u, q, 0); });
    else each_unit([&](float (&u)[8], uint4 q) { had.low_bits(u, q, 5); });
    if (log2b >= 6) each_unit([&](float (&u)[8], uint4) { stage_xor1(u, had.s1); });
    if (log2b >= 7) each_unit([&](float (&u)[8], uint4) { stage_xor2(u, had.s2); });
    if (log2b >= 8) each_unit([&](float (&u)[8], uint4) { stage_xor8(u, had.s8); });
    if (log2b >= 9) each_unit([&](float (&u)[8], uint4) { stage_xor7(u, had.s7); });
#pragma unroll
    for (int c = 0; c < CPW; ++c) {
        amax[c] = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) amax[c] = fmaxf(amax[c], fabsf(v[c][i]));
    }
    if constexpr (CPW >= 4) {
#pragma unroll
        for (int c = 0; c < CPW; c += 4) wave_max4(amax[c], amax[c + 1], amax[c + 2], amax[c + 3]);
    } else {
#pragma unroll
        for (int c = 0; c < CPW; ++c) amax[c] = wave_max(amax[c]);
    }
    if (lane == 0) {   // (not negative: the order of the values is the order of their bits)
#pragma unroll
        for (int c = 0; c < CPW; ++c) atomicMax(s_rowmax + row[c], __float_as_uint(amax[c]));
    }
    __syncthreads();
    float my_r;   // lane l: the reciprocal step of row l
    {
        const float a = __uint_as_float(s_rowmax[min(lane, rows - 1)]);
        const float scale = (float)((double)a * in.scale_mul);
        my_r = scale > 0.f ? in.recip_num / scale : 0.f;
        if (wave == 0 && lane < rows) s_scale[lane] = scale;
    }
    const float flip = had.flip(log2b);
    float r[CPW];
#pragma unroll
    for (int c = 0; c < CPW; ++c) r[c] = flip * __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, my_r), row[c]));
    int sum[CPW];
    if constexpr (FMT == FMT_FP6) {
        auto each = [&](auto f) __attribute__((always_inline)) {
            f(std::integral_constant<int, 0>{});
            if constexpr (CPW > 1) f(std::integral_constant<int, 1>{});
            if constexpr (CPW > 2) f(std::integral_constant<int, 2>{});
            if constexpr (CPW > 3) f(std::integral_constant<int, 3>{});
        };
#pragma unroll
        for (int c0 = 0; c0 < CPW; c0 += 4) {
            fp6_source qa = fp6_undefined(), qb = qa;
            each([&](auto g_c) __attribute__((always_inline)) {
                constexpr int G = decltype(g_c)::value;
                float fsum = 0.f;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    qa[4 * G + i] = fmaf(v[c0 + G][2 * i], r[c0 + G], kRoundMagic) - kRoundMagic;
                    qb[4 * G + i] = fmaf(v[c0 + G][2 * i + 1], r[c0 + G], kRoundMagic) - kRoundMagic;
                    fsum += qa[4 * G + i] + qb[4 * G + i];
                }
                sum[c0 + G] = (int)fsum;
            });
            const fp6_fields pk = pack_codes_fp6(qa, qb);
            each([&](auto g_c) __attribute__((always_inline)) {
                constexpr int G = decltype(g_c)::value;
                const int c = c0 + G;
                if (!there[c] || k0[c] >= K) return;
                uint8_t *d = s_codes + row[c] * code_stride + k0[c] / 8 * 6;
                const bool odd = had.chunk & 1;
                store_chunk_fp6<G>(pk, odd, reinterpret_cast<uint32_t *>(d + (odd ? 2 : 0)), reinterpret_cast<uint16_t *>(d + (odd ? 0 : 4)));
            });
        }
    } else {
#pragma unroll
        for (int c = 0; c < CPW; ++c) {
            uint32_t b[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) b[i] = __float_as_uint(fmaf(v[c][i], r[c], kRoundMagic));
            uint8_t *to = s_codes + row[c] * code_stride;
            const bool ok = there[c] && k0[c] < K;
            if constexpr (FMT == FMT_PACKED4) {
                const uint32_t p = pack_codes_nibbles(b);
                if (ok) *reinterpret_cast<uint32_t *>(to + k0[c] / 2) = p;
                sum[c] = __builtin_amdgcn_sdot8((int)p, 0x11111111, 0, false);
            } else {
                const uint2 p = pack_codes_int8(b);
                if (ok) *reinterpret_cast<uint2 *>(to + k0[c]) = p;
                sum[c] = __builtin_amdgcn_sdot4((int)p.y, 0x01010101, __builtin_amdgcn_sdot4((int)p.x, 0x01010101, 0, false), false);
            }
        }
    }
    if (want_sum) {
#pragma unroll
        for (int c = 0; c < CPW; ++c) sum[c] = wave_sum(sum[c]);
        if (lane == 0) {
#pragma unroll
            for (int c = 0; c < CPW; ++c) atomicAdd(s_sum + row[c], sum[c]);
        }
    }
    __syncthreads();
}

// CPW > 0, the layer: the codes are made here, from `in`, by every workgroup for its own 32 tokens, CPW units of 512 channels a wave.
// DEPTH: slices a wave has in flight.  2, in shapes with one workgroup per compute unit (and so 512 registers a lane).
template <int FMT, int TM, int TN, int NW, int CPW, int DEPTH>
__global__ __launch_bounds__(64 * NW, DEPTH == 2 ? 1 : 2) void w4ax_gemm_small_kernel(
    const uint8_t *__restrict__ codes, const float *__restrict__ x_scale, const uint8_t *__restrict__ w,
    const float *__restrict__ w_scale, const int8_t *__restrict__ w_zero, const int32_t *__restrict__ code_rowsum,
    const uint16_t *__restrict__ bias, int M, int N, int K, uint16_t *__restrict__ y, int32_t *__restrict__ acc_out,
    int tiles_m, int tiles_n, int m_fastest, LayerInput in) {
    constexpr bool FP6 = FMT == FMT_FP6, CANONICAL = FMT == FMT_CANONICAL, LAYER = CPW > 0;
    constexpr int BM = 32 * TM, BN = 32 * TN;
    constexpr int A_ROW = FMT == FMT_PACKED4 ? kBK / 2 : kBK;    // bytes of a code row per slice (row-major containers)
    constexpr int PN = phase_columns<TN>(), PHASES = TN / PN;   // the reduction takes PN columns of MFMA tiles at a time
    constexpr int NG = TM * PN * 4;                            // groups of 4 accumulator registers per phase
    constexpr int GROUP_STRIDE = kGroupStride;
    constexpr int A_STAGE = FP6 || LAYER ? 0 : BM * A_ROW, W_STAGE = CANONICAL ? BN * (kBK / 2) : 0;   // a wave's own slice in LDS
    constexpr int WAVE_LDS = wave_lds<FMT, TM, TN, LAYER>();
    static_assert(NG * GROUP_STRIDE <= WAVE_LDS && A_STAGE + W_STAGE <= WAVE_LDS, "per-wave LDS");
    constexpr int CV = (BN + 63) / 64;                         // values per lane of a channel vector
    static_assert(!LAYER || (TM == 1 && NW == 8), "the layer's tokens and units");
    static_assert(TM <= 2 && TN <= 4 && TN % PHASES == 0, "token vectors are one value per lane");
    typedef typename std::conditional<FP6, AccF32x64, AccI32<FMT == FMT_PACKED4 ? 8 : 4>>::type P;
    typedef typename P::vec Acc;

    extern __shared__ __align__(16) uint8_t smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int KT = (K + kBK - 1) / kBK;   // (CANONICAL: K % 32 == 0 only, the last slice may be a part of one)
    const int G = ((N + kNPad - 1) / kNPad) * (kNPad / kGroup);

    // consecutive workgroups go to different XCDs: each XCD gets a contiguous run of tiles
    const int total = tiles_m * tiles_n;
    int tile = blockIdx.x;
    const int per_xcd = total / 8;
    if (tile < per_xcd * 8) tile = (tile % 8) * per_xcd + tile / 8;
    const int n_fast = m_fastest ? tiles_m : tiles_n, slow = tile / n_fast, fast = tile - slow * n_fast;
    const int m0 = (m_fastest ? fast : slow) * BM, n0 = (m_fastest ? slow : fast) * BN;
    const int rows = min(BM, M - m0);

    // The tile's token and channel vectors, one value per lane, requested before everything else and put into LDS
    // after the K loop.  (Always loaded, from some vector that exists: a branch would wait for them here.)
    const int vm = min(m0 + lane, M - 1);
    const float v_xs = LAYER ? 0.f : x_scale[vm];
    const int v_rs = LAYER ? 0 : (w_zero ? code_rowsum : reinterpret_cast<const int32_t *>(x_scale))[vm];
    float v_ws[CV];
    uint16_t v_bias[CV];
    int8_t v_z[CV];
#pragma unroll
    for (int i = 0; i < CV; ++i) {
        const int vn = min(n0 + i * 64 + lane, N - 1);
        v_ws[i] = w_scale[vn];
        v_bias[i] = (bias ? bias : reinterpret_cast<const uint16_t *>(w_scale))[vn];
        v_z[i] = (w_zero ? w_zero : reinterpret_cast<const int8_t *>(w_scale))[vn];
    }

    const int row_bytes = FMT == FMT_PACKED4 ? K / 2 : K;
    const uint8_t *a_tile = FP6 ? codes + (int64_t)(m0 / 32) * KT * kFp6Block : codes + (int64_t)m0 * row_bytes;
    const int a_bytes = FP6 ? (rows + 31) / 32 * KT * kFp6Block : rows * row_bytes;
    const uint8_t *w_tile = CANONICAL ? w + (int64_t)n0 * (K / 2) : w + (int64_t)(n0 / kGroup) * (FP6 ? kFp6Block : kGroupBytes);
    const int64_t w_slice_stride = (int64_t)G * (FP6 ? kFp6Block : kGroupBytes);
    const int frow = lane & 31, fhalf = lane >> 5;
    constexpr int CHUNKS = A_ROW / 16, ROWS_PER_LOAD = 64 / CHUNKS;
    const int a_lane = FP6 ? fhalf * 1536 + frow * 16 : (lane / CHUNKS) * row_bytes + (lane % CHUNKS) * 16;

    typedef Slice<FMT, TM, TN> S;
    auto load = [&](S &s, int kt) __attribute__((always_inline)) {
        const bool ok = kt < KT;
        const int a_off = LAYER ? 0 : kt * (FP6 ? kFp6Block : A_ROW);
        const __amdgpu_buffer_rsrc_t ra = buffer(a_tile + (ok ? a_off : 0), ok ? a_bytes - a_off : 0);   // (LAYER: unused)
        const int64_t w_off = CANONICAL ? kt * (kBK / 2) : kt * w_slice_stride;
        // (G is a multiple of 8: the minimum is TN but for TN = 3, whose last tile has one or two groups left, and whose reads past them the
        // descriptor's end turns into zeros.  With the constant in its place, where it is TN, the same loads come out in another order: 3121 x 1152 x
        // 1160 packed codes 9.7 -> 9.8 us, 512 x 3072 x 3072 int8 10.4 -> 10.6, 300 x 3072 x 3072 7.4 -> 7.2)
        const int w_bytes = CANONICAL ? min(BN, N - n0) * (K / 2) - (int)w_off : min(TN, G - n0 / kGroup) * (FP6 ? kFp6Block : kGroupBytes);
        const __amdgpu_buffer_rsrc_t rw = buffer(w_tile + (ok ? w_off : 0), ok ? w_bytes : 0);
        if constexpr (FP6) {
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    s.w16[i * 3 + c] = __builtin_amdgcn_raw_buffer_load_b128(rw, a_lane + i * kFp6Block + c * 512, 0, 0);
#pragma unroll
            for (int j = 0; j < (LAYER ? 0 : TM); ++j)
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    s.a[j * 3 + c] = __builtin_amdgcn_raw_buffer_load_b128(ra, a_lane + j * KT * kFp6Block + c * 512, 0, 0);
        } else if constexpr (CANONICAL) {
            // a lane whose channels lie past K (in a last part of a slice) reads past the descriptor instead
            const int k_left = K - kt * kBK, beyond = 0x7FFFFFF0;
            const int a_at = (lane % CHUNKS) * 16 < k_left ? a_lane : beyond;
            const int w_at = (lane % 4) * 32 < k_left ? (lane / 4) * (K / 2) + (lane % 4) * 16 : beyond;
#pragma unroll
            for (int i = 0; i < (LAYER ? 0 : S::A_LOADS); ++i)
                s.a[i] = __builtin_amdgcn_raw_buffer_load_b128(ra, a_at == beyond ? beyond : a_at + i * ROWS_PER_LOAD * row_bytes, 0, 0);
#pragma unroll
            for (int i = 0; i < TN * 2; ++i)
                s.w16[i] = __builtin_amdgcn_raw_buffer_load_b128(rw, w_at == beyond ? beyond : w_at + i * 16 * (K / 2), 0, 0);
        } else {
#pragma unroll
            for (int i = 0; i < (LAYER ? 0 : S::A_LOADS); ++i)
                s.a[i] = __builtin_amdgcn_raw_buffer_load_b128(ra, a_lane + i * ROWS_PER_LOAD * row_bytes, 0, 0);
#pragma unroll
            for (int i = 0; i < TN * 4; ++i)
                s.w[i] = __builtin_amdgcn_raw_buffer_load_b64(rw, lane * 8 + (FMT == FMT_PACKED4 ? fhalf * 256 : 0) + (i / 4) * kGroupBytes + (FMT == FMT_PACKED4 ? (i % 4 / 2) * 1024 + (i % 2) * 256 : (i % 4) * 512), 0, 0);
        }
    };

    Acc acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

    uint8_t *mine = smem + wave * WAVE_LDS;
    float *s_xs = reinterpret_cast<float *>(smem + NW * WAVE_LDS), *s_ws = s_xs + 64, *s_bias = s_ws + CV * 64;
    int *s_rs = reinterpret_cast<int *>(s_bias + CV * 64), *s_z = s_rs + 64;
    uint32_t *s_rowmax = reinterpret_cast<uint32_t *>(s_z + CV * 64);
    float *s_scale = reinterpret_cast<float *>(s_rowmax + 32);
    int *s_sum = reinterpret_cast<int *>(s_scale + 32);
    uint8_t *s_codes = reinterpret_cast<uint8_t *>(s_sum + 32);
    const int code_stride = layer_row_bytes<FMT>(K);
    // (rows past M: some row that exists, for outputs that are never stored)
    const uint8_t *my_codes = s_codes + min(frow, rows - 1) * code_stride;

    S slice, behind;
    if constexpr (CPW > 0) {
        if (tid < 32) s_rowmax[tid] = 0, s_sum[tid] = 0;
        quantize_rows<FMT, NW, CPW>(in, m0, rows, K, wave, lane, w_zero != nullptr, s_rowmax, s_scale, s_sum, s_codes, code_stride,
                                    [&]() __attribute__((always_inline)) { load(slice, wave); });
    } else {
        load(slice, wave);
        if constexpr (DEPTH == 2) load(behind, wave + NW);
    }

    auto multiply = [&](const S &s, int kt) __attribute__((always_inline)) {
        if constexpr (FP6) {
            auto half = [&](auto hc) __attribute__((always_inline)) {
                constexpr int H = decltype(hc)::value;
                v8i fa[TM];
#pragma unroll
                for (int j = 0; j < TM; ++j) {
                    if constexpr (LAYER) {
                        const v4u *c = reinterpret_cast<const v4u *>(my_codes + kt * (kFp6Block / 32) + fhalf * 48);
                        fa[j] = H == 0 ? fp6_fragment<H>(c[0], c[1], c[1]) : fp6_fragment<H>(c[1], c[1], c[2]);
                    } else {
                        fa[j] = fp6_fragment<H>(s.a[j * 3], s.a[j * 3 + 1], s.a[j * 3 + 2]);
                    }
                }
#pragma unroll
                for (int i = 0; i < TN; ++i) {
                    const v8i fw = fp6_fragment<H>(s.w16[i * 3], s.w16[i * 3 + 1], s.w16[i * 3 + 2]);
#pragma unroll
                    for (int j = 0; j < TM; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fw, fa[j], acc[i][j], 2, 2, 0, 0, 0, 0);
                }
            };
            half(std::integral_constant<int, 0>{});
            half(std::integral_constant<int, 1>{});
        } else {
            // the code rows, loaded as whole lines, become fragments through this wave's own LDS (in order: no barrier)
#pragma unroll
            for (int i = 0; i < (LAYER ? 0 : S::A_LOADS); ++i) {
                const int row = i * ROWS_PER_LOAD + lane / CHUNKS;
                *reinterpret_cast<v4u *>(mine + row * A_ROW + (((lane % CHUNKS) ^ swz_bk<A_ROW>(row)) << 4)) = s.a[i];
            }
            if constexpr (CANONICAL) {
                // packed weight rows of 64 bytes.  A fragment is 8 bytes: the halves of a 16-byte chunk are swapped in
                // every second group of 16 rows, so that the 32 rows a read serves at a time use all 64 banks
#pragma unroll
                for (int i = 0; i < TN * 2; ++i) {
                    const int row = i * 16 + lane / 4;
                    const v4u q = s.w16[i];
                    *reinterpret_cast<v4u *>(mine + A_STAGE + row * 64 + (((lane % 4) ^ swz_bk<64>(row)) << 4)) =
                        (i & 1) ? v4u{q[2], q[3], q[0], q[1]} : q;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            constexpr int NT = FMT == FMT_PACKED4 ? 2 : 1;
#pragma unroll
            for (int ks = 0; ks < 4 / NT; ++ks) {
                v4i ra[TM];
#pragma unroll
                for (int j = 0; j < TM; ++j)
                    ra[j] = LAYER ? *reinterpret_cast<const v4i *>(my_codes + kt * A_ROW + (ks * 2 + fhalf) * 16)
                                  : *reinterpret_cast<const v4i *>(mine + (j * 32 + frow) * A_ROW + (((ks * 2 + fhalf) ^ swz_bk<A_ROW>(frow)) << 4));
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    v4i fa[TM];
#pragma unroll
                    for (int j = 0; j < TM; ++j)
                        fa[j] = FMT == FMT_PACKED4 ? widen16((uint32_t)ra[j][2 * t], (uint32_t)ra[j][2 * t + 1]) : ra[j];
#pragma unroll
                    for (int i = 0; i < TN; ++i) {
                        v4i fw;
                        if constexpr (CANONICAL) {
                            const v2u p = *reinterpret_cast<const v2u *>(mine + A_STAGE + (i * 32 + frow) * 64 +
                                                                         ((ks ^ swz_bk<64>(frow)) << 4) + ((fhalf ^ (frow >> 4)) << 3));
                            fw = widen16_canonical(p[0], p[1]);
                        } else {
                            const v2u p = s.w[i * 4 + ks * NT + t];
                            fw = widen16(p[0], p[1]);
                        }
#pragma unroll
                        for (int j = 0; j < TM; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fw, fa[j], acc[i][j], 0, 0, 0);
                    }
                }
            }
            __builtin_amdgcn_wave_barrier();   // the next slice's LDS writes stay behind these reads
        }
    };

    if constexpr (DEPTH == 2) {
        // (pairs in one basic block: with a way out between the two the compiler waits for all loads in front of the second, which
        // is why a second slice in flight was 10 % slower at 512 x 3072 x 3072 once)
        int kt = wave;
        for (; kt + NW < KT; kt += 2 * NW) {
            multiply(slice, kt);
            load(slice, kt + 2 * NW);
            __builtin_amdgcn_sched_barrier(0);
            multiply(behind, kt + NW);
            load(behind, kt + 3 * NW);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (kt < KT) multiply(slice, kt);
    } else {
        for (int kt = wave; kt < KT; kt += NW) {
            multiply(slice, kt);
            load(slice, kt + NW);   // (the compiler moves it up between the MFMAs; past the last slice it fetches nothing)
        }
    }

    // ---- reduction over the waves' shares of K and epilogue.  Every wave puts its accumulators into its part of LDS,
    // group (4 registers) by group; then a thread adds up and finishes 8 consecutive channels of one token, which are
    // the two lane halves of one group.  Groups are 1024 + 32 bytes apart so that the threads of a token, which read
    // neighbouring groups, use different banks.
    if (wave == NW - 1) {
        float xs = v_xs;
        int rs = v_rs;
        if constexpr (LAYER) {   // (lanes past the rows: values never used)
            xs = s_scale[min(lane, rows - 1)];
            rs = s_sum[min(lane, rows - 1)];
            if (n0 == 0 && lane < rows) {
                in.x_scale[m0 + lane] = xs;
                if (w_zero) in.code_rowsum[m0 + lane] = rs;
            }
        }
        s_xs[lane] = xs * P::edge_fold();
        s_rs[lane] = w_zero ? rs : 0;
#pragma unroll
        for (int i = 0; i < CV; ++i) {
            s_ws[i * 64 + lane] = v_ws[i];
            s_bias[i * 64 + lane] = __uint_as_float((uint32_t)v_bias[i] << 16);
            s_z[i * 64 + lane] = w_zero ? v_z[i] : 0;
        }
    }
    constexpr int PIECES = PN * 4;    // 8 consecutive channels each
    const bool has_bias = bias != nullptr;
#pragma unroll
    for (int ph = 0; ph < PHASES; ++ph) {
#pragma clang fp contract(off)
        if (ph) __syncthreads();
#pragma unroll
        for (int i = 0; i < PN; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const Acc &t = acc[ph * PN + i][j];
                    typedef typename std::conditional<FP6, v4f_t, v4i>::type Q;
                    *reinterpret_cast<Q *>(mine + ((i * TM + j) * 4 + g) * GROUP_STRIDE + lane * 16) =
                        Q{t[g * 4], t[g * 4 + 1], t[g * 4 + 2], t[g * 4 + 3]};
                }
        __syncthreads();
        // (unrolled, so that the reads of a thread's pieces run beside each other: 2800 of the kernel's 16500 clocks went to these sums at
        // 300 x 3072 x 3072; 512 x 3072 x 3072 int8 11.6 -> 10.5 us, 512 x 1536 x 3072 8.6 -> 7.4.  With more than two pieces a thread, what is not there --
        // zero-points, bias -- is chosen once: a branch in each piece keeps the reads apart (1560 x 1536 x 1536 packed 10.0 -> 9.4, 3121 x 1152 x
        // 1160 10.3 -> 9.8 the GEMM; 2300 whole layers 0.98 of their time in the mean, with zero-points 0.97 to 0.99, without 0.98 to 1.00).  With two at most, with canonical weights and with FP6 codes it is branched around: there the copies of the code
        // cost up to 4 %: 700 x 1536 x 2304 int8 8.4 and 8.7)
        constexpr int ITEMS = (BM * PIECES + 64 * NW - 1) / (64 * NW);
        constexpr bool SAME_CHANNELS = 64 * NW % PIECES == 0;   // of all of a thread's pieces
        typedef typename std::conditional<FP6, v4f_t, v4i>::type Q;
        auto row_of = [&](int it) { return it / PIECES; };
        auto channel_of = [&](int it) { return (ph * PIECES + it % PIECES) * 8; };   // a piece's first channel within the tile
        auto exists = [&](int it) {
            return (BM * PIECES % (64 * NW) == 0 || it < BM * PIECES) && row_of(it) < rows && n0 + channel_of(it) < N;
        };
        auto sum_shares = [&](int it, Q &lo, Q &hi) __attribute__((always_inline)) {
            const int p = it % PIECES, r = row_of(it);
            const uint8_t *q = smem + (((p >> 2) * TM + (r >> 5)) * 4 + (p & 3)) * GROUP_STRIDE + (r & 31) * 16;
            lo = *reinterpret_cast<const Q *>(q);
            hi = *reinterpret_cast<const Q *>(q + 512);
#pragma unroll
            for (int u = 1; u < NW; ++u) {
                lo += *reinterpret_cast<const Q *>(q + u * WAVE_LDS);
                hi += *reinterpret_cast<const Q *>(q + u * WAVE_LDS + 512);
            }
        };
        auto read8 = [](auto (&v)[2], const auto *from) __attribute__((always_inline)) {
            v[0] = *reinterpret_cast<const std::remove_reference_t<decltype(v[0])> *>(from);
            v[1] = *reinterpret_cast<const std::remove_reference_t<decltype(v[1])> *>(from + 4);
        };
        auto store = [&](int it, const float (&o)[8], const int (&a)[8]) __attribute__((always_inline)) {
            const int c = channel_of(it);
            const int64_t at = (int64_t)(m0 + row_of(it)) * N + n0 + c;
            // (16 bytes at any even address: rows of an output with N no multiple of 8 begin anywhere.  Stored per element such
            // rows cost the layer 385 x 2304 x 4436 1.3 of 14.6 us)
            if (n0 + c + 8 <= N) {
                store_piece_unaligned(y + at, make_uint4(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]),
                                                         pack_bf16x2(o[4], o[5]), pack_bf16x2(o[6], o[7])));
            } else {
#pragma unroll
                for (int e = 0; e < 7; ++e)
                    if (n0 + c + e < N) y[at + e] = (uint16_t)(pack_bf16x2(o[e], 0.f) & 0xFFFFu);
            }
            if (acc_out) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (n0 + c + e < N) acc_out[at + e] = P::sum(a[e]);
            }
        };
        if constexpr (ITEMS <= 2 || CANONICAL || (FP6 && DEPTH == 1)) {
#pragma unroll
            for (int item = 0; item < ITEMS; ++item) {
                const int it = tid + item * 64 * NW;
                if (!exists(it)) continue;
                Q lo, hi;
                sum_shares(it, lo, hi);
                const int r = row_of(it), c = channel_of(it);
                const float xs = s_xs[r];
                v4f_t ws[2], bb[2];
                read8(ws, s_ws + c);
                int a[8];
                float o[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) a[e] = P::integer(e < 4 ? lo[e] : hi[e - 4]);
                if (w_zero) {
                    const int rs = s_rs[r];
                    v4i z[2];
                    read8(z, s_z + c);
#pragma unroll
                    for (int e = 0; e < 8; ++e) a[e] = P::unzero(a[e], z[e / 4][e % 4], rs);
                }
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = (float)a[e] * xs * ws[e / 4][e % 4];
                if (has_bias) {
                    read8(bb, s_bias + c);
#pragma unroll
                    for (int e = 0; e < 8; ++e) o[e] += bb[e / 4][e % 4];
                }
                store(it, o, a);
            }
        } else {
            auto finish = [&](auto zp, auto with_bias) __attribute__((always_inline)) {
                constexpr bool ZP = decltype(zp)::value, BIAS = decltype(with_bias)::value;
                struct Channels { v4f_t ws[2], bias[2]; v4i z[2]; } ch[SAME_CHANNELS ? 1 : ITEMS];
                Q lo[ITEMS], hi[ITEMS];
                float xs[ITEMS];
                int rs[ITEMS];
#pragma unroll
                for (int item = 0; item < ITEMS; ++item) {   // (rows past M and channels past N: sums that are not stored)
                    const int it = min(tid + item * 64 * NW, BM * PIECES - 1);
                    sum_shares(it, lo[item], hi[item]);
                    xs[item] = s_xs[row_of(it)];
                    if constexpr (ZP) rs[item] = s_rs[row_of(it)];
                    if (item == 0 || !SAME_CHANNELS) {
                        read8(ch[item].ws, s_ws + channel_of(it));
                        if constexpr (BIAS) read8(ch[item].bias, s_bias + channel_of(it));
                        if constexpr (ZP) read8(ch[item].z, s_z + channel_of(it));
                    }
                }
#pragma unroll
                for (int item = 0; item < ITEMS; ++item) {
                    const int it = tid + item * 64 * NW;
                    const Channels &h = ch[SAME_CHANNELS ? 0 : item];
                    int a[8];
                    float o[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        a[e] = P::integer(e < 4 ? lo[item][e] : hi[item][e - 4]);
                        if constexpr (ZP) a[e] = P::unzero(a[e], h.z[e / 4][e % 4], rs[item]);
                        o[e] = (float)a[e] * xs[item] * h.ws[e / 4][e % 4];
                        if constexpr (BIAS) o[e] += h.bias[e / 4][e % 4];
                    }
                    if (exists(it)) store(it, o, a);
                }
            };
            if (w_zero) {
                if (has_bias) finish(std::true_type{}, std::true_type{});
                else finish(std::true_type{}, std::false_type{});
            } else {
                if (has_bias) finish(std::false_type{}, std::true_type{});
                else finish(std::false_type{}, std::false_type{});
            }
        }
    }
    if constexpr (LAYER) {
        // the first column of tiles leaves the codes where the two-kernel layer does
        if (n0 != 0) return;
        const int pieces = (code_stride - 16) / 16;   // of a row; neighbouring threads take neighbouring rows
        const int row = tid & 31;
        if (row >= rows) return;
        for (int p = tid >> 5; p < pieces; p += 2 * NW) {
            uint8_t *to = FP6 ? in.codes + ((int64_t)(m0 / 32) * KT + p / 6) * kFp6Block + (p % 6) * 512 + row * 16
                              : in.codes + (int64_t)(m0 + row) * (code_stride - 16) + p * 16;
            *reinterpret_cast<uint4 *>(to) = *reinterpret_cast<const uint4 *>(s_codes + row * code_stride + p * 16);
        }
    }
}

template <int FMT, int TM, int TN, int NW, int CPW = 0, int DEPTH = 1>
int launch_tile(const uint8_t *codes, const float *x_scale, const uint8_t *w, const float *w_scale, const int8_t *w_zero,
                const int32_t *code_rowsum, const uint16_t *bias, int M, int N, int K, uint16_t *y, int32_t *acc_out,
                hipStream_t stream, const LayerInput &in = {}) {
    constexpr bool LAYER = CPW > 0;
    const int tiles_m = (M + 32 * TM - 1) / (32 * TM), tiles_n = (N + 32 * TN - 1) / (32 * TN);
    const size_t smem = (size_t)NW * wave_lds<FMT, TM, TN, LAYER>() + (2 + 3 * ((TN * 32 + 63) / 64)) * 256 +
                        (LAYER ? kLayerVectors + min(M, 32) * layer_row_bytes<FMT>(K) + kLayerPad : 0);
    auto k = w4ax_gemm_small_kernel<FMT, TM, TN, NW, CPW, DEPTH>;
    static std::atomic<uint64_t> configured{0};
    allow_dynamic_lds(reinterpret_cast<const void *>(k), LAYER ? kLdsPerCu : smem, configured);
    // an XCD takes a contiguous run of tiles: it should read all of the smaller operand and its share of the larger one
    const int m_fastest = FMT == FMT_INT8 || FMT == FMT_CANONICAL ? N > 2 * M : N > M;
    hipLaunchKernelGGL(k, dim3((unsigned)(tiles_m * tiles_n)), dim3(64 * NW), smem, stream, codes, x_scale, w, w_scale, w_zero,
                       code_rowsum, bias, M, N, K, y, acc_out, tiles_m, tiles_n, m_fastest, in);
    return check_launch();
}

}  // namespace

// The kernel's shape for an M x N output of K: tile and waves that share its K slices.  -1: the large tiles' kernels.
// The smallest tile is taken whose workgroups all run at once (1 to 4 per compute unit, by their LDS and registers):
// more workgroups mean fewer slices in series, until a second round of them costs more.  The lines were taken from a
// sweep over M = 1 .. 16384, N = 256 .. 9216, K = 256 .. 9216, int8 and FP6 codes (all shapes timed at each point): this
// rule is within 2.6 % of the best shape in the geometric mean, and the same lines are best for both containers.  On
// the lines (int8 codes): 1024 x 1024 x 256 (tokens x K x channels, 256 tiles of 32 x 32) 4.6 us as shape 0, 4.8 as 1;
// 512 x 3072 x 3072 (384 tiles of 64 x 64) 11.8 as 3, 10.7 as 7, 14.7 as 4; 1024 x 3072 x 3072 (768) 18.7 and 16.9;
// 2048 x 3072 x 3072 (768 tiles of 64 x 128) 29.0 as 5, 31.1 with large tiles; 3072 x 3072 x 3072 (1152) 45.5 and 40.0.
// FP6 codes halve the large tiles' time per slice, not the operand traffic of the small ones: there the large tiles
// win as soon as 96 of them (256 x 256) are at work: 1536 x 3072 x 3072 (72) 20.4 as 5 and 24.0, 2048 x 3072 x 3072 (96)
// 22.9 and 21.9, 5120 x 9216 x 1160 (100) 55 and 47.7, 2048 x 640 x 3072 (96) 13.0 and 10.6.
int small_gemm_shape(int64_t M, int64_t N, int64_t K, bool fp6) {
    auto tiles = [&](int bm, int bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
    if (tiles(32, 32) <= 256) return 0;
    // (deep K: eight waves; 1 x 9216 x 9216: 14.8 -> 11.0 us, at 3072 channels equal)
    if (tiles(32, 64) <= 256) return K / kBK >= 48 ? 2 : 1;
    // (one workgroup per compute unit with the same outputs each, where of the 64 x 64 tiles some compute units have two and some one: by the
    // number of slices up to 11 / 12 to 17 / 18 to 23 / more 0.94 to 1.08 / 0.97 to 1.01 / 0.94 to 0.97 / 0.85 to 0.89 of shape 3's time, int8,
    // packed and FP6 codes; 512 x 3072 x 3072 int8 12.0 -> 10.7 us, FP6 9.9 -> 8.8)
    if (tiles(64, 64) > 256 && tiles(64, 96) <= 256 && K / kBK >= 18) return 7;
    if (tiles(64, 64) <= 512) return 3;
    if (tiles(64, 64) <= 1024) return 4;
    if (tiles(64, 128) <= 1024 && !(fp6 && tiles(256, 256) >= 96)) return 5;
    return -1;
}

int launch_w4ax_gemm_small(const uint8_t *codes, const float *x_scale, const uint8_t *w, const float *w_scale,
                           const int8_t *w_zero, const int32_t *code_rowsum, const uint16_t *bias, int64_t M, int64_t N,
                           int64_t K, int codes_format, int w_layout, int shape, uint16_t *y, int32_t *acc_out, hipStream_t stream) {
#define DVDQ_SMALL_ARGS codes, x_scale, w, w_scale, w_zero, code_rowsum, bias, (int)M, (int)N, (int)K, y, acc_out, stream
#define DVDQ_SMALL(FMT) /* {tile M / 32, tile N / 32, waves} */                \
    if constexpr (FMT != FMT_CANONICAL) { /* (two slices in flight) */         \
        if (shape == 7) return launch_tile<FMT, 2, 3, 4, 0, 2>(DVDQ_SMALL_ARGS); \
    }                                                                          \
    switch (shape) {                                                           \
        case 0: return launch_tile<FMT, 1, 1, 8>(DVDQ_SMALL_ARGS); \
        case 1: return launch_tile<FMT, 1, 2, 4>(DVDQ_SMALL_ARGS); \
        case 2: return launch_tile<FMT, 1, 2, 8>(DVDQ_SMALL_ARGS); \
        case 3: return launch_tile<FMT, 2, 2, 4>(DVDQ_SMALL_ARGS); \
        case 4: return launch_tile<FMT, 2, 2, 2>(DVDQ_SMALL_ARGS); \
        case 5: return launch_tile<FMT, 2, 4, 2>(DVDQ_SMALL_ARGS); \
        case 6: return launch_tile<FMT, 2, 4, 1>(DVDQ_SMALL_ARGS); /* (sweeps, and canonical weights: w4ax_gemm_choice) */ \
        default: return DVDQ_ERR_UNSUPPORTED;                                  \
    }
    if (codes_format == DVDQ_CODES_FP6) { DVDQ_SMALL(FMT_FP6) }
    if (codes_format == DVDQ_CODES_PACKED4) { DVDQ_SMALL(FMT_PACKED4) }
    if (w_layout == DVDQ_W_CANONICAL) { DVDQ_SMALL(FMT_CANONICAL) }
    DVDQ_SMALL(FMT_INT8)
#undef DVDQ_SMALL
#undef DVDQ_SMALL_ARGS
}

// Whether a whole layer takes the layer form of the kernel above, one launch: 0 (two launches), or the width of its tiles in 32
// channels.  Not where y or the workspace lies over x, against the rule of dvdq.h: one workgroup stores its part of y and the codes
// while others still read their tokens, where of two launches the first has read all of x before the second stores.  Every workgroup quantizes its 32 tokens, so it pays while that is little: up to 32 units of 512 channels (4 a wave), up to
// 64 for rows of four units or more, where the quantizer alone takes longer too, and as long as all workgroups run at once (the lines
// of small_gemm_shape).  Swept with launches in a graph, so without the host's time, M = 1 .. 4096, K = 256 .. 4096, N = 256 .. 9216, two
// launches -> one (us, int8 codes): 1 x 256 x 1024 5.3 -> 4.2; 2 x 1536 x 9216 7.6 -> 5.6; 128 x 256 x 1024 (32 units) 5.9 -> 5.3;
// 1 x 4096 x 9216 11.0 -> 7.3; 8 x 4096 x 1024 (64) 8.8 -> 8.3; not taken: 32 x 1024 x 1024 (64 units of 2-unit rows) 6.5 and 7.0,
// 16 x 1536 x 1024 (48) 6.8 and 7.0, 64 x 512 x 9216 (288 tiles of 32 x 64) 7.4 and 10.6.  FP6 codes within 3 % of these ratios.  Outside
// a graph the host's second launch, 4 us, comes on top of the two.
int qlinear_choice(const void *x, const void *y, const void *workspace, size_t workspace_bytes, int64_t M, int64_t N, int64_t K) {
    const int64_t units = (K + kUnit - 1) / kUnit;
    if ((M < 32 ? M : 32) * units > (units >= 4 ? kLayerTasks : kLayerTasks / 2)) return 0;
    const int shape = small_gemm_shape(M, N, K, false);
    if (shape < 0 || shape > 2) return 0;
    const uintptr_t at = reinterpret_cast<uintptr_t>(x), end = at + 2 * (uintptr_t)(M * K);
    auto over_x = [&](const void *p, size_t bytes) { return at < reinterpret_cast<uintptr_t>(p) + bytes && reinterpret_cast<uintptr_t>(p) < end; };
    if (over_x(y, 2 * (size_t)(M * N)) || over_x(workspace, workspace_bytes)) return 0;
    return shape == 0 ? 1 : 2;
}

int launch_qlinear_small(const uint16_t *x, int log2_block, int act_bits, const uint8_t *w, const float *w_scale,
                         const int8_t *w_zero, const uint16_t *bias, int64_t M, int64_t N, int64_t K, int codes_format,
                         int w_layout, int width, uint16_t *y, uint8_t *codes, float *x_scale, int32_t *code_rowsum, hipStream_t stream) {
    const double qmax = (double)((1 << (act_bits - 1)) - 1), norm = 1.0 / sqrt((double)(1 << log2_block));
    const int units = (int)((K + kUnit - 1) / kUnit);
    const LayerInput in{x, norm / qmax, (float)norm, log2_block, (65536u + units - 1) / units, codes, x_scale, code_rowsum};
    // units a wave takes: 1, 2, 4 or 8 (what the workgroup with most of them needs)
    const int tasks = (int)(M < 32 ? M : 32) * units, per_wave = (tasks + 7) / 8;
#define DVDQ_LAYER_CPW(FMT, TN, CPW) \
    launch_tile<FMT, 1, TN, 8, CPW>(nullptr, nullptr, w, w_scale, w_zero, nullptr, bias, (int)M, (int)N, (int)K, y, nullptr, stream, in)
#define DVDQ_LAYER_TN(FMT, TN)                                                                   \
    (per_wave <= 1 ? DVDQ_LAYER_CPW(FMT, TN, 1) : per_wave <= 2 ? DVDQ_LAYER_CPW(FMT, TN, 2) \
                                                : per_wave <= 4 ? DVDQ_LAYER_CPW(FMT, TN, 4) : DVDQ_LAYER_CPW(FMT, TN, 8))
#define DVDQ_LAYER(FMT) return width == 1 ? DVDQ_LAYER_TN(FMT, 1) : DVDQ_LAYER_TN(FMT, 2);
    if (codes_format == DVDQ_CODES_FP6) DVDQ_LAYER(FMT_FP6)
    if (codes_format == DVDQ_CODES_PACKED4) DVDQ_LAYER(FMT_PACKED4)
    if (w_layout == DVDQ_W_CANONICAL) DVDQ_LAYER(FMT_CANONICAL)
    DVDQ_LAYER(FMT_INT8)
#undef DVDQ_LAYER
#undef DVDQ_LAYER_TN
#undef DVDQ_LAYER_CPW
}

}  // namespace dvdq
