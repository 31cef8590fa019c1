// Device pieces of the quantizer (rotate_quant.hip), shared with the layer of few tokens (w4ax_gemm_small.hip): the block
// Hadamard transform of a 512-channel unit by one wave, a row's maximum, and the packing of codes.  rotate_quant.hip says how the
// transform is split between the matrix cores and lane exchanges.
#pragma once
#include "dvdq_internal.h"

namespace dvdq {

constexpr int kWave = 64;
constexpr int kUnit = 512;  // channels a wave handles per step (64 lanes x 8)
constexpr float kRoundMagic = 12582912.f;   // 1.5 * 2^23: adding it rounds to integer, ties to even

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

// One butterfly stage over a lane pairing with a single DPP operand, 8 values, one
// instruction per value: v = own + sign * partner, sign = +1 in the lane whose stage bit
// is clear and -1 in the other.  The lane with the bit set therefore holds MINUS the
// butterfly's difference; the caller tracks that sign and folds it into the quantizer.
// (The compiler does not fuse a DPP move into an fma, so this is inline assembly.  The
// leading s_nop covers the 2 wait states a DPP read needs after a VALU write of the same
// register.  PRE is put in front of that: the first stage reads registers that an MFMA may have written
// directly, whose longer read-after-write distance the compiler does not see through inline assembly.)
#define DVDQ_FMAC_DPP8(PRE, CTRL)                                                                              \
    asm volatile(PRE "s_nop 1\n\t"                                                                             \
                 "v_fmac_f32_dpp %0, %0, %8 " CTRL " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"              \
                 "v_fmac_f32_dpp %1, %1, %8 " CTRL " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"              \
                 "v_fmac_f32_dpp %2, %2, %8 " CTRL " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"              \
                 "v_fmac_f32_dpp %3, %3, %8 " CTRL " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"              \
                 "v_fmac_f32_dpp %4, %4, %8 " CTRL " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"              \
                 "v_fmac_f32_dpp %5, %5, %8 " CTRL " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"              \
                 "v_fmac_f32_dpp %6, %6, %8 " CTRL " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"              \
                 "v_fmac_f32_dpp %7, %7, %8 " CTRL " row_mask:0xf bank_mask:0xf bound_ctrl:1"                  \
                 : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), "+v"(v[7]) \
                 : "v"(sign))

// (first of the lane-pairing stages: its values come straight from the 8-pass MFMAs, whose results a vector
// instruction may read 12 wait states after the MFMA issued; 20 are kept)
static __device__ __forceinline__ void stage_xor1(float (&v)[8], float sign) { DVDQ_FMAC_DPP8("s_nop 15\n\ts_nop 1\n\t", "quad_perm:[1,0,3,2]"); }
static __device__ __forceinline__ void stage_xor2(float (&v)[8], float sign) { DVDQ_FMAC_DPP8("", "quad_perm:[2,3,0,1]"); }
static __device__ __forceinline__ void stage_xor8(float (&v)[8], float sign) { DVDQ_FMAC_DPP8("", "row_ror:8"); }

static __device__ __forceinline__ void stage_xor7(float (&v)[8], float sign) { DVDQ_FMAC_DPP8("", "row_half_mirror"); }

// Maximum of a non-negative value over the wave, the same in every lane: two quad permutes and two row
// mirrors leave each 16-lane row's maximum in all its lanes, two row broadcasts carry it on into lane 63.
// (Inline assembly: the compiler keeps a move, two canonicalizing maxima and the maximum per step instead of one
// maximum with a DPP operand.  s_nop 1: the 2 wait states between a vector write and a DPP read of a register.)
static __device__ __forceinline__ float wave_max(float a) {
    asm volatile("s_nop 1\n\t"
                 "v_max_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
                 "s_nop 1\n\t"
                 "v_max_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
                 "s_nop 1\n\t"
                 "v_max_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
                 "s_nop 1\n\t"
                 "v_max_f32_dpp %0, %0, %0 row_mirror row_mask:0xf bank_mask:0xf\n\t"
                 "s_nop 1\n\t"
                 "v_max_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"   // into rows 1, 3
                 "s_nop 1\n\t"
                 "v_max_f32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf"          // into rows 2, 3
                 : "+v"(a));
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, a), 63));
}

// The same of four values at once: the chains run between each other's steps, so none waits.
static __device__ __forceinline__ void wave_max4(float &a, float &b, float &c, float &d) {
#define DVDQ_MAX4(CTRL)                                             \
    "v_max_f32_dpp %0, %0, %0 " CTRL " bank_mask:0xf\n\t"           \
    "v_max_f32_dpp %1, %1, %1 " CTRL " bank_mask:0xf\n\t"           \
    "v_max_f32_dpp %2, %2, %2 " CTRL " bank_mask:0xf\n\t"           \
    "v_max_f32_dpp %3, %3, %3 " CTRL " bank_mask:0xf\n\t"
    asm volatile("s_nop 1\n\t"
                 DVDQ_MAX4("quad_perm:[1,0,3,2] row_mask:0xf")
                 DVDQ_MAX4("quad_perm:[2,3,0,1] row_mask:0xf")
                 DVDQ_MAX4("row_half_mirror row_mask:0xf")
                 DVDQ_MAX4("row_mirror row_mask:0xf")
                 DVDQ_MAX4("row_bcast:15 row_mask:0xa")
                 DVDQ_MAX4("row_bcast:31 row_mask:0xc")
                 : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
#undef DVDQ_MAX4
    auto last = [](float v) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63)); };
    a = last(a), b = last(b), c = last(c), d = last(d);
}

// entry (r, k) of the 32 x 32 matrix that applies H to the index bits in `mask` and the
// identity to the others, as a bf16 bit pattern (+1, -1 or 0)
static __device__ __forceinline__ uint32_t had5_bf16(int r, int k, int mask) {
    if ((r ^ k) & ~mask & 31) return 0u;
    return (__builtin_popcount(r & k & mask) & 1) ? 0xBF80u : 0x3F80u;
}

// A lane's place in the transform: its 16-byte chunk within a unit (u5 .. u8: the lane's coordinates over the pairings 1, 2, 8,
// 7 = channel-index bits 5 .. 8 of its chunk), the constant MFMA operands and the signs of its butterflies.
// mask5: the channel-index bits 0 .. 4 that the transform covers.
struct HadamardLane {
    int u5, u6, u7, u8, chunk;
    float s1, s2, s8, s7;   // signs of the lane-pairing stages (the lane with the stage's bit set takes the difference)
    bf16x8 tmat[2];
    __device__ __forceinline__ HadamardLane(int lane, int mask5) {
        u8 = (lane >> 2) & 1, u7 = (lane >> 3) & 1, u6 = ((lane >> 1) & 1) ^ u8, u5 = (lane & 1) ^ u8;
        chunk = ((lane >> 4) & 3) | (u5 << 2) | (u6 << 3) | (u7 << 4) | (u8 << 5);
        s1 = u5 ? -1.f : 1.f, s2 = u6 ? -1.f : 1.f, s8 = u7 ? -1.f : 1.f, s7 = u8 ? -1.f : 1.f;
        // rows r = 8 (m / 4) + 4 h + (m % 4) of the 32 x 32 transform, m = lane % 16,
        // columns k = 8 (lane / 16) + t.  MFMA h then yields transformed channels 4h .. 4h+3 of this lane's chunk.
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int m = lane & 15, r = 8 * (m >> 2) + 4 * h + (m & 3);
            uint32_t w[4];
#pragma unroll
            for (int t = 0; t < 8; t += 2) {
                const int k = 8 * (lane >> 4) + t;
                w[t / 2] = had5_bf16(r, k, mask5) | (had5_bf16(r, k + 1, mask5) << 16);
            }
            tmat[h] = __builtin_bit_cast(bf16x8, make_uint4(w[0], w[1], w[2], w[3]));
        }
    }
    // every stage leaves MINUS the difference in the lane whose coordinate is set
    __device__ __forceinline__ float flip(int log2b) const {
        return (((log2b >= 6) & u5) ^ ((log2b >= 7) & u6) ^ ((log2b >= 8) & u7) ^ ((log2b >= 9) & u8)) ? -1.f : 1.f;
    }
    // channel-index bits 0 .. 4 of the lane's 8 values (log2b = 0: the values as they are)
    __device__ __forceinline__ void low_bits(float (&v)[8], uint4 raw, int log2b) const {
        if (log2b == 0) {
            const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[2 * i] = __uint_as_float(w[i] << 16);
                v[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
            }
        } else {
            const bf16x8 data = __builtin_bit_cast(bf16x8, raw);
            const v4f zero = {0.f, 0.f, 0.f, 0.f};
            const v4f d0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tmat[0], data, zero, 0, 0, 0);
            const v4f d1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(tmat[1], data, zero, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[i] = d0[i];
                v[4 + i] = d1[i];
            }
        }
    }
    // bits 5 .. 8
    __device__ __forceinline__ void high_bits(float (&v)[8], int log2b) const {
        if (log2b >= 6) stage_xor1(v, s1);
        if (log2b >= 7) stage_xor2(v, s2);
        if (log2b >= 8) stage_xor8(v, s8);
        if (log2b >= 9) stage_xor7(v, s7);
    }
};

// rounded values (bit patterns of v * r + kRoundMagic) -> 8 int8 codes
static __device__ __forceinline__ uint2 pack_codes_int8(const uint32_t (&b)[8]) {
    uint2 out;   // low bytes of b[0..3] / b[4..7] -> one dword each
    out.x = __builtin_amdgcn_perm(__builtin_amdgcn_perm(b[3], b[2], 0x0c0c0400u),
                                  __builtin_amdgcn_perm(b[1], b[0], 0x0c0c0400u), 0x05040100u);
    out.y = __builtin_amdgcn_perm(__builtin_amdgcn_perm(b[7], b[6], 0x0c0c0400u),
                                  __builtin_amdgcn_perm(b[5], b[4], 0x0c0c0400u), 0x05040100u);
    return out;
}

// -> two codes per byte, in the nibble order the GEMM widens with two masks: byte b of the dword = code[b] (bits 0-3) |
// code[b + 4] (bits 4-7), two's complement
static __device__ __forceinline__ uint32_t pack_codes_nibbles(const uint32_t (&b)[8]) {
    uint32_t u[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) u[i] = (b[i] & 0xFu) | (b[i + 4] << 4);
    return __builtin_amdgcn_perm(__builtin_amdgcn_perm(u[3], u[2], 0x0c0c0400u),
                                 __builtin_amdgcn_perm(u[1], u[0], 0x0c0c0400u), 0x05040100u);
}

// FP6 container: code c as the E2M3 pattern (c < 0) << 5 | |c|, a lane's 8 fields = 48 bits, made by the chip's packed f32 ->
// FP6 conversion: exact integers -7 .. 7 divided by 8 (its scale operand) are E2M3 subnormals m / 8, whose patterns sign << 5 | m are
// the container's fields.  One conversion takes 32 values, field 2 i from element i of its first source and field 2 i + 1 from
// element i of its second: four chunks of a lane at a time, chunk g's even channels in elements 4 g .. 4 g + 3 of the first source and
// its odd channels in those of the second, so that chunk g comes out as bits 48 g .. 48 g + 47.  The instruction reads its sources
// while it writes its result, so the result must not share registers with them (the early-clobber output; the compiler's own
// builtin does not keep them apart).
typedef float fp6_source __attribute__((ext_vector_type(16)));
typedef uint32_t fp6_fields __attribute__((ext_vector_type(6)));
static __device__ __forceinline__ fp6_source fp6_undefined() {   // (don't-cares: left undefined, they cost no instruction)
    const v4f none = {0.f, 0.f, 0.f, 0.f};
    return __builtin_shufflevector(none, none, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1);
}
static __device__ __forceinline__ fp6_fields pack_codes_fp6(fp6_source even, fp6_source odd) {
    fp6_fields pk;
    asm volatile("v_cvt_scalef32_2xpk16_fp6_f32 %0, %1, %2, %3\n\ts_nop 1" : "=&v"(pk) : "v"(even), "v"(odd), "v"(8.0f));
    return pk;
}
// Chunk g's 6 bytes into LDS, at `word` and `half`: an even chunk sits 4-byte aligned in the row's bytes and stores bytes 0-3
// and 4-5, an odd one (2 mod 4) bytes 0-1 and 2-5.
template <int G>
static __device__ __forceinline__ void store_chunk_fp6(fp6_fields pk, bool odd, uint32_t *word, uint16_t *half) {
    // the chunk's three 16-bit pieces h0 h1 h2: an even chunk stores (h0 h1) and h2, an odd one h0 and (h1 h2)
    const uint32_t w0 = pk[3 * (G / 2) + (G & 1)], w1 = pk[3 * (G / 2) + (G & 1) + 1];
    uint32_t h01, h12, h0, h2;
    if (G & 1) {   // bits 16 .. 63 of (w0, w1)
        h01 = __builtin_amdgcn_alignbit(w1, w0, 16); h12 = w1; h0 = w0 >> 16; h2 = w1 >> 16;
    } else {       // bits 0 .. 47
        h01 = w0; h12 = __builtin_amdgcn_alignbit(w1, w0, 16); h0 = w0; h2 = w1;
    }
    *word = odd ? h12 : h01;
    *half = (uint16_t)(odd ? h0 : h2);
}

}  // namespace dvdq
