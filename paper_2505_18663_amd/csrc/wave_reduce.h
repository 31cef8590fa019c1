// Reductions over the 64 lanes of a wave (or over groups of them) in registers: quad permutes and row mirrors as DPP
// operands within 16 lanes, gfx950's row swaps across them.  A shuffle (__shfl_xor) goes through the LDS permute unit,
// with its latency at each of the six levels.
// The mirrors pair lanes as l ^ 7 and l ^ 15; the lanes of a quad (of 8) already agree by then, so these are the
// missing l ^ 4 and l ^ 8 for any reduction that leaves its result in all lanes.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dvdq {

enum { DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141, DPP_MIRROR = 0x140, DPP_ROR8 = 0x128 };

template <int CTRL, typename T>
static __device__ __forceinline__ T dpp(T v) {
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
    } else {
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xF, 0xF, true);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, true);
        return __builtin_bit_cast(T, ((uint64_t)hi << 32) | lo);
    }
}

// op(value of lane l, value of lane l ^ 16), the same in both; likewise l ^ 32
template <bool ROWS32, class Op, typename T>
static __device__ __forceinline__ T swap_rows(T v, Op op) {
    auto swap = [](uint32_t x) {
        if constexpr (ROWS32) return __builtin_amdgcn_permlane32_swap(x, x, false, false);
        else return __builtin_amdgcn_permlane16_swap(x, x, false, false);
    };
    if constexpr (sizeof(T) == 4) {
        const auto r = swap(__builtin_bit_cast(uint32_t, v));
        return op(__builtin_bit_cast(T, (uint32_t)r[0]), __builtin_bit_cast(T, (uint32_t)r[1]));
    } else {
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        const auto lo = swap((uint32_t)u), hi = swap((uint32_t)(u >> 32));
        return op(__builtin_bit_cast(T, ((uint64_t)hi[0] << 32) | lo[0]), __builtin_bit_cast(T, ((uint64_t)hi[1] << 32) | lo[1]));
    }
}

// sum over the wave, the same in every lane (a fixed order of additions)
template <typename T>
static __device__ __forceinline__ T wave_sum(T v) {
    auto add = [](T a, T b) { return a + b; };
    v += dpp<DPP_XOR1>(v);
    v += dpp<DPP_XOR2>(v);
    v += dpp<DPP_HALF_MIRROR>(v);
    v += dpp<DPP_MIRROR>(v);
    v = swap_rows<false>(v, add);
    return swap_rows<true>(v, add);
}

}  // namespace dvdq
