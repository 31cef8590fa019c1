// Device helpers shared by the persistent GEMM kernels (INT8 matrix path in w4ax_gemm.hip, FP6 matrix
// path in w4a4_fp6_gemm.hip, both operand types with one wave per SIMD in w4ax_gemm_wide.hip): LDS-direct
// loads, hand-kept vmcnt waits, streaming stores, tile order, tile draws.
#pragma once
#include "dvdq_internal.h"

namespace dvdq {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int kBK = 128;      // K slice (bytes of int8 codes per row)
constexpr int kGroup = 32;    // weight rows per native-layout group
constexpr int kGroupBytes = kGroup * kBK / 2;  // 2048: one group, one K slice, packed
constexpr int kNPad = 256;    // native layout pads N to a multiple of this

#define DVDQ_LDS(p) ((__attribute__((address_space(3))) void *)(p))

static __device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
    typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
    v2bf p = {(__bf16)a, (__bf16)b};  // round-to-nearest-even conversions
    return __builtin_bit_cast(uint32_t, p);
}

// Stores of a staged chunk, output the kernel never reads again: 16 bytes per lane in each of four rows 8 apart, from byte
// `off` of the tile's buffer (output_tile below) on; 8 lanes make 128 bytes of a row.
// Non-temporal where rows begin at a multiple of 64 bytes (N of 32): the output stream then bypasses the L2 instead of
// evicting code and weight panels and leaving dirty lines to flush at the kernel's end (FP6, 118800 x 768 x 1536: 121.5 us,
// cached 170.3; 32760 x 1536 x 4608: 163.3 and 175.9).  Where they do not, the 128 bytes begin and end within a line, and
// every part of a line becomes a write to memory of its own: cached stores, which meet in the L2 (118800 x 256 x 952: 155.1
// us non-temporal, 59.5 cached; 32760 x 1536 x 9704: 535.8 and 476.6; int8 codes 118800 x 768 x 1160: 191.3 and 161.9).
// WHICH: the kernel is compiled for one of the two, or tests N at every chunk (a branch there cost the wide INT8 kernel, whose
// epilogue nothing hides, 1 %: 32760 x 1536 x 8960 468.3 and 463.5 us).
enum StoreKind { STORE_BY_PITCH, STORE_STREAMING, STORE_CACHED, STORE_UNALIGNED };
static inline bool streaming_pitch(int64_t N) { return (N & 31) == 0; }
template <StoreKind WHICH = STORE_BY_PITCH>
static __device__ __forceinline__ void store_chunk(__amdgpu_buffer_rsrc_t tile, uint32_t off, int N, const uint4 (&v)[4]) {
    typedef uint32_t v4u __attribute__((ext_vector_type(4)));
    if (WHICH == STORE_STREAMING || (WHICH == STORE_BY_PITCH && (N & 31) == 0)) {
#pragma unroll
        for (int pass = 0; pass < 4; ++pass)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, v[pass]), tile, (int)(off + pass * 16 * N), 0, 2 /* nt */);
    } else {
#pragma unroll
        for (int pass = 0; pass < 4; ++pass)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, v[pass]), tile, (int)(off + pass * 16 * N), 0, 0);
    }
}

// 16 bytes at an address that is only a multiple of 2 (global stores take any)
static __device__ __forceinline__ void store_piece_unaligned(uint16_t *p, uint4 v) {
    struct __attribute__((packed, aligned(2))) Piece { uint32_t d[4]; };
    *reinterpret_cast<Piece *>(p) = Piece{{v.x, v.y, v.z, v.w}};
}

// The chunk of an output whose rows begin at any even address (N no multiple of 8): the piece across a row's end goes out by
// element.  (m, n): the lane's first row and channel.  Cached: parts of lines meet in the L2.  Stored per element, 64 stores of
// 2 bytes in place of 8 of 16 per 32 tokens x 32 channels, these outputs were bound by the stores: whole layers, before -> now,
// FP6 39026 x 256 x 5627 716 -> 210 us (3.4 TB/s of everything moved), int8 74402 x 128 x 239 130 -> 53, 21054 x 3456 x 1827 284 -> 182.
static __device__ __forceinline__ void store_chunk_unaligned(uint16_t *y, int m, int n, int M, int N, const uint4 (&v)[4]) {
    uint16_t *p = y + (int64_t)m * N + n;
#pragma unroll
    for (int pass = 0; pass < 4; ++pass, p += 8 * N) {
        if (m + pass * 8 >= M) continue;
        if (n + 8 <= N) {
            store_piece_unaligned(p, v[pass]);
        } else {
            const uint32_t d[4] = {v[pass].x, v[pass].y, v[pass].z, v[pass].w};
#pragma unroll
            for (int e = 0; e < 7; ++e)
                if (n + e < N) p[e] = (uint16_t)(d[e / 2] >> (16 * (e & 1)));
        }
    }
}

// Buffer of the output rows from m0 on, starting at channel n0, at most bm of them: what lies past row M is past the
// buffer's end, so that a tile at the lower edge of the output is stored by the same instructions as any other (lanes
// past the end are dropped).  Channels past N are the caller's to drop: kPastTile as the offset of a column group does,
// whatever row offset is added to it.  Offsets are 32 bits: N below kMaxTileN.
constexpr uint32_t kPastTile = 0x80000000u;
static __device__ __forceinline__ __amdgpu_buffer_rsrc_t output_tile(uint16_t *y, int m0, int n0, int M, int N, int bm) {
    const int rows = min(bm, M - m0);
    return __builtin_amdgcn_make_buffer_rsrc(y + (int64_t)m0 * N + n0, 0, (rows * N - n0) * 2, 0x00020000);
}

// vmcnt-only wait (leave expcnt / lgkmcnt alone): gfx9 encoding, vmcnt = {imm[15:14], imm[3:0]}
template <int N>
static __device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt is 6 bits");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// One LDS-direct load: 16 bytes per lane from global address `sbase` + `voff` (sbase
// wave-uniform, voff per lane) to LDS address `lds_base` + 16 * lane (lds_base
// wave-uniform).  Written as inline assembly so that the compiler's waitcnt insertion
// does not know about it: with the builtin it makes every later LDS read wait for ALL
// outstanding LDS-direct loads (it cannot tell the ring buffers apart), which
// serializes the pipeline.  Completion is awaited by hand (wait_vmcnt) before the
// workgroup barrier that publishes a buffer.
// (The wait states cover two hazards the compiler cannot see inside the statement: M0 written by the s_mov
// needs one before an LDS-direct load, and a scalar register written by a vector instruction -- a base address
// the compiler has just reloaded with v_readlane or made uniform with v_readfirstlane -- needs five before a
// vector memory instruction reads it: the load would otherwise go to whatever address the register pair held
// before.)
static __device__ __forceinline__ void lds_direct_load16(const void *sbase, uint32_t voff, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(voff), "s"(sbase), "s"(lds_base)
                 : "memory");
}

// Follow-up of lds_direct_load16 with the same M0: the instruction offset OFF is added to the global address
// and to the LDS address alike (checked on the hardware), so a run of loads whose source and destination
// advance by the same number of bytes needs one M0 and one base address.  No other M0 write may stand
// between it and the load that set M0, and the base address must not have been written by a vector instruction
// within the last five wait states (it is the register pair the run's first load used; tests/test_kernel_asm.py
// checks both on the kernels' assembly).
template <int OFF>
static __device__ __forceinline__ void lds_direct_load16_more(const void *sbase, uint32_t voff) {
    static_assert(OFF > 0 && OFF < 4096, "13-bit signed instruction offset");
    asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" : : "v"(voff), "s"(sbase), "n"(OFF) : "memory");
}

// chunk swizzle of a code row in LDS (see the kernel).  A 16-byte read is served 16 lanes = 16 rows at a
// time by the 64 banks (256 bytes), and rows 128 bytes apart alternate between the two halves of the
// banks: the 8 rows of a half take 8 different chunk slots with (row >> 1) & 7.  With 64-byte rows four
// rows share a quarter of the banks and take its 4 slots with (row >> 2) & 3.
template <int BK>
static __device__ __forceinline__ int swz_bk(int row) { return BK == 128 ? ((row >> 1) & 7) : ((row >> 2) & 3); }

// Same, 4 bytes per lane (LDS address lds_base + 4 * lane): used for the per-tile scale vectors.
static __device__ __forceinline__ void lds_direct_load4(const void *sbase, uint32_t voff, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 3\n\tglobal_load_lds_dword %0, %1"
                 :
                 : "v"(voff), "s"(sbase), "s"(lds_base)
                 : "memory");
}

static __device__ __forceinline__ uint32_t lds_address(const void *p) {
    return (uint32_t)(uintptr_t)DVDQ_LDS(p);
}

// make a 64-bit pointer provably wave-uniform (lives in SGPRs)
template <typename T>
static __device__ __forceinline__ const T *uniform_ptr(const T *p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<const T *>(((uint64_t)hi << 32) | lo);
}

// Tile order.  Tiles are numbered so that `group_n` output-column tiles run fastest,
// then token tiles, then column groups: tiles with neighbouring numbers share code
// panels and a bounded set of weight panels, which is what stays in an XCD's L2.
static __device__ __forceinline__ void tile_origin(int t, int tiles_m, int tiles_n, int group_n, int BM, int BN, int &m0,
                                            int &n0) {
    const int per_group = tiles_m * group_n;
    const int grp = t / per_group;
    const int in_grp = t - grp * per_group;
    const int gw = min(group_n, tiles_n - grp * group_n);  // columns in this (possibly last, narrower) group
    const int tile_m = in_grp / gw;
    m0 = tile_m * BM;
    n0 = (grp * group_n + (in_grp - tile_m * gw)) * BN;
}


// ---- tile numbers of a persistent launch
// Workgroup ids are dealt round-robin to the 8 XCDs, and the workgroups of one XCD work on one contiguous
// run of tile numbers at a time.
//   ctr != nullptr: XCD x owns tile numbers [x total / 8, (x + 1) total / 8).  Its i-th workgroup starts with the
//     i-th of them and goes on with the one its neighbour in a pair would take of the next n (n workgroups per XCD); the
//     others are drawn in order through one counter word (an atomic add).  (A workgroup has to
//     know its second tile when it starts.  When it drew both, the workgroups that started first took two tiles
//     each and, with fewer than two tiles per workgroup, left none to the last ones: 732 tiles on 512 workgroups
//     took 65.7 us instead of 52.9, 125 tiles on 128 workgroups 39 instead of 21.  When it drew the second, that draw's
//     reply stood at the start of every launch, and where columns of tiles differ in cost and alternate, as with 343
//     channels, some workgroups took two dear ones: 58675 x 512 x 343 95.3 -> 107.6 us, now 88.5; 9000 x 640 x 3072 35.2
//     -> 31.1, with packed codes 9000 x 1536 x 4608 74.1 -> 64.4, 32760 x 1536 x 8960 474.9 -> 469.9.)  The word is zero when the kernel starts: whatever
//     runs on the stream right before the GEMM clears the slot (the quantizer kernel, if that is what the
//     library enqueued last on the stream, else a small kernel the GEMM's launcher puts in front), so no
//     launch depends on what an earlier one -- finished or not -- left behind, and nothing has to be put back
//     at the end.
//     With at most two tiles per workgroup there is nothing to draw: such a launch is handed words that no one clears and no one
//     counts in (idle_slot), so a GEMM called on its own has no clearing kernel in front of it, and its workgroups no atomics to wait for
//     (with bias and zero-points, GEMM alone, us: 15600 x 768 x 1536 packed codes 32.8 -> 28.3, 20000 x 1024 x 1024 int8 37.3 -> 32.2,
//     12000 x 3072 x 2048 FP6 54.0 -> 49.6; without the clearing kernel only, 31.0, 35.4, 52.4).  One that is captured, and that several
//     graph instances may run at once, starts with the same two tiles.
//     Up to kCusPerXcd tiles more than workgroups are fixed shares all the same: those tiles go to the first XCD, one to a compute unit,
//     and beside their neighbours' shared panels that is 1 to 2 % faster than one here and there (in graphs, 120 launches of up to 32 such
//     tiles: 0.96 to 1.10 of the time as fixed shares, 1.01 in the mean; from 33 on, two to a compute unit, 0.80 to 1.08, 0.93 in the mean).
//   ctr == nullptr: fixed shares, the j-th tile of workgroup b is number j * grid + (b % 8) * (grid / 8) + b / 8.
struct TileSource {
    int total, grid, xcd, first_tile, run_lo;
    unsigned run_len, wgs, fixed;   // tiles and workgroups of this XCD; tiles the workgroups start with, two each
    unsigned *ctr;        // this XCD's counter (nullptr: fixed shares)
    unsigned *draw_ctr;   // the same where there is something to draw

    // stride: words between the XCDs' counters
    __device__ __forceinline__ TileSource(int tiles_m, int tiles_n, unsigned *sched, int stride = kSchedStride) {
        total = tiles_m * tiles_n;
        grid = gridDim.x;   // a multiple of 8
        xcd = blockIdx.x % 8;
        first_tile = xcd * (grid / 8) + blockIdx.x / 8;
        run_lo = (int)((int64_t)xcd * total / 8);
        run_len = (unsigned)((int64_t)(xcd + 1) * total / 8) - (unsigned)run_lo;
        wgs = gridDim.x / 8;
        fixed = min(run_len, 2 * wgs);
        ctr = sched ? sched + xcd * stride : nullptr;
        draw_ctr = run_len > fixed ? ctr : nullptr;
    }
    // the tile a draw's reply stands for (drawn mode), or the workgroup's ordinal-th tile (fixed shares); -1: none left
    __device__ __forceinline__ int tile(unsigned reply, int ordinal) const {
        if (ctr) return reply < run_len - fixed ? run_lo + (int)(fixed + reply) : -1;
        const int t = first_tile + ordinal * grid;
        return t < total ? t : -1;
    }
    // one further tile (one lane; drawn mode only).  The reply may be awaited as late as the caller likes.
    __device__ __forceinline__ unsigned draw() const { return atomicAdd(ctr, 1u); }
    // the workgroup's first two tiles (one lane; either mode)
    __device__ __forceinline__ void first_two(int &t0, int &t1) const {
        if (ctr) {
            const unsigned i = blockIdx.x / 8, second = wgs + ((i ^ 1u) < wgs ? i ^ 1u : i);
            t0 = i < run_len ? run_lo + (int)i : -1;
            t1 = second < run_len ? run_lo + (int)second : -1;
        } else {
            t0 = tile(0u, 0);
            t1 = tile(0u, 1);
        }
    }
};

// ---- epilogues of the two-waves-per-SIMD kernels (INT8 matrix path and FP6 matrix path)
// Both kernels end a tile the same way; what differs is how an accumulator register turns into the integer sum
// of code products, which an accumulator policy states:
//   AccI32<SHIFT>: int32 registers holding 2^SHIFT times the sum (the widened operands' factor);
//   AccF32x64:     fp32 registers holding the sum / 64 exactly (FP6 values are codes / 8).
// Accumulator register r = 4 g + e of MFMA tile (i, j) in lane l is
//   n = n0 + wn + 32 i + 8 g + 4 (l / 32) + e,   m = m0 + wm + 32 j + (l % 32).
// With weight zero-points, sum q (c - z) = acc - z * rs (rs the token's code sum) is taken with a 24-bit
// multiply: operands and product are in range (checked by the C ABI), so it is exact.
template <int SHIFT>
struct AccI32 {
    typedef v16i vec;
    // factor folded into the token scale (a power of two: exact)
    static __device__ __forceinline__ constexpr float fold(bool) { return 1.f / (float)(1 << SHIFT); }
    template <bool ZP>
    static __device__ __forceinline__ float scaled(int a, int z, int rs, float xs_folded) {
        if constexpr (ZP) a -= __mul24(z * (1 << SHIFT), rs);
        return (float)a * xs_folded;
    }
    // per-element path: the register's integer (still times 2^SHIFT), its zero-point term, the plain sum
    static __device__ __forceinline__ int integer(int a) { return a; }
    static __device__ __forceinline__ int unzero(int v, int z, int rs) { return v - __mul24(z * (1 << SHIFT), rs); }
    static __device__ __forceinline__ int sum(int v) { return v >> SHIFT; }
    static __device__ __forceinline__ constexpr float edge_fold() { return 1.f / (float)(1 << SHIFT); }
};

struct AccF32x64 {
    typedef v16f vec;
    // without zero-points the token scale times 64 multiplies the fp32 accumulator directly
    static __device__ __forceinline__ constexpr float fold(bool zp) { return zp ? 1.f : 64.f; }
    template <bool ZP>
    static __device__ __forceinline__ float scaled(float a, int z, int rs, float xs_folded) {
        if constexpr (ZP) return (float)((int)(a * 64.f) - __mul24(z, rs)) * xs_folded;
        else return a * xs_folded;
    }
    static __device__ __forceinline__ int integer(float a) { return (int)(a * 64.f); }
    static __device__ __forceinline__ int unzero(int v, int z, int rs) { return v - __mul24(z, rs); }
    static __device__ __forceinline__ int sum(int v) { return v; }
    static __device__ __forceinline__ constexpr float edge_fold() { return 1.f; }
};

// LDS image of a tile's epilogue vectors (staged by LDS-direct loads with the tile's first slice): token scales
// fp32 [BM], channel scales fp32 [BN], bias bf16 [BN], code sums int32 [BM], zero-points int8 [BN]
template <int BM, int BN>
struct TileVectors {
    static constexpr int OFF_BIAS = (BM + BN) * 4, OFF_RSUM = OFF_BIAS + BN * 2, OFF_ZERO = OFF_RSUM + BM * 4;
    static constexpr int BYTES = OFF_ZERO + (BN < 256 ? 256 : BN);   // (zero-points come 256 at a time)
};

// The bias and zero-points of the last N % 4 channels, in the image of the tile at n0: the LDS-direct loads bring whole dwords
// of channels below N only.  (Every wave writes them, the same values, and reads its own.)
template <int BM, int BN>
static __device__ __forceinline__ void fill_vector_tail(uint8_t *s_tile, const uint16_t *bias, const int8_t *w_zero, int lane,
                                                        int n0, int N) {
    if ((N & 3) == 0 || n0 + BN <= N) return;
    const int n = (N & ~3) + lane;
    if (n < N) {
        if (bias) reinterpret_cast<uint16_t *>(s_tile + TileVectors<BM, BN>::OFF_BIAS)[n - n0] = bias[n];
        if (w_zero) reinterpret_cast<int8_t *>(s_tile + TileVectors<BM, BN>::OFF_ZERO)[n - n0] = w_zero[n];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Any tile of an output with N a multiple of 8, or of any other with STORE_UNALIGNED (below kMaxTileN; tiles at the edges included: see output_tile; specialized on zero-points and, where the caller
// can afford the code, on bias: a run-time test inside the unrolled loops costs a branch per register group): no predicates, every
// vector the epilogue needs comes from LDS, one row offset per lane.  (Edge tiles used to go through epilogue_edge, per
// element with a global load per zero-point; on outputs whose token count is no multiple of the tile the last tiles of a
// launch then ran several times as long as the others: 5000 x 512 x 3072 with zero-points 27.7 us, now 17.5 (int8 codes).)  The bf16 tile goes through LDS so that every store instruction
// writes whole 128-byte lines: in the accumulator layout a lane owns one token and 8 consecutive channels per
// register group, so a direct store touches 32 token rows with 32 bytes each.  32 tokens x 64 channels at a
// time are staged in `stg` (this wave's 4 KB of the ring buffer whose slice was consumed last: after the
// barrier no wave reads it any more, and the next loads into it are only issued after the next K loop's first
// barrier; 16-byte pieces, piece index xor-ed with the row against bank conflicts) and read back with 8 lanes
// per token row.  A lane's channel vectors (4 channel scales, bias, zero-points) for register group g of MFMA
// tile column i are fetched one group ahead of their use: a read issued where its value is needed would
// expose the LDS latency once per group, 32 times per tile.  The accumulators are left at zero.
// BIAS: 1 / 0 = with / without bias, fixed at compile time; -1 = `has_bias` decides at run time (for kernels
// whose register budget does not survive four inlined copies of this function).
template <class P, int BM, int BN, int TM, int TN, bool ZP, int BIAS, StoreKind STORE>
static __device__ __forceinline__ void epilogue_interior(typename P::vec (&acc)[TN][TM], const uint8_t *s_tile, bool has_bias,
                                                         int lane, int wm, int wn, uint8_t *stg, uint16_t *y, int m0,
                                                         int n0, int M, int N) {
    // (scale, then add the bias, each rounded: a fused multiply-add would differ from the per-element path in the last bit)
#pragma clang fp contract(off)
    if constexpr (BIAS >= 0) has_bias = BIAS != 0;
    typedef TileVectors<BM, BN> TV;
    const int frow = lane & 31, fhalf = lane >> 5;
    const float *s_xs = reinterpret_cast<const float *>(s_tile);
    const float *ws_l = s_xs + BM + wn + fhalf * 4;
    const int32_t *s_rsum = reinterpret_cast<const int32_t *>(s_tile + TV::OFF_RSUM);
    const uint32_t *bias_l = reinterpret_cast<const uint32_t *>(s_tile + TV::OFF_BIAS) + (wn + fhalf * 4) / 2;
    const uint32_t *zero_l = reinterpret_cast<const uint32_t *>(s_tile + TV::OFF_ZERO) + (wn + fhalf * 4) / 4;
    float xs_l[TM];
    int rsum[TM];
#pragma unroll
    for (int j = 0; j < TM; ++j) {
        xs_l[j] = s_xs[wm + j * 32 + frow] * P::fold(ZP);
        rsum[j] = ZP ? s_rsum[wm + j * 32 + frow] : 0;
    }
    const int rd_row = lane >> 3, rd_piece = lane & 7;
    const __amdgpu_buffer_rsrc_t tile = output_tile(y, m0, n0, M, N, BM);
    const uint32_t lane_off = ((wm + rd_row) * N + wn + rd_piece * 8) * 2;
    struct ChannelVec { float4 ws; uint2 bb; uint32_t zq; };
    auto fetch = [&] __device__(ChannelVec &cv, int i, int g) {
        const int c = i * 32 + g * 8;
        cv.ws = *reinterpret_cast<const float4 *>(ws_l + c);
        if (has_bias) cv.bb = *reinterpret_cast<const uint2 *>(bias_l + c / 2);
        if constexpr (ZP) cv.zq = zero_l[c / 4];
    };
    ChannelVec cv[2];   // group k of the tile's groups lives in cv[k & 1]
    fetch(cv[0], 0, 0);
    int k = 0;
#pragma unroll
    for (int ip = 0; ip < TN / 2; ++ip) {
#pragma unroll
        for (int j = 0; j < TM; ++j) {
#pragma unroll
            for (int ii = 0; ii < 2; ++ii) {
                const int i = 2 * ip + ii;
#pragma unroll
                for (int g = 0; g < 4; g += 2) {
                    uint32_t pk[2][2];
#pragma unroll
                    for (int h = 0; h < 2; ++h, ++k) {
                        {   // the group after this one, in this loop nest's order
                            int gn = g + h + 1, iin = ii, jn = j, ipn = ip;
                            if (gn == 4) { gn = 0; if (++iin == 2) { iin = 0; if (++jn == TM) { jn = 0; ++ipn; } } }
                            if (ipn < TN / 2) fetch(cv[(k + 1) & 1], 2 * ipn + iin, gn);
                        }
                        const ChannelVec &c = cv[k & 1];
                        const int r = (g + h) * 4;
                        float o[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            o[e] = P::template scaled<ZP>(acc[i][j][r + e], (int)(int8_t)(c.zq >> (8 * e)), rsum[j], xs_l[j]);
                            acc[i][j][r + e] = 0;
                        }
                        o[0] *= c.ws.x;
                        o[1] *= c.ws.y;
                        o[2] *= c.ws.z;
                        o[3] *= c.ws.w;
                        if (has_bias) {
                            o[0] += __uint_as_float(c.bb.x << 16);
                            o[1] += __uint_as_float(c.bb.x & 0xFFFF0000u);
                            o[2] += __uint_as_float(c.bb.y << 16);
                            o[3] += __uint_as_float(c.bb.y & 0xFFFF0000u);
                        }
                        pk[h][0] = pack_bf16x2(o[0], o[1]);
                        pk[h][1] = pack_bf16x2(o[2], o[3]);
                    }
                    // lanes l and l+32 hold channels (8g .. 8g+3) and (8g+4 .. 8g+7): swap the upper half
                    // of group g with the lower half of group g+1 so each lane owns 8 consecutive channels
#pragma unroll
                    for (int d = 0; d < 2; ++d) {
                        auto sw = __builtin_amdgcn_permlane32_swap(pk[0][d], pk[1][d], false, false);
                        pk[0][d] = sw[0];
                        pk[1][d] = sw[1];
                    }
                    const int piece = ii * 4 + g + fhalf;   // 16-byte piece of the 64-channel row
                    *reinterpret_cast<uint4 *>(stg + frow * 128 + ((piece ^ (frow & 7)) << 4)) =
                        make_uint4(pk[0][0], pk[0][1], pk[1][0], pk[1][1]);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const uint32_t off = n0 + wn + ip * 64 + rd_piece * 8 < N ? lane_off + (j * 32 * N + ip * 64) * 2 : kPastTile;
            uint4 v[4];
#pragma unroll
            for (int pass = 0; pass < 4; ++pass) {
                const int row = pass * 8 + rd_row;
                v[pass] = *reinterpret_cast<const uint4 *>(stg + row * 128 + ((rd_piece ^ (row & 7)) << 4));
            }
            if constexpr (STORE != STORE_UNALIGNED) store_chunk<STORE>(tile, off, N, v);
            else store_chunk_unaligned(y, m0 + wm + j * 32 + rd_row, n0 + wn + ip * 64 + rd_piece * 8, M, N, v);
            __builtin_amdgcn_wave_barrier();   // the next chunk's LDS writes stay behind these reads
        }
    }
}

// N below 8 or kMaxTileN and more, the accumulator hook, and N no multiple of 8 in the kernels without STORE_UNALIGNED: predicated
// per element, through the integer accumulator (same values and rounding order as the interior path).  The accumulators are left at zero.
template <class P, int BM, int BN, int TM, int TN>
static __device__ __forceinline__ void epilogue_edge(typename P::vec (&acc)[TN][TM], const uint8_t *s_tile, const uint16_t *bias,
                                                     const int8_t *w_zero, int lane, int wm, int wn, uint16_t *y,
                                                     int32_t *acc_out, int m0, int n0, int M, int N) {
    typedef TileVectors<BM, BN> TV;
    const int frow = lane & 31, fhalf = lane >> 5;
    const float *s_xs = reinterpret_cast<const float *>(s_tile);
    const float *s_ws = s_xs + BM;
    const int32_t *s_rsum = reinterpret_cast<const int32_t *>(s_tile + TV::OFF_RSUM);
    const bool vec8 = (N & 7) == 0;
#pragma unroll
    for (int j = 0; j < TM; ++j) {
        const int m = m0 + wm + j * 32 + frow;
        const bool m_ok = m < M;
        const float xs = s_xs[wm + j * 32 + frow] * P::edge_fold();
        const int rs = w_zero ? s_rsum[wm + j * 32 + frow] : 0;
#pragma unroll
        for (int i = 0; i < TN; ++i) {
            const int nb = n0 + wn + i * 32;   // this MFMA tile's first output channel
            int a[16];
#pragma unroll
            for (int g = 0; g < 4; ++g)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // (channels past N: some valid zero-point, for values that are never stored)
                    const int z = w_zero ? (int)w_zero[min(nb + g * 8 + fhalf * 4 + e, N - 1)] : 0;
                    a[g * 4 + e] = P::unzero(P::integer(acc[i][j][g * 4 + e]), z, rs);
                    acc[i][j][g * 4 + e] = 0;
                }
            if (acc_out && m_ok) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int n = nb + g * 8 + fhalf * 4;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (n + e < N) acc_out[(int64_t)m * N + n + e] = P::sum(a[g * 4 + e]);
                }
            }
            if (vec8) {
                uint32_t pk[4][2];
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int n = nb + g * 8 + fhalf * 4;
                    float o[4];
                    if (n < N) {  // N % 8 == 0 and n % 4 == 0: n + 3 < N as well
                        const float4 ws = *reinterpret_cast<const float4 *>(s_ws + (n - n0));
                        o[0] = (float)a[g * 4 + 0] * xs * ws.x;
                        o[1] = (float)a[g * 4 + 1] * xs * ws.y;
                        o[2] = (float)a[g * 4 + 2] * xs * ws.z;
                        o[3] = (float)a[g * 4 + 3] * xs * ws.w;
                        if (bias) {
                            const uint2 bb = *reinterpret_cast<const uint2 *>(bias + n);
                            o[0] += __uint_as_float(bb.x << 16);
                            o[1] += __uint_as_float(bb.x & 0xFFFF0000u);
                            o[2] += __uint_as_float(bb.y << 16);
                            o[3] += __uint_as_float(bb.y & 0xFFFF0000u);
                        }
                    } else {
                        o[0] = o[1] = o[2] = o[3] = 0.f;
                    }
                    pk[g][0] = pack_bf16x2(o[0], o[1]);
                    pk[g][1] = pack_bf16x2(o[2], o[3]);
                }
                // lanes l and l+32 hold channels (8g .. 8g+3) and (8g+4 .. 8g+7): swap the upper half of
                // group g with the lower half of group g+1 so each lane owns 8 consecutive channels
#pragma unroll
                for (int g = 0; g < 4; g += 2) {
#pragma unroll
                    for (int d = 0; d < 2; ++d) {
                        auto r = __builtin_amdgcn_permlane32_swap(pk[g][d], pk[g + 1][d], false, false);
                        pk[g][d] = r[0];
                        pk[g + 1][d] = r[1];
                    }
                    const int n = nb + g * 8 + fhalf * 8;
                    if (m_ok && n < N)
                        *reinterpret_cast<uint4 *>(y + (int64_t)m * N + n) =
                            make_uint4(pk[g][0], pk[g][1], pk[g + 1][0], pk[g + 1][1]);
                }
            } else if (m_ok) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int n = nb + g * 8 + fhalf * 4;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if (n + e >= N) break;
                        float o = (float)a[g * 4 + e] * xs * s_ws[n + e - n0];
                        if (bias) o += __uint_as_float((uint32_t)bias[n + e] << 16);
                        y[(int64_t)m * N + n + e] = (uint16_t)(pack_bf16x2(o, 0.f) & 0xFFFFu);
                    }
                }
            }
        }
    }
}

// Enqueues the kernel that zeroes a counter slot (sched_slot; defined in w4ax_gemm.hip).
int clear_sched_slot(unsigned *slot, hipStream_t stream);

}  // namespace dvdq
