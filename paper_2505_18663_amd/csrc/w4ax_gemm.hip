// W4Ax GEMM for gfx950, fast path for pre-packed ("native") weights: int8
// activation codes x packed INT4 weights on the INT8 matrix cores, exact int32
// accumulation, dequantizing epilogue to bf16 (Sec. 3.2: Y = X^ Lambda W^^T;
// Sec. 3.1 DeQuant with zero-point 0).
//
// Data movement.  Both operands travel HBM/L2 -> LDS with LDS-direct loads
// (16 bytes per lane, no VGPR staging) through a ring of STAGES buffers; K is
// consumed in slices of 128.  Completion is tracked by hand with s_waitcnt vmcnt
// because the compiler does not order LDS reads after LDS-direct loads.
//   codes  : [row][128 B], the 16-byte chunk index xor-ed with (row & 7), so the 8 lanes
//            that read the same chunk of 8 consecutive rows cover a whole 128-byte LDS
//            bank line; a wave's load instruction covers 8 full 128-byte rows.
//   weights: stay packed (two codes per byte) in LDS; the native layout is the LDS
//            image itself, so a slice is one linear, fully coalesced copy:
//            [k128 slice][32-row group][k32 step][k16 half][row][8 B].
//            The 8 bytes hold 16 consecutive channels; byte b of dword d carries
//            channel 8d+b in its low and channel 8d+b+4 in its high nibble, so that
//            (p << 4) & 0xF0F0F0F0 and p & 0xF0F0F0F0 are int8 lanes of 16*code in
//            channel order.  The MFMA then accumulates 16*acc exactly; the factor
//            is folded into the token scale (a power of two) or shifted out.
//
// Compute.  A workgroup of WAVES_M x WAVES_N waves owns a BM x BN tile; a wave a
// (BM/WAVES_M) x (BN/WAVES_N) sub-tile of 32x32x32 MFMAs.  The weight fragment is
// the MFMA's row operand and the code fragment its column operand, so a lane holds
// 4 consecutive output channels of one token; lane halves are exchanged
// (v_permlane32_swap) so that every lane stores 16 contiguous bytes of bf16.
#include <mutex>
#include <type_traits>
#include <unordered_map>
#include <vector>

#include "gemm_common.h"

namespace dvdq {

// Operands: int8 codes, or packed 4-bit codes, with native weights; int8 codes with canonical weights ([N, K/2] as an offline
// quantizer hands them over, K any multiple of 32).
enum Operands { OPS_INT8, OPS_PACKED4, OPS_CANONICAL };

// STORE: how tiles are stored (see store_chunk).  STORE_UNALIGNED is the kernel for N >= 8 no multiple of 8 (without
// the accumulator hook); the others store such outputs per element.
template <int BM, int BN, int BK, int WAVES_M, int WAVES_N, int STAGES, int OCC, Operands OPS, StoreKind STORE>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N, OCC) void w4ax_gemm_native_kernel(
    const int8_t *__restrict__ codes, const float *__restrict__ x_scale, const uint8_t *__restrict__ w,
    const float *__restrict__ w_scale, const int8_t *__restrict__ w_zero, const int32_t *__restrict__ code_rowsum,
    const uint16_t *__restrict__ bias, int M, int N, int K, uint16_t *__restrict__ y, int32_t *__restrict__ acc_out,
    int tiles_m, int tiles_n, int group_n, unsigned *__restrict__ sched) {
    constexpr bool UNALIGNED = STORE == STORE_UNALIGNED, A4 = OPS == OPS_PACKED4, CANON = OPS == OPS_CANONICAL;
    constexpr int NW = WAVES_M * WAVES_N;
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;  // wave sub-tile
    constexpr int TM = WM / 32, TN = WN / 32;            // MFMA tiles per wave
    // A4: the codes arrive packed two per byte (same nibble order as the weights) and are
    // widened to int8 lanes of 16 * code in registers like the weights.  A lane's 16-byte code
    // fragment then spans 32 channels, so one pipeline step covers 64 channels = 2 MFMAs per tile.
    constexpr int A_ROW = A4 ? BK / 2 : BK;              // bytes of one code row per item
    // CANON: the packed weights of a row are loaded as they are, 16 bytes = 32 channels a piece, and such a piece is a lane's weight
    // fragment of a 64-channel step likewise; the code fragments are put into its order (see deal_codes).
    constexpr int NT = A4 || CANON ? 2 : 1;              // MFMAs along K per step and output tile
    constexpr int KS = BK / (32 * NT);                   // pipeline steps per item
    constexpr int A_STAGE = BM * A_ROW, W_STAGE = BN * BK / 2, STAGE = A_STAGE + W_STAGE;
    constexpr int A_DMA = A_STAGE / 1024 / NW;           // LDS-direct loads per wave per item (1 KB each)
    constexpr int W_DMA = W_STAGE / 1024 / NW;
    constexpr int DMA = A_DMA + W_DMA;
    constexpr int CHUNKS = A_ROW / 16;                   // 16-byte chunks per code row in LDS
    constexpr int ROWS_PER_DMA = 1024 / A_ROW;           // code rows one wave-wide load covers
    constexpr int W_GROUP = kGroup * BK / 2;             // bytes of one 32-row weight group per item
    // With 3 or more buffers the item after the current one is already published, so the
    // first fragments of item q+1 are fetched while the last MFMAs of item q run.
    constexpr int AHEAD = STAGES >= 3 ? 1 : 0;
    // one tile's epilogue vectors in LDS: token scales, channel scales (fp32), bias (bf16), and for
    // weights with zero-points the tokens' code sums (int32) and the channels' zero-points (int8)
    typedef TileVectors<BM, BN> TV;
    constexpr int OFF_BIAS = TV::OFF_BIAS, OFF_RSUM = TV::OFF_RSUM, OFF_ZERO = TV::OFF_ZERO, SCALES = TV::BYTES;
    constexpr int SHIFT = A4 ? 8 : 4;                    // log2 of the factor the widened operands carry
    constexpr int STORES = TM * TN * 2;                  // 16-byte store instructions per wave per full tile
    static_assert((STAGES - 2 - AHEAD) * DMA + STORES < 64, "store-aware wait exceeds vmcnt");
    static_assert(BK == 64 || BK == 128, "K slice per item");
    static_assert(A_ROW == 64 || A_ROW == 128, "code row bytes per item");
    static_assert(A_DMA >= 1 && W_DMA >= 1 && A_DMA * 1024 * NW == A_STAGE && W_DMA * 1024 * NW == W_STAGE,
                  "tile does not split over the waves");
    static_assert(STAGES >= 2 && (STAGES - 1) * DMA < 64, "too many loads in flight for vmcnt");
    static_assert(NW * 4096 <= STAGE && TN % 2 == 0, "the epilogue stages 4 KB per wave in one ring buffer");

    extern __shared__ __align__(16) uint8_t smem[];
    const uint32_t smem_base = lds_address(smem);

    auto swz = [] __device__(int row) { return swz_bk<A_ROW>(row); };
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = (wave % WAVES_M) * WM, wn = (wave / WAVES_M) * WN;
    const int KT = CANON ? (K + BK - 1) / BK : K / BK;
    const int k_tail = CANON ? K - (KT - 1) * BK : BK;   // channels of the last slice (CANON: 32 .. BK)
    const int G = ((N + kNPad - 1) / kNPad) * (kNPad / kGroup);  // 32-row groups in the padded weight buffer
    const int64_t w_slice_stride = (int64_t)G * kGroupBytes;
    const int code_row_bytes = A4 ? K / 2 : K;

    // Persistent workgroups take tiles until none is left: drawn per XCD through counters (sched), or in
    // fixed shares (see TileSource).  The two workgroups of a compute unit do not run at the same speed (the
    // older one wins the issue arbitration), so equal shares would leave the faster ones idle for the last
    // tenth of the kernel.
    // The tile numbers a workgroup has drawn go through an 8-entry ring in LDS (s_tiles; -1 = no
    // tile left).  Wave 0 draws tile n + 2 while the loads of tile n are being enqueued and writes the
    // number into the ring one item later, before that item's barrier: the atomic's reply is then
    // older than loads the wave has already awaited, so the draw never stalls anything.
    const TileSource tiles(tiles_m, tiles_n, sched);
    typedef volatile __attribute__((address_space(3))) int lds_int;   // (explicitly LDS: a generic volatile access would be a flat one)
    lds_int *s_tiles = (lds_int *)DVDQ_LDS(smem + STAGES * STAGE + 2 * SCALES);
    int draws = 0;           // tiles drawn so far (the same in every wave)
    unsigned drawn = 0;      // wave 0, lane 0: reply of the draw not yet written into the ring
    bool draw_pending = false;
    auto draw = [&] __device__() {
        if (wave == 0 && tiles.draw_ctr && lane == 0) drawn = tiles.draw();
        ++draws;
        draw_pending = true;
    };
    auto publish_draw = [&] __device__() {   // before a workgroup barrier
        if (wave == 0) {
            if (lane == 0) s_tiles[(draws - 1) & 7] = tiles.tile(drawn, draws - 1);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
        draw_pending = false;
    };
    // the first two tiles follow from the workgroup's number
    if (wave == 0 && lane == 0) {
        int t0, t1;
        tiles.first_two(t0, t1);
        s_tiles[0] = t0;
        s_tiles[1] = t1;
    }
    draws = 2;
    __syncthreads();
    int comp_tile = __builtin_amdgcn_readfirstlane(s_tiles[0]);   // tile being multiplied
    if (comp_tile < 0) return;   // (whole workgroup: nothing below is reached, no barrier is missed)

    // ---- LDS-direct load addressing: wave-uniform base pointer + per-lane 32-bit offset.
    // codes: load slot i of this wave fills ROWS_PER_DMA consecutive LDS rows of the stage;
    // LDS position p of a row holds the row's 16-byte chunk p ^ swz(row), where swz spreads
    // the 16 rows that one quarter-wave reads over the 64 banks (see swz_bk).
    int a_row[A_DMA];
    uint32_t a_voff[A_DMA];
#pragma unroll
    for (int i = 0; i < A_DMA; ++i) a_row[i] = (wave * A_DMA + i) * ROWS_PER_DMA + lane / CHUNKS;
    // weights: per item and 32-row group a contiguous run of W_GROUP bytes in the native buffer, so the
    // 1 KB piece p of the stage's weight image starts at byte p * W_PIECE of the item's slice: a
    // wave-uniform term (added to the scalar base) plus 16 bytes per lane
    constexpr int W_PIECE = 1024 / W_GROUP * kGroupBytes + 1024 % W_GROUP;
    static_assert(W_GROUP == kGroupBytes || W_GROUP == 1024, "piece offsets are linear for whole slices or one group per piece");
    const uint32_t lane16 = lane * 16;
    // CANON: a load of weights is 16 rows of 4 pieces, swizzled like code rows of 64 bytes
    uint32_t w_voff[CANON ? W_DMA : 1];
    const int w_chunk = (lane & 3) ^ swz_bk<64>(lane >> 2);
    const int8_t *a_base = codes;   // start of the tile's first code row, advanced by BK per item
    const uint8_t *w_base = w;      // start of the tile's weight image for the item
    int issue_tile = 0, issue_kt = 0;   // next item to enqueue: K slice issue_kt of this workgroup's tile issue_tile
    bool issue_live = true;             // false once the ring says there is no further tile
    const int draw_kt = KT > 1 ? 1 : 0; // slice at whose enqueueing the tile after next is drawn
    uint32_t issue_sa = 0;                          // LDS address of the buffer being filled
    // The loads of one item are enqueued one at a time (issue_one) so they can be spread
    // between the MFMAs of the slice being multiplied.  Past the last item the same slice
    // is enqueued again (harmless, keeps the load count per item uniform for vmcnt).
    auto issue_prepare = [&] __device__(int buf) {
        int issue_no = -1;
        if (issue_live && issue_kt == 0) {
            issue_no = __builtin_amdgcn_readfirstlane(s_tiles[issue_tile & 7]);
            issue_live = issue_no >= 0;
        }
        if (issue_live && issue_kt == draw_kt) draw();
        if (issue_no >= 0) {
            int m0, n0;
            tile_origin(issue_no, tiles_m, tiles_n, group_n, BM, BN, m0, n0);
            a_base = uniform_ptr(codes + (int64_t)m0 * code_row_bytes);
            w_base = uniform_ptr(CANON ? w + (int64_t)n0 * (K / 2) : w + (int64_t)(n0 / kGroup) * kGroupBytes);
            if constexpr (CANON) {
#pragma unroll
                for (int i = 0; i < W_DMA; ++i)   // (rows past N re-read the last one)
                    w_voff[i] = (uint32_t)min((wave * W_DMA + i) * 16 + (lane >> 2), N - 1 - n0) * (K / 2) + w_chunk * 16;
            }
#pragma unroll
            for (int i = 0; i < A_DMA; ++i) {
                const int row = min(a_row[i], M - 1 - m0);   // rows past M re-read the last valid row
                a_voff[i] = (uint32_t)row * code_row_bytes + (((lane % CHUNKS) ^ swz(a_row[i])) << 4);
            }
            // The tile's scales go to LDS as well ([BM token scales][BN channel scales], two tiles
            // deep), so that the epilogue needs no vector-memory load: such a load would queue
            // behind the LDS-direct loads in flight.  Indices past M / N repeat the last valid one.
            // They are issued ahead of the tile's first data loads and are therefore complete
            // whenever that item is published.
            const uint32_t sc = smem_base + STAGES * STAGE + (issue_tile & 1) * SCALES;
#pragma unroll
            for (int j = 0; j < (BM + BN) / 64; ++j) {
                if (j % NW != wave) continue;
                if (j < BM / 64)
                    lds_direct_load4(x_scale, (uint32_t)min(m0 + j * 64 + lane, M - 1) * 4, sc + j * 256);
                else
                    lds_direct_load4(w_scale, (uint32_t)min(n0 + (j - BM / 64) * 64 + lane, N - 1) * 4, sc + j * 256);
            }
            // (bias and zero-points go to LDS, pairs and fours of channels at a time, where N is a multiple of 8 or, with STORE_UNALIGNED,
            // any other; the last N % 4 channels follow in front of the epilogue, see fill_vector_tail.  Elsewhere the epilogue reads them
            // from memory)
            if (bias && (UNALIGNED || (N & 7) == 0)) {
#pragma unroll
                for (int j = 0; j < BN / 128; ++j)
                    if (j % NW == wave)
                        lds_direct_load4(bias, (uint32_t)min(n0 / 2 + j * 64 + lane, N / 2 - 1) * 4, sc + OFF_BIAS + j * 256);
            }
            if (w_zero) {
#pragma unroll
                for (int j = 0; j < BM / 64; ++j)
                    if (j % NW == wave)
                        lds_direct_load4(code_rowsum, (uint32_t)min(m0 + j * 64 + lane, M - 1) * 4, sc + OFF_RSUM + j * 256);
                if (UNALIGNED || (N & 7) == 0) {
#pragma unroll
                    for (int j = 0; j < (BN + 255) / 256; ++j)
                        if (j % NW == wave)
                            lds_direct_load4(w_zero, (uint32_t)min(n0 / 4 + j * 64 + lane, N / 4 - 1) * 4, sc + OFF_ZERO + j * 256);
                }
            }
        }
        if constexpr (CANON) {
            // the last slice of a tile: pieces past the rows' ends re-read the last one (their weights are taken as zeros)
            if (issue_live && issue_kt == KT - 1 && k_tail < BK) {
#pragma unroll
                for (int i = 0; i < A_DMA; ++i)
                    a_voff[i] -= max(((((lane % CHUNKS) ^ swz(a_row[i])) + 1) << 4) - k_tail, 0);
#pragma unroll
                for (int i = 0; i < W_DMA; ++i) w_voff[i] -= max((w_chunk + 1) * 16 - k_tail / 2, 0);
            }
        }
        issue_sa = smem_base + buf * STAGE;
    };
    // (idx is a constant wherever this is called.  With 128-channel slices the weight pieces of a wave are one
    // run in memory and in LDS: the first sets M0, the others reuse it and move by the instruction offset; the
    // loops below issue a wave's pieces in ascending order, weight pieces last, so nothing comes between them.)
    auto issue_one = [&] __device__(int idx) __attribute__((always_inline)) {
        if (idx < A_DMA) {
            lds_direct_load16(a_base, a_voff[idx], issue_sa + (wave * A_DMA + idx) * 1024);
        } else if constexpr (CANON) {
            lds_direct_load16(w_base, w_voff[idx - A_DMA], issue_sa + A_STAGE + (wave * W_DMA + idx - A_DMA) * 1024);
        } else if (W_PIECE != 1024 || W_DMA > 4 || idx == A_DMA) {
            lds_direct_load16(w_base + (wave * W_DMA + idx - A_DMA) * W_PIECE, lane16,
                              issue_sa + A_STAGE + (wave * W_DMA + idx - A_DMA) * 1024);
        } else {
            const uint8_t *run = w_base + wave * W_DMA * 1024;
            switch (idx - A_DMA) {
                case 1: lds_direct_load16_more<1024>(run, lane16); break;
                case 2: lds_direct_load16_more<2048>(run, lane16); break;
                default: lds_direct_load16_more<3072>(run, lane16); break;
            }
        }
    };
    auto issue_advance = [&] __device__() {
        if (!issue_live) return;
        if (issue_kt + 1 < KT) {
            a_base += A_ROW;
            // items alternate between the halves of a 128-channel slice of the native layout when BK = 64
            w_base += CANON ? BK / 2 : (BK == 128 || (issue_kt & 1)) ? w_slice_stride - (kBK - BK) * (kGroup / 2) : (int64_t)W_GROUP;
            ++issue_kt;
        } else {   // next: slice 0 of the next tile, whose addresses issue_prepare sets (or none: stay on this slice)
            issue_kt = 0;
            ++issue_tile;
        }
    };

    v16i acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

    // ---- fragment addressing: MFMA operand row = lane % 32, K half = lane / 32
    const int frow = lane & 31, fhalf = lane >> 5;
    int a_row_off[TM];
#pragma unroll
    for (int j = 0; j < TM; ++j) a_row_off[j] = (wm + j * 32 + frow) * A_ROW;
    const int a_xor = swz(frow);  // == swz(row): wm and 32 j are multiples of 32
    // Weight fragment of MFMA t of step ks: the 16 channels at 32 (NT ks + t) + 16 fhalf of the slice
    // with int8 codes; with packed codes lane half fhalf owns channels 64 ks + 32 fhalf + 16 t
    // (what its 16-byte code fragment holds), i.e. k32 step 2 ks + fhalf, k16 half t of the layout.
    // (CANON: likewise, from the piece 2 ks + fhalf of its row)
    const int w_off = (wn / kGroup) * W_GROUP + (CANON ? frow * 64 : frow * 8 + fhalf * (A4 ? 512 : 256));
    const int w_xor = swz_bk<64>(frow);

    // fragments of one step: TM code fragments (16 B) and NT x TN packed weight fragments (8 B)
    // (CANON: NT code fragments each, and 16 bytes of weights for both MFMAs of a step)
    struct Frags { v4i a[CANON ? NT * TM : TM]; uint2 w[NT][TN]; };
    auto load_frags = [&] __device__(Frags &f, int buf, int ks) {
        const uint8_t *sa = smem + buf * STAGE, *sw = sa + A_STAGE;
        if constexpr (CANON) {
#pragma unroll
            for (int i = 0; i < TN; ++i) {
                const uint4 p = *reinterpret_cast<const uint4 *>(sw + w_off + i * W_GROUP + (((ks * 2 + fhalf) ^ w_xor) << 4));
                f.w[0][i] = make_uint2(p.x, p.y);
                f.w[1][i] = make_uint2(p.z, p.w);
            }
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int j = 0; j < TM; ++j)
                    f.a[t * TM + j] = *reinterpret_cast<const v4i *>(sa + a_row_off[j] + (((ks * 4 + fhalf * 2 + t) ^ a_xor) << 4));
            return;
        }
#pragma unroll
        for (int j = 0; j < TM; ++j) {
            f.a[j] = *reinterpret_cast<const v4i *>(sa + a_row_off[j] + (((ks * 2 + fhalf) ^ a_xor) << 4));
        }
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int i = 0; i < TN; ++i) {
                f.w[t][i] = *reinterpret_cast<const uint2 *>(sw + w_off + i * W_GROUP +
                                                             (A4 ? ks * 1024 + t * 256 : ks * 512));
            }
    };
    // two packed dwords (16 codes) -> int8 lanes of 16 * code, channel order
    auto widen = [] __device__(uint32_t lo, uint32_t hi) {
        v4i f;
        f[0] = (int)((lo << 4) & 0xF0F0F0F0u);
        f[1] = (int)(lo & 0xF0F0F0F0u);
        f[2] = (int)((hi << 4) & 0xF0F0F0F0u);
        f[3] = (int)(hi & 0xF0F0F0F0u);
        return f;
    };

    // canonical nibble order (nibble i of a dword = channel i): the masks of `widen` give the even and the odd channels of 8, and
    // the codes of 8 channels are dealt the same way (the order of channels within an MFMA is free)
    auto deal_codes = [] __device__(v4i c) {
        v4i r;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            r[2 * h] = (int)__builtin_amdgcn_perm((uint32_t)c[2 * h + 1], (uint32_t)c[2 * h], 0x06040200u);
            r[2 * h + 1] = (int)__builtin_amdgcn_perm((uint32_t)c[2 * h + 1], (uint32_t)c[2 * h], 0x07050301u);
        }
        return r;
    };

    // ---- prologue: fill STAGES-1 buffers; with look-ahead also publish slice 0 and fetch its first fragments
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s) {
        issue_prepare(s);
#pragma unroll
        for (int d = 0; d < DMA; ++d) issue_one(d);
        issue_advance();
    }
    Frags f0, f1;
    if (AHEAD) {
        wait_vmcnt<(STAGES - 2) * DMA>();
        __builtin_amdgcn_s_barrier();
        load_frags(f0, 0, 0);
    }

    int kt = 0, tile_j = 0, store_credit = 0;
    for (int q = 0;; ++q) {
        // Publish slice q + AHEAD: it has landed once at most the loads of the
        // (STAGES - 2 - AHEAD) younger slices are outstanding (a wave's vector memory
        // operations complete in issue order).  The barrier also means that everyone is
        // done reading slice q-1, whose buffer the next loads overwrite.
        {
            // Right after the epilogue of a full tile exactly STORES stores are this wave's youngest
            // operations (for the next STAGES-1-AHEAD items the awaited loads are older than them):
            // do not wait for their acknowledgement.
            if (store_credit > 0) {
                wait_vmcnt<(STAGES - 2 - AHEAD) * DMA + STORES>();
                --store_credit;
            } else {
                wait_vmcnt<(STAGES - 2 - AHEAD) * DMA>();
            }
            if (draw_pending) publish_draw();
            __builtin_amdgcn_s_barrier();
        }
        issue_prepare((q + STAGES - 1) % STAGES);
        // A wave feeding the matrix cores outranks one that converts and stores a finished tile (the
        // two workgroups of a compute unit are in different phases most of the time).
        if (kt == 0) __builtin_amdgcn_s_setprio(2);

        // Software pipeline over the K=32 steps of the item: the fragments of step s+1 (or of
        // step 0 of the next item) are requested before the MFMAs of step s are issued, and the
        // LDS-direct loads of item q+STAGES-1 are dealt out between the MFMA groups.  The
        // scheduling barriers keep the compiler from regrouping any of it.
        const int buf = q % STAGES;
        if (!AHEAD) load_frags(f0, buf, 0);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            Frags &cur = (ks & 1) ? f1 : f0;
            Frags &nxt = (ks & 1) ? f0 : f1;
            if (ks + 1 < KS) load_frags(nxt, buf, ks + 1);
            else if (AHEAD) load_frags(nxt, (q + 1) % STAGES, 0);   // after the last item: stale but in-bounds, unused
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (CANON) {
                if (kt == KT - 1 && (ks * 2 + 2) * 32 > k_tail) {   // a step with channels past K
                    const bool past = (ks * 2 + fhalf) * 32 >= k_tail;
#pragma unroll
                    for (int i = 0; i < TN; ++i)
#pragma unroll
                        for (int t = 0; t < NT; ++t) {
                            cur.w[t][i].x = past ? 0u : cur.w[t][i].x;
                            cur.w[t][i].y = past ? 0u : cur.w[t][i].y;
                        }
                }
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                v4i fa[TM];
#pragma unroll
                for (int j = 0; j < TM; ++j)
                    fa[j] = A4 ? widen((uint32_t)cur.a[j][2 * t], (uint32_t)cur.a[j][2 * t + 1])
                               : CANON ? deal_codes(cur.a[t * TM + j]) : cur.a[j];
#pragma unroll
                for (int i = 0; i < TN; ++i) {
                    const v4i fw = widen(cur.w[t][i].x, cur.w[t][i].y);
#pragma unroll
                    for (int j = 0; j < TM; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fw, fa[j], acc[i][j], 0, 0, 0);
#pragma unroll
                    for (int d = (ks * NT + t) * TN + i; d < DMA; d += KS * NT * TN) issue_one(d);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        issue_advance();
        if (++kt < KT) continue;
        __builtin_amdgcn_s_setprio(0);   // the epilogue yields issue slots to the other workgroup's K loop

        // ---- epilogue of tile tile_j (shared with the FP6 kernel: see epilogue_interior / epilogue_edge; here the
        // accumulators hold 2^SHIFT times the sum of code products)
        int m0, n0;
        tile_origin(comp_tile, tiles_m, tiles_n, group_n, BM, BN, m0, n0);
        kt = 0;
        ++tile_j;
        comp_tile = __builtin_amdgcn_readfirstlane(s_tiles[tile_j & 7]);   // the next one (its loads are under way)
        uint8_t *s_tile = smem + STAGES * STAGE + ((tile_j - 1) & 1) * SCALES;
        typedef AccI32<SHIFT> Acc;
        int lane_e = lane;   // (keeps the epilogue's lane-dependent addresses out of the K loop's registers)
        asm volatile("" : "+v"(lane_e));
        if (UNALIGNED || ((N & 7) == 0 && !acc_out && N < kMaxTileN)) {
            // Every wave issues the same number of stores, whatever its tile (see the store-aware wait above).
            if (KT >= STAGES && (!UNALIGNED || (m0 + BM <= M && n0 + BN <= N))) store_credit = STAGES - 1 - AHEAD;
            uint8_t *stg = smem + (q % STAGES) * STAGE + wave * 4096;
            __builtin_amdgcn_s_barrier();   // every wave is done reading the last slice: its buffer stages the tile
            if constexpr (UNALIGNED) fill_vector_tail<BM, BN>(s_tile, bias, w_zero, lane_e, n0, N);
            // Two specializations, with and without weight zero-points, chosen once per tile (with four, bias as
            // well, this kernel spills).
            if (w_zero) epilogue_interior<Acc, BM, BN, TM, TN, true, -1, STORE>(acc, s_tile, bias != nullptr, lane_e, wm, wn, stg, y, m0, n0, M, N);
            else epilogue_interior<Acc, BM, BN, TM, TN, false, -1, STORE>(acc, s_tile, bias != nullptr, lane_e, wm, wn, stg, y, m0, n0, M, N);
        } else {
            epilogue_edge<Acc, BM, BN, TM, TN>(acc, s_tile, bias, w_zero, lane_e, wm, wn, y, acc_out, m0, n0, M, N);
        }
        if (comp_tile < 0) break;
    }
    wait_vmcnt<0>();   // no LDS-direct load may still be in flight when the workgroup's LDS is released
}

namespace {

// canonical [N, K/2] -> native layout (see the top of this file).  One thread per
// output dword (8 channels).  Rows >= N and channels >= K are written as zero.
__global__ __launch_bounds__(256) void w4_prepack_kernel(const uint8_t *__restrict__ src, uint32_t *__restrict__ dst,
                                                         int N, int K, int G, int KT) {
    const int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t words = (int64_t)KT * G * (kGroupBytes / 4);
    if (o >= words) return;
    int64_t v = o;
    const int d = (int)(v & 1); v >>= 1;
    const int r = (int)(v & 31); v >>= 5;
    const int half = (int)(v & 1); v >>= 1;
    const int ks = (int)(v & 3); v >>= 2;
    const int g = (int)(v % G);
    const int kt = (int)(v / G);
    const int n = g * kGroup + r;
    const int k = kt * kBK + ks * 32 + half * 16 + d * 8;
    uint32_t p = 0;
    if (n < N && k < K) p = *reinterpret_cast<const uint32_t *>(src + (int64_t)n * (K / 2) + k / 2);
    // nibble i of p is channel k+i; wanted: byte b = channel b (low nibble) | channel b+4 (high nibble)
    uint32_t q = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        q |= ((p >> (4 * b)) & 0xFu) << (8 * b);
        q |= ((p >> (4 * (b + 4))) & 0xFu) << (8 * b + 4);
    }
    dst[o] = q;
}

std::atomic<int> g_variant{-1};   // -1: pick by shape; set by the benchmark's sweep hook
std::atomic<int> g_schedule{-1};  // -1: tiles drawn from counters where possible; 0: fixed shares (benchmark hook)
std::atomic<int> g_grid_limit{0}; // 0: persistent grids fill the chip; else at most this many workgroups (benchmark hook)

// Tile counters of the persistent kernels: one slot per stream;
// kernels of one stream run one after the other.  What a slot holds between launches does not matter (see
// TileSource): it is cleared on the stream right before every kernel that counts in it.
constexpr int kSchedSlots = 512;
__device__ __align__(64) unsigned g_sched[kSchedSlots + 1][kSchedWords];   // (the last one: idle_slot)

struct SchedTable {
    unsigned *base = nullptr;
    std::unordered_map<uint64_t, int> slot_of;   // stream handle -> slot
    std::vector<int> free_slots;                 // released slots, reused before fresh ones
    int fresh = 0;                               // slots never handed out yet
    bool clear[kSchedSlots] = {};                // the last library kernel enqueued on the slot's stream zeroes the slot
};
std::mutex g_sched_mu;
SchedTable g_sched_table[64];

__global__ void fill_sched_kernel(unsigned *p, unsigned value, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = value;
}

}  // namespace

static bool find_base(SchedTable &t) {
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(g_sched)) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    t.base = static_cast<unsigned *>(p);
    return true;
}

bool drawing_enabled() { return g_schedule.load(std::memory_order_relaxed) != 0; }

bool tiles_drawn(hipStream_t stream) {
    if (!drawing_enabled()) return false;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &cap) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return cap == hipStreamCaptureStatusNone;
}

// The counter slot of `stream`, or nullptr (fixed shares): when the stream is being captured into a graph
// -- the same node may later run in several graph instances at once, which must not share counters -- or
// when all slots are taken.  *index: the slot's number.
static unsigned *slot_of_stream(hipStream_t stream, int *dev_out, int *index) {
    if (!tiles_drawn(stream)) return nullptr;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    SchedTable &t = g_sched_table[dev];
    if (!t.base && !find_base(t)) return nullptr;
    auto it = t.slot_of.find(reinterpret_cast<uint64_t>(stream));
    if (it == t.slot_of.end()) {
        int slot;
        if (!t.free_slots.empty()) {
            slot = t.free_slots.back();
            t.free_slots.pop_back();
        } else if (t.fresh < kSchedSlots) {
            slot = t.fresh++;
        } else {
            return nullptr;
        }
        t.clear[slot] = false;
        it = t.slot_of.emplace(reinterpret_cast<uint64_t>(stream), slot).first;
    }
    *dev_out = dev;
    *index = it->second;
    return t.base + it->second * kSchedWords;
}

// For a GEMM about to be enqueued on `stream`: its counter slot (or nullptr: fixed shares), and whether the
// library kernel enqueued last on the stream zeroes it (a quantizer; then the GEMM needs no clearing kernel
// of its own).  The GEMM leaves the slot dirty.  (Calls on one stream are in the caller's order, as the
// stream's own semantics require.)
unsigned *sched_slot(hipStream_t stream, bool *is_clear) {
    std::lock_guard<std::mutex> lock(g_sched_mu);
    int dev = 0, index = 0;
    *is_clear = false;
    unsigned *slot = slot_of_stream(stream, &dev, &index);
    if (slot) {
        *is_clear = g_sched_table[dev].clear[index];
        g_sched_table[dev].clear[index] = false;
    }
    return slot;
}

// For a GEMM whose workgroups start with every tile there is: draws come back empty whatever the words hold, so all streams share
// them.  (Not looked up for the first time while a stream is being captured.)
unsigned *idle_slot(hipStream_t stream) {
    if (g_schedule.load(std::memory_order_relaxed) == 0) return nullptr;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    std::lock_guard<std::mutex> lock(g_sched_mu);
    SchedTable &t = g_sched_table[dev];
    if (!t.base) {
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(stream, &cap) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        if (cap != hipStreamCaptureStatusNone || !find_base(t)) return nullptr;
    }
    return t.base + kSchedSlots * kSchedWords;
}

// For a quantizer about to be enqueued on `stream`: the slot it should zero (or nullptr), noted as zeroed by it;
// if it could not be enqueued, the note is taken back.
unsigned *sched_slot_to_clear(hipStream_t stream) {
    std::lock_guard<std::mutex> lock(g_sched_mu);
    int dev = 0, index = 0;
    unsigned *slot = slot_of_stream(stream, &dev, &index);
    if (slot) g_sched_table[dev].clear[index] = true;
    return slot;
}
void sched_slot_not_cleared(hipStream_t stream) {
    std::lock_guard<std::mutex> lock(g_sched_mu);
    int dev = 0, index = 0;
    if (slot_of_stream(stream, &dev, &index)) g_sched_table[dev].clear[index] = false;
}

int clear_sched_slot(unsigned *slot, hipStream_t stream) {
    hipLaunchKernelGGL(fill_sched_kernel, dim3(1), dim3(kSchedWords), 0, stream, slot, 0u, kSchedWords);
    return check_launch();
}

int fill_sched_slots(uint32_t value, hipStream_t stream) {
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(g_sched)) != hipSuccess) return DVDQ_ERR_HIP;
    const int n = kSchedSlots * kSchedWords;
    hipLaunchKernelGGL(fill_sched_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, static_cast<unsigned *>(p), value, n);
    {
        std::lock_guard<std::mutex> lock(g_sched_mu);
        for (auto &t : g_sched_table)
            for (bool &c : t.clear) c = false;
    }
    return check_launch();
}

// Forget `stream` on the current device (its slot goes to the next stream that needs one).
void release_sched_slot(hipStream_t stream) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return;
    std::lock_guard<std::mutex> lock(g_sched_mu);
    SchedTable &t = g_sched_table[dev];
    auto it = t.slot_of.find(reinterpret_cast<uint64_t>(stream));
    if (it == t.slot_of.end()) return;
    t.free_slots.push_back(it->second);
    t.slot_of.erase(it);
}

namespace {

template <int BM, int BN, int BK, int WAVES_M, int WAVES_N, int STAGES, int OCC, Operands OPS = OPS_INT8, StoreKind STORE = STORE_BY_PITCH>
int launch_native(const int8_t *codes, const float *x_scale, const uint8_t *w, const float *w_scale,
                  const int8_t *w_zero, const int32_t *code_rowsum, const uint16_t *bias, int M, int N, int K,
                  uint16_t *y, int32_t *acc_out, hipStream_t stream) {
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    // column tiles per L2 sharing group: balanced groups of at most 16
    const int n_groups = (tiles_n + 15) / 16;
    const int group_n = (tiles_n + n_groups - 1) / n_groups;
    const int total = tiles_m * tiles_n;
    // persistent: OCC workgroups per compute unit (256 CUs), grid a multiple of the 8 XCDs
    int grid = 256 * OCC;
    if (total < grid) grid = (total + 7) / 8 * 8;
    grid = limited_grid(grid);
    // the ring, then two tiles' epilogue vectors (scales, bias, code sums, zero-points; see the kernel)
    const size_t smem = (size_t)STAGES * (BM * (OPS == OPS_PACKED4 ? BK / 2 : BK) + BN * BK / 2) +
                        2 * TileVectors<BM, BN>::BYTES + 8 * sizeof(int);   // + the ring of tile numbers
    auto k = w4ax_gemm_native_kernel<BM, BN, BK, WAVES_M, WAVES_N, STAGES, OCC, OPS, STORE>;
    static std::atomic<uint64_t> configured{0};   // one per template instantiation
    allow_dynamic_lds(reinterpret_cast<const void *>(k), smem, configured);
    bool is_clear = false;
    // (two tiles per workgroup at most: nothing to draw, no counter to clear)
    unsigned *sched = nullptr;
    if (total > 2 * grid) sched = sched_slot(stream, &is_clear);
    else if (total > grid + kCusPerXcd) sched = idle_slot(stream), is_clear = true;
    if (sched && !is_clear && clear_sched_slot(sched, stream) != DVDQ_OK) return DVDQ_ERR_HIP;
    hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(64 * WAVES_M * WAVES_N), smem, stream, codes, x_scale, w,
                       w_scale, w_zero, code_rowsum, bias, M, N, K, y, acc_out, tiles_m, tiles_n, group_n, sched);
    return check_launch();
}

}  // namespace

void set_gemm_variant(int v) { g_variant.store(v, std::memory_order_relaxed); }
int gemm_variant() { return g_variant.load(std::memory_order_relaxed); }
void set_gemm_schedule(int v) { g_schedule.store(v, std::memory_order_relaxed); }
void set_gemm_grid_limit(int v) { g_grid_limit.store(v, std::memory_order_relaxed); }
int limited_grid(int grid) {
    const int limit = g_grid_limit.load(std::memory_order_relaxed);
    if (limit <= 0 || grid <= limit) return grid;
    return limit < 8 ? 8 : limit / 8 * 8;
}

// The tile variant for a size and the number of vectors, bias and zero-points (variants 2 and 5 below; 10 + shape: the small-output kernel; kCanonicalVariant: the two-wave kernel
// with canonical weights, kCanonicalShape6Variant: the small-output kernel beyond its outputs, a wave per 64 x 128 tile).
// Variant 5 is the wide kernel of w4ax_gemm_wide.hip (int8 codes only), taken
//   - from 12 K slices on (from 8 with both vectors, bias and zero-points, where its one or two rounds of tiles end more than half full but
//     not full: 0.97 of variant 2's time there in the mean of 61 outputs of 129 to 511 tiles at 8 to 11 slices, 0.93 to 1.04; with one
//     vector 1.00, up to 1.19, with none 1.01, up to 1.07; with 256 or 512 tiles 1.01 in the mean of 16, and 1.03 to 1.07 in one column);
//   - where N is a multiple of 8.  For others variant 2 has the stores (STORE_UNALIGNED); per element, as the wide kernel stores
//     them, a tile takes several times as long with no second workgroup to multiply meanwhile (before variant 2 had them the
//     wide kernel was already 4-24 % slower at K = 1536 .. 6144, with bias and zero-points 20-53 %);
//   - unless its last round of tiles, one per compute unit, is at most half full: variant 2's tiles are half as large, so it ends
//     half a round earlier, if the rest is spread over the chip, as drawn tiles are.  Fixed shares (a stream under capture) deal it to the
//     first XCDs, compute units with two tiles each beyond the first 16 tiles (32 of variant 2's): variant 2 has 0.84 to 0.95 of variant 5's time
//     there below two rounds and, from two to five, at 16 and fewer (14897 x 1536 x 2200, 531 tiles: 69.1 and 78.3 us), else 1.00 to 1.09 up to
//     fifteen rounds (41486 x 4480 x 1704, 1141 tiles: 325 and 306).  Drawn: time of variant 5 over that of variant 2 (bias and zero-points, 1536 to 3072 channels, 12 to 60 slices) by the
//     number of 256 x 256 tiles: 1.11-1.15 at 264 to 384 (15600 x 1536 x 1536, 366 tiles: 48.3 and 43.0 us), 0.94-0.97 at 432 to 512,
//     1.08-1.12 at 516 to 640, 0.95-0.99 at 672 to 768, 1.04-1.10 at 1026 to 1400, 1.02-1.07 at 2064 to 2172, 1.01-1.05 at 3100 to 3200.
//     One column of tiles: 1.02 to 1.14 up to two fifths of a round; the line stays there, and below four rounds, as
//     tests/test_dispatch.py states it.
// The lines between 2 and 5 are from before variant 2 had 128 x 128 tiles (narrow_tiles).  Where variant 5 is
// taken and those take no more rounds of 768 than it of 256, they have 0.91 of its time in the mean of 383 outputs of one round (1.03 at most), 0.89 of 59 of two
// (1.01), 0.91 of 25 of three (the GEMM alone, drawn, 8 to 47 slices, with the wide kernel of before it transposed tiles with zero-points first, which
// takes 1 to 2 % off): a line there would pay (25805 x 2560 x 320: 37.1 and 30.8 us).
int w4ax_gemm_choice(int64_t M, int64_t N, int64_t K, int codes_format, int w_layout, int vectors, bool drawn) {
    const int shape = small_gemm_shape(M, N, K, false);
    if (w_layout == DVDQ_W_CANONICAL && shape < 0) {
        // a second round of the two-wave kernel's tiles where the waves, eight per compute unit, take one
        const bool one_round = ((M + 63) / 64) * ((N + 127) / 128) <= 2048;
        return one_round && ((M + 127) / 128) * ((N + 255) / 256) > 512 ? kCanonicalShape6Variant : kCanonicalVariant;
    }
    if (shape == 5 && w_layout != DVDQ_W_CANONICAL && narrow_for_small_outputs(M, N, K, codes_format)) return 2;
    if (shape == 7 && w_layout == DVDQ_W_CANONICAL) return kFirstSmallVariant + 3;   // (variant 17 is another thing there)
    if (shape >= 0) return kFirstSmallVariant + shape;
    if (codes_format != DVDQ_CODES_INT8 || K / 128 < 8 || !whole_line_tiles(N)) return 2;
    const int64_t tiles = ((M + 255) / 256) * ((N + 255) / 256), last = tiles % 256;
    if (K / 128 < 12) return vectors == 2 && tiles < 512 && last > 128 ? 5 : 2;
    if (N <= 256) return tiles > 256 && tiles < 1024 && last != 0 && 5 * last < 2 * 256 ? 2 : 5;
    const int64_t most = drawn ? (tiles < 4096 ? 128 : 0) : tiles < 512 ? 128 : tiles < 1536 ? 16 : 0;
    return last != 0 && last <= most ? 2 : 5;
}

int launch_w4ax_gemm(const int8_t *codes, const float *x_scale, const uint8_t *w, const float *w_scale,
                     const int8_t *w_zero, const int32_t *code_rowsum, const uint16_t *bias, int64_t M, int64_t N,
                     int64_t K, int codes_format, int w_layout, uint16_t *y, int32_t *acc_out, hipStream_t stream) {
    if (w_layout == DVDQ_W_CANONICAL) {
        if (codes_format != DVDQ_CODES_INT8 || w_zero) return DVDQ_ERR_UNSUPPORTED;
        const int f = gemm_variant(), v = f >= kFirstSmallVariant || f == 6 ? f : w4ax_gemm_choice(M, N, K, codes_format, w_layout, bias != nullptr, true);
        if (v != kCanonicalVariant && v != 6)
            return launch_w4ax_gemm_small(reinterpret_cast<const uint8_t *>(codes), x_scale, w, w_scale, nullptr, nullptr, bias, M, N, K,
                                          codes_format, w_layout, v == kCanonicalShape6Variant ? 6 : v - kFirstSmallVariant, y, acc_out, stream);
        // Variant 2 with the weights as they come.  A slice of a weight row is 64 bytes, half a cache line, so twice the weight bytes
        // leave the L2, but once per 256 channels x 128 tokens: a wave per 64 x 128 tile, its operands for itself, was bound by
        // that traffic.  Before -> now: 7800 x 1440 x 1440 40.1 -> 27.8 us, 32760 x 1536 x 4608 342 -> 247 (1.9 POP/s), 32760 x 13824 x 5120
        // 2708 -> 1993, 27510 x 11552 x 7296 3282 -> 2266, 32760 x 1440 x 1441 170 -> 92.  The waves keep what they take in one round
        // (eight per compute unit, 2048) and variant 2 in two: a wave per tile 0.81 to 0.98 of its time there (22528 x 96 x 592 15.1 and 12.2 us,
        // 5910 x 160 x 2680 18.5 and 15.6, 16734 x 1120 x 792 36.0 and 33.1), from 2050 waves on 1.01 to 1.4 (12021 x 64 x 1328 15.7 and 15.9).
#define DVDQ_CANONICAL_ARGS codes, x_scale, w, w_scale, nullptr, nullptr, bias, (int)M, (int)N, (int)K, y, acc_out, stream
        const bool unaligned = unaligned_tiles(N) && !acc_out;
        if (v == 6 || (f < 0 && narrow_tiles(M, N, K, codes_format, w_layout, stream)))
            return unaligned ? launch_native<128, 128, 128, 2, 2, 2, 3, OPS_CANONICAL, STORE_UNALIGNED>(DVDQ_CANONICAL_ARGS)
                             : launch_native<128, 128, 128, 2, 2, 2, 3, OPS_CANONICAL>(DVDQ_CANONICAL_ARGS);
        return unaligned ? launch_native<128, 256, 128, 2, 2, 2, 2, OPS_CANONICAL, STORE_UNALIGNED>(DVDQ_CANONICAL_ARGS)
                         : launch_native<128, 256, 128, 2, 2, 2, 2, OPS_CANONICAL>(DVDQ_CANONICAL_ARGS);
#undef DVDQ_CANONICAL_ARGS
    }
    const int m = (int)M, n = (int)N, k = (int)K;
#define DVDQ_GEMM_ARGS codes, x_scale, w, w_scale, w_zero, code_rowsum, bias, m, n, k, y, acc_out, stream
    // Tile variants: {tile M, tile N, K slice, waves M x N, ring depth, workgroups per compute unit}.
    // Outputs of few tiles go to w4ax_gemm_small.hip (small_gemm_shape).  Variant 2 is the default of the two-wave kernels: two independent 4-wave workgroups per compute unit,
    // each owning a 128 x 256 tile (64 x 128 per wave) with K slices of 128 through two buffers.  In
    // interleaved sweeps over the DiT shapes (K = 1536 ... 13824) it was fastest or within 1 % of the
    // fastest: while one workgroup converts and stores its tile the other keeps the matrix cores busy,
    // which the one-workgroup 256 x 256 variants cannot do.  Variant 6 is the same with 128 x 128 tiles (64 x 64 per wave) and three
    // workgroups per compute unit, taken in place of variant 2 by narrow_tiles.  The others remain for sweeps; a shape with
    // fewer K slices than a variant's ring needs falls back to variant 2, which always qualifies.
    const bool unaligned = unaligned_tiles(N) && !acc_out;
    const int forced = gemm_variant();
    int v = forced;
    if (forced < 0) {
        const int vectors = (bias != nullptr) + (w_zero != nullptr);
        v = w4ax_gemm_choice(M, N, K, codes_format, w_layout, vectors, true);
        const int fixed = w4ax_gemm_choice(M, N, K, codes_format, w_layout, vectors, false);
        if (fixed != v && !tiles_drawn(stream)) v = fixed;
        if (v == 2 && narrow_tiles(M, N, K, codes_format, w_layout, stream)) v = 6;
    }
    if (v >= kFirstSmallVariant)
        return launch_w4ax_gemm_small(reinterpret_cast<const uint8_t *>(codes), x_scale, w, w_scale, w_zero, code_rowsum,
                                      bias, M, N, K, codes_format, w_layout, v - kFirstSmallVariant, y, acc_out, stream);
    if (codes_format == DVDQ_CODES_PACKED4) {
        if ((v == 1 && k / 128 < 2) || (v > 2 && v < 6 && k / 128 < 3)) v = 2;
        switch (v) {
            case 1: return launch_native<256, 256, 128, 2, 4, 3, 1, OPS_PACKED4>(DVDQ_GEMM_ARGS);
            case 2:
                return unaligned ? launch_native<128, 256, 128, 2, 2, 2, 2, OPS_PACKED4, STORE_UNALIGNED>(DVDQ_GEMM_ARGS)
                                 : launch_native<128, 256, 128, 2, 2, 2, 2, OPS_PACKED4>(DVDQ_GEMM_ARGS);
            case 3: return launch_native<256, 256, 128, 2, 4, 4, 1, OPS_PACKED4>(DVDQ_GEMM_ARGS);
            case 4: return launch_native<256, 256, 128, 4, 2, 4, 1, OPS_PACKED4>(DVDQ_GEMM_ARGS);
            case 6:
                return unaligned ? launch_native<128, 128, 128, 2, 2, 2, 3, OPS_PACKED4, STORE_UNALIGNED>(DVDQ_GEMM_ARGS)
                                 : launch_native<128, 128, 128, 2, 2, 2, 3, OPS_PACKED4>(DVDQ_GEMM_ARGS);
            default: return DVDQ_ERR_UNSUPPORTED;
        }
    }
    if (v == 5)
        return launch_w4ax_gemm_wide(reinterpret_cast<const uint8_t *>(codes), x_scale, w, w_scale, w_zero, code_rowsum, bias,
                                     M, N, K, false, y, acc_out, stream);
    {
        const int bk = v == 4 ? 64 : 128, stages = v == 2 || v == 6 ? 2 : (v == 4 ? 4 : 3);
        if (k / bk < stages - 1) v = 2;
    }
    switch (v) {
        case 1: return launch_native<256, 256, 128, 4, 2, 3, 1>(DVDQ_GEMM_ARGS);
        case 2:
            return unaligned ? launch_native<128, 256, 128, 2, 2, 2, 2, OPS_INT8, STORE_UNALIGNED>(DVDQ_GEMM_ARGS)
                             : launch_native<128, 256, 128, 2, 2, 2, 2>(DVDQ_GEMM_ARGS);
        case 3: return launch_native<256, 256, 128, 2, 4, 3, 1>(DVDQ_GEMM_ARGS);
        case 4: return launch_native<128, 256, 64, 2, 2, 4, 2>(DVDQ_GEMM_ARGS);
        case 6:
            return unaligned ? launch_native<128, 128, 128, 2, 2, 2, 3, OPS_INT8, STORE_UNALIGNED>(DVDQ_GEMM_ARGS)
                             : launch_native<128, 128, 128, 2, 2, 2, 3>(DVDQ_GEMM_ARGS);
        default: return DVDQ_ERR_UNSUPPORTED;
    }
#undef DVDQ_GEMM_ARGS
}

size_t w4_native_bytes(int64_t N, int64_t K) {
    const int64_t npad = (N + kNPad - 1) / kNPad * kNPad, kpad = (K + kBK - 1) / kBK * kBK;
    return (size_t)(npad * kpad / 2);
}

int launch_w4_prepack(const uint8_t *w_canonical, int64_t N, int64_t K, uint8_t *w_native, hipStream_t stream) {
    const int G = (int)((N + kNPad - 1) / kNPad * (kNPad / kGroup));
    const int KT = (int)((K + kBK - 1) / kBK);
    const int64_t words = (int64_t)KT * G * (kGroupBytes / 4);
    const int64_t blocks = (words + 255) / 256;
    hipLaunchKernelGGL(w4_prepack_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, w_canonical,
                       reinterpret_cast<uint32_t *>(w_native), (int)N, (int)K, G, KT);
    return check_launch();
}

}  // namespace dvdq
