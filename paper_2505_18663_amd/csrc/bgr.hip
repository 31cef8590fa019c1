// Bounded-init Grid Refinement (Sec. 3.1, Alg. 1): the offline INT4 weight quantizer.
// For every weight row (output channel) it searches clipped MinMax starts, refines each
// start's grid (least-squares step size, relaxed zero-point, re-quantization) round after
// round, and keeps the grid with the smallest row error: either as Alg. 1 prints it (starts
// i = 1, 2, ..., a start's result is the grid of its last round) or as a superset search (i = 0,
// plain MinMax, is a start too and every grid evaluated competes).  Runs once per layer, off the
// inference path; everything that decides is fp64 or better, so that its decisions (roundings, comparisons)
// match a plain fp64 implementation up to the rounding of that one's sums.
//
// One workgroup per row.  A row is evaluated on several hundred grids (Delta, z), and what an evaluation needs of
// it are only four sums over c = clamp(rint(w / Delta) + z, 0, 15), d = c - z:
//   e2 = sum (w - Delta d)^2,  num = sum d w,  den = sum d^2,  sq = sum c.
// c takes 16 values, and it is monotone in w: on the SORTED row an evaluation is 15 positions
//   pos_j = #{w : rint(w / Delta) <= j - z},  j = 0 .. 14,
// and, with P(p) the sum of the p smallest weights, Abel summation gives
//   sq  = 15 K - sum_j pos_j
//   den = (15 - z)^2 K - sum_j (2 (j - z) + 1) pos_j          (both exact integers)
//   num = (15 - z) P(K) - sum_j P(pos_j)
//   e2  = sum w^2 - 2 Delta num + Delta^2 den
// The last two are differences of larger numbers: for rows quantized well, several digits of e2 cancel.  So nothing
// in them is rounded before the end.  The prefix sums are 64-bit integers, the weights in units of 2^-43 .. 2^-47 of
// the row's largest (FixedPoint below): a weight is exact in them unless it is more than 2^20 times smaller than the
// largest, and then d is 0 on every grid that does not clip the largest away.  sum w^2 is held in two doubles and the
// expression evaluated in them.  One rounding to fp64 remains (the row error is within 1.3e-16 of what
// sums in 80 bits give).  Below 2^-40 sum w^2, where the two doubles would run out, e2 is taken from the row.
// So the row is sorted once, its prefix sums are kept, and an evaluation costs 15 lookups instead of a pass over
// the row with a division per weight.  A lookup is three dependent LDS reads (the cell of values the threshold falls
// in, the block of 4 .. 16 weights there, its weights and prefix sum).  The division survives only where it decides:
// for a float that sits on a threshold to within fp64 rounding, so every weight is classified by exactly the quotient
// and rounding of the definition.  The starts of the search are independent of each other: 8 lanes take one start, two
// positions each, with no barrier inside the search.  (What a round does once per start, divisions, square root and the
// expression of e2, all lanes of the start do, some 100 of its 300 instructions; bgr_choice says where 4 lanes with four positions are better.)
//
// Cost.  1536 rows of 8960 weights, 100 steps, 10 rounds: 0.140 ms; a pass over the row per evaluation, one workgroup of
// 256 threads per row, took 8.7 ms.  Bound by latencies and the issue of fp64 instructions, not by memory (62 MB): of the
// 104 K clocks a row is in work (two rows per compute unit, each beside another one's phases) 10 K are the load, 25 K the two
// dealing passes with the counts between them (LDS atomics and barriers) and the sum of squares, 13 K the windows, 4 K the
// prefix sums, 46 K the search, 6 K the codes.  The search is eleven rounds of 4 K, bound by issue: three to four waves per SIMD,
// some 300 instructions each.  (The clocks are from when the row took 0.145 ms; since then the search got 4 to 9 % of the whole cheaper:
// sq / K without the division's steps, weights chosen before they are converted, unsigned block numbers, 24-bit products: 8960 rows of 1536
// 587 -> 539 us, 13824 of 256 837 -> 763, 1536 of 8960 146 -> 140.)  That the sums are not rounded costs 7 K: with sums in fp64 0.136 ms for
// 0.145 (8960 rows of 1536: 0.517 for 0.586) and a squared error off by 1e-14, up to 1e-12 where a grid fits a row to a hundredth.
#include "dvdq_internal.h"
#include "wave_reduce.h"

#pragma clang fp contract(off)   // every product and sum rounded on its own, like a plain C loop

namespace dvdq {
namespace {

constexpr double kQmax = 15.0;           // INT4
constexpr int kCellLimit = 1024; // fullest cell that is sorted in windows (see the kernel)

// Sum over 4 or 8 neighbouring lanes; every lane gets it.
template <int LANES, typename T>
__device__ __forceinline__ T sum_lanes(T v) {
    static_assert(LANES == 4 || LANES == 8);
    v += dpp<DPP_XOR1>(v);
    v += dpp<DPP_XOR2>(v);
    if constexpr (LANES == 8) v += dpp<DPP_HALF_MIRROR>(v);
    return v;
}

// A sum held in two doubles: hi + lo.
struct TwoDoubles { double hi, lo; };
// a + b without an error, |a| >= |b|: hi = a + b rounded, lo the rest
__device__ __forceinline__ TwoDoubles fast_two_sum(double a, double b) {
    const double s = a + b;
    return {s, b - (s - a)};
}

// Weights as multiples of `unit` = 2^e, summed in 64-bit integers.  A running sum of a few weights is kept as a double
// near `bias` = 1.5 * 2^52 units, where neighbouring doubles are one unit apart: every addition rounds the weight added
// to whole units, and the sum's bits less the bias's bits are the integer.  (The weights of a block are always added
// in the same order from its first one, so that each has one rounded value, whatever position the sum ends at.)
struct FixedPoint {
    double bias, unit;
    __device__ __forceinline__ int64_t integer(double sum) const {
        return __builtin_bit_cast(int64_t, sum) - __builtin_bit_cast(int64_t, bias);
    }
};

__device__ __forceinline__ double clamp_d(double v, double lo, double hi) { return v < lo ? lo : (v > hi ? hi : v); }

// the float right after v (toward +inf)
__device__ __forceinline__ float next_up(float v) {
    const uint32_t u = __float_as_uint(v);
    return __uint_as_float(v == 0.f ? 1u : (u & 0x80000000u) ? u - 1u : u + 1u);
}

// Value cells: `cells` equal parts of the row's range; monotone in v (every step rounds monotonically).
struct CellMap {
    float lo, inv;
    int last;
    __device__ __forceinline__ int operator()(float v) const { return max((int)fminf((v - lo) * inv, (float)last), 0); }
};

struct Sums { double e2, num, den, sq; };

// What a start of the search looks the row up in (LDS).
template <int BLK>
struct Row {
    const float *sorted;      // the weights, ascending, then +infinity up to a multiple of BLK (at least one)
    const int64_t *prefix;    // prefix[b] = sum of the first b * BLK of them, in units
    const uint32_t *cells;    // cells[c] = number of weights in the cells before c
    CellMap cell;
    int K;
    FixedPoint fixed;
    int64_t sum;              // of all weights, in units
    TwoDoubles sw2;           // sum of their squares
};

// The four sums on the grid (delta, z), by the LANES lanes of a group (j = lane % LANES takes positions j, j + LANES, ...): every
// lane gets all of them.
template <int BLK, int LANES>
__device__ __forceinline__ Sums evaluate(const Row<BLK> &r, int j, double delta, double z) {
    constexpr int P = 16 / LANES;
    float bound[P];      // pos_j = #{w < bound}
    unsigned lo[P], hi[P];
#pragma unroll
    for (int i = 0; i < P; ++i) {
        // With t the threshold (j - z + 1/2) Delta and c the float nearest to it, every smaller float is below t and
        // every larger one above it by at least a quarter of a float's ulp, which the roundings of t and of a
        // quotient (fp64) cannot bridge.  So is c itself unless it equals t to within a few of those roundings:
        // then its own quotient decides.
        const double u = (double)(j + i * LANES) - z, t = (u + 0.5) * delta;
        const float c = (float)t;
        const double off = (double)c - t;
        bool below = off < 0.0;
        if (fabs(off) <= fabs(t) * 0x1p-48) below = rint((double)c / delta) <= u;
        bound[i] = below ? next_up(c) : c;
        const int cb = r.cell(bound[i]);
        const unsigned first = r.cells[cb], past = r.cells[cb + 1];
        lo[i] = first / BLK;
        hi[i] = (past > first ? past - 1 : first) / BLK;
    }
    // the last block of each cell that starts below the bound (or the cell's first)
    auto searching = [&] __device__ {
        bool any = false;
#pragma unroll
        for (int i = 0; i < P; ++i) any |= lo[i] < hi[i];
        return any;
    };
    while (searching()) {
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const unsigned mid = (lo[i] + hi[i] + 1) >> 1;
            const bool up = r.sorted[mid * BLK] < bound[i] || lo[i] >= hi[i];
            lo[i] = up ? mid : lo[i];   // (mid = lo where the range is a single block)
            hi[i] = up ? hi[i] : mid - 1;
        }
    }
    int64_t p = 0;              // this lane's share of the sums over the positions: of P(pos_j),
    int moment = 0, count = 0;  // (2 (j - z) + 1) pos_j and pos_j
    const int zi = (int)z;
#pragma unroll
    for (int i = 0; i < P; ++i) {
        double run = r.fixed.bias;
        int pos = (int)(lo[i] * BLK);
        const float4 *blk = reinterpret_cast<const float4 *>(r.sorted + lo[i] * BLK);
#pragma unroll
        for (int b = 0; b < BLK / 4; ++b) {
            const float4 v = blk[b];
            const float q[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                const bool in = q[h] < bound[i];
                pos += in ? 1 : 0;
                float w = in ? q[h] : 0.f;
                asm("" : "+v"(w));   // (chosen as a float: the compiler would choose among the converted doubles, twice the work)
                run += (double)w;
            }
        }
        int64_t sum = r.prefix[lo[i]] + r.fixed.integer(run);
        if (i == P - 1 && j == LANES - 1) { pos = 0; sum = 0; }   // (15 positions)
        p += sum;
        moment += __mul24(2 * (j + i * LANES - zi) + 1, pos);   // (24 bits: pos <= K, the row fits the LDS)
        count += pos;
    }
    Sums s;
    const int64_t num = (int64_t)((uint64_t)(uint32_t)(15 - zi) * (uint64_t)r.sum) - sum_lanes<LANES>(p);
    s.den = (double)(__mul24(__mul24(15 - zi, 15 - zi), r.K) - sum_lanes<LANES>(moment));
    s.sq = (double)(15 * r.K - sum_lanes<LANES>(count));
    // num in two doubles: its upper and lower 32 bits are exact (and the upper ones, if any, are the larger)
    const double upper = (double)(int32_t)(num >> 32) * (0x1p32 * r.fixed.unit), lower = (double)(uint32_t)num * r.fixed.unit;
    s.num = upper + lower;
    const double num_lo = (upper - s.num) + lower;
    // e2 = sum w^2 + Delta (Delta den - 2 num), both sums from the larger term on (where it is not the larger one, no
    // digits cancel: such a grid is worse than no grid at all)
    const double q = delta * s.den, q_lo = __builtin_fma(delta, s.den, -q);
    const TwoDoubles t = fast_two_sum(-2.0 * s.num, q);
    const double t_lo = t.lo + (q_lo - 2.0 * num_lo);
    const double u = delta * t.hi, u_lo = __builtin_fma(delta, t.hi, -u) + delta * t_lo;
    const TwoDoubles e = fast_two_sum(r.sw2.hi, u);
    s.e2 = e.hi + (e.lo + (u_lo + r.sw2.lo));
    // A (nearly) exact fit: the sum over the row instead, as slow as it is.
    if (!(s.e2 > 0x1p-40 * r.sw2.hi)) {
        double e2 = 0.0;
        for (int k = j; k < r.K; k += LANES) {
            const double w = (double)r.sorted[k];
            const double d = w - delta * (clamp_d(rint(w / delta) + z, 0.0, kQmax) - z);
            e2 += d * d;
        }
        s.e2 = sum_lanes<LANES>(e2);
    }
    return s;
}

// ---- sorting
// Order-preserving integers for floats (and back: the map is its own inverse), so that a comparator is one integer
// minimum and one maximum.
__device__ __forceinline__ int order_key(float v) { const int u = __float_as_int(v); return u ^ ((u >> 31) & 0x7FFFFFFF); }
__device__ __forceinline__ float from_key(int k) { return __int_as_float(k ^ ((k >> 31) & 0x7FFFFFFF)); }

// Bitonic network over 32 registers whose comparators all put the smaller value first (the first step of a merge pairs
// mirrored positions).  FROM = 2: a full sort; FROM = 32: merges two sorted halves.
template <int FROM>
__device__ __forceinline__ void network32(int (&k)[32]) {
#pragma unroll
    for (int span = FROM; span <= 32; span *= 2)
#pragma unroll
        for (int dist = span / 2; dist >= 1; dist /= 2)
#pragma unroll
            for (int i = 0; i < 32; ++i) {
                const int l = dist == span / 2 ? i ^ (span - 1) : i ^ dist;
                if (l > i) {
                    const int a = min(k[i], k[l]), b = max(k[i], k[l]);
                    k[i] = a;
                    k[l] = b;
                }
            }
}

// Sorts or merges the 32 floats at `a` (16-byte aligned), in one thread.
template <int FROM>
__device__ __forceinline__ void window32(float *a) {
    int k[32];
    float4 *q = reinterpret_cast<float4 *>(a);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float4 v = q[i];
        k[4 * i] = order_key(v.x);
        k[4 * i + 1] = order_key(v.y);
        k[4 * i + 2] = order_key(v.z);
        k[4 * i + 3] = order_key(v.w);
    }
    network32<FROM>(k);
#pragma unroll
    for (int i = 0; i < 8; ++i)
        q[i] = make_float4(from_key(k[4 * i]), from_key(k[4 * i + 1]), from_key(k[4 * i + 2]), from_key(k[4 * i + 3]));
}

// floats the row takes in LDS: up to a whole window and one more, of which the last K .. are +infinity
__host__ __device__ constexpr int row_floats(int K) { return (K / 32 + 2) * 32; }

// Sorts a[0 .. n): the same network in LDS, where positions past n act as +infinity without being there.
template <int T>
__device__ void bitonic_sort(float *a, int n) {
    int span = 2;
    for (;; span <<= 1) {
        for (int dist = span >> 1; dist >= 1; dist >>= 1) {
            const bool mirror = dist == span >> 1;
            for (int t = threadIdx.x;; t += T) {
                const int i = ((t & ~(dist - 1)) << 1) | (t & (dist - 1));
                if (i >= n) break;
                const int l = mirror ? i ^ (span - 1) : i + dist;
                if (l < n) {
                    const float x = a[i], y = a[l];
                    if (y < x) { a[i] = y; a[l] = x; }
                }
            }
            __syncthreads();
        }
        if (span >= n) break;
    }
}

// T threads, a prefix sum every BLK weights.  HELD > 0: the threads hold the row in registers, HELD pairs of weights
// each (K <= 2 HELD T); 0: it is read again for every step that needs it in its own order.
// (128 registers per lane at most: 16 waves per compute unit, one workgroup of 1024 threads, two of 512, or as many of 256, up to four, as
// their LDS lets be resident.)
template <int T, int BLK, int HELD, int LANES>
__global__ __launch_bounds__(T, 4) void bgr_kernel(const float *__restrict__ w, int K, int cells, int n_steps, int max_refine,
                                                double eps, int search, uint8_t *__restrict__ w_packed,
                                                float *__restrict__ w_scale, int8_t *__restrict__ w_zero,
                                                double *__restrict__ row_error) {
    constexpr bool REGS = HELD > 0;   // the row is held
    constexpr int WAVES = T / 64, PAIRS = REGS ? HELD : 4;
    // LDS: the row fp32 [row_floats(K)], prefix sums int64 [blocks], the cells uint32 [cells + 1]
    extern __shared__ __align__(16) uint8_t smem_raw[];
    const int blocks = K / BLK + 1;
    float *row = reinterpret_cast<float *>(smem_raw);
    int64_t *prefix = reinterpret_cast<int64_t *>(row + row_floats(K));
    uint32_t *first = reinterpret_cast<uint32_t *>(prefix + blocks);   // first[c]: weights before cell c
    __shared__ double s_a[WAVES], s_b[WAVES], s_c[WAVES], s_d[WAVES];
    __shared__ int64_t s_sum[WAVES];
    __shared__ int s_i[WAVES], s_max[WAVES];
    __shared__ double s_best[3];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t n = blockIdx.x;
    const float2 *src = reinterpret_cast<const float2 *>(w + n * K);   // (K is even, w 16-byte aligned)
    const int pairs = K / 2;

    // f(pair number, pair) for this thread's pairs; the loads of PAIRS pairs are in flight together
    float2 held[PAIRS];
    auto load = [&] __device__(int base) {
#pragma unroll
        for (int i = 0; i < PAIRS; ++i)
            if (base + i * T < pairs) held[i] = src[base + i * T];
    };
    auto for_row = [&] __device__(auto f) {
        for (int base = tid;; base += PAIRS * T) {
            if (!REGS) load(base);
#pragma unroll
            for (int i = 0; i < PAIRS; ++i)
                if (base + i * T < pairs) f(base + i * T, held[i]);
            if (REGS || base + PAIRS * T >= pairs) break;
        }
    };
    if (REGS) load(tid);

    // ---- minimum, maximum, sum and sum of squares
    float lo_f = INFINITY, hi_f = -INFINITY;
    double sw = 0.0;
    for (int c = tid; c <= cells; c += T) first[c] = 0u;
    for_row([&] __device__(int, float2 v) {
        lo_f = fminf(lo_f, fminf(v.x, v.y));
        hi_f = fmaxf(hi_f, fmaxf(v.x, v.y));
        const double a = (double)v.x, b = (double)v.y;
        sw += a;
        sw += b;
    });
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        lo_f = fminf(lo_f, __shfl_xor(lo_f, m, 64));
        hi_f = fmaxf(hi_f, __shfl_xor(hi_f, m, 64));
    }
    sw = wave_sum(sw);
    if (lane == 0) {
        s_a[wave] = sw;
        s_c[wave] = __builtin_bit_cast(double, make_float2(lo_f, hi_f));
    }
    __syncthreads();
    sw = wave_sum(lane < WAVES ? s_a[lane] : 0.0);
#pragma unroll
    for (int i = 0; i < WAVES; ++i) {
        const float2 r = __builtin_bit_cast(float2, s_c[i]);
        lo_f = fminf(lo_f, r.x);
        hi_f = fmaxf(hi_f, r.y);
    }
    const double lo0 = (double)lo_f, hi0 = (double)hi_f;
    const bool constant = !(hi0 > lo0);

    // constant row c, represented exactly: Delta = |c| (1 if c = 0), z = (c < 0), q = (c > 0)
    double best = 0.0;
    double best_delta = lo0 == 0.0 ? 1.0 : fabs(lo0);
    double best_z = lo0 < 0.0 ? 1.0 : 0.0;

    if (!constant) {   // (the whole workgroup takes the same side: every thread has the same range)
        // ---- sort.  The row is dealt into cells of equal width (counting with LDS atomics, whose order decides
        // nothing in the end), which leaves every weight within a cell's length of its place.  Windows of 32 then
        // put it there, one thread each: sorted once where they are aligned, then merged alternately half a window
        // further on and aligned again, an odd-even transposition over blocks of 16 (a cell of m weights lies in
        // (m - 2) / 16 + 2 of them at most and needs as many passes).  Rows whose weights crowd into few cells
        // (many equal weights, one enormous outlier) take a bitonic sort instead.
        const CellMap cell = {lo_f, (float)cells / (hi_f - lo_f), cells - 1};
        // The sum of squares comes in two parts meanwhile: rounded to units so coarse that all K of them add up without an
        // error (as in FixedPoint), and the rest.  (In this pass, which waits for LDS atomics: summed in two doubles in the
        // first one it cost 2 to 4 % of the whole.)
        const int exponent = __builtin_amdgcn_frexp_expf(fmaxf(fabsf(lo_f), fabsf(hi_f))), log2_k = 32 - __builtin_clz(K);
        const double square_bias = ldexp(0x1.8p52, 2 * exponent + log2_k - 51);
        double coarse = square_bias;
        TwoDoubles sw2 = {0.0, 0.0};
        for_row([&] __device__(int, float2 v) {
            atomicAdd(&first[1 + cell(v.x)], 1u);
            atomicAdd(&first[1 + cell(v.y)], 1u);
            for (int h = 0; h < 2; ++h) {
                const double w = (double)(h ? v.y : v.x), q = w * w, sum = coarse + q;   // (the square of a float is exact)
                sw2.lo += q - (sum - coarse);
                coarse = sum;
            }
        });
        sw2 = {wave_sum(coarse - square_bias), wave_sum(sw2.lo)};
        if (lane == 0) { s_b[wave] = sw2.hi; s_d[wave] = sw2.lo; }
        __syncthreads();
        sw2 = {wave_sum(lane < WAVES ? s_b[lane] : 0.0), wave_sum(lane < WAVES ? s_d[lane] : 0.0)};
        uint32_t *mine = first + 1 + tid * (cells / T);   // this thread's consecutive cells
        int count = 0, fullest = 0;
        for (int i = 0; i < cells / T; ++i) {
            count += (int)mine[i];
            fullest = max(fullest, (int)mine[i]);
        }
        int upto = count;   // inclusive scan over the threads
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) {
            const int o = __shfl_up(upto, m, 64);
            if (lane >= m) upto += o;
            fullest = max(fullest, __shfl_xor(fullest, m, 64));
        }
        if (lane == 63) s_i[wave] = upto;
        if (lane == 0) s_max[wave] = fullest;
        __syncthreads();
        int before = upto - count;
        fullest = 0;
#pragma unroll
        for (int i = 0; i < WAVES; ++i) {
            if (i < wave) before += s_i[i];
            fullest = max(fullest, s_max[i]);
        }
        const bool by_cells = fullest <= kCellLimit;
        // by cells: the first position of each cell, which the scatter below turns into its end; else the end
        for (int i = 0; i < cells / T; ++i) {
            const int c = (int)mine[i];
            mine[i] = (uint32_t)(by_cells ? before : before + c);
            before += c;
        }
        for (int k = K + tid; k < row_floats(K); k += T) row[k] = INFINITY;
        if (by_cells) {
            __syncthreads();
            for_row([&] __device__(int, float2 v) {
                row[atomicAdd(&first[1 + cell(v.x)], 1u)] = v.x;
                row[atomicAdd(&first[1 + cell(v.y)], 1u)] = v.y;
            });
            __syncthreads();
            for (int i = tid * 32; i < K; i += T * 32) window32<2>(row + i);
            __syncthreads();
            for (int pass = 1; pass <= (fullest + 14) / 16; ++pass) {
                for (int i = tid * 32 + (pass & 1) * 16; i < K; i += T * 32) window32<32>(row + i);
                __syncthreads();
            }
        } else {
            for_row([&] __device__(int p, float2 v) {
                row[2 * p] = v.x;
                row[2 * p + 1] = v.y;
            });
            __syncthreads();
            bitonic_sort<T>(row, K);
        }

        // ---- prefix sums, one every BLK weights.  A unit is 2^-bits of the power of two above the largest weight: the
        // sums of up to BLK weights stay below 2^51 units, those of 15 prefix sums of K weights below 2^63.
        const int bits = min(47, 59 - log2_k);
        const double unit = ldexp(1.0, exponent - bits);
        const FixedPoint fixed = {0x1.8p52 * unit, unit};
        int64_t total;   // all K weights
        {
            const int full = K / BLK, nb = (full + T - 1) / T;   // whole blocks, consecutive ones of this thread
            const int b0 = min(tid * nb, full), b1 = min(b0 + nb, full);
            auto block_sum = [&] __device__(int b) {
                const float4 *blk = reinterpret_cast<const float4 *>(row + b * BLK);
                double s = fixed.bias;
#pragma unroll
                for (int i = 0; i < BLK / 4; ++i) {
                    const float4 v = blk[i];
                    s += (double)v.x;
                    s += (double)v.y;
                    s += (double)v.z;
                    s += (double)v.w;
                }
                return fixed.integer(s);
            };
            int64_t s = 0;
            for (int b = b0; b < b1; ++b) {
                prefix[b + 1] = s;   // (for now: within the thread's blocks, before block b)
                s += block_sum(b);
            }
            int64_t incl = s;
#pragma unroll
            for (int m = 1; m < 64; m <<= 1) {
                const int64_t o = __shfl_up((long long)incl, m, 64);
                if (lane >= m) incl += o;
            }
            if (lane == 63) s_sum[wave] = incl;
            __syncthreads();
            int64_t run = incl - s;   // the lanes before this one, then the waves before
            for (int i = 0; i < wave; ++i) run += s_sum[i];
            for (int b = b0; b < b1; ++b) prefix[b + 1] = run + (b + 1 < b1 ? prefix[b + 2] : s);   // up to block b's end
            if (tid == 0) prefix[0] = 0;
            __syncthreads();
            double rest = fixed.bias;
            for (int k = full * BLK; k < K; ++k) rest += (double)row[k];
            total = prefix[full] + fixed.integer(rest);
        }

        // ---- search: LANES lanes per start, no barrier
        const Row<BLK> r = {row, prefix, first, cell, K, fixed, total, sw2};
        const int j = lane & (LANES - 1);
        const bool all = search == DVDQ_BGR_BEST_OF_ALL;
        const double step = (hi0 - lo0) / (double)n_steps;
        const double mean = sw / (double)K;
        // sq / K, rounded as the division does: with r exact, the quotient before its last rounding is off by 2^-52 of an ulp
        // at most, and a quotient of integers below 2^19 and 2^15 is no closer to the middle between two doubles than 2^-16 ulp.
        const double per_k = 1.0 / (double)K;
        auto over_k = [&] __device__(double sq) {
            const double q = sq * per_k, rest = __builtin_fma(-q, (double)K, sq);
            return __builtin_fma(rest, per_k, q);
        };
        int best_i = 0x7FFFFFFF;
        best = INFINITY;
        best_delta = 1.0;
        best_z = 0.0;
        for (int64_t i = (all ? 0 : 1) + tid / LANES; i <= n_steps; i += T / LANES) {
            const double lo = lo0 + (double)i * step, hi = hi0 - (double)i * step;
            if (!(lo < hi)) break;   // the range has collapsed (from i = n_steps / 2 on)
            // clipped MinMax start
            double delta = (hi - lo) / kQmax;
            double z = clamp_d(rint(-(lo / delta)), 0.0, kQmax);
            Sums s = evaluate<BLK, LANES>(r, j, delta, z);
            double e = sqrt(s.e2);
            if (all && e < best) { best = e; best_delta = delta; best_z = z; best_i = (int)i; }
            for (int round = 0; round < max_refine; ++round) {
                if (s.den == 0.0 || e != e) break;   // (e: a NaN among the weights)
                const double dn = s.num / s.den;
                if (!(dn > 0.0)) break;
                const double zn = clamp_d(rint(over_k(s.sq) - mean / dn), 0.0, kQmax);
                if (dn == delta && zn == z) break;   // a fixed point: every further round is this grid again
                s = evaluate<BLK, LANES>(r, j, dn, zn);
                const double en = sqrt(s.e2);
                if (all && en < best) { best = en; best_delta = dn; best_z = zn; best_i = (int)i; }
                const double gain = e - en;
                e = en;
                delta = dn;
                z = zn;   // the start's current (last) grid
                if (gain < eps) break;
            }
            // as printed in Alg. 1: only the grid of the start's last round competes
            if (!all && e < best) { best = e; best_delta = delta; best_z = z; best_i = (int)i; }
        }
        // ---- the smallest error, ties to the earliest start: across the wave's groups, then the waves
#pragma unroll
        for (int m = LANES; m <= 32; m <<= 1) {
            const double oe = __shfl_xor(best, m, 64), od = __shfl_xor(best_delta, m, 64), oz = __shfl_xor(best_z, m, 64);
            const int oi = __shfl_xor(best_i, m, 64);
            if (oe < best || (oe == best && oi < best_i)) { best = oe; best_delta = od; best_z = oz; best_i = oi; }
        }
        if (lane == 0) { s_a[wave] = best; s_b[wave] = best_delta; s_c[wave] = best_z; s_i[wave] = best_i; }
        __syncthreads();
        if (tid == 0) {
            for (int i = 1; i < WAVES; ++i)
                if (s_a[i] < best || (s_a[i] == best && s_i[i] < best_i)) {
                    best = s_a[i];
                    best_delta = s_b[i];
                    best_z = s_c[i];
                    best_i = s_i[i];
                }
            s_best[0] = best;
            s_best[1] = best_delta;
            s_best[2] = best_z;
        }
        if (REGS) load(tid);   // (again, from the L2: kept through the search they would cost registers)
        __syncthreads();
        best = s_best[0];
        best_delta = s_best[1];
        best_z = s_best[2];
    }

    // ---- the codes on the best grid, as signed nibbles (unsigned code - 8), two per byte
    for_row([&] __device__(int p, float2 v) {
        int c[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const double wv = (double)(h ? v.y : v.x);
            const double q = constant ? (lo0 > 0.0 ? 1.0 : 0.0) : clamp_d(rint(wv / best_delta) + best_z, 0.0, kQmax);
            c[h] = (int)q - 8;
        }
        w_packed[n * pairs + p] = (uint8_t)((c[0] & 0xF) | ((c[1] & 0xF) << 4));
    });
    if (tid == 0) {
        w_scale[n] = (float)best_delta;
        w_zero[n] = (int8_t)((int)best_z - 8);
        if (row_error) row_error[n] = best;
    }
}

size_t lds_bytes(int64_t K, int blk, int cells) {
    return row_floats((int)K) * sizeof(float) + (size_t)(K / blk + 1) * sizeof(int64_t) + (size_t)(cells + 1) * sizeof(uint32_t);
}

template <int T, int BLK, int HELD, int LANES>
int launch(const float *w, int64_t N, int K, int cells, int n_steps, int max_refine, double eps, int search,
           uint8_t *w_packed, float *w_scale, int8_t *w_zero, double *row_error, hipStream_t stream) {
    auto k = bgr_kernel<T, BLK, HELD, LANES>;
    static std::atomic<uint64_t> configured{0};   // one per template instantiation
    allow_dynamic_lds(reinterpret_cast<const void *>(k), 158 * 1024, configured);
    // (a launch has fewer than 2^32 threads: more rows than that in several)
    constexpr int64_t kRows = ((int64_t)1 << 32) / T / 2;
    for (int64_t n = 0; n < N; n += kRows) {
        const unsigned rows = (unsigned)(N - n < kRows ? N - n : kRows);
        hipLaunchKernelGGL(k, dim3(rows), dim3(T), lds_bytes(K, BLK, cells), stream, w + n * K, K, cells, n_steps, max_refine, eps,
                           search, w_packed + n * (K / 2), w_scale + n, w_zero + n, row_error ? row_error + n : nullptr);
        const int rc = check_launch();
        if (rc != DVDQ_OK) return rc;
    }
    return DVDQ_OK;
}

}  // namespace

// Threads per workgroup for N rows of K weights: 256 (short rows), 512 or 1024.
// Bound by the issue of instructions, most of them fp64, of which a start's own (the same in all its lanes) weigh less the fewer lanes
// take it: rows short enough go as workgroups of 256 threads, four lanes a start, three to four at a time on a compute unit and not
// held in registers (100 steps, 10 rounds; as workgroups of 512 with eight lanes a start -> now: 13824 rows of 256 763 -> 504 us, 8960 of
// 1536 539 -> 369, 3000 of 4096 212 -> 161, 520 of 6144 63.5 -> 58.9).  Longer ones leave no room for a third beside two (780 rows of 6656:
// level).  Beyond 5376 weights three instead of four are resident, and the sorting, in which fewer threads take longer, needs many starts to
// outweigh: time over that of 512 threads at 4 to 50 steps up to 1.10 (1019 rows of 5604, 20 steps, 66.8 -> 73.6 us; up to 5376 weights at
// most 0.96), at 100 and more 0.76 to 1.00.
// With at most two rows per compute unit the time is one row's own, and the same holds for shorter rows, a start's rounds being shorter
// with eight lanes: at 3 to 20 steps 0.92 to 1.33 (454 rows of 2798, 10 steps, 16.5 -> 18.0 us; 413 of 4318, 6 steps, 32.8 -> 40.4), at 50 and
// 64 up to 1.17 (the starts, 24 and 31, still fill few waves), at 80 0.89 to 1.00 up to 2048 weights and 0.96 to 1.02 beyond, at 100 and more
// 0.80 to 0.96 with three rounds and 0.85 to 1.03 with fewer.
// 512 threads, two rows at a time per compute unit, while their LDS allows (half of 160 KB each; longer rows with coarser prefix sums
// and cells): 0.145 ms against 0.20 as workgroups of 1024 for 1536 rows of 8960.  1024 where there is no second row to put
// beside it: with no more rows than compute units (32 rows of 8960: level at 100 steps, 46.7 us against 50.8 at 200;
// 200 rows of 13824: 41.7 against 46.0), and from 14 K weights on.
int bgr_choice(int64_t N, int64_t K, int n_steps, int max_refine) {
    if (N > 512 ? K <= 5376 || (K <= 6144 && n_steps >= 100)
                : N > 256 && (K <= 2048 ? n_steps >= 80 : K <= 4608 && n_steps >= 100 && max_refine >= 3))
        return 256;
    return N > 256 && K <= 14336 ? 512 : 1024;
}

int launch_bgr(const float *w, int64_t N, int64_t K, int n_steps, int max_refine, double eps, int search,
               uint8_t *w_packed, float *w_scale, int8_t *w_zero, double *row_error, hipStream_t stream) {
#define DVDQ_BGR_ARGS(CELLS) \
    w, N, (int)K, CELLS, n_steps, max_refine, eps, search, w_packed, w_scale, w_zero, row_error, stream
    // (a few weights per cell: 1024 .. 4096 cells)
    const int threads = bgr_choice(N, K, n_steps, max_refine), cells = K <= 2048 ? 1024 : (K <= 4096 ? 2048 : 4096);
    if (threads == 256) return launch<256, 4, 0, 4>(DVDQ_BGR_ARGS(2048));
    if (threads == 512) return K <= 10240 ? launch<512, 4, 10, 8>(DVDQ_BGR_ARGS(cells)) : launch<512, 8, 14, 8>(DVDQ_BGR_ARGS(2048));
    return K > 16384 ? launch<1024, 16, 0, 8>(DVDQ_BGR_ARGS(2048)) : launch<1024, 4, 8, 8>(DVDQ_BGR_ARGS(cells));
#undef DVDQ_BGR_ARGS
}

}  // namespace dvdq
