// delta-Guided Bit Switching (Sec. 3.3): the relative L1 change between successive model
// outputs, L1(F, t) = ||F_t - F_{t-1}||_1 / ||F_{t-1}||_1, and the controller update that
// turns the running sum of these changes into the activation bit-width of the next
// denoising step.  No read-modify-write atomics, fixed summation order (bit-reproducible).
//
// HBM-bound partial sums: every thread reads 16 bytes of each tensor per step, accumulates |a - b| and |b| in fp32,
// workgroups reduce and write fp64 partials; one workgroup adds the partials in fp64, one per thread, forms the ratio
// and updates the state.  A step is ONE launch: the last workgroup waits for the other partials and adds them itself.
// (As a second launch the update was 5.2 us, as long as the pass over two 7.6 M element tensors, and 2.8 us of host
// time; three steps and a reset: 34.5 us with two launches per step.)  How it knows that a partial has arrived, with no
// counter that somebody would have to zero first (the caller's scratch holds anything): each launch carries a tag of
// its own, and a partial is three words, both sums and tag + k1 * sum + k2 * sum, that are valid only together.  The
// words may arrive in any order; a mixture with what lay there before fails the test unless it holds the same sums.
// A launch captured into a graph would repeat its tag, so under capture a step is two launches.
#include <chrono>
#include <unistd.h>

#include "dvdq_internal.h"
#include "wave_reduce.h"

namespace dvdq {
namespace {

constexpr int kThreads = 512;
constexpr int kMaxBlocks = 512;
constexpr int kWorkspaceSlots = 1024;   // partial-sum slots a caller's workspace has room for
static_assert(kMaxBlocks <= kThreads && 3 * kMaxBlocks <= 2 * kWorkspaceSlots, "one partial per thread of the update");

struct GbsState {      // 16 bytes in device memory, layout documented in dvdq.h
    double acc;        // running sum of relative L1 changes since the last reset
    float last_l1;     // the change computed by the latest step (for logging)
    int32_t bits;      // activation bit-width for the next denoising step
};

__device__ __forceinline__ void accum8(const uint4 a, const uint4 b, float &num, float &den) {
    const uint32_t aw[4] = {a.x, a.y, a.z, a.w}, bw[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float a0 = __uint_as_float(aw[i] << 16), a1 = __uint_as_float(aw[i] & 0xFFFF0000u);
        const float b0 = __uint_as_float(bw[i] << 16), b1 = __uint_as_float(bw[i] & 0xFFFF0000u);
        num += fabsf(a0 - b0) + fabsf(a1 - b1);
        den += fabsf(b0) + fabsf(b1);
    }
}

constexpr uint64_t kMixNum = 0x9E3779B97F4A7C15ull, kMixDen = 0xC2B2AE3D27D4EB4Full;   // odd, no simple ratio

// sums over the workgroup of one double2 per thread, the same in every thread; s_num, s_den: one slot per wave
__device__ __forceinline__ double2 workgroup_sum(double2 p, double *s_num, double *s_den) {
    const double num = wave_sum(p.x), den = wave_sum(p.y);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) { s_num[wave] = num; s_den[wave] = den; }
    __syncthreads();
    double2 s = make_double2(0.0, 0.0);
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) { s.x += s_num[w]; s.y += s_den[w]; }
    return s;
}

__device__ __forceinline__ void update_state(double2 s, double before, double delta, int b_low, int b_high, GbsState *state) {
    const double l1 = s.y > 0.0 ? s.x / s.y : (s.x > 0.0 ? (double)INFINITY : 0.0);
    double acc = before + l1;
    int bits = b_low;
    if (acc >= delta) { acc = 0.0; bits = b_high; }   // the sum reached the threshold: high precision, restart
    state->acc = acc;
    state->last_l1 = (float)l1;
    state->bits = bits;
}

// WHOLE: the step in one launch (see the top of this file); else the partials only, for gbs_update_kernel.
// partial: WHOLE [3][kMaxBlocks] words, else [blocks] pairs of doubles.
template <bool WHOLE>
__global__ __launch_bounds__(kThreads) void gbs_partial_kernel(const uint16_t *__restrict__ ft,
                                                               const uint16_t *__restrict__ fp, int64_t n,
                                                               uint64_t *partial, uint64_t tag, uint64_t wait_tag,
                                                               uint64_t wait_ticks, double delta, int b_low, int b_high,
                                                               GbsState *state) {
    __shared__ double s_num[kThreads / 64], s_den[kThreads / 64];
    __shared__ int s_lost;
    const int64_t nvec = n / 8;
    const uint4 *a = reinterpret_cast<const uint4 *>(ft), *b = reinterpret_cast<const uint4 *>(fp);
    float num = 0.f, den = 0.f;
    const int64_t stride = (int64_t)gridDim.x * kThreads;
    int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    // two independent loads in flight per tensor
    for (; i + stride < nvec; i += 2 * stride) {
        const uint4 a0 = a[i], b0 = b[i], a1 = a[i + stride], b1 = b[i + stride];
        accum8(a0, b0, num, den);
        accum8(a1, b1, num, den);
    }
    if (i < nvec) accum8(a[i], b[i], num, den);
    if (blockIdx.x == 0 && threadIdx.x == 0) {   // ragged tail of fewer than 8 elements
        for (int64_t e = nvec * 8; e < n; ++e) {
            const float x = __uint_as_float((uint32_t)ft[e] << 16), y = __uint_as_float((uint32_t)fp[e] << 16);
            num += fabsf(x - y);
            den += fabsf(y);
        }
    }
    // (fp32 within a wave, fp64 from there)
    num = wave_sum(num);
    den = wave_sum(den);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) { s_num[wave] = (double)num; s_den[wave] = (double)den; }
    if (threadIdx.x == 0) s_lost = 0;
    __syncthreads();
    if (threadIdx.x == 0) {
        double dn = 0.0, dd = 0.0;
        for (int w = 0; w < kThreads / 64; ++w) { dn += s_num[w]; dd += s_den[w]; }
        const uint64_t a = __builtin_bit_cast(uint64_t, dn), b = __builtin_bit_cast(uint64_t, dd);
        if constexpr (WHOLE) {
            __hip_atomic_store(partial + blockIdx.x, a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(partial + kMaxBlocks + blockIdx.x, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(partial + 2 * kMaxBlocks + blockIdx.x, tag + kMixNum * a + kMixDen * b, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        } else {
            partial[2 * blockIdx.x] = a;
            partial[2 * blockIdx.x + 1] = b;
        }
    }
    if constexpr (WHOLE) {
        if (blockIdx.x != gridDim.x - 1) return;
        // (Nothing waits for this workgroup: the others finish whatever it does, so the loop below ends.  Two steps at
        // once on one scratch buffer, which it is not for, would overwrite each other's partials: then it ends after
        // `wait_ticks` of the constant 100 MHz clock, and the step says that it has no result: NaN as the change, the
        // running sum as it was, and the higher bit-width, the safe choice.  wait_tag is `tag`; another in the test of this.)
        const uint64_t deadline = wall_clock64() + wait_ticks;
        const double before = state->acc;
        double2 p = make_double2(0.0, 0.0);
        if (threadIdx.x < gridDim.x) {
            uint64_t a, b, c;
            for (;;) {
                a = __hip_atomic_load(partial + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                b = __hip_atomic_load(partial + kMaxBlocks + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                c = __hip_atomic_load(partial + 2 * kMaxBlocks + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (c == wait_tag + kMixNum * a + kMixDen * b) break;
                if (wall_clock64() > deadline) {
                    s_lost = 1;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
            p = make_double2(__builtin_bit_cast(double, a), __builtin_bit_cast(double, b));
        }
        __syncthreads();   // s_num, s_den are read above
        if (s_lost) {
            if (threadIdx.x == 0) {
                state->last_l1 = __builtin_nanf("");
                state->bits = b_high;
            }
            return;
        }
        p = workgroup_sum(p, s_num, s_den);
        if (threadIdx.x == 0) update_state(p, before, delta, b_low, b_high, state);
    }
}

__global__ __launch_bounds__(kThreads) void gbs_update_kernel(const double2 *__restrict__ partial, int blocks, double delta,
                                                              int b_low, int b_high, GbsState *state) {
    __shared__ double s_num[kThreads / 64], s_den[kThreads / 64];
    const double before = state->acc;   // (requested here: its latency passes with the reduction's)
    const double2 p = workgroup_sum((int)threadIdx.x < blocks ? partial[threadIdx.x] : make_double2(0.0, 0.0), s_num, s_den);
    if (threadIdx.x == 0) update_state(p, before, delta, b_low, b_high, state);
}

__global__ void gbs_reset_kernel(GbsState *state, int bits) {
    state->acc = 0.0;
    state->last_l1 = 0.f;
    state->bits = bits;
}

// A tag per launch: consecutive numbers from a start that differs between processes (time and process number, mixed),
// so that neither an earlier launch of this process nor memory that another one left behind holds partials of the same
// tag.
uint64_t next_tag() {
    static std::atomic<uint64_t> tag{[] {
        uint64_t z = (uint64_t)std::chrono::system_clock::now().time_since_epoch().count() * kMixNum + (uint64_t)getpid() * kMixDen;
        z = (z ^ (z >> 31)) * kMixDen;
        return z ^ (z >> 29);
    }()};
    return tag.fetch_add(1, std::memory_order_relaxed);
}

constexpr int64_t kWaitTicks = 1000000000;   // ten seconds: longer than any step takes, also on a GPU shared with others
std::atomic<int64_t> g_wait{-1};             // test hook: wait this long for partials that do not come; -1: off

}  // namespace

void set_gbs_wait(int64_t ticks) { g_wait.store(ticks, std::memory_order_relaxed); }

size_t gbs_workspace_bytes() { return sizeof(double) * 2 * kWorkspaceSlots; }

int launch_gbs_reset(void *state, int bits, hipStream_t stream) {
    hipLaunchKernelGGL(gbs_reset_kernel, dim3(1), dim3(1), 0, stream, static_cast<GbsState *>(state), bits);
    return check_launch();
}

int launch_gbs_step(const uint16_t *ft, const uint16_t *fp, int64_t n, double delta, int b_low, int b_high,
                    void *state, void *workspace, hipStream_t stream) {
    int64_t blocks = (n / 8 + kThreads - 1) / kThreads;
    if (blocks < 1) blocks = 1;
    if (blocks > kMaxBlocks) blocks = kMaxBlocks;
    uint64_t *partial = static_cast<uint64_t *>(workspace);
    GbsState *st = static_cast<GbsState *>(state);
    const dim3 grid((unsigned)blocks), block(kThreads);
    hipStreamCaptureStatus cap = hipStreamCaptureStatusActive;
    if (hipStreamIsCapturing(stream, &cap) != hipSuccess) {
        (void)hipGetLastError();
        cap = hipStreamCaptureStatusActive;
    }
    if (cap == hipStreamCaptureStatusNone) {
        const int64_t hook = g_wait.load(std::memory_order_relaxed);
        const uint64_t tag = next_tag();
        hipLaunchKernelGGL(gbs_partial_kernel<true>, grid, block, 0, stream, ft, fp, n, partial, tag, hook < 0 ? tag : ~tag,
                           (uint64_t)(hook < 0 ? kWaitTicks : hook), delta, b_low, b_high, st);
        return check_launch();
    }
    hipLaunchKernelGGL(gbs_partial_kernel<false>, grid, block, 0, stream, ft, fp, n, partial, (uint64_t)0, (uint64_t)0, (uint64_t)0, delta,
                       b_low, b_high, st);
    const int rc = check_launch();
    if (rc != DVDQ_OK) return rc;
    hipLaunchKernelGGL(gbs_update_kernel, dim3(1), block, 0, stream, static_cast<const double2 *>(workspace), (int)blocks, delta,
                       b_low, b_high, st);
    return check_launch();
}

}  // namespace dvdq
