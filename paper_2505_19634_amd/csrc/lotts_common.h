// Shared by the HIP translation units of liblotts.so: status codes, launch checking and
// wavefront helpers.  gfx950 only (64-wide wavefronts).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>
#include "lotts.h"

namespace lotts {

constexpr int kWave = 64;
// MI355X: 256 compute units in 8 XCDs.  Launch plans are sized for this part and do not depend
// on the device the process happens to see, so workspace queries agree everywhere.
constexpr int kNumCU = 256;
constexpr int kNumXCD = 8;

// Kernel timer (lotts_timer_start / lotts_timer_stop, kernel_timer.hip).  While it runs on the calling
// host thread, timer_take hands out one pair of events per launch and the launch carries them, so
// the pair reads that kernel's own start and end on the device.
bool timer_take(hipEvent_t* start, hipEvent_t* stop);

// Tag of a call whose workgroups exchange tagged words through the workspace (spec_accept,
// spec_accept_logits): different for every such call of the process whichever entry point makes it, so one
// buffer can serve both without either taking the other's leftovers for its own.  The top bit is always set: cleared
// words hold 0 above, and the 64-bit weight sums that earlier calls leave untagged in the same buffer (at most 2^50 for
// a row of logits, about 2^40 for a row of probabilities) never show a tag in their upper half.
unsigned next_word_tag();

// Polls after which a workgroup that waits for another one's words stops waiting.  The end of such a wait is not certain:
// every XCD dispatches its own share of a grid, so with two launches in flight one XCD can be full of the first one's
// waiting workgroups and another one full of the second's.  So nobody depends on it: after these polls (about a
// millisecond; ordinary waits are a few microseconds) a workgroup does the missing part itself, or leaves its own part to
// whoever comes last, and gives its place up.  Results are the same either way.  The test build sets 0: everything
// takes the other way.
#ifndef LOTTS_WAIT_POLLS
#define LOTTS_WAIT_POLLS 1024
#endif
constexpr int kWaitPolls = LOTTS_WAIT_POLLS;

// Every launch of the library goes through here: no dynamic LDS, the caller's stream.
#define LOTTS_LAUNCH(kernel, grid, block, stream, ...)                                                        \
    do {                                                                                                      \
        hipEvent_t lotts_e0_, lotts_e1_;                                                                      \
        if (lotts::timer_take(&lotts_e0_, &lotts_e1_))                                                        \
            hipExtLaunchKernelGGL(kernel, grid, block, 0, stream, lotts_e0_, lotts_e1_, 0, __VA_ARGS__);     \
        else                                                                                                  \
            hipLaunchKernelGGL(kernel, grid, block, 0, stream, __VA_ARGS__);                                  \
    } while (0)

inline int check_launch() {
    return hipGetLastError() == hipSuccess ? LOTTS_OK : LOTTS_ERR_LAUNCH;
}

// Division of 0 <= x < 2^31 by a divisor that the host knows: q = (2 x m) >> 32 >> l with l = ceil(log2 d), m = ceil(2^(31 + l) / d)
// <= 2^32 - 1 (m = 2^31 for powers of two).  Exact: m d = 2^(31 + l) + e with 0 <= e < d <= 2^l, so x m / 2^(31 + l) = x / d + x e / (d
// 2^(31 + l)) and the second term is below 1 / d.  Three instructions, scalar where x is; the compiler's own division by a
// run-time value is about twenty vector instructions in one dependent chain, 0.1 us at one wavefront per SIMD.
struct FastDiv {
    unsigned m, l;
};
static inline FastDiv fast_div(unsigned d) {
    FastDiv f = {0x80000000u, 0};
    while ((1ull << f.l) < d) ++f.l;
    f.m = (unsigned)(((1ull << (31 + f.l)) + d - 1) / d);
    return f;
}
__host__ __device__ __forceinline__ int quot(int x, FastDiv f) {
    return (int)((unsigned)(((unsigned long long)((unsigned)x << 1) * f.m) >> 32) >> f.l);
}

__device__ __forceinline__ float shfl_xor_f(float v, int mask) { return __shfl_xor(v, mask, kWave); }

__device__ __forceinline__ unsigned long long shfl_down_u64(unsigned long long v, int delta) {
    unsigned lo = (unsigned)v, hi = (unsigned)(v >> 32);
    lo = __shfl_down(lo, delta, kWave);
    hi = __shfl_down(hi, delta, kWave);
    return ((unsigned long long)hi << 32) | lo;
}
__device__ __forceinline__ unsigned long long shfl_up_u64(unsigned long long v, int delta) {
    unsigned lo = (unsigned)v, hi = (unsigned)(v >> 32);
    lo = __shfl_up(lo, delta, kWave);
    hi = __shfl_up(hi, delta, kWave);
    return ((unsigned long long)hi << 32) | lo;
}
__device__ __forceinline__ unsigned long long shfl_u64(unsigned long long v, int src) {
    unsigned lo = (unsigned)v, hi = (unsigned)(v >> 32);
    lo = __shfl(lo, src, kWave);
    hi = __shfl(hi, src, kWave);
    return ((unsigned long long)hi << 32) | lo;
}
// sum over the wavefront; the total is valid in lane 0
__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += shfl_down_u64(v, d);
    return v;
}
// inclusive prefix sum over the wavefront
__device__ __forceinline__ unsigned long long wave_incl_scan_u64(unsigned long long v, int lane) {
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        unsigned long long o = shfl_up_u64(v, d);
        if (lane >= d) v += o;
    }
    return v;
}

// Adds a lane's neighbour's value in one instruction: the wavefront-wide steps of a scan without a trip through LDS.  Lanes
// without a source, and rows that ROWS masks out, add nothing.
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned dpp_add(unsigned v) {
    return v + (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
// inclusive prefix sum over the wavefront of 32-bit values whose total fits 32 bits; lane 63 holds the total
__device__ __forceinline__ unsigned wave_incl_scan_u32(unsigned v) {
    v = dpp_add<0x111, 0xf>(v);  // row_shr 1, 2, 4, 8: inside each row of 16 lanes
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    v = dpp_add<0x142, 0xa>(v);  // row_bcast 15: rows 1 and 3 take the last lane of the row before
    return dpp_add<0x143, 0xc>(v);  // row_bcast 31: rows 2 and 3 take lane 31
}

template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned dpp_max(unsigned v) {
    return max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false));
}
// maximum over the wavefront
__device__ __forceinline__ unsigned wave_max_u31(unsigned v) {
    v = dpp_max<0x111, 0xf>(v);
    v = dpp_max<0x112, 0xf>(v);
    v = dpp_max<0x114, 0xf>(v);
    v = dpp_max<0x118, 0xf>(v);
    v = dpp_max<0x142, 0xa>(v);
    v = dpp_max<0x143, 0xc>(v);
    return __builtin_amdgcn_readlane(v, kWave - 1);
}

}  // namespace lotts
