// spec_accept_logits: speculative-sampling acceptance straight from target / draft LOGITS, so
// that the V-wide softmax outputs p and q are never written to memory (for the 32B-shaped
// workload: 34 MB of bf16 logits read instead of 34 MB read + 68 MB written + 13-19 MB re-read).
// The rule is the one of spec_accept (paper Section 2 / 3.2: draft proposes, target verifies,
// losslessly); the distributions are softmax(z * inv_temperature).
//
// To be independent of summation order and of any exp() implementation, the softmax is defined on
// integers: y_v = fp32(z_v) * inv_temp, m = max_v y_v, t_v = (y_v - m) * log2(e),
//   E_v = trunc(P(frac(-t_v)) * 2^(30 - floor(-t_v)))   (0 when floor(-t_v) >= 31),
// P a fixed degree-6 polynomial for 2^-f evaluated with fused multiply-adds, S = sum_v E_v, and the
// probability of v is E_v / S exactly.  Accept x iff U * Eq(x) * Sp < 2^24 * Ep(x) * Sq with
// U = trunc(u * 2^24); residual weights W_v = max(0, Ep_v * Sq - Eq_v * Sp); bonus weights Ep_v;
// token = first v whose prefix sum exceeds floor(U_k * sum W / 2^24).  128-bit integers.
//
// Two launches:
//   lg_stat_kernel      grid (pieces of 8192 to 16384 logits, B * (2k + 1) rows, the pieces of a row next to each other): a
//                       workgroup reads its piece ONCE into registers, publishes the piece's maximum under this call's tag (two words),
//                       collects the maxima of the row's other pieces (one that stays out for long it forms itself, from
//                       the logits), and stores the piece's integer weight sum, formed from the registers; the piece that
//                       holds the row's drafted token stores its weight too.
//   lg_scan_pick_kernel grid (chunks, B): accept tests -> n; 128-bit chunk sums of the weights of row n, published as
//                       six 8-byte words that each carry 32 bits of a sum and this call's tag.  The workgroup of a
//                       branch's LAST chunk then collects the branch's sums (one that stays out for long it forms itself)
//                       and finds the chunk and the token where the integer CDF crosses the threshold, re-reading that one
//                       chunk.
// Rows start anywhere (the vocabulary need not be a multiple of anything): 16-byte loads take any alignment of the element
// type, and only the last group of a row is read element by element.
// Every floating-point operation in this file is rounded on its own, as the definition of the integer weights
// says: the compiler's default for device code would otherwise be free to merge a multiplication and a
// following addition or subtraction into one fused operation (one rounding), depending on how the
// surrounding code happens to be shaped.  Fused multiply-adds are written out where the definition has them.
#pragma clang fp contract(off)
#include "lotts_common.h"

namespace lotts {

typedef unsigned __int128 u128;

constexpr int kLgThreads = 256;
constexpr int kLgWaves = kLgThreads / kWave;
constexpr int kLgGroup = kLgThreads * 8;  // logits a workgroup reads in one round of 16-byte loads (two rounds for fp32)
constexpr int kLgMaxPieces = 64;     // pieces of a row: one wavefront collects their maxima
constexpr int kLgChunk = 2048;       // tokens per chunk: 8 per thread
constexpr int kLgMaxChunks = 512;    // V <= 2^20
constexpr int kLgMaxK = kLgThreads;
constexpr unsigned long long kLgNoSum = ~0ull;  // no sum of a chunk: those are below 2^41

struct RowStat {
    float m;               // row maximum of y
    unsigned long long S;  // sum of the integer weights
};

// 16 bytes of logits at any alignment of the element type: one load instruction on this part, whatever the address
typedef unsigned l_u32x4 __attribute__((ext_vector_type(4)));
typedef l_u32x4 l_u32x4_any __attribute__((aligned(2)));

// One multiplication / subtraction, rounded to nearest.  Defined here, under the pragma above: the toolkit's
// __fmul_rn / __fsub_rn are plain operators compiled under the default mode, and a product and a difference taken
// through them were merged into one fused operation once the two were inlined next to each other.
__device__ __forceinline__ float mul_rn(float a, float b) { return a * b; }
__device__ __forceinline__ float sub_rn(float a, float b) { return a - b; }

__device__ __forceinline__ float bf16_bits_to_float(unsigned short h) { return __uint_as_float((unsigned)h << 16); }

// 2^30 * 2^-f on [0, 1): the polynomial of the definition (c0 = 1 exactly), fused multiply-adds only, with every
// coefficient scaled by 2^30.  Scaling by a power of two commutes with each rounding (no result comes near the
// ends of the exponent range), so this is 2^30 times the definition's P(f), bit for bit.
__device__ __forceinline__ float pow2_neg_poly_2p30(float f) {
    float g = 0x1.e243bep+16f;
    g = __fmaf_rn(g, f, -0x1.52a284p+20f);
    g = __fmaf_rn(g, f, 0x1.3a7ae4p+23f);
    g = __fmaf_rn(g, f, -0x1.c6a66cp+25f);
    g = __fmaf_rn(g, f, 0x1.ebfbaap+27f);
    g = __fmaf_rn(g, f, -0x1.62e430p+29f);
    g = __fmaf_rn(g, f, 0x1p+30f);
    return g;
}

// The conversions that truncate, with the instruction's results outside the integers' range (NaN: 0; beyond: the nearest end):
// written out, because C++ leaves those results open.
__device__ __forceinline__ int to_i32(float v) {
    int r;
    asm("v_cvt_i32_f32 %0, %1" : "=v"(r) : "v"(v));
    return r;
}
__device__ __forceinline__ unsigned to_u32(float v) {
    unsigned r;
    asm("v_cvt_u32_f32 %0, %1" : "=v"(r) : "v"(v));
    return r;
}
// E = trunc(2^t * 2^30) through the definition's steps; every operation individually rounded.  With n = floor(-t) = -trunc(t) the
// definition's trunc(P * 2^(30 - n)) is one scaling by a power of two (exact: P * 2^30 >= 2^29, a result below the normal numbers
// truncates to 0 as the definition's does) and one truncation.  From n = 31 on the result is 0 by itself; -inf logits
// (n = the lowest integer) and NaN (rows that are -inf throughout, or hold +inf) truncate to 0 as well: no clamp, branch or select.
__device__ __forceinline__ unsigned logit_weight(float y, float m) {
    const float t = mul_rn(sub_rn(y, m), 0x1.715476p+0f);
    const float f = __builtin_amdgcn_fractf(-t);  // -t - floor(-t) in one instruction, exact
    return to_u32(__builtin_ldexpf(pow2_neg_poly_2p30(f), to_i32(t)));
}

template <bool BF16>
__device__ __forceinline__ float load_y(const void* z, size_t idx, float inv_temp) {
    const float v = BF16 ? bf16_bits_to_float(static_cast<const unsigned short*>(z)[idx])
                         : static_cast<const float*>(z)[idx];
    return mul_rn(v, inv_temp);
}

// 8 consecutive logits of a row, raw: tokens i .. i + 7, -inf from hi on
template <bool BF16>
struct Raw8 {
    l_u32x4 v[BF16 ? 1 : 2];
};
template <bool BF16>
__device__ __forceinline__ Raw8<BF16> load_raw8(const void* z, size_t base, int i, int hi) {
    Raw8<BF16> r;
    if (BF16) {
        const unsigned short* src = static_cast<const unsigned short*>(z) + base + i;
        if (i + 8 <= hi) {
            r.v[0] = *reinterpret_cast<const l_u32x4_any*>(src);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {  // bf16 -inf is 0xff80
                const unsigned a = i + 2 * e < hi ? src[2 * e] : 0xff80u, b = i + 2 * e + 1 < hi ? src[2 * e + 1] : 0xff80u;
                r.v[0][e] = a | (b << 16);
            }
        }
    } else {
        const float* src = static_cast<const float*>(z) + base + i;
        if (i + 8 <= hi) {
            r.v[0] = *reinterpret_cast<const l_u32x4_any*>(src);
            r.v[BF16 ? 0 : 1] = *reinterpret_cast<const l_u32x4_any*>(src + 4);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) r.v[BF16 ? 0 : e / 4][e % 4] = __float_as_uint(i + e < hi ? src[e] : -INFINITY);
        }
    }
    return r;
}
template <bool BF16>
__device__ __forceinline__ void scale8(const Raw8<BF16>& r, float inv_temp, float (&y)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float v = BF16 ? __uint_as_float(e % 2 ? r.v[0][e / 2] & 0xffff0000u : r.v[0][e / 2] << 16)
                             : __uint_as_float(r.v[BF16 ? 0 : e / 4][e % 4]);
        y[e] = mul_rn(v, inv_temp);
    }
}

// Inclusive prefix sum over the wavefront of values whose total is below 2^104, as four limbs (24, 24, 24, 32 bits) in
// independent 32-bit chains of one-instruction steps.  (A weight is at most 2^30 * 2^50, a chunk's sum 2^91, a row's 2^100.)
__device__ __forceinline__ u128 wave_incl_scan_u128(u128 v) {
    const unsigned l0 = wave_incl_scan_u32((unsigned)v & 0xffffffu), l1 = wave_incl_scan_u32((unsigned)(v >> 24) & 0xffffffu);
    const unsigned l2 = wave_incl_scan_u32((unsigned)(v >> 48) & 0xffffffu), l3 = wave_incl_scan_u32((unsigned)(v >> 72));
    return (u128)l0 + ((u128)l1 << 24) + ((u128)l2 << 48) + ((u128)l3 << 72);
}
// exclusive prefix sum in thread order over a 256-thread workgroup; the total in every thread
__device__ __forceinline__ u128 block_excl_scan_u128(u128 v, u128* sh /*[kLgWaves]*/, u128& total) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    const u128 incl = wave_incl_scan_u128(v);
    __syncthreads();
    if (lane == kWave - 1) sh[w] = incl;
    __syncthreads();
    u128 base = 0;
    total = 0;
#pragma unroll
    for (int i = 0; i < kLgWaves; ++i) {
        base += (i < w) ? sh[i] : (u128)0;
        total += sh[i];
    }
    return base + incl - v;
}

// row index of target row (b, j) and of draft row (b, j) in the stats array
__device__ __forceinline__ int trow(int b, int j, int k) { return b * (k + 1) + j; }
__device__ __forceinline__ int drow(int B, int b, int j, int k) { return B * (k + 1) + b * k + j; }

// one published word: 32 bits of a value under the call's tag
__device__ __forceinline__ void lg_publish(unsigned long long* slot, unsigned part, unsigned tag) {
    __hip_atomic_store(slot, ((unsigned long long)tag << 32) | part, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long lg_peek(const unsigned long long* slot) {
    return __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Row statistics in one sweep.  The weights need the row maximum, so the pieces of a row exchange their maxima inside the
// launch while their logits stay in registers; what a launch boundary and a second read of all logits cost before is one trip
// through memory now.  A row's pieces are neighbours in the grid, so the others' words are mostly there when they are looked
// for; that they come at all is not relied on (kWaitPolls).  The words are cleared by the next launch.
// Bound by the vector unit: 16 instructions a logit that the integer definition fixes (12 for the weight, the rest unpacking, scaling,
// maximum and sum), 7 us of the chip's rate for 112 rows x 152064 logits, behind the read that all workgroups start with: a unit returns
// loads in order, so the words of the exchange wait behind the logits that the unit's other workgroups have asked for (fewer
// workgroups at a time are no way out: 28.7 us with five to a unit, 30.4 with four, against 27.4).  In a captured graph, us, as three launches
// (maxima, sums, scan) -> two -> now: 16 x 7 rows x 152064 bf16 30.8 -> 27.5 -> 23.1, fp32 40.5 -> 31.3 -> 27.7; 5 x 15 rows x 50257 fp32
// (rows off a 16-byte boundary) 48.0 -> 15.7 -> 13.5; 32 x 17 x 151936 bf16 68.3 -> 55.6.
template <bool BF16, int IT>
__global__ __launch_bounds__(kLgThreads) void lg_stat_kernel(int B, int k, int V, int npieces, unsigned tag,
                                                             const void* __restrict__ zt, const void* __restrict__ zd,
                                                             float inv_temp, unsigned long long* __restrict__ words,
                                                             float* __restrict__ rmax, unsigned long long* __restrict__ psum,
                                                             unsigned long long* __restrict__ slots, long long nslots,
                                                             const int32_t* __restrict__ draft, unsigned* __restrict__ draft_e,
                                                             FastDiv d_pieces, FastDiv d_targets) {
    __shared__ float sh_m[kLgWaves];
    __shared__ float sh_row;
    __shared__ unsigned long long sh_miss, sh_s[kLgWaves];
    const int r = quot(blockIdx.x, d_pieces), pc = blockIdx.x - r * npieces, tid = threadIdx.x, lane = tid & (kWave - 1);
    const int nt = B * (k + 1);
    // the token that was drafted where this row stands (a branch's last target row: none)
    const int rb = quot(r, d_targets), rj = r - rb * (k + 1);
    const int dx = r < nt ? (rj < k ? rb * k + rj : -1) : r - nt;
    const int drafted = dx >= 0 ? ((const __attribute__((address_space(4))) int32_t*)draft)[dx] : -1;
    const void* z = r < nt ? zt : zd;
    const size_t base = (size_t)(r < nt ? r : r - nt) * V;
    const int lo = pc * (IT * kLgGroup);
    // The next launch's words are cleared, so that a captured call (same tags) can be replayed.  (A piece is at most 8 chunks of
    // a row, 48 words: a word per thread is enough.)
    const long long slot = (long long)blockIdx.x * kLgThreads + tid;
    if (slot < nslots) slots[slot] = 0ull;
    // the whole piece is requested before any of it is used
    Raw8<BF16> raw[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) raw[it] = load_raw8<BF16>(z, base, lo + it * kLgGroup + tid * 8, V);
    // Its weight is formed here, where the row's maximum is met anyway: the next launch's accept tests would reach its logit
    // only behind the drafted token, two dependent trips through memory.
    const int x = drafted < 0 ? 0 : (drafted >= V ? V - 1 : drafted);
    const bool mine = dx >= 0 && x >= lo && x < lo + IT * kLgGroup;  // uniform
    float yx = 0.f;
    if (mine) yx = load_y<BF16>(z, base + x, inv_temp);
    float y[IT][8], m = -INFINITY;
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        scale8<BF16>(raw[it], inv_temp, y[it]);
#pragma unroll
        for (int e = 0; e < 8; ++e) m = fmaxf(m, y[it][e]);
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, kWave));
    if (lane == 0) sh_m[tid / kWave] = m;
    __syncthreads();
    if (tid < kWave) {
#pragma unroll
        for (int w = 0; w < kLgWaves; ++w) m = fmaxf(m, sh_m[w]);
        // A piece's maximum stands in two words, under the tag and under its complement, and counts only when both agree: no
        // single leftover of an earlier call -- a row sum, a maximum, a word of another size's layout -- reads as one.
        unsigned long long* row = words + (size_t)r * npieces * 2;
        if (tid == 0) {
            lg_publish(row + pc * 2, __float_as_uint(m), tag);
            lg_publish(row + pc * 2 + 1, __float_as_uint(m), ~tag);
        }
        bool missing = lane < npieces && lane != pc;
        for (int polls = 0; missing && polls < kWaitPolls; ++polls) {
            const unsigned long long w0 = lg_peek(row + lane * 2), w1 = lg_peek(row + lane * 2 + 1);
            if ((unsigned)(w0 >> 32) == tag && (unsigned)(w1 >> 32) == ~tag && (unsigned)w0 == (unsigned)w1) {
                m = fmaxf(m, __uint_as_float((unsigned)w0));
                missing = false;
            } else {
                __builtin_amdgcn_s_sleep(1);
            }
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, kWave));
        const unsigned long long miss = __ballot(missing);
        if (tid == 0) {
            sh_row = m;
            sh_miss = miss;
        }
    }
    __syncthreads();
    m = sh_row;
    if (sh_miss) {  // uniform over the workgroup: the maxima that have not come, from the logits
        for (unsigned long long left = sh_miss; left; left &= left - 1) {
            const int at = (__ffsll((long long)left) - 1) * (IT * kLgGroup);
#pragma unroll 1
            for (int it = 0; it < IT; ++it) {
                float v[8];
                scale8<BF16>(load_raw8<BF16>(z, base, at + it * kLgGroup + tid * 8, V), inv_temp, v);
#pragma unroll
                for (int e = 0; e < 8; ++e) m = fmaxf(m, v[e]);
            }
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, kWave));
        if (lane == 0) sh_m[tid / kWave] = m;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kLgWaves; ++w) m = fmaxf(m, sh_m[w]);
    }
    unsigned long long s = 0;
#pragma unroll
    for (int it = 0; it < IT; ++it)
#pragma unroll
        for (int e = 0; e < 8; e += 3) {  // three weights (each at most 2^30) fit 32 bits together
            unsigned part = logit_weight(y[it][e], m);
            if (e + 1 < 8) part += logit_weight(y[it][e + 1], m);
            if (e + 2 < 8) part += logit_weight(y[it][e + 2], m);
            s += part;
        }
    // at most 64 weights a lane: s < 2^37; two limbs whose wavefront sums fit 32 bits
    const unsigned s0 = wave_incl_scan_u32((unsigned)s & 0xffffffu), s1 = wave_incl_scan_u32((unsigned)(s >> 24));
    if (lane == kWave - 1) sh_s[tid / kWave] = (unsigned long long)s0 + ((unsigned long long)s1 << 24);
    __syncthreads();
    if (tid == 0) {
        unsigned long long tot = 0;
#pragma unroll
        for (int w = 0; w < kLgWaves; ++w) tot += sh_s[w];
        psum[(size_t)r * npieces + pc] = tot;
        if (pc == 0) rmax[r] = m;
        if (mine) draft_e[r] = logit_weight(yx, m);
    }
}

// Statistics of branch b's 2k + 1 rows (targets 0 .. k, then drafts) into LDS, from what lg_stat_kernel leaves: the row
// maxima and the sums of the rows' pieces.  As many lanes to a row as the workgroup has, so that one load latency covers
// nearly all of it (a thread per row, 16 loads at a time, cost a 16 x 7 rows x 152064 call 1.5 us more).  lg: log2 of the lanes.
__device__ __forceinline__ void lg_row_stats(int B, int b, int k, int npieces, int lg, const float* rmax, const unsigned long long* psum,
                                             RowStat* sh_stat) {
    const int rows = 2 * k + 1;
    const int sub = threadIdx.x & ((1 << lg) - 1);
    for (int j = threadIdx.x >> lg; j < rows; j += kLgThreads >> lg) {
        const int row = j <= k ? trow(b, j, k) : drow(B, b, j - k - 1, k);
        const unsigned long long* src = psum + (size_t)row * npieces;
        RowStat st;
        st.m = rmax[row];
        st.S = 0;
        if (npieces <= (2 << lg)) {  // one or two pieces a lane: no load that is not needed
            const int next = sub + (1 << lg);
            const unsigned long long v0 = sub < npieces ? src[sub] : 0ull, v1 = next < npieces ? src[next] : 0ull;
            st.S = v0 + v1;
        } else {
            for (int i0 = sub; i0 < npieces; i0 += 8 << lg) {  // eight loads in flight
                unsigned long long v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = src[min(i0 + (e << lg), npieces - 1)];
#pragma unroll
                for (int e = 0; e < 8; ++e) st.S += i0 + (e << lg) < npieces ? v[e] : 0ull;
            }
        }
        // a row's lanes are here together: their sum (below 2^50, two limbs) in the last of them
        unsigned s0 = (unsigned)st.S & 0xffffffu, s1 = (unsigned)(st.S >> 24);
        if (lg > 0) { s0 = dpp_add<0x111, 0xf>(s0); s1 = dpp_add<0x111, 0xf>(s1); }  // row_shr 1, 2, 4, 8
        if (lg > 1) { s0 = dpp_add<0x112, 0xf>(s0); s1 = dpp_add<0x112, 0xf>(s1); }
        if (lg > 2) { s0 = dpp_add<0x114, 0xf>(s0); s1 = dpp_add<0x114, 0xf>(s1); }
        if (lg > 3) { s0 = dpp_add<0x118, 0xf>(s0); s1 = dpp_add<0x118, 0xf>(s1); }
        if (lg > 4) { s0 = dpp_add<0x142, 0xa>(s0); s1 = dpp_add<0x142, 0xa>(s1); }  // row_bcast 15, 31
        if (lg > 5) { s0 = dpp_add<0x143, 0xc>(s0); s1 = dpp_add<0x143, 0xc>(s1); }
        st.S = ((unsigned long long)s1 << 24) + s0;
        if (sub == (1 << lg) - 1) sh_stat[j] = st;
    }
}

// Accepted length of branch b; every thread of the 256-thread workgroup gets it, and the statistics of the two rows at n (of
// the target row alone when every draft was accepted) with it.
__device__ __forceinline__ int lg_accepted_length(int B, int b, int k, const unsigned* draft_e, const float* u, const float* rmax,
                                                  const unsigned long long* psum, int npieces, int lg, int* sh_first,
                                                  RowStat* sh_stat, RowStat& sp, RowStat& sq) {
    const int tid = threadIdx.x;
    float uv = 0.f;
    unsigned Ep = 0, Eq = 0;
    if (tid < k) {  // one trip together with the sums
        uv = u[(size_t)b * (k + 1) + tid];
        Ep = draft_e[trow(b, tid, k)];
        Eq = draft_e[drow(B, b, tid, k)];
    }
    lg_row_stats(B, b, k, npieces, lg, rmax, psum, sh_stat);
    __syncthreads();
    bool rejected = false;
    if (tid < k) {
        const RowStat p = sh_stat[tid], q = sh_stat[k + 1 + tid];
        const u128 U = (u128)(unsigned)(uv * 16777216.0f);
        rejected = !(U * Eq * p.S < ((u128)1 << 24) * Ep * q.S);
    }
    const unsigned long long mask = __ballot(rejected);
    if ((tid & (kWave - 1)) == 0) sh_first[tid / kWave] = mask ? (tid + __ffsll((long long)mask) - 1) : k;
    __syncthreads();
    int n = k;
#pragma unroll
    for (int w = 0; w < kLgWaves; ++w) n = sh_first[w] < n ? sh_first[w] : n;
    sp = sh_stat[n];
    sq = n < k ? sh_stat[k + 1 + n] : sp;
    return n;
}

// Sampling weights are below 2^80 and a thread's sum of eight below 2^83: three 32-bit limbs and their carries, not the four of
// 128 bits with a comparison and a selection of their own.
struct U96 {
    unsigned v[3];
};
__device__ __forceinline__ u128 widen(U96 a) { return (u128)a.v[0] | ((u128)a.v[1] << 32) | ((u128)a.v[2] << 64); }
// a weight (at most 2^30) times a row's sum (below 2^50): two products
__device__ __forceinline__ U96 mul_e_s(unsigned e, unsigned long long s) {
    const unsigned long long lo = (unsigned long long)e * (unsigned)s;
    const unsigned long long hi = (unsigned long long)e * (unsigned)(s >> 32) + (lo >> 32);
    return U96{{(unsigned)lo, (unsigned)hi, (unsigned)(hi >> 32)}};
}
__device__ __forceinline__ U96 add_96(U96 a, U96 b) {
    unsigned c;
    U96 r;
    r.v[0] = __builtin_addc(a.v[0], b.v[0], 0u, &c);
    r.v[1] = __builtin_addc(a.v[1], b.v[1], c, &c);
    r.v[2] = __builtin_addc(a.v[2], b.v[2], c, &c);
    return r;
}
// max(0, a - b)
__device__ __forceinline__ U96 sub_sat_96(U96 a, U96 b) {
    unsigned c;
    U96 r;
    r.v[0] = __builtin_subc(a.v[0], b.v[0], 0u, &c);
    r.v[1] = __builtin_subc(a.v[1], b.v[1], c, &c);
    r.v[2] = __builtin_subc(a.v[2], b.v[2], c, &c);
#pragma unroll
    for (int i = 0; i < 3; ++i) r.v[i] = c ? 0u : r.v[i];
    return r;
}

// the 8 weights a thread owns in a chunk (tokens lo .. lo+7, clipped to V): residual or plain
template <bool BF16>
__device__ __forceinline__ void lg_weights8(const void* zt_row, const void* zd_row, int lo, int V, float inv_temp,
                                            bool residual, RowStat sp, RowStat sq, U96 (&W)[8], unsigned (&Ep)[8]) {
    float yp[8], yq[8];
    const Raw8<BF16> rp = load_raw8<BF16>(zt_row, 0, lo, V);
    if (residual) {
        const Raw8<BF16> rq = load_raw8<BF16>(zd_row, 0, lo, V);
        scale8<BF16>(rq, inv_temp, yq);
    }
    scale8<BF16>(rp, inv_temp, yp);
#pragma unroll
    for (int e = 0; e < 8; ++e) {  // (beyond V the logits are -inf and weigh 0: a branch for each cost more than the weights)
        Ep[e] = logit_weight(yp[e], sp.m);
        if (residual) {
            const unsigned Eq = logit_weight(yq[e], sq.m);
            W[e] = sub_sat_96(mul_e_s(Ep[e], sq.S), mul_e_s(Eq, sp.S));
        } else {
            W[e] = U96{{Ep[e], 0u, 0u}};
        }
    }
}

template <bool BF16>
__global__ __launch_bounds__(kLgThreads) void lg_scan_pick_kernel(int B, int k, int V, int nchunks, int npieces, int lg, unsigned tag,
                                                                  const void* __restrict__ zt, const void* __restrict__ zd,
                                                                  float inv_temp, const unsigned* __restrict__ draft_e,
                                                                  const float* __restrict__ u,
                                                                  const float* __restrict__ rmax,
                                                                  const unsigned long long* __restrict__ psum,  // [rows][npieces]
                                                                  int32_t* __restrict__ accept_len,
                                                                  unsigned long long* __restrict__ words,  // [rows][npieces][2]
                                                                  unsigned long long* __restrict__ slots,  // [B][nchunks][6]
                                                                  int32_t* __restrict__ next_token,
                                                                  int32_t* __restrict__ priv_len) {
    __shared__ int sh_first[kLgWaves];
    __shared__ u128 sh_w[kLgWaves];
    __shared__ u128 sh_base;
    __shared__ int sh_chunk, sh_missing;
    __shared__ u128 sh_wsum[kLgMaxChunks];
    __shared__ unsigned long long sh_psum[kLgMaxChunks];
    const int b = blockIdx.y, c = blockIdx.x, tid = threadIdx.x;
    __shared__ RowStat sh_stat[2 * kLgMaxK + 1];
    const float u_last = u[(size_t)b * (k + 1) + k];
    RowStat sp, sq;
    const int n = lg_accepted_length(B, b, k, draft_e, u, rmax, psum, npieces, lg, sh_first, sh_stat, sp, sq);
    bool residual = n < k;
    const size_t es = BF16 ? 2 : 4;
    const void* zt_row = static_cast<const char*>(zt) + (size_t)trow(b, n, k) * V * es;
    const void* zd_row = residual ? static_cast<const char*>(zd) + ((size_t)b * k + n) * V * es : zt_row;
    U96 W[8];
    unsigned Ep[8];
    __shared__ unsigned long long sh_e[kLgWaves];
    // sums of a chunk's weights (residual after a rejection) and of its plain ones; complete in thread 0 only
    auto chunk_sums = [&](int chunk, u128& w, unsigned long long& e) {
        lg_weights8<BF16>(zt_row, zd_row, chunk * kLgChunk + tid * 8, V, inv_temp, n < k, sp, sq, W, Ep);
        U96 sum = W[0];
        e = Ep[0];
#pragma unroll
        for (int i = 1; i < 8; ++i) {
            sum = add_96(sum, W[i]);
            e += Ep[i];
        }
        w = widen(sum);
        // both sums over the workgroup at once: the totals stand in lane 63 of every wavefront
        w = wave_incl_scan_u128(w);
        const unsigned e0 = wave_incl_scan_u32((unsigned)e & 0xffffffu), e1 = wave_incl_scan_u32((unsigned)(e >> 24));
        if ((tid & (kWave - 1)) == kWave - 1) {
            sh_w[tid / kWave] = w;
            sh_e[tid / kWave] = (unsigned long long)e0 + ((unsigned long long)e1 << 24);
        }
        __syncthreads();
        if (tid == 0) {
            w = 0;
            e = 0;
#pragma unroll
            for (int i = 0; i < kLgWaves; ++i) {
                w += sh_w[i];
                e += sh_e[i];
            }
        }
    };
    u128 w;
    unsigned long long e;
    chunk_sums(c, w, e);
    unsigned long long* mine = slots + ((size_t)b * nchunks + c) * 6;
    if (tid == 0) {
        lg_publish(mine + 0, (unsigned)w, tag);
        lg_publish(mine + 1, (unsigned)(w >> 32), tag);
        lg_publish(mine + 2, (unsigned)(w >> 64), tag);
        lg_publish(mine + 3, (unsigned)(w >> 96), tag);
        lg_publish(mine + 4, (unsigned)e, tag);
        lg_publish(mine + 5, (unsigned)(e >> 32), tag);   // the plain sum of a chunk is below 2^41
    }
    // the words of the launch before are consumed: cleared, so that a captured call (same tags) can be replayed
    for (int i = c * kLgThreads + tid; i < (2 * k + 1) * npieces * 2; i += nchunks * kLgThreads) {
        const int j = i / (npieces * 2);
        const int row = j <= k ? trow(b, j, k) : drow(B, b, j - k - 1, k);
        words[(size_t)row * npieces * 2 + (i - j * npieces * 2)] = 0ull;
    }
    if (c != nchunks - 1) return;  // uniform over the workgroup

    // ---- the branch's last chunk collects ----
    if (tid == 0) {
        accept_len[b] = n;
        if (priv_len) priv_len[b] -= k - n;  // the rejected drafts leave the branch's KV cache
        sh_wsum[c] = w;
        sh_psum[c] = e;
        sh_missing = 0;
    }
    __syncthreads();
    for (int j = tid; j < c; j += kLgThreads) {
        const unsigned long long* en = slots + ((size_t)b * nchunks + j) * 6;
        unsigned long long v[6] = {};
        bool ok = false;
        for (int polls = 0; !ok && polls < kWaitPolls; ++polls) {
            ok = true;
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                v[i] = lg_peek(en + i);
                ok = ok && (unsigned)(v[i] >> 32) == tag;
            }
            if (!ok) __builtin_amdgcn_s_sleep(1);
        }
        if (!ok) sh_missing = 1;
        sh_wsum[j] = (u128)(unsigned)v[0] | ((u128)(unsigned)v[1] << 32) | ((u128)(unsigned)v[2] << 64) | ((u128)(unsigned)v[3] << 96);
        sh_psum[j] = ok ? (unsigned long long)(unsigned)v[4] | ((unsigned long long)(unsigned)v[5] << 32) : kLgNoSum;
    }
    __syncthreads();
    if (sh_missing) {  // uniform over the workgroup: the sums that have not come, from the logits
        for (int j = 0; j < c; ++j) {
            if (sh_psum[j] != kLgNoSum) continue;
            chunk_sums(j, w, e);
            __syncthreads();  // everybody has seen the mark of chunk j, thread 0 has read the wavefronts' parts
            if (tid == 0) {
                sh_wsum[j] = w;
                sh_psum[j] = e;
            }
        }
        __syncthreads();
    }
    // kLgMaxChunks = 2 * kLgThreads: every thread owns two consecutive chunk sums
    const int c0 = tid * 2;
    u128 w0 = 0, w1 = 0;
    unsigned long long p0 = 0, p1 = 0;
    if (c0 < nchunks) {
        w0 = sh_wsum[c0];
        p0 = sh_psum[c0];
    }
    if (c0 + 1 < nchunks) {
        w1 = sh_wsum[c0 + 1];
        p1 = sh_psum[c0 + 1];
    }
    u128 Z, excl = block_excl_scan_u128(w0 + w1, sh_w, Z);
    if (residual && Z == 0) {  // empty residual: sample the target row itself (uniform branch: n and Z are)
        residual = false;
        w0 = p0;
        w1 = p1;
        excl = block_excl_scan_u128(w0 + w1, sh_w, Z);
    }
    if (Z == 0) {  // a row without any weight (all logits -inf, or +inf / NaN among them): no token; uniform
        if (tid == 0) next_token[b] = -1;
        return;
    }
    unsigned m24 = (unsigned)(u_last * 16777216.0f);
    m24 = m24 > 16777215u ? 16777215u : m24;  // u must be < 1; keeps T < Z regardless
    const u128 T = ((u128)m24 * Z) >> 24;
    if (excl <= T && T < excl + w0 + w1) {  // exactly one thread: T < Z and Z > 0
        const bool second = !(T < excl + w0);
        sh_chunk = c0 + (second ? 1 : 0);
        sh_base = second ? excl + w0 : excl;
    }
    __syncthreads();
    const int cc = sh_chunk;
    const u128 base = sh_base;
    const void* zd_row2 = residual ? zd_row : zt_row;
    const RowStat sq2 = residual ? sq : sp;
    const int lo = cc * kLgChunk + tid * 8;
    lg_weights8<BF16>(zt_row, zd_row2, lo, V, inv_temp, residual, sp, sq2, W, Ep);
    U96 sum = W[0];
#pragma unroll
    for (int i = 1; i < 8; ++i) sum = add_96(sum, W[i]);
    const u128 local = widen(sum);
    u128 total;
    const u128 run = base + block_excl_scan_u128(local, sh_w, total);
    if (run <= T && T < run + local) {  // exactly one thread
        // its first token whose inclusive prefix exceeds T
        const u128 rest = T - run;  // below local
        const U96 t = {{(unsigned)rest, (unsigned)(rest >> 32), (unsigned)(rest >> 64)}};
        U96 pre = W[0];
        int passed = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (i > 0) pre = add_96(pre, W[i]);
            passed += widen(pre) > widen(t) ? 0 : 1;
        }
        const int tok = lo + passed;
        next_token[b] = tok;
    }
}


struct LgLayout {
    size_t off_psum, off_chunks, off_words, off_draft, total;
    size_t asked;  // what the workspace query answers, >= total
    int nchunks, npieces, iters;
};
// [row maxima][sums of the pieces][tagged words of the chunks: 6 per (branch, chunk)][tagged words of the pieces: 2 per (row, piece)]
// [weights of the drafted tokens: one per row]
static inline LgLayout lg_layout(int B, int k, int V) {
    LgLayout l;
    l.nchunks = (V + kLgChunk - 1) / kLgChunk;
    const size_t rows = (size_t)B * (2 * k + 1);
    // Loads a thread (a piece is that many times 2048 logits): of four, five and six what leaves the least to read to the fullest
    // unit, with a workgroup's fixed part counted as one load; eight where a row would have more than 64 pieces, or one grid (of
    // fewer than 2^32 threads) could not hold them.  With four throughout, the 2128 pieces of 112 rows x 152064 were 80 more than
    // are resident at once, and those ended 2.8 us after the others: 26.4 us, 25.2 with five.  544 x 151936 64.2 -> 58.9, 72 x 151936
    // 20.2 -> 19.5 (six), 75 x 50257 fp32 15.8 -> 15.3, 72 x 65537 17.0 -> 16.3; four stays where it is 55 x 72936 (15.1, five 15.7), 63 x
    // 49153 (15.5, 16.1).  Eight for one workgroup to a unit instead of two of four loses: 63 x 49153 17.2.
    size_t best = 0;
    l.iters = 8;
    for (int it = 4; it <= 6; ++it) {
        const size_t pieces = (V + it * kLgGroup - 1) / (it * kLgGroup);
        if (pieces > kLgMaxPieces || rows * pieces * kLgThreads > 0xffffffffu) continue;
        const size_t cost = (rows * pieces + kNumCU - 1) / kNumCU * (it + 1);
        if (best == 0 || cost < best) {
            best = cost;
            l.iters = it;
        }
    }
    l.npieces = (V + l.iters * kLgGroup - 1) / (l.iters * kLgGroup);
    // The query asks for the smallest pieces' words whichever are taken: by the pieces' number alone 14 branches would ask for less
    // than 13, and a workspace sized for the larger batch would be too small for the smaller one.
    const size_t smallest = (V + 4 * kLgGroup - 1) / (4 * kLgGroup);
    const size_t most = rows * smallest * kLgThreads > 0xffffffffu ? (size_t)l.npieces : smallest;
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    auto bytes = [&](size_t pieces) {
        l.off_psum = up(rows * sizeof(float));
        l.off_chunks = l.off_psum + up(rows * pieces * sizeof(unsigned long long));
        l.off_words = l.off_chunks + up((size_t)B * l.nchunks * 6 * sizeof(unsigned long long));
        l.off_draft = l.off_words + up(rows * pieces * 2 * sizeof(unsigned long long));
        return l.off_draft + up(rows * sizeof(unsigned));
    };
    l.asked = bytes(most);
    l.total = bytes(l.npieces);
    return l;
}
static inline bool lg_sizes_ok(int B, int k, int V) {
    if (!(B >= 1 && B <= 65535 && k >= 0 && k <= kLgMaxK && V >= 1 && V <= (1 << 20))) return false;
    // the documented limit: pieces of 16384 logits over all rows
    const long long pieces = (V + 16383) / 16384;
    return pieces * B * (2 * k + 1) <= 0x7fffffffLL;
}

template <bool BF16>
static int lg_launch(int B, int k, int V, const void* zt, const void* zd, float inv_temp, const int32_t* draft,
                     const float* u, int32_t* accept_len, int32_t* next_token, int32_t* priv_len, void* workspace,
                     hipStream_t s) {
    const LgLayout l = lg_layout(B, k, V);
    char* ws = static_cast<char*>(workspace);
    float* rmax = reinterpret_cast<float*>(ws);
    unsigned long long* psum = reinterpret_cast<unsigned long long*>(ws + l.off_psum);
    unsigned long long* chunks = reinterpret_cast<unsigned long long*>(ws + l.off_chunks);
    unsigned long long* words = reinterpret_cast<unsigned long long*>(ws + l.off_words);
    unsigned* draft_e = reinterpret_cast<unsigned*>(ws + l.off_draft);
    const unsigned tag_s = next_word_tag(), tag_c = next_word_tag();
    const long long nslots = (long long)B * l.nchunks * 6;
    const dim3 sgrid((unsigned)((long long)l.npieces * B * (2 * k + 1)));  // (piece, row) pairs, row-major
    const FastDiv d_pieces = fast_div(l.npieces), d_targets = fast_div(k + 1);
    auto stat = [&](auto kernel) {
        LOTTS_LAUNCH(kernel, sgrid, dim3(kLgThreads), s, B, k, V, l.npieces, tag_s, zt, zd, inv_temp, words, rmax, psum, chunks, nslots, draft,
                     draft_e, d_pieces, d_targets);
    };
    switch (l.iters) {
        case 4: stat(lg_stat_kernel<BF16, 4>); break;
        case 5: stat(lg_stat_kernel<BF16, 5>); break;
        case 6: stat(lg_stat_kernel<BF16, 6>); break;
        default: stat(lg_stat_kernel<BF16, 8>); break;
    }
    const int rc = check_launch();
    if (rc != LOTTS_OK) return rc;
    int lg = 6;  // lanes that add up a row's pieces: not more than there are pieces, all rows at once if they fit
    while (lg > 0 && (((2 * k + 1) << lg) > kLgThreads || (1 << lg) >= 2 * l.npieces)) --lg;
    LOTTS_LAUNCH((lg_scan_pick_kernel<BF16>), dim3(l.nchunks, B), dim3(kLgThreads), s, B, k, V, l.nchunks, l.npieces, lg, tag_c, zt,
                 zd, inv_temp, draft_e, u, rmax, psum, accept_len, words, chunks, next_token, priv_len);
    return check_launch();
}

}  // namespace lotts

extern "C" size_t spec_accept_logits_workspace_bytes(int32_t B, int32_t k, int32_t V) {
    if (!lotts::lg_sizes_ok(B, k, V)) return 0;
    return lotts::lg_layout(B, k, V).asked;
}

extern "C" int spec_accept_logits(int32_t B, int32_t k, int32_t V, const void* target_logits, const void* draft_logits,
                                  int32_t logit_dtype, float inv_temperature, const int32_t* draft, const float* u,
                                  int32_t* accept_len, int32_t* next_token, int32_t* priv_len, void* workspace,
                                  size_t workspace_bytes, void* stream) {
    using namespace lotts;
    if (!lg_sizes_ok(B, k, V)) return LOTTS_ERR_SHAPE;
    if (logit_dtype != LOTTS_F32 && logit_dtype != LOTTS_BF16) return LOTTS_ERR_DTYPE;
    if (!(inv_temperature > 0.0f) || inv_temperature > 3.0e38f) return LOTTS_ERR_SHAPE;
    if (!target_logits || !u || !accept_len || !next_token || !workspace) return LOTTS_ERR_NULL;
    if (k > 0 && (!draft_logits || !draft)) return LOTTS_ERR_NULL;
    if (workspace_bytes < lg_layout(B, k, V).total) return LOTTS_ERR_WORKSPACE;
    if (((uintptr_t)workspace & 15) != 0) return LOTTS_ERR_SHAPE;
    const bool bf16 = logit_dtype == LOTTS_BF16;
    const uintptr_t es = bf16 ? 2 : 4;
    if (((uintptr_t)target_logits | (uintptr_t)draft_logits) & (es - 1)) return LOTTS_ERR_SHAPE;
    hipStream_t s = (hipStream_t)stream;
    if (bf16)
        return lg_launch<true>(B, k, V, target_logits, draft_logits, inv_temperature, draft, u, accept_len, next_token, priv_len,
                               workspace, s);
    return lg_launch<false>(B, k, V, target_logits, draft_logits, inv_temperature, draft, u, accept_len, next_token, priv_len,
                            workspace, s);
}
