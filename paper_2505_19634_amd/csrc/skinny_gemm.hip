// skinny_gemm: Y[M][N] = X[M][K] W[N][K]^T for the B * (k + 1) new tokens of a verify forward (M up to
// 256) against one weight matrix (paper Section 3.1: the step is bound by loading the weights; Appendix:
// 64 GB of weights for the 32B model).  bf16 in, fp32 accumulate on the matrix cores, bf16 out.
// HBM-bound on streaming W once: 2 * M flop per weight byte is far below the MFMA balance.
//
//   skinny_gemm_stream_kernel<MT, RT, WAVES, KG>  grid (blocks of weight rows, K splits).  A workgroup walks its K range
//       in steps of half a chunk (64 k); W and X both go from global memory straight into LDS stages, with no registers
//       in between; Y^T[n][m] accumulates in registers over the whole K range.  Three forms: 256 weight rows (eight
//       wavefronts side by side), 128 (four) and 64 (two row wavefronts x two groups that share every stage and take half
//       of its k each; their accumulators are added up through LDS at the end).  PARTS: 128 weight rows and half of the tokens.
//   skinny_gemm_reduce_kernel  only when K is split across workgroups (few weight rows): sums the fp32
//       partials in a fixed order and converts.
//   skinny_gemm_direct_kernel<RN, TT, WAVES, UB>  small matrices: a workgroup owns 16 * RN weight rows and 16 * TT tokens for
//       the WHOLE K range, its wavefronts a share of K each; no partials, no second launch.
// skinny_gemm_append, for the QKV projection, also puts its K and V columns into the branches' caches: the kernel that writes Y (the
// direct or the reduce kernel) stores them twice.
#include <algorithm>

#include "lotts_common.h"

namespace lotts {

typedef __bf16 g_bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 g_bf16x4 __attribute__((ext_vector_type(4)));
typedef float g_f32x16 __attribute__((ext_vector_type(16)));
typedef float g_f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned g_u32x4 __attribute__((ext_vector_type(4)));

constexpr int kGemmRows = 32;    // weight rows per wavefront = M of the MFMA
constexpr int kGemmChunk = 128;  // K elements per chunk
constexpr int kGemmMaxM = 256;
constexpr int kGemmMaxSplit = 32;
constexpr int kGemmTileFloats = 32 * 32;  // one accumulator tile: 32 weight rows x 32 tokens
// W row strides (elements) at which every row of a step starts in the same few memory channels: with all blocks at the same k
// they queue there.  Starting the blocks at different steps: 152064 x 2048 at 3 / 40 / 192 tokens 127 / 139 / 176 us -> 103 / 115 /
// 162; 28672 x 4096 49.5 / 48.9 / 65.3 -> 37.5 / 37.9 / 62.7; 22016 x 2048 19.3 / 20.4 / 31.4 -> 17.4 / 18.7 / 31.7.  At other strides
// it gives nothing and X is shared worse (55296 x 5120 87.1 / 128 -> 88.9 / 131 us at 40 / 192 tokens; 33280 x 3072 level).
constexpr int kStaggerStride = 2048;
// Bytes of X from which the workgroups of an XCD are given a run of the K splits instead of every eighth block of all of them, so that its
// 4 MB of L2 see only their share of X.  Staggered blocks walk that share at different places: 8192 x 28672 at 80 / 96 / 128 / 192 tokens
// 93.6 / 103 / 129 / 166 us, dealt by runs 93.8 / 92 / 95 / 115; below the line 4096 x 14336 at 96 tokens 30.8 / 32.0.  Unstaggered blocks pass
// X in step: dealt by runs, all of an XCD are at the same lines at once (7168 x 5120 at 192 tokens 28.7 -> 32.1, 5120 x 27648 level), so
// they stay as they were -- but for two token parts, which have twice the workgroups at X: 1024 x 18944 at 174 tokens 22.7 -> 20.8, 2048 x
// 28672 at 230 52.7 -> 47.7, while 920 x 10240 at 218 tokens (4.5 MB) 17.3 -> 18.9.
constexpr long long kXcdTokens = 5 << 20;
constexpr int kPartsMaxK = 12288;         // two token parts from 129 tokens up to this K, from 161 beyond
static inline int tokens_in_one_part(int K) { return K <= kPartsMaxK ? 128 : 160; }
constexpr int kGemmOutRow = 80;           // bytes per token row of a 32 x 32 bf16 tile on its way out through LDS (64 + pad)

struct GemmParams {  // (in the order in which the kernels come to need it)
    const __bf16 *X, *W;
    long long ldx, ldw;
    int M, N, K;
    int tokens;  // direct form, and stream forms with two token parts: tokens a workgroup owns
    int ksplit;
    int rows;     // weight rows a wavefront owns: 32, or fewer (a multiple of 4) when that fills the chip better
    FastDiv d_ksplit;           // by ksplit
    FastDiv d_nblocks;          // by nblocks
    FastDiv d_steps[2];         // by the half-chunk steps of a K split: all splits have one of two numbers of them, 2 apart
    int stagger;                // stream forms: blocks start their K loop at different steps
    int nblocks;                // blocks of weight rows
    short items;                // blocks x K splits
    bool by_xcd;                // each XCD takes a run of them
    unsigned char parts;        // token parts (1 or 2)
    unsigned char roww, rt, tt; // for the reduce kernel: row wavefronts, row / token tiles per wavefront
    __bf16* Y;
    long long ldy;
    float* part;  // fp32 partials when ksplit > 1: [ksplit][token part][block of weight rows][row wavefront][tile][quad][lane] float4
};

// Where the K and V columns of a QKV projection go beside Y: token m = b * R + r of branch b to position len[b] - R + r of its caches.
// A launch of its own for these few KB is all fixed cost (4.3 us between two launches of a graph); the threads that hold the columns
// store them a second time for next to nothing: a 36-layer step of 8 branches x 5 tokens 2534 -> 2426 us, 3 us a layer.
struct GemmAppend {
    __bf16 *Kpriv, *Vpriv;
    const int32_t* len;
    long long sb, sh, st;  // strides in elements
    int n_new, D, Hkv, R, Lmax;  // the first of the K columns
    FastDiv d_R, d_D;
};

struct GemmAppendParams : GemmParams {
    GemmAppend a;
};
template <typename P>
constexpr bool kAppends = std::is_same<P, GemmAppendParams>::value;

// The position of token m in its branch's caches, negative if there is none.  The epilogues read it ahead of the sums that they wait for.
__device__ __forceinline__ int append_position(const GemmAppend& a, int m) {
    const int b = quot(m, a.d_R), t = a.len[b] - a.R + (m - b * a.R);
    return t < a.Lmax ? t : -1;
}
// Columns n .. n + 3 of token m; D a multiple of 8 keeps them in one head.
__device__ __forceinline__ void append_store(const GemmAppend& a, int m, int t, int n, g_bf16x4 v) {
    if (n < a.n_new || t < 0) return;
    const int head = quot(n - a.n_new, a.d_D), d = n - a.n_new - head * a.D;
    const bool k = head < a.Hkv;
    __bf16* row = (k ? a.Kpriv : a.Vpriv) + quot(m, a.d_R) * a.sb + (k ? head : head - a.Hkv) * a.sh + t * a.st + d;
    *reinterpret_cast<g_bf16x4*>(row) = v;
}

enum GemmForm { kStream256, kStream128, kStream64, kDirect };

struct GemmPlan {
    GemmForm form;
    int mt, rt;            // stream forms: token tiles of 32; row tiles per wavefront (2: pairs split the token tiles)
    int rows, roww;        // weight rows per wavefront; wavefronts side by side over the rows
    int nblocks, ksplit, parts;
    int rn, tt, nby;       // direct: 16-row and 16-token tiles per workgroup, workgroups over the tokens
};

// Largest number of K splits that keeps the launch at or below one workgroup per compute unit (a count just above is the
// worst choice: a few units run two and everybody waits for them), with at least 4 chunks per workgroup.
static inline int plan_ksplit(int nblocks, int chunks) {
    int ks = kNumCU / nblocks;
    const int max_ks = chunks / 4 > 0 ? chunks / 4 : 1;
    if (ks > max_ks) ks = max_ks;
    if (ks > kGemmMaxSplit) ks = kGemmMaxSplit;
    return ks < 1 ? 1 : ks;
}

// Fewest weight rows per wavefront (20 .. 32) that still give at most one workgroup per unit: up to 96 tokens the launch
// is bound by how fast each unit takes in its share of W and X, not by the padded MFMA rows.  Measured at 40 tokens, before
// the staggered starts: 22016 x 2048 in 230 workgroups of 96 rows 21.6 us, in 172 of 128 rows 22.2; 33280 x 3072 in 208 of 160 rows 41.7 us, in
// 130 of 256 48.9.
static inline int plan_rows(int N, int roww, int mt) {
    if (mt > 3) return kGemmRows;
    for (int rows = 20; rows < kGemmRows; rows += 4)
        if ((N + roww * rows - 1) / (roww * rows) <= kNumCU) return rows;
    return kGemmRows;
}

// Direct form: wavefronts of a workgroup, and 32-wide k steps of a batch of loads, by weight and token tiles (of 16).
static inline int direct_waves(int rn) { return rn == 4 ? 4 : 8; }
static inline int direct_batch(int rn, int tt) { return rn == 4 ? 2 : (tt == 1 ? 8 : 4); }

// Direct form: the tile that leaves the fewest bytes (its weight rows plus its tokens, over the whole K) to a workgroup with at most one
// workgroup per unit.  Tokens are dealt in even shares: 40 tokens in two workgroups are 20 and 20, not 32 and 8 (60 sizes whose tile
// or shares that changes: 5 % faster; but 6784 .. 7424 x 768 at 33 .. 36 tokens, in tiles of 64 rows then, 7.5 -> 8.0 us).  Returns those
// KB, with a wavefront's share of K in whole batches, or 0 if no tile fits; `filled`: the fewest KB with tiles full of tokens.
static inline double plan_direct(int M, int N, int K, GemmPlan* pl, double* filled) {
    static const int tiles[][2] = {{1, 1}, {1, 2}, {2, 1}, {2, 2}, {2, 3}, {4, 2}, {4, 3}};
    double best = 0.0;
    *filled = 0.0;
    for (const auto& t : tiles) {
        const long long nx = (N + 16 * t[0] - 1) / (16 * t[0]), ny = (M + 16 * t[1] - 1) / (16 * t[1]);
        if (nx * ny > kNumCU) continue;
        const int unit = direct_waves(t[0]) * direct_batch(t[0], t[1]) * 32;
        const double row_kb = ((K + unit - 1) / unit * unit) * 2.0 / 1024.0;
        const double kb = (16.0 * t[0] + (double)((M + ny - 1) / ny)) * row_kb;
        const double kb_filled = (16.0 * t[0] + (16 * t[1] < M ? 16 * t[1] : M)) * row_kb;
        if (*filled == 0.0 || kb_filled < *filled) *filled = kb_filled;
        if (best == 0.0 || kb < best) {
            best = kb;
            pl->rn = t[0]; pl->tt = t[1]; pl->nblocks = (int)nx; pl->nby = (int)ny;
        }
    }
    return best;
}

// Which form, and how it is cut.  Measured on 16 matrices between 1536 x 1536 and 152064 x 5120 at 1 .. 256 tokens, calls
// back to back over rotated weights, reduce launch included.
//   Direct, up to K = 4096 and 8192 rows: 3.4 us + 0.022 us per KB of a workgroup's W and X (whole batches of loads) + 0.14 us per
//     MB of W, against 7 us + 0.125 us per MB of W + 7e-6 us per token and (N + K) of the split stream forms; both fitted to 1188
//     sizes (1536 .. 14336 rows, K 512 .. 4096, 1 .. 192 tokens) with tiles full of tokens, where the choice costs 0.4 % over the better
//     form: 2560 x 2048 at 1 / 40 tokens 5.1 / 7.6 us against 7.9 / 9.2; 4736 x 1280 at 24 tokens 12.4 against 9.7; 6144
//     x 4096 at 2 tokens 17.7 against 13.2.  Even shares are fewer KB, but not all of what is counted less is time saved: where only they
//     put the direct form ahead, 0.034 us per KB + 0.15 us per MB of W have to stay below 6.7 us (6.3 with 64 weight rows to a
//     workgroup) + 10e-6 us per token and (N + K), fitted to 492 such sizes: always direct is 5.3 % over the better form there (3968 x
//     2176 at 168 tokens 20.0 us, streamed 17.3), never direct 2.5 % (2176 x 1408 at 66 tokens 8.7 us, streamed 10.1), so 0.2 %, and 0.2 ..
//     0.5 % on 430 sizes beside them.  (Calls that are not captured have one launch less to make by it, too: 3328 x 1536 and 1536 x 3072
//     at 36 tokens, level in a graph.)
//     With more rows only the tile of 64 rows is left, four wavefronts with many small batches: 11904 x 1280 at 48 tokens 16.5 us
//     against 13.2.  Beyond K = 4096 the wavefronts wait for their loads in batches: 5120 x 5120 at 1 token 19.8 us against 13.8.
//   256-row stream form: more than 256 blocks of 128 rows; an X chunk in LDS serves the most rows.  55296 x 5120 at 64
//     tokens 92 us, 128-row form 104.
//   Two token parts, N <= 4608 and more than 128 tokens: blocks of 128 rows x half of the tokens instead of 64 x all, as many K splits.
//     A unit takes in W and X at some 50 KB/us together, and 128 + M / 2 rows are fewer than 64 + M; the parts of a block lie on one
//     XCD, side by side, and W comes from HBM once.  2048 x 11008 at 144 / 192 / 256 tokens 22.8 / 24.0 / 27.4 -> 21.5 / 22.7 / 24.8 us; 4608 x
//     4480 22.4 / 25.6 / 28.6 -> 20.7 / 22.2 / 24.8; 50 sizes of K > 4096 17 % faster.  With a K beyond 12288 and up to 160 tokens level or
//     slower (3584 x 18944 at 144 tokens 46.7 -> 48.0), with up to 128 tokens too (3264 x 14336 at 123 31.5 -> 36.7).  The same for more rows, 256 x
//     half of the tokens without a split, loses (22016 x 2048 at 160 / 192 tokens 27.5 / 29.6 -> 29.9 / 30.6).  Beside it the direct form stays
//     while 0.03 us per KB are below 6.75 us + 4e-6 us per token and (N + K): fitted to 402 sizes (32 .. 4608 rows, K 1024 .. 4096), 0.16 %
//     over the better form (always direct 9.4 %, never 24 %; a line of 4.75 us + 0.1 us per MB of W + 6.5e-6 us, from fewer sizes and none
//     below 600 rows, 1.2 %: 200 x 2176 at 146 tokens 7.4 us direct, streamed 9.9).  2184 x 2304 at 245 tokens 18.4 -> 16.0 us, 1536 x 4096 at
//     244 18.4 -> 14.5, 2560 x 2048 at 150 / 192 / 240 14.2 / 14.6 / 16.8 -> 12.9 / 14.0 / 15.9.
//   128-row form below that, 64-row form when it would have to be split more than sevenfold (N <= 4608): the fewer splits,
//     the fewer fp32 partials, but the more often a unit reads X.  2048 x 11008 at 40 / 192 tokens in 64-row blocks x 8
//     splits 14.8 / 24.3 us, 128 x 16 17.1 / 26.5; 5120 x 5120 at 64 / 192 tokens 128 x 6 17.9 / 26.0, 64 x 3 17.4 / 28.6; 6144 x 6144
//     21.5 / 31.0 against 23.4 / 38.1.
static inline GemmPlan plan_gemm(int M, int N, int K, bool may_be_direct = true) {
    GemmPlan pl = {};
    const int chunks = K / kGemmChunk;
    pl.mt = (M + 31) / 32;
    // An even number of token tiles from 4 on: pairs of wavefronts own two row tiles together and half of the token tiles each.
    pl.rt = pl.mt >= 4 && pl.mt % 2 == 0 ? 2 : 1;
    pl.ksplit = pl.parts = 1;
    const int nb128 = (N + 127) / 128, ks_parts = plan_ksplit(2 * nb128, chunks);
    const bool parts = nb128 <= 36 && M > tokens_in_one_part(K) && ks_parts > 1;
    if (may_be_direct && K <= 4096 && N <= 8192) {
        double filled;
        const double kb = plan_direct(M, N, K, &pl, &filled), mb = 2e-6 * N * K, tokens = 1e-6 * M * (N + K);
        auto ahead = [&](double k) { return 3.4 + 0.022 * k + 0.14 * mb < 7.0 + 0.125 * mb + 7.0 * tokens; };
        if (kb > 0.0 && (parts ? 0.03 * kb < 6.75 + 4.0 * tokens
                               : ahead(filled) || (ahead(kb) && 0.034 * kb + 0.15 * mb < (pl.rn == 4 ? 6.3 : 6.7) + 10.0 * tokens))) {
            pl.form = kDirect;
            return pl;
        }
    }
    if (nb128 > kNumCU) {
        pl.form = kStream256;
        pl.roww = 8;
        pl.rows = plan_rows(N, 8, pl.mt);
        const int nb32 = (N + 255) / 256, nb28 = (N + 223) / 224;
        // several rounds of workgroups: 28 rows instead of 32 where that fills the last round visibly better
        auto fill = [](int wgs) { return (double)wgs / (double)(((wgs + kNumCU - 1) / kNumCU) * kNumCU); };
        if (pl.mt <= 3 && nb32 > kNumCU && fill(nb28) > fill(nb32) + 0.03) pl.rows = 28;
    } else if (nb128 > 36) {
        pl.form = kStream128;
        pl.roww = 4;
        pl.ksplit = plan_ksplit(nb128, chunks);
        pl.rows = pl.ksplit == 1 ? plan_rows(N, 4, pl.mt) : kGemmRows;
    } else if (parts) {
        pl.form = kStream128;
        pl.roww = 4;
        pl.rows = kGemmRows;
        pl.parts = 2;
        pl.ksplit = ks_parts;
        pl.mt = ((M + 1) / 2 + 31) / 32;
        pl.rt = pl.mt == 4 ? 2 : 1;
    } else {
        pl.form = kStream64;
        pl.roww = 2;
        pl.rows = kGemmRows;
        pl.ksplit = plan_ksplit((N + 63) / 64, chunks);
    }
    pl.nblocks = (N + pl.roww * pl.rows - 1) / (pl.roww * pl.rows);
    return pl;
}

// Workspace of a plan: the fp32 partials of its K splits, 256 bytes at least.
static inline size_t plan_bytes(const GemmPlan& pl) {
    const size_t bytes = pl.ksplit > 1 ? sizeof(float) * pl.ksplit * pl.parts * pl.nblocks * pl.roww * pl.mt * kGemmTileFloats : 0;
    return bytes < 256 ? 256 : bytes;
}

// The streaming kernel.  WAVES = ROWW * KG wavefronts, 32 * ROWW weight rows per workgroup: a row wavefront owns one MFMA row
// tile of 32 weight rows and all M tokens -- or, for an even number of token tiles from 4 on (97..128, 161..192,
// 225..256 tokens), two neighbouring ones own two row tiles together and half of the token tiles each: a k step then
// reads 2 + MT / 2 fragments for MT MFMAs instead of 1 + MT, and LDS reads are what bounds the loop at these token counts
// (measured 1..11 % faster on the 32B-shaped layers).
// KG = 2: two groups of row wavefronts share every stage; group g multiplies k steps 2 g and 2 g + 1 of its four.  That puts two
// wavefronts of a 64-row block on every row tile without more LDS or more transfers, so a matrix of few rows makes twice the
// workgroups of the 128-row form from half the K splits.
// Neither operand passes through registers: global-to-LDS loads (16 bytes per lane, landing at a wavefront-uniform
// LDS base + 16 * lane) fill stages of half a chunk (64 k) --
//   X: XS stages per workgroup, one multiplied while the others are filled, one barrier per stage; rows of 8 tokens that
//      are all past the last one stay out (an MFMA column is one token: what their LDS holds reaches no output; with 40 tokens
//      24 of 64 rows, 22016 x 2048 20.6 -> 19.7 us, 55296 x 5120 at 64 tokens 91 -> 89);
//   W: XS + 1 stages per row wavefront (32 rows x 64 k, 4 KB): one multiplied, XS on their way; non-temporal; private to the wavefront, or to those that share its rows
//      (pair and groups: each fills its part; the step barrier that publishes X publishes these too).
// A stage keeps rows of 128 bytes back to back (a load instruction fills 8 whole rows), so the 16-byte pieces of a
// row are stored permuted -- piece p of row r at slot p ^ ((r >> 1) & 7) -- which spreads the 16 lanes of a
// fragment read over all 64 banks without padding.  With no staging registers there is room for two fragment sets
// beside the accumulators of 256 tokens: the LDS reads of k step s + 1 run under the MFMAs of step s.
//
// The loads are written out as instructions.  Through the compiler's builtin every later LDS access of the kernel
// would wait for ALL loads in flight (the compiler cannot tell which LDS bytes a transfer writes), which stalls the
// transfers that are meant to stay in flight; and without a "memory" clobber, with which the same wait comes
// back: the barrier statements of the step loop, which have it, fence every read of a stage against the transfer
// that refills it, and volatile statements keep their order among themselves.  M0 carries the LDS base.  Since the
// compiler does not know of the loads, the waits are written out too: before the barrier of a step, vmcnt(n) -- the
// step's X transfers have landed, and with them the older W stage; only the n transfers issued after them (stages of later
// steps) may still be in flight -- counted down to vmcnt(0) in the last step.
// XS = 2 for the 128- and 256-row forms (with 3 or 4 they are level within 1 us: one workgroup has 32 KB of W in flight as it is);
// XS = 4 for the 64-row form up to 96 tokens, whose two stages of W are half of that: 2048 x 11008 at 3 / 40 / 96 tokens 15.4 /
// 15.9 / 19.3 -> 13.7 / 14.8 / 18.5 us; beyond, X stages of 16 KB and more crowd the LDS and it loses (192 tokens 23.9 -> 24.4).
//
// The way out.  Accumulator lanes hold one token and scattered weight rows, so stores straight from them write 16 bytes
// per row of Y (32 of a row of fp32 partials), and the launch ended on them: 2560 x 2048 at 192 tokens took 18.6 us for 8
// steps.  Partials now go out as they lie in the registers, 1 KB per store, and the reduce kernel reads them back the same
// way; Y tiles turn through LDS into 64-byte row pieces.  With the forms above (before: 128 / 256 rows only), reduce launch
// included, 40 / 192 tokens: 2048 x 11008 20.2 / 34.5 -> 16.8 / 24.5 us; 7168 x 5120 21.5 / 40 -> 20.0 / 29.7; 22016 x 2048
// 25.4 / 41.5 -> 21.6 / 31.0 (with what came since 14.8 / 24.3, 19.2 / 29.9, 18.8 / 31.7).
template <int MT, int RT, int WAVES, int KG, int XS, bool PARTS = false>
__global__ __launch_bounds__(WAVES * kWave, 2) void skinny_gemm_stream_kernel(const GemmParams p) {
    static_assert(RT == 1 || (RT == 2 && MT % 2 == 0), "a pair of wavefronts splits the token tiles evenly");
    constexpr int WS = XS + 1;        // W stages
    constexpr int ROWW = WAVES / KG;  // wavefronts side by side over the weight rows
    constexpr int WI = 4 / KG;        // W transfers per wavefront and stage
    constexpr int TT = MT / RT;  // token tiles per wavefront
    constexpr int XROWS = 32 * MT;
    constexpr int XINSTR = XROWS / 8;
    // X transfers per wavefront and stage: the most, and the fewest (of 8 token rows each; rows past the last token stay out)
    constexpr int XI = (XINSTR + WAVES - 1) / WAVES, XMIN = (XINSTR - 3) / WAVES;
    constexpr int kStageRow = 128;
    constexpr int XSTAGE = XROWS * kStageRow, WSTAGE = 32 * kStageRow;
    constexpr int TILES = RT * TT;   // accumulator tiles per wavefront
    constexpr int TILE_Q = kGemmTileFloats / 4;
    constexpr int STAGES = XS * XSTAGE + ROWW * WS * WSTAGE, PARK = ROWW * TILES * (KG - 1) * TILE_Q * 16;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[STAGES > PARK ? STAGES : PARK];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid & (kWave - 1);
    const int kgrp = KG == 1 ? 0 : wave / ROWW, wr = KG == 1 ? wave : wave % ROWW;
    const int ln = lane & 31, hh = lane >> 5;
    // RT = 1: row wavefront w owns row tile w and all tokens.  RT = 2: row wavefronts 2j and 2j + 1 own row tiles 2j and
    // 2j + 1 together, each half of the token tiles, and share the W stages of their 64 rows.
    const int grp = RT == 1 ? wr : wr >> 1, th = RT == 1 ? 0 : wr & 1;
    int block = blockIdx.x, split = blockIdx.y, part = 0;
    if (PARTS || p.by_xcd) {  // workgroups of one XCD, in the order in which they start: both parts of an item, then its next one
        const int xcd = blockIdx.x % kNumXCD, i = (int)blockIdx.x / (PARTS ? 2 * kNumXCD : kNumXCD);
        part = PARTS ? (int)(blockIdx.x / kNumXCD) & 1 : 0;
        int item = i * kNumXCD + xcd, end = p.items;  // of the list [split][block]: every eighth one,
        if (p.by_xcd) {                               // or a run of it
            const int each = p.items / kNumXCD, more = p.items % kNumXCD, first = xcd * each + min(xcd, more);
            item = first + i;
            end = first + each + (xcd < more);
        }
        if (item >= end) return;
        split = quot(item, p.d_nblocks);
        block = item - split * p.nblocks;
    }
    const int M = PARTS ? p.tokens : p.M, m0 = part ? p.M - p.tokens : 0;  // the second part starts early enough to be as long as the first
    const int n0 = block * (p.rows * ROWW) + grp * (p.rows * RT);  // pairs always own 2 x 32 rows
    const int chunks = p.K / kGemmChunk;
    // (Through host-made divisors: the run-time divisions here, two of them of 64 bits, stood 0.5 us in front of the first load.)
    const int c_lo = quot(split * chunks, p.d_ksplit);
    const int c_hi = quot((split + 1) * chunks, p.d_ksplit);
    const int G = 2 * (c_hi - c_lo);  // half-chunk steps
    // Staggered start: block x begins 5 x steps into its K range and wraps around; the pointers go back once, at that step.  (A
    // select of the offset in every transfer instead cost 2 % of 55296 x 5120.)
    int first = 0;
    if (p.stagger && G > 0) {
        const FastDiv d = G == 2 * quot(chunks, p.d_ksplit) ? p.d_steps[0] : p.d_steps[1];
        const int turn = block * 5, at = turn + quot(turn, d);
        first = at - quot(at, d) * G;
    }
    const int wrap = first > 0 ? G - first : -1;  // the step that is back at the start of the range
    unsigned char* xs = lds;
    unsigned char* wsl = lds + XS * XSTAGE + grp * (WS * RT * WSTAGE);

    // Per-lane source addresses of the transfers, for step 0: 64-bit, so that neither
    // operand is limited to 4 GB.  lane -> (row of the instruction's 8, slot); the piece fetched for a slot is
    // slot ^ swizzle(row).
    const int l_row = lane >> 3, l_slot = lane & 7;
    const __bf16* x_src[XI];
    const __bf16* w_src[WI];
#pragma unroll
    for (int i = 0; i < XI; ++i) {
        const int r = (wave + i * WAVES) * 8 + l_row;
        const int m = r < M ? r : M - 1;
        x_src[i] = p.X + (long long)(m0 + m) * p.ldx + (long long)c_lo * kGemmChunk + first * 64 + (l_slot ^ ((r >> 1) & 7)) * 8;
    }
#pragma unroll
    for (int i = 0; i < WI; ++i) {
        const int r = th * 32 + (kgrp * WI + i) * 8 + l_row;  // of a pair, each wavefront brings in 32 of the 64 rows
        int n = n0 + (RT == 1 && r >= p.rows ? p.rows - 1 : r);  // a short tile re-reads its last row
        n = n < p.N ? n : p.N - 1;  // rows past the end re-read the last row; never stored
        w_src[i] = p.W + (long long)n * p.ldw + (long long)c_lo * kGemmChunk + first * 64 + (l_slot ^ ((r >> 1) & 7)) * 8;
    }
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"  // M0 is on the clobber list on purpose
    auto fetch_x = [&](int g) {
        if (g == wrap) {
#pragma unroll
            for (int i = 0; i < XI; ++i) x_src[i] -= (long long)G * 64;
        }
        unsigned char* stage = xs + (g % XS) * XSTAGE;
#pragma unroll
        for (int i = 0; i < XI; ++i) {
            const int j = wave + i * WAVES;
            if ((i + 1) * WAVES <= XINSTR - 3 || j * 8 < M) {  // (all but the last 3 are rows of tokens that exist)
                const unsigned lds_base = __builtin_amdgcn_readfirstlane(
                    (unsigned)(uintptr_t)(__attribute__((address_space(3))) void*)(stage + j * 8 * kStageRow));
                asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                             :
                             : "v"(x_src[i] + (long long)g * 64), "s"(lds_base)
                             : "m0");
            }
        }
    };
    auto fetch_w = [&](int g) {
        if (g == wrap) {
#pragma unroll
            for (int i = 0; i < WI; ++i) w_src[i] -= (long long)G * 64;
        }
        unsigned char* stage = wsl + (g % WS) * (RT * WSTAGE) + th * WSTAGE;
#pragma unroll
        for (int i = 0; i < WI; ++i) {
            const unsigned lds_base = __builtin_amdgcn_readfirstlane(
                (unsigned)(uintptr_t)(__attribute__((address_space(3))) void*)(stage + (kgrp * WI + i) * 8 * kStageRow));
            if (PARTS)
                asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                             :
                             : "v"(w_src[i] + (long long)g * 64), "s"(lds_base)
                             : "m0");
            else
                asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt"
                             :
                             : "v"(w_src[i] + (long long)g * 64), "s"(lds_base)
                             : "m0");
        }
    };
#pragma clang diagnostic pop
    g_f32x16 acc[RT][TT];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int t = 0; t < TT; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[r][t][i] = 0.f;

    const int swz = (ln >> 1) & 7;
    auto multiply = [&](const unsigned char* xst, const unsigned char* wst) {
        g_bf16x8 fa[2][RT], fb[2][TT];
        auto frags = [&](int s, g_bf16x8 (&a)[RT], g_bf16x8 (&b)[TT]) {
#pragma unroll
            for (int r = 0; r < RT; ++r)
                a[r] = *reinterpret_cast<const g_bf16x8*>(wst + (r * 32 + ln) * kStageRow + (((2 * s + hh) ^ swz) * 16));
#pragma unroll
            for (int t = 0; t < TT; ++t)
                b[t] = *reinterpret_cast<const g_bf16x8*>(xst + ((th * TT + t) * 32 + ln) * kStageRow +
                                                          (((2 * s + hh) ^ swz) * 16));
        };
        frags(kgrp * WI, fa[0], fb[0]);
#pragma unroll
        for (int s = 0; s < WI; ++s) {
            if (s + 1 < WI) frags(kgrp * WI + s + 1, fa[(s + 1) & 1], fb[(s + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int t = 0; t < TT; ++t)
                    acc[r][t] =
                        __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[s & 1][r], fb[s & 1][t], acc[r][t], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (G > 0) fetch_w(0);
#pragma unroll
    for (int i = 0; i + 1 < XS; ++i) {
        if (i < G) fetch_x(i);
        if (i + 1 < G) fetch_w(i + 1);
    }
    // Arguments that are still on their way share the LDS reads' counter and come in any order: with one outstanding, every wait of
    // the loop for a fragment would be a wait for all of them (192 tokens x 22016 x 2048 29.4 -> 30.1 us, 256 36.5 -> 38.2).
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0) alone
    for (int g = 0; g < G; ++g) {
        // issued after step g's X: W of the steps up to g + XS - 1 and X of those up to g + XS - 2, as far as there are any
        if (g + XS - 1 < G)
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((XS - 1) * WI + (XS - 2) * XMIN) : "memory");
        else if (XS > 3 && g + 2 < G)
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * (WI + XMIN)) : "memory");
        else if (XS > 2 && g + 1 < G)
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(WI + XMIN) : "memory");
        else
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (g + XS - 1 < G) fetch_x(g + XS - 1);
        if (g + XS < G) fetch_w(g + XS);
        multiply(xs + (g % XS) * XSTAGE, wsl + (g % WS) * (RT * WSTAGE));
    }
    // KG = 2: the groups add up.  Group g finishes the tiles j with j % KG == g; each wavefront parks the others in LDS (the
    // stages are free: no transfer is in flight after the last step) and adds what its partner parked, groups in order.
    if (KG > 1) {
        __syncthreads();
        float4* park = reinterpret_cast<float4*>(lds);
#pragma unroll
        for (int j = 0; j < TILES; ++j) {
            const int dst = j % KG;
            if (dst != kgrp) {
                float4* slot = park + (size_t)((wr * TILES + j) * (KG - 1) + (kgrp < dst ? kgrp : kgrp - 1)) * TILE_Q + lane;
                const g_f32x16& a = acc[j / TT][j % TT];
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4)
                    slot[q4 * kWave] = make_float4(a[q4 * 4 + 0], a[q4 * 4 + 1], a[q4 * 4 + 2], a[q4 * 4 + 3]);
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < TILES; ++j) {
            const int dst = j % KG;
            if (dst == kgrp) {
                g_f32x16& a = acc[j / TT][j % TT];
                g_f32x16 sum;
#pragma unroll
                for (int i = 0; i < 16; ++i) sum[i] = 0.f;
#pragma unroll
                for (int g = 0; g < KG; ++g) {
                    if (g == dst) {
                        sum += a;
                    } else {
                        const float4* slot = park + (size_t)((wr * TILES + j) * (KG - 1) + (g < dst ? g : g - 1)) * TILE_Q + lane;
#pragma unroll
                        for (int q4 = 0; q4 < 4; ++q4) {
                            const float4 v = slot[q4 * kWave];
                            sum[q4 * 4 + 0] += v.x; sum[q4 * 4 + 1] += v.y; sum[q4 * 4 + 2] += v.z; sum[q4 * 4 + 3] += v.w;
                        }
                    }
                }
                a = sum;
            }
        }
    }
    // register i of accumulator (r, t) of this lane: output row m = (th * TT + t) * 32 + ln,
    // column n = n0 + r * 32 + (i / 4) * 8 + hh * 4 + i % 4
    if (PARTS || p.ksplit > 1) {
        float4* dst = reinterpret_cast<float4*>(p.part) +
                      ((long long)((split * (PARTS ? 2 : 1) + part) * p.nblocks + block) * ROWW + wr) * (TILES * TILE_Q) + lane;
#pragma unroll
        for (int j = 0; j < TILES; ++j) {
            if (KG > 1 && j % KG != kgrp) continue;
            if ((th * TT + j % TT) * 32 + ln >= M) continue;
            const g_f32x16& a = acc[j / TT][j % TT];
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                if (RT == 1 && q4 * 8 >= p.rows) continue;  // beyond a short tile
                dst[j * TILE_Q + q4 * kWave] = make_float4(a[q4 * 4 + 0], a[q4 * 4 + 1], a[q4 * 4 + 2], a[q4 * 4 + 3]);
            }
        }
        return;
    }
    // Y tiles turn through LDS, 32 tokens x 32 weight rows at a time, wavefront-private: a token's 64 bytes leave together
    __syncthreads();  // nobody reads a stage or a parked tile any more
    unsigned char* tr = lds + wave * (32 * kGemmOutRow);
#pragma unroll
    for (int j = 0; j < TILES; ++j) {
        if (KG > 1 && j % KG != kgrp) continue;
        const int m_base = (th * TT + j % TT) * 32;
        if (m_base >= M) continue;
        const g_f32x16& a = acc[j / TT][j % TT];
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            g_bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (__bf16)a[q4 * 4 + e];
            *reinterpret_cast<g_bf16x4*>(tr + ln * kGemmOutRow + (q4 * 8 + hh * 4) * 2) = o;
        }
        const int nc = (lane & 7) * 4, n = n0 + (j / TT) * 32 + nc;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ml = i * 8 + (lane >> 3);
            const g_bf16x4 o = *reinterpret_cast<const g_bf16x4*>(tr + ml * kGemmOutRow + nc * 2);
            if (m_base + ml < M && n < p.N && (RT > 1 || nc < p.rows))  // N a multiple of 8: 4 columns are in or out together
                *reinterpret_cast<g_bf16x4*>(p.Y + (long long)(m_base + ml) * p.ldy + n) = o;
        }
    }
}

// One workgroup per accumulator tile of 32 tokens x 32 weight rows: thread (quad, lane) adds up the tile's partials as the stream
// kernel's lanes left them, in split order (deterministic), and the bf16 tile turns through LDS into 64-byte row pieces of Y.
template <typename P>
__global__ __launch_bounds__(256) void skinny_gemm_reduce_kernel(const P p) {
    __shared__ __attribute__((aligned(16))) unsigned char tr[32 * kGemmOutRow];
    const int tiles = p.rt * p.tt;
    const int j = blockIdx.x % tiles, wb = blockIdx.x / tiles;
    const int wr = wb % p.roww, blocks = wb / p.roww;
    const int part = blocks >= p.nblocks, block = part ? blocks - p.nblocks : blocks;  // (two parts at most; a run-time division is 0.05 .. 0.1 us)
    const int M = p.parts > 1 ? p.tokens : p.M, m0 = part ? p.M - p.tokens : 0;
    const int grp = p.rt == 1 ? wr : wr >> 1, th = p.rt == 1 ? 0 : wr & 1;
    const int m_base = (th * p.tt + j % p.tt) * 32;
    const int n_base = block * (p.rows * p.roww) + grp * (p.rows * p.rt) + (j / p.tt) * 32;
    if (m_base >= M || n_base >= p.N) return;  // uniform over the workgroup
    const int q4 = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1), ln = lane & 31, hh = lane >> 5;
    const bool in = m_base + ln < M && (p.rt > 1 || q4 * 8 < p.rows);  // what the stream kernel has stored
    const int ml = threadIdx.x >> 3, nc = (threadIdx.x & 7) * 4, m = m0 + m_base + ml, n = n_base + nc;
    int t = -1;
    if constexpr (kAppends<P>)
        if (n_base + 32 > p.a.n_new) t = append_position(p.a, min(m, p.M - 1));
    const long long stride = (long long)p.nblocks * p.parts * p.roww * tiles * (kGemmTileFloats / 4);
    const float4* src = reinterpret_cast<const float4*>(p.part) + (long long)blockIdx.x * (kGemmTileFloats / 4) + threadIdx.x;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (in) {
        for (int k0 = 0; k0 < p.ksplit; k0 += 8) {  // eight loads in flight
            float4 v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (k0 + e < p.ksplit) v[e] = src[(k0 + e) * stride];
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (k0 + e < p.ksplit) {
                    s.x += v[e].x;
                    s.y += v[e].y;
                    s.z += v[e].z;
                    s.w += v[e].w;
                }
        }
    }
    g_bf16x4 o;
    o[0] = (__bf16)s.x;
    o[1] = (__bf16)s.y;
    o[2] = (__bf16)s.z;
    o[3] = (__bf16)s.w;
    *reinterpret_cast<g_bf16x4*>(tr + ln * kGemmOutRow + (q4 * 8 + hh * 4) * 2) = o;
    __syncthreads();
    if (m_base + ml < M && n < p.N && (p.rt > 1 || nc < p.rows)) {
        const g_bf16x4 y = *reinterpret_cast<const g_bf16x4*>(tr + ml * kGemmOutRow + nc * 2);
        *reinterpret_cast<g_bf16x4*>(p.Y + (long long)m * p.ldy + n) = y;
        if constexpr (kAppends<P>) append_store(p.a, m, t, n, y);
    }
}

// The direct form.  Small matrices are bound by fixed costs -- launch, first data, the exchange of partials -- so the whole K
// range stays in one workgroup and both operands go straight from memory into fragment registers: with 16x16x32 MFMA a load
// covers 64 contiguous bytes of 16 rows, and a wavefront's share of K at K = 2048 is one or two batches of UB steps with tiles of
// up to 32 rows (all of it in flight at once), eight batches with 64.  The wavefronts' sums meet in LDS, added in wavefront order.  W is non-temporal when a single
// workgroup column reads it (NT); with several over the tokens the later ones find it in the L2.
template <int RN, int TT, int WAVES, int UB, bool NT, typename P>
__global__ __launch_bounds__(WAVES * kWave) void skinny_gemm_direct_kernel(const P p) {
    constexpr int TILES = RN * TT, TURNS = (TILES + WAVES - 1) / WAVES, ROLL = kAppends<P> ? TURNS : 1;  // of the last loop
    __shared__ __attribute__((aligned(16))) float4 red[WAVES][TILES][kWave];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid & (kWave - 1);
    const int lr = lane & 15, kg = lane >> 4;
    const int n0 = blockIdx.x * (16 * RN), m0 = blockIdx.y * p.tokens, m_end = min(m0 + p.tokens, p.M);
    int to[TURNS];
    if constexpr (kAppends<P>) {
#pragma unroll
        for (int e = 0; e < TURNS; ++e) to[e] = -1;
        if (n0 + 16 * RN > p.a.n_new) {
#pragma unroll
            for (int e = 0; e < TURNS; ++e) to[e] = append_position(p.a, min(m0 + (wave + e * WAVES) % TT * 16 + lr, p.M - 1));
        }
    }
    const int S = p.K / 32;
    const int s_lo = (int)((long long)wave * S / WAVES), s_hi = (int)((long long)(wave + 1) * S / WAVES);
    const __bf16 *wp[RN], *xp[TT];
#pragma unroll
    for (int i = 0; i < RN; ++i) wp[i] = p.W + (long long)min(n0 + i * 16 + lr, p.N - 1) * p.ldw + kg * 8;
#pragma unroll
    for (int t = 0; t < TT; ++t) xp[t] = p.X + (long long)min(m0 + t * 16 + lr, m_end - 1) * p.ldx + kg * 8;
    g_f32x4 acc[RN][TT];
#pragma unroll
    for (int i = 0; i < RN; ++i)
#pragma unroll
        for (int t = 0; t < TT; ++t) acc[i][t] = g_f32x4{0.f, 0.f, 0.f, 0.f};
    union frag { g_u32x4 u; g_bf16x8 v; };
    struct buf { frag w[UB][RN], x[UB][TT]; };
    auto load = [&](int s0, buf& b) {
#pragma unroll
        for (int j = 0; j < UB; ++j) {
            const int s = min(s0 + j, s_hi - 1);
#pragma unroll
            for (int i = 0; i < RN; ++i) {
                const g_u32x4* a = reinterpret_cast<const g_u32x4*>(wp[i] + s * 32);
                b.w[j][i].u = NT ? __builtin_nontemporal_load(a) : *a;
            }
#pragma unroll
            for (int t = 0; t < TT; ++t) b.x[j][t].u = *reinterpret_cast<const g_u32x4*>(xp[t] + s * 32);
        }
    };
    auto mul = [&](int s0, buf& b) {
#pragma unroll
        for (int j = 0; j < UB; ++j) {
            if (s0 + j < s_hi) {
#pragma unroll
                for (int i = 0; i < RN; ++i)
#pragma unroll
                    for (int t = 0; t < TT; ++t)
                        acc[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b.w[j][i].v, b.x[j][t].v, acc[i][t], 0, 0, 0);
            }
        }
    };
    if (s_lo < s_hi) {  // with few chunks some wavefronts have no share
        buf A, B;
        load(s_lo, A);
        for (int s = s_lo; s < s_hi; s += 2 * UB) {
            if (s + UB < s_hi) load(s + UB, B);
            __builtin_amdgcn_sched_barrier(0);
            mul(s, A);
            if (s + 2 * UB < s_hi) load(s + 2 * UB, A);
            __builtin_amdgcn_sched_barrier(0);
            if (s + UB < s_hi) mul(s + UB, B);
        }
    }
#pragma unroll
    for (int i = 0; i < RN; ++i)
#pragma unroll
        for (int t = 0; t < TT; ++t) red[wave][i * TT + t][lane] = make_float4(acc[i][t][0], acc[i][t][1], acc[i][t][2], acc[i][t][3]);
    __syncthreads();
    // (Tiles by the thread's number, not by the wavefront's, which is in a scalar register from the start: with it the compiler laid the registers out
    // so that the second batch's addresses waited for the first batch's last loads, 2048 x 2048 at 192 tokens 12.6 -> 12.9 us, 2560 x 2048 at
    // 128 12.3 -> 12.6.  Unrolled where the append's positions are in registers.)
#pragma unroll ROLL
    for (int e = 0; e < TURNS; ++e) {
        const int at = tid + e * WAVES * kWave, tile = at / kWave, l = at % kWave;
        if (at >= TILES * kWave) break;
        float4 s = red[0][tile][l];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) {
            const float4 v = red[w][tile][l];
            s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
        }
        const int i = tile / TT, t = tile % TT;
        const int m = m0 + t * 16 + (l & 15), n = n0 + i * 16 + (l >> 4) * 4;
        if (m < m_end && n < p.N) {
            g_bf16x4 o;
            o[0] = (__bf16)s.x; o[1] = (__bf16)s.y; o[2] = (__bf16)s.z; o[3] = (__bf16)s.w;
            *reinterpret_cast<g_bf16x4*>(p.Y + (long long)m * p.ldy + n) = o;
            if constexpr (kAppends<P>) append_store(p.a, m, to[e], n, o);
        }
    }
}
static inline bool gemm_sizes_ok(int M, int N, int K) {
    return M >= 1 && M <= kGemmMaxM && N >= 8 && (N % 8) == 0 && K >= kGemmChunk && (K % kGemmChunk) == 0 &&
           (long long)M * N < (1LL << 40);
}

// XS stages of X up to 96 tokens, XSM beyond
template <int WAVES, int KG, int XS, int XSM>
static void launch_stream(int mt, dim3 grid, hipStream_t s, const GemmParams& p) {
    const dim3 block(WAVES * kWave);
    switch (mt) {
        case 1: LOTTS_LAUNCH((skinny_gemm_stream_kernel<1, 1, WAVES, KG, XS>), grid, block, s, p); break;
        case 2: LOTTS_LAUNCH((skinny_gemm_stream_kernel<2, 1, WAVES, KG, XS>), grid, block, s, p); break;
        case 3: LOTTS_LAUNCH((skinny_gemm_stream_kernel<3, 1, WAVES, KG, XS>), grid, block, s, p); break;
        case 4: LOTTS_LAUNCH((skinny_gemm_stream_kernel<4, 2, WAVES, KG, XSM>), grid, block, s, p); break;
        case 5: LOTTS_LAUNCH((skinny_gemm_stream_kernel<5, 1, WAVES, KG, XSM>), grid, block, s, p); break;
        case 6: LOTTS_LAUNCH((skinny_gemm_stream_kernel<6, 2, WAVES, KG, XSM>), grid, block, s, p); break;
        case 7: LOTTS_LAUNCH((skinny_gemm_stream_kernel<7, 1, WAVES, KG, XSM>), grid, block, s, p); break;
        default: LOTTS_LAUNCH((skinny_gemm_stream_kernel<8, 2, WAVES, KG, XSM>), grid, block, s, p); break;
    }
}

template <int WAVES, int KG, int XS>
static void launch_parts(int mt, dim3 grid, hipStream_t s, const GemmParams& p) {
    const dim3 block(WAVES * kWave);
    if (mt == 3) LOTTS_LAUNCH((skinny_gemm_stream_kernel<3, 1, WAVES, KG, XS, true>), grid, block, s, p);
    else LOTTS_LAUNCH((skinny_gemm_stream_kernel<4, 2, WAVES, KG, XS, true>), grid, block, s, p);
}

template <int RN, int TT, int WAVES, int UB, typename P>
static void launch_direct(dim3 grid, hipStream_t s, const P& p) {
    const dim3 block(WAVES * kWave);
    if (grid.y == 1) LOTTS_LAUNCH((skinny_gemm_direct_kernel<RN, TT, WAVES, UB, true, P>), grid, block, s, p);
    else LOTTS_LAUNCH((skinny_gemm_direct_kernel<RN, TT, WAVES, UB, false, P>), grid, block, s, p);
}

// What both entry points check and prepare.
static int prepare(int M, int N, int K, const void* X, int64_t ldx, const void* W, int64_t ldw, void* Y, int64_t ldy, void* workspace,
                   size_t workspace_bytes, GemmPlan* plan, GemmParams* params) {
    if (!gemm_sizes_ok(M, N, K)) return LOTTS_ERR_SHAPE;
    if (!X || !W || !Y || !workspace) return LOTTS_ERR_NULL;
    if (ldx < K || ldw < K || ldy < N || (ldx % 8) || (ldw % 8) || (ldy % 4)) return LOTTS_ERR_SHAPE;
    if ((((uintptr_t)X | (uintptr_t)W | (uintptr_t)workspace) & 15) || ((uintptr_t)Y & 7)) return LOTTS_ERR_SHAPE;
    const GemmPlan pl = *plan = plan_gemm(M, N, K);
    if (workspace_bytes < plan_bytes(pl)) return LOTTS_ERR_WORKSPACE;
    GemmParams& p = *params;
    p.X = static_cast<const __bf16*>(X);
    p.W = static_cast<const __bf16*>(W);
    p.Y = static_cast<__bf16*>(Y);
    p.part = static_cast<float*>(workspace);
    p.M = M; p.N = N; p.K = K; p.ksplit = pl.ksplit; p.rows = pl.rows;
    p.nblocks = pl.nblocks; p.roww = pl.roww; p.rt = pl.rt; p.tt = pl.mt / pl.rt; p.parts = pl.parts;
    p.stagger = ldw % kStaggerStride == 0;
    p.by_xcd = pl.ksplit > 1 && (pl.parts > 1 || p.stagger) && 2LL * M * K > kXcdTokens;
    p.items = (short)(pl.ksplit > 1 ? pl.nblocks * pl.ksplit : 0);
    p.tokens = pl.form == kDirect ? (M + pl.nby - 1) / pl.nby : (M + pl.parts - 1) / pl.parts;
    p.d_ksplit = fast_div(pl.ksplit);
    p.d_nblocks = fast_div(pl.nblocks);
    const int steps = 2 * (K / kGemmChunk / pl.ksplit);  // of the shorter splits
    p.d_steps[0] = fast_div(steps > 0 ? steps : 1);
    p.d_steps[1] = fast_div(steps + 2);
    p.ldx = ldx; p.ldw = ldw; p.ldy = ldy;
    return LOTTS_OK;
}

// The launches of a plan: the one that writes Y gets p as it is.
template <typename P>
static int launch_plan(const GemmPlan& pl, hipStream_t s, const P& p) {
    const dim3 grid = p.by_xcd || pl.parts > 1 ? dim3((p.items + kNumXCD - 1) / kNumXCD * kNumXCD * pl.parts)
                                               : dim3(pl.nblocks, pl.form == kDirect ? pl.nby : pl.ksplit);
    switch (pl.form) {
        case kStream256:
            launch_stream<8, 1, 2, 2>(pl.mt, grid, s, p);
            break;
        case kStream128:
            if (pl.parts > 1) launch_parts<4, 1, 2>(pl.mt, grid, s, p);
            else launch_stream<4, 1, 2, 2>(pl.mt, grid, s, p); break;
        case kStream64: launch_stream<4, 2, 4, 2>(pl.mt, grid, s, p); break;
        case kDirect:
            switch (pl.rn * 10 + pl.tt) {
                case 11: launch_direct<1, 1, 8, 8>(grid, s, p); break;
                case 12: launch_direct<1, 2, 8, 4>(grid, s, p); break;
                case 21: launch_direct<2, 1, 8, 8>(grid, s, p); break;
                case 22: launch_direct<2, 2, 8, 4>(grid, s, p); break;
                case 23: launch_direct<2, 3, 8, 4>(grid, s, p); break;
                case 42: launch_direct<4, 2, 4, 2>(grid, s, p); break;
                default: launch_direct<4, 3, 4, 2>(grid, s, p); break;
            }
            break;
    }
    const int rc = check_launch();
    if (rc != LOTTS_OK || pl.ksplit == 1) return rc;
    LOTTS_LAUNCH(skinny_gemm_reduce_kernel<P>, dim3((unsigned)(pl.parts * pl.nblocks * pl.roww * pl.mt)), dim3(256), s, p);
    return check_launch();
}

}  // namespace lotts

// The query asks for the K splits of the stream form also where the direct form is taken: which one is faster changes back and forth with
// the tokens, and a workspace sized for the most of them would be too small for fewer.  The same where the tokens come to be in two parts:
// 161 of them beside 3208 weight rows and K = 12416 have 2 % fewer bytes of partials than 160 in one part.
extern "C" size_t skinny_gemm_workspace_bytes(int32_t M, int32_t N, int32_t K) {
    using namespace lotts;
    if (!gemm_sizes_ok(M, N, K)) return 0;
    const GemmPlan pl = plan_gemm(M, N, K, false);
    const size_t bytes = plan_bytes(pl);
    return pl.parts > 1 ? std::max(bytes, plan_bytes(plan_gemm(tokens_in_one_part(K), N, K, false))) : bytes;
}

extern "C" int skinny_gemm(int32_t M, int32_t N, int32_t K, const void* X, int64_t ldx, const void* W, int64_t ldw,
                           void* Y, int64_t ldy, void* workspace, size_t workspace_bytes, void* stream) {
    using namespace lotts;
    GemmPlan pl;
    GemmParams p;
    const int rc = prepare(M, N, K, X, ldx, W, ldw, Y, ldy, workspace, workspace_bytes, &pl, &p);
    return rc != LOTTS_OK ? rc : launch_plan(pl, (hipStream_t)stream, p);
}

extern "C" int skinny_gemm_append(int32_t B, int32_t k, int32_t Hkv, int32_t D, int32_t N, int32_t K, const void* X, int64_t ldx,
                                  const void* W, int64_t ldw, void* Y, int64_t ldy, void* Kpriv, void* Vpriv, int64_t priv_stride_b,
                                  int64_t priv_stride_h, int64_t priv_stride_t, int32_t Lmax, const int32_t* priv_len, void* workspace,
                                  size_t workspace_bytes, void* stream) {
    using namespace lotts;
    if (B < 1 || B > kGemmMaxM || k < 0 || k > 255 || Hkv < 1 || D < 8 || (D % 8) || 2LL * Hkv * D > N || Lmax < k + 1) return LOTTS_ERR_SHAPE;
    if (!Kpriv || !Vpriv || !priv_len) return LOTTS_ERR_NULL;
    for (int64_t s : {priv_stride_b, priv_stride_h, priv_stride_t})
        if (s < 0 || (s % 8)) return LOTTS_ERR_SHAPE;
    if (priv_stride_t < D || (ldy % 8) || (((uintptr_t)Y | (uintptr_t)Kpriv | (uintptr_t)Vpriv) & 15)) return LOTTS_ERR_SHAPE;
    GemmPlan pl;
    GemmAppendParams p;
    int rc = prepare(B * (k + 1), N, K, X, ldx, W, ldw, Y, ldy, workspace, workspace_bytes, &pl, &p);
    if (rc != LOTTS_OK) return rc;
    const int n_new = N - 2 * Hkv * D;
    // The stream kernel writes Y itself only where K is not split: matrices beyond the direct form with 129 blocks of rows or more, or
    // short in K.  There the append stays its own launch, 4 us behind a product of 25 and more, and the kernel without a twin.
    if (pl.form != kDirect && pl.ksplit == 1) {
        rc = launch_plan<GemmParams>(pl, (hipStream_t)stream, p);
        if (rc != LOTTS_OK) return rc;
        const __bf16* fresh = static_cast<const __bf16*>(Y) + n_new;
        return kv_append(B, k, Hkv, D, LOTTS_BF16, fresh, fresh + (long long)Hkv * D, (k + 1) * ldy, ldy, D, Kpriv, Vpriv, priv_stride_b,
                         priv_stride_h, priv_stride_t, Lmax, priv_len, stream);
    }
    p.a = {static_cast<__bf16*>(Kpriv), static_cast<__bf16*>(Vpriv), priv_len, priv_stride_b, priv_stride_h, priv_stride_t,
           n_new, D, Hkv, k + 1, Lmax, fast_div(k + 1), fast_div(D)};
    return launch_plan(pl, (hipStream_t)stream, p);
}
