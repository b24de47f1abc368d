// verify_attention: causal attention of the k + 1 new positions of every branch against the
// branch's KV cache, which sits behind a prompt prefix shared by all branches (paper
// Section 3.2: B branches of one question; Section 2: the target model verifies the drafts in
// one parallel forward; Section 3.1: the step is bound by loading the KV cache).
//
// bf16 path (MFMA, gfx950), normally ONE launch:
//   attn_kernel           one launch over "work items", one workgroup each: 4 wavefronts for up to 32
//       query rows, 8 for up to 64 (two groups of 4, one row tile each; wavefront w of either group
//       streams the same key tiles, so the two load half a tile each into a slab both read).  An item
//       is a share of the keys of one KV segment and a stack of up to 32*NQT query rows that all
//       read those keys:
//         - private item: the G*R rows (G = Hq/Hkv query heads x R = k+1 positions) of one branch
//           and KV head, against a share of that branch's private keys;
//         - prefix item ("stacked" plan): rows of SEVERAL branches stacked on the MFMA N dimension
//           against a share of the shared prefix, so a prefix tile is fetched once per row stack
//           instead of once per branch;
//         - "folded" plan (prefix short next to the private caches): there are no prefix items;
//           each private item first runs its share of the prefix keys for its own rows (served by
//           the L2 after the first touch, so HBM still sees the prefix once) and continues into
//           the private keys with the same running state -- no extra partial, no extra workgroups.
//       The 32-key tiles of a segment are dealt round-robin to all wavefronts working on it; a
//       wavefront streams its tiles with coalesced non-temporal 16-byte loads into registers one
//       tile ahead, staged through a wavefront-private LDS slab
//       (K read back row-wise as the MFMA A operand, V with the transposing LDS load), S^T = K Q^T
//       and O^T += V^T P^T on 32x32x16 bf16 MFMA, flash-style running (max, sum, O).  Where no wavefront gets more than
//       one tile, a form of its own (ONE): the wavefronts publish their tiles' weights, and each forms a block of the item's output
//       over all of them.  The 4 states
//       are combined through LDS after one barrier and the item's un-normalised partial goes to
//       the workspace -- or, if the item holds whole rows (no key shares, no prefix items), straight to O.
//       Who merges the partials of a row depends on how many there are (of dealt tiles, below: on how many there may be): of two, or of
//       up to eight with few bytes, the item that finishes last (arrivals are counted per (KV head, branch) in a cell that carries the call's tag: what an earlier
//       call left there, complete or not, counts as zero arrivals); of more, merge workgroups at the end of the grid, which wait for a flag of
//       every partial they read and share the rows among them; one whose flags stay out for long leaves, and the item that
//       delivers the last partial merges in its place.  Partials cross workgroups -- and XCDs,
//       each with its own L2 -- inside one launch, so they are written and read with 16-byte
//       buffer accesses that carry the device-scope cache policy (performed at the memory side of
//       the L2s); nothing is ever flushed or invalidated cache-wide.
//       For long calls the shares of a branch follow its length (the "flat" plan, see FlatCuts): every item takes an equal piece of
//       its KV head's tiles, branch after branch, and starts with the cuts, from all branches' lengths, on the device.
//   attn_merge_kernel     second launch, where prefix items or several row groups add partials of their own (but for the
//       smallest batches, where the last arriver merges).
// fp32 path: attn_f32_kernel, plain fp32 VALU arithmetic, one workgroup per output row; it
// exists for exactness checks on small fp32 problems.
// Two entry points share all of this: verify_attention (the caller brings the workspace) and
// verify_attention_noalloc (arrival cells and partials in a static device array of this file).
#include <algorithm>
#include <atomic>
#include <cmath>

#include "lotts_common.h"

namespace lotts {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

constexpr int kAttnThreads = 256;
constexpr int kAttnWaves = kAttnThreads / kWave;
constexpr int kTile = 32;      // keys per tile = M of one 32x32x16 MFMA
constexpr int kRowTile = 32;   // query rows per row tile = N of the MFMA
constexpr int kMaxSplit = 64;       // key shares of a segment whose partials are merged by merge workgroups or a launch of
                                    // their own: one wavefront polls the flags of a row's partials
constexpr int kMaxSplitStack = 16;  // the same when prefix items or several row groups add partials of their own

constexpr int kMaxCounters = 16384;  // 64-bit cells at the start of the workspace
// Flat plan (below): places of a head's sequence that stand for what starting on a branch costs an item (its states meet, its rows go
// out, Q and a first tile come in: about two tiles of each wavefront; 6 is level, without any 44 x 2 heads x 1310 .. 5243 tokens
// took 2 % more).
constexpr int kStartTiles = 8;
// Flat plan: from this many tiles of each wavefront on.  (A build of the tests sets 0, and deals whatever lengths differ: calls as short as
// theirs would not gain by it.)
#ifndef LOTTS_FLAT_STEPS
#define LOTTS_FLAT_STEPS 18
#endif

struct AttnPlan {
    int n_pre_items, n_priv_items;
    int fold;           // 1: private items also run their share of the prefix (no prefix items)
    int n_rg_priv;      // row groups per (branch, KV head)
    int nsplit_priv;    // key splits of a private segment
    int nsplit_pre;     // key splits of the prefix (stacked plan; 0 otherwise)
    int nslots;         // partials per output row
    int merge;          // who merges a row's partials: one of the five below
    int rpm, mpp;       // merge workgroups: rows each of them takes (a power of two), their number per (KV head, branch)
    int n_merge;
    int nqt;            // row tiles per item: 1 or 2
    int n_rg_pre;       // row groups per KV head over all branches' stacked rows (stacked plan)
    int one;            // 1: no wavefront of an item gets more than one key tile
    int runs;           // runs of key tiles of an item
};
struct AttnPlans : AttnPlan {
    int flat;     // 0: shares of fixed number; 1: the items deal the tiles by the branches' lengths where that gains; 2: always; 3: where lengths differ
    int workers;  // flat: items per KV head
    int flat_merge;  // who merges where the tiles are dealt by the lengths: kMergeLast or kMergeGroups
};
constexpr int kMergeLast = 0;    // the last-arriving workgroup of a (KV head, branch), inside the attention launch
constexpr int kMergeGroups = 1;  // merge workgroups at the end of the attention launch's grid
constexpr int kMergeLaunch = 2;  // a launch of its own
constexpr int kMergeNone = 3;    // an item holds whole rows: it stores the output itself
constexpr int kMergePair = 4;    // two items, one row tile: the later one reads the other's partial, its own is in registers

struct AttnParams {
    // first what every item needs before its first tile, together: few loads, few trips
    const void *Q, *Kpre, *Vpre, *Kpriv, *Vpriv;
    const int32_t* priv_len;
    long long q_stride_b, q_stride_r, q_stride_h;
    long long kpre_stride_h, kpre_stride_t;
    long long kpriv_stride_b, kpriv_stride_h, kpriv_stride_t;
    FastDiv d_hkv, d_nsp, d_rgp, d_wpriv, d_g;  // by Hkv, nsplit_priv, n_rg_priv, the wavefronts that share a private segment, G
    int k, R, Hkv, G, GR, P, Lmax;
    int near_rows;              // a tile's key rows lie within 2^31 bytes of its first one, prefix and private
    int tiles_pre, first_wave;  // prefix tiles; folded plan: the wavefront of a segment that gets the first private tile
    AttnPlan plan;
    FastDiv d_npre, d_wpre, d_gr, d_mpp;  // by nsplit_pre, the wavefronts that share the prefix, GR, mpp
    int B, Hq, D;
    float scale_log2;  // scale * log2(e)
    void* ws;                  // workspace base; everything below lives in it
    unsigned ws_bytes;
    unsigned off_o, off_ml;    // byte offsets: partial O [Hkv][B*GR][nslots][D] fp32,
                               //               partial (running max in log2 units, sum) [Hkv][B*GR][nslots][2] fp32
    unsigned long long* counters;  // [Hkv][B] arrival cells at the start of the workspace: (call tag << 16) | arrivals
    unsigned long long tag;        // this call's tag, shifted into place: larger than that of any earlier call
    void* O;
    float* lse;
    long long o_stride_b, o_stride_r, o_stride_h;
    // flat plans only (behind everything else: a call that is not captured reads its arguments from far away, 0.2 us for every line more)
    int flat, workers, flat_merge;
    FastDiv d_workers;  // by workers
};

static inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Launch plan.  Depends on the descriptor only (never on device data), so the workspace query
// and the launch agree.  The HBM stream runs best with one streaming workgroup per compute
// unit, so the private caches are cut into just enough key shares to give every CU one item.
static inline AttnPlans plan_attention(const lotts_attn_desc& d, bool may_be_flat = true) {
    AttnPlans pl = {};
    const int GR = (d.Hq / d.Hkv) * (d.k + 1);
    pl.nqt = GR > kRowTile ? 2 : 1;
    const int rows_per_item = kRowTile * pl.nqt;
    pl.n_rg_priv = ceil_div(GR, rows_per_item);
    pl.n_rg_pre = ceil_div(d.B * GR, rows_per_item);
    const int tiles_priv = ceil_div(d.Lmax, kTile), tiles_pre = ceil_div(d.P, kTile);
    const long long base = (long long)d.B * d.Hkv * pl.n_rg_priv;
    // A prefix that is short next to the private caches is folded into the private items.
    pl.fold = (d.P > 0 && (long long)d.P * 4 <= d.Lmax) ? 1 : 0;
    const bool simple = pl.n_rg_priv == 1 && (d.P == 0 || pl.fold);  // an item's rows are one branch's rows
    // At least about one tile per wavefront.  Few branches: the folded prefix tiles count as well, and the last share may be
    // ragged -- from three shares on; below, a share more costs the merge more than it saves (8 x 8 heads x 137 tokens, D = 64:
    // 5.0 us in one share, 5.8 in two; 6 x 8 x 307 6.3 in two, 7.0 in three).  (With more branches, one share more would double the
    // items and with them the partials; the built-in scratch of the allocation-free entry point has to hold what it held.)
    const bool few = simple && base <= kNumCU / 2;
    const int tiles_all = tiles_priv + (pl.fold ? tiles_pre : 0);
    int max_split = !few ? tiles_priv / kAttnWaves : tiles_all < 3 * kAttnWaves ? tiles_all / kAttnWaves : ceil_div(tiles_all, kAttnWaves);
    const int cap_split = simple ? kMaxSplit : kMaxSplitStack;
    if (max_split > cap_split) max_split = cap_split;
    if (max_split < 1) max_split = 1;
    // Prefix shares beside s private ones (stacked plan): items of about the same length.
    auto pre_shares = [&](int s) {
        if (d.P == 0 || pl.fold) return 0;
        const int tiles_per_item = ceil_div(tiles_priv, s);
        int q = (tiles_pre + tiles_per_item / 2) / tiles_per_item;
        int cap = tiles_pre / kAttnWaves;
        if (cap > kMaxSplitStack) cap = kMaxSplitStack;
        if (q > cap) q = cap;
        return q < 1 ? 1 : q;
    };
    // A count of items just above one per unit is the worst choice: a few units run two and everybody waits for them (48
    // branches x 2 heads x 4300 tokens in 3 shares, 288 items, 48.6 us; in 2 shares, 192 items, 36.7).  Prefix items count (8 x 8
    // heads x 512 tokens behind 2048: 26.7 us in 4 shares, 896 items with the prefix's, 15.2 in one, 224; 16 x 8 x 1500 behind 1100
    // 33.5 us in 2, 336 items, 25.9 in one).  Branches of different lengths lose by it where few items are left for many units: 11 x 8 heads x 669 + 6418 / 4
    // .. 6418 tokens 39.5 us in 3 shares, 44.1 in 2, at equal lengths 68.1 and 50.2.
    // At D = 64 and one row tile an item has half the bytes in flight and two of them fit a unit with ease, so where one per
    // unit leaves many units without an item, two per unit are dealt (12 branches x 8 heads x 2461 tokens, D = 64: 5 shares 15.9
    // us, 2 shares 16.7; of different lengths 13.8 against 15.4; 24 x 8 x 2000 behind 900, where one share a branch
    // and the prefix's are more than one per unit already, 21.5 against 24.2).  Where two do not
    // fill the units either, branches of different lengths still need more items than units, from 40 tiles on (9 x 16 heads x 375
    // .. 1500 tokens 12.1 us in two shares, 14.5 in one, at equal lengths 15.3 and 15.2; 12 x 16 x 1250 .. 5000 32.1 and 37.5).
    auto items = [&](long long s) { return base * s + (long long)d.Hkv * pl.n_rg_pre * pre_shares((int)s); };
    auto shares = [&](int units) {
        long long s = base < units ? units / base : 1;
        if (!simple && s > max_split) s = max_split;
        while (s > 1 && items(s) > units) --s;
        return s;
    };
    auto fills = [&](int units) {
        const long long n = items(shares(units));
        return n * 20 >= (long long)units * 17 && n <= units;
    };
    long long want = shares(kNumCU);
    if (d.D == 64 && pl.nqt == 1 && (simple ? !fills(kNumCU) : items(want) > kNumCU)) {
        if (fills(2 * kNumCU)) want = shares(2 * kNumCU);
        else if (simple && base < kNumCU && want == 1 && tiles_all >= 40) want = 2;
    }
    pl.nsplit_priv = (int)(want > max_split ? max_split : want);
    if (simple) {  // the fewest shares (partials) that leave the longest wavefront the same number of tiles
        const int per_wave = ceil_div(tiles_all, kAttnWaves * pl.nsplit_priv);
        pl.nsplit_priv = ceil_div(tiles_all, kAttnWaves * per_wave);
    }
    pl.nsplit_pre = pre_shares(pl.nsplit_priv);
    // A form of its own where no wavefront gets more than one tile: four wavefronts to a row tile, eight to two (14 branches x 4
    // heads x 448 tokens 9.9 -> 9.3 us, 12 x 1 x 736 9.7 -> 9.2, 8 x 2 heads x 2560 with 40 rows 12.8 -> 12.3).  Taking several tiles in
    // rounds of it is level at two (20 x 4 .. 88 x 1: -2.5 .. +2.8 %) and loses from three on, and so do eight wavefronts that share four
    // tiles (2 x 1 heads x 1888, 35 rows, 11.8 -> 12.6).  Not at D = 64, where the output has fewer blocks than there are
    // wavefronts: level with one tile, 1 x 8 x 2600 behind 960 with two 9.7 -> 10.1.
    int longest = ceil_div(tiles_all, kAttnWaves * pl.nsplit_priv);
    if (pl.nsplit_pre > 0) {
        const int longest_pre = ceil_div(tiles_pre, kAttnWaves * pl.nsplit_pre);
        longest = longest > longest_pre ? longest : longest_pre;
    }
    pl.one = d.D == 128 && longest == pl.nqt;
    pl.runs = pl.one ? kAttnWaves * pl.nqt : kAttnWaves;
    pl.nslots = pl.nsplit_pre + pl.nsplit_priv;
    // Who merges (measured with calls back to back, kernel + what merges, when items started and ended about 1 us later than now,
    // on either side of each comparison):
    //  - an item that holds whole rows stores the output: 32 branches x 8 KV heads x 3168 tokens 57.3 -> 53.3 us;
    //  - of two items the later one merges and reads only the other's partial (16 x 8 heads x 4096 tokens: 0.5 us less than
    //    with merge workgroups);
    //  - merge workgroups at the end of the grid share the rows of a (KV head, branch) and wait for the flags of its partials:
    //    1 x 2 heads x 8192 tokens, 64 shares, 10.6 us against 11.7 with a launch of its own (and 15.6 with 16 shares);
    //    8 x 8 heads x 4300 tokens, 4 shares, 27.4 us against 29.3 with the merge by the last arriver; short contexts too:
    //    2 x 2 heads x 4064 tokens 10.2 us against 11.0 with a launch of its own, 1 x 2 x 800 9.2 either way;
    //  - the last arriver, where one round of its loads is all (up to eight partials of a row) and there are few bytes of them: up
    //    to 32 KB it is 2 .. 17 % ahead of merge workgroups (7 x 8 x 646 tokens 10.1 us against 11.0, 10 x 8 x 605, D = 64, 8.0
    //    against 9.2), with more partials or bytes 3 .. 15 % behind (1 x 16 x 7834, D = 64, 12 KB in 16 partials 13.1 against 12.1;
    //    8 x 8 x 1222, 60 KB, 15.0 against 13.7);
    //  - a second launch where prefix items or several row groups add partials of their own -- an item then brings in rows of
    //    several branches, and its last arriver would merge them one after the other: 3 x 8 heads x 1264 tokens behind 505, D = 64,
    //    9.2 us against 15.1, 37 x 4 x 65 behind 300 10.1 against 23.5 -- but for the smallest batches (4 x 8 x 300 behind 200,
    //    D = 64, 8.9 against 7.5).
    const long long part_bytes = (long long)pl.nslots * GR * d.D * 4;  // of a (KV head, branch)
    const bool last_arriver = pl.nslots <= 8 && (simple ? pl.nqt == 1 && part_bytes <= 32 * 1024
                                                        : d.B * GR <= 2 * kRowTile && part_bytes <= 48 * 1024);
    if (pl.nslots == 1) pl.merge = kMergeNone;  // no prefix items, no key shares
    else if (simple && pl.nslots == 2 && pl.nqt == 1) pl.merge = kMergePair;
    else if (last_arriver) pl.merge = kMergeLast;
    else pl.merge = simple ? kMergeGroups : kMergeLaunch;
    // rows per merge workgroup: as few as leave at most one merge workgroup per unit (items are not counted, so with two row tiles,
    // whose items leave no room for another workgroup, some mergers start when an item ends)
    auto rows_per_merger = [&](int threads) {
        pl.rpm = 1;
        while (pl.rpm * 2 * (d.D / 4) <= threads && (long long)d.B * d.Hkv * ceil_div(GR, pl.rpm) > kNumCU) pl.rpm *= 2;
        pl.mpp = ceil_div(GR, pl.rpm);
    };
    if (pl.merge == kMergeGroups) {
        const int threads = kAttnThreads * pl.nqt;
        rows_per_merger(threads);
        // Cells of the merge workgroups: a flag per key share and a count.  Where only the counts are too many (64 shares for 256
        // merge workgroups), twice the rows for half of the workgroups.
        auto cells = [&](int per_merger) { return (long long)d.B * d.Hkv * pl.mpp * per_merger; };
        const bool flags_fit = cells(pl.nslots) <= kMaxCounters;
        while (flags_fit && cells(pl.nslots + 1) > kMaxCounters && pl.rpm * 2 * (d.D / 4) <= threads) {
            pl.rpm *= 2;
            pl.mpp = ceil_div(GR, pl.rpm);
        }
        if (cells(pl.nslots + 1) > kMaxCounters) pl.merge = kMergeLaunch;
    }
    if (pl.merge == kMergeLaunch) {
        rows_per_merger(kAttnThreads);
        // a thread takes four partials of a row at least: more groups of threads only meet again in LDS (2 x 1 heads x 72 rows, 4
        // partials, 12.9 -> 12.4 us)
        while (pl.rpm * 2 * (d.D / 4) <= kAttnThreads && kAttnThreads / (pl.rpm * 2 * (d.D / 4)) * 4 >= pl.nslots) pl.rpm *= 2;
        pl.mpp = ceil_div(GR, pl.rpm);
    }
    // Branches of different lengths.  Fixed shares leave the longest branches' items behind: the host does not know the lengths, so the
    // number of shares cannot follow them.  In the flat plan the items deal a head's tiles among themselves on the device (see FlatCuts),
    // unless that would gain too little for these lengths, and then the same kernel runs the fixed shares, with their own merge and the same bits.
    // An item finds that out before its first tile, 0.5 .. 0.8 us, so it is for long calls only: from 18 tiles a wavefront on, 26 x 2 heads x 1086 +
    // 2399 .. 9596 tokens 43.2 -> 39.0 us, 19 x 4 x 1051 + 2722 .. 10890 67.1 -> 59.8, 64 x 2 x 1003 + 1792 .. 7168 63.9 -> 58.3.  Equal lengths
    // are told at once: over 60 sizes 1.6 % slower to 2.6 % faster than without a flat plan, on average 0.1 % slower at D = 128, 0.4 % at D = 64
    // (dealt all the same, or merged as dealt tiles are, up to 9 % slower: 7 x 16 heads x 15408 tokens, D = 64, 70.6 us against 64.8).  (Of 14 .. 17 tiles a wavefront different lengths gain as much, but those that are not dealt lose a larger part of their time.)  At D = 64
    // with a third more items of whole rows than units the few units with two of them hold up everybody, whatever the lengths: always dealt
    // (17 x 16 heads x 897 + 4635 tokens 78.5 -> 64.0, 42 x 8 x 390 + 5137 86.8 -> 83.6; 36 sizes of equal lengths 12 % faster, the worst, 42 x 8 x
    // 3702, 3 % slower, of different ones 12 .. 43 %; with more items than that fixed shares even out).
    const int units = d.D == 64 && pl.nqt == 1 ? 2 * kNumCU : kNumCU;  // (two items to a unit there)
    const int workers = units / d.Hkv;
    const long long farthest = std::max((d.Lmax + 32LL) * d.kpriv_stride_t, (d.P + 32LL) * d.kpre_stride_t) * 2;  // bytes
    const long long flat_bytes = (long long)d.Hkv * (workers + d.B) * GR * (d.D * 4 + 8) + kMaxCounters * 8 + 512;
    if (may_be_flat && simple && !pl.one && pl.merge != kMergeLaunch && d.B > 1 && d.B <= kWave && workers > 0 && (pl.nsplit_priv == 1 || d.B * pl.nsplit_priv <= workers) &&
        (long long)d.B * tiles_all >= (long long)LOTTS_FLAT_STEPS * kAttnWaves * workers &&
        (long long)d.B * (tiles_all + kStartTiles) * workers < (1LL << 31) && farthest < (1LL << 31) && flat_bytes <= (16 << 20)) {
        pl.flat = d.D == 64 && pl.nqt == 1 && base * pl.nsplit_priv > kNumCU && base * pl.nsplit_priv * 3 <= 4 * kNumCU ? 2 : LOTTS_FLAT_STEPS > 0 ? 1 : 3;
        pl.workers = workers;
        // Where an item has whole branches of its own, the last arriver merges the few that are cut; where branches have several items each,
        // merge workgroups, however few bytes their partials would be in fixed shares: a branch that is longer than the others has up to
        // all items' partials, which one arriver adds up in a chain.  44 sizes with up to 8 KB, one branch longer than the others 30 x 2
        // heads, 10030 tokens 25.0 -> 12.1 us, on average 19 % (D = 64) and 37 %, a quarter of them longer 4 and 9 %, lengths between
        // a quarter and all 0.2 and 2 %; the workgroups that are left over cost calls in fixed shares 0.1 %.
        pl.flat_merge = kMergeLast;
        if (workers > d.B) {
            if (pl.merge != kMergeGroups) rows_per_merger(kAttnThreads * pl.nqt);  // (fixed shares have the same ones)
            if ((long long)d.Hkv * (workers + 2 * d.B) * pl.mpp <= kMaxCounters) pl.flat_merge = kMergeGroups;
        }
    }
    pl.n_merge = pl.merge == kMergeGroups || (pl.flat && pl.flat_merge == kMergeGroups) ? d.B * d.Hkv * pl.mpp : 0;
    pl.n_pre_items = d.Hkv * pl.n_rg_pre * pl.nsplit_pre;
    pl.n_priv_items = pl.flat ? d.Hkv * std::max(pl.workers, d.B * pl.nsplit_priv) : d.B * d.Hkv * pl.n_rg_priv * pl.nsplit_priv;
    return pl;
}

static inline size_t part_rows(const lotts_attn_desc& d, const AttnPlans& pl) {
    return (size_t)(d.Hq / d.Hkv) * (d.k + 1) * d.Hkv * (pl.flat ? pl.workers + d.B : d.B * pl.nslots);
}
static inline size_t part_o_elems(const lotts_attn_desc& d, const AttnPlans& pl) {
    return part_rows(d, pl) * d.D;
}
static inline size_t part_ml_elems(const lotts_attn_desc& d, const AttnPlans& pl) {
    return part_rows(d, pl) * 2;
}

// Workspace: [arrival cells][partial O][partial (max, sum)], each part 256-byte aligned.  The
// cell block has the same place and size for every geometry, so a buffer stays usable when the
// geometry changes: partials of one call never land where another counts.
//
// An arrival cell holds (tag << 16) | arrivals.  Every call draws a tag larger than all earlier ones
// of this process; an arriving workgroup first raises the cell to (tag, 0) with an atomic maximum,
// then adds one.  A cell left at zero (a fresh zero-filled buffer, or the reset the last arriver
// does) and a cell left behind by an earlier call that never completed both start the new call
// at zero arrivals, so no call can poison the buffer for the next one.  With merge workgroups the same cells are, for
// every merge workgroup of a (KV head, branch), one flag per key share (flat plan: per partial) and one arrival cell.  An item sets its flag of every
// merge workgroup that reads its partial to (tag << 16) | 1; a merge workgroup that leaves sets its flags to (tag << 16) | 2;
// whoever merges puts the zeros back.  Any other content counts as not arrived.
constexpr int kTagShift = 16;            // arrivals per cell < 2^16, checked on the host
static std::atomic<unsigned long long> g_call_tag{0};
static inline size_t workspace_layout(const lotts_attn_desc& d, const AttnPlans& pl, size_t* off_o, size_t* off_ml) {
    size_t bytes = (size_t)kMaxCounters * sizeof(unsigned long long);
    if (off_o) *off_o = bytes;
    bytes += part_o_elems(d, pl) * sizeof(float);
    bytes = (bytes + 255) & ~(size_t)255;
    if (off_ml) *off_ml = bytes;
    bytes += part_ml_elems(d, pl) * sizeof(float);
    return (bytes + 255) & ~(size_t)255;
}

// 16- and 8-byte accesses to the workspace, with the device-scope cache policy (sc0 sc1) when the
// data crosses workgroups inside one launch, plain otherwise.
constexpr int kDevScope = 17;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t ws_rsrc(const AttnParams& prm) {
    return __builtin_amdgcn_make_buffer_rsrc(prm.ws, 0, (int)prm.ws_bytes, 0x00020000);
}
template <bool DEV>
__device__ __forceinline__ void ws_store4(__amdgpu_buffer_rsrc_t r, unsigned byte_off, float4 v) {
    u32x4 u;
    u[0] = __float_as_uint(v.x); u[1] = __float_as_uint(v.y); u[2] = __float_as_uint(v.z); u[3] = __float_as_uint(v.w);
    __builtin_amdgcn_raw_buffer_store_b128(u, r, (int)byte_off, 0, DEV ? kDevScope : 0);
}
template <bool DEV>
__device__ __forceinline__ void ws_store2(__amdgpu_buffer_rsrc_t r, unsigned byte_off, float2 v) {
    u32x2 u;
    u[0] = __float_as_uint(v.x); u[1] = __float_as_uint(v.y);
    __builtin_amdgcn_raw_buffer_store_b64(u, r, (int)byte_off, 0, DEV ? kDevScope : 0);
}
template <bool DEV>
__device__ __forceinline__ float4 ws_load4(__amdgpu_buffer_rsrc_t r, unsigned byte_off) {
    const u32x4 u = __builtin_amdgcn_raw_buffer_load_b128(r, (int)byte_off, 0, DEV ? kDevScope : 0);
    return make_float4(__uint_as_float(u[0]), __uint_as_float(u[1]), __uint_as_float(u[2]), __uint_as_float(u[3]));
}
template <bool DEV>
__device__ __forceinline__ float2 ws_load2(__amdgpu_buffer_rsrc_t r, unsigned byte_off) {
    const u32x2 u = __builtin_amdgcn_raw_buffer_load_b64(r, (int)byte_off, 0, DEV ? kDevScope : 0);
    return make_float2(__uint_as_float(u[0]), __uint_as_float(u[1]));
}

// Output quad c4 of row rl (0 .. G*R-1) of a (KV head, branch): normalise, convert, store; the first quad's thread stores LSE.
__device__ __forceinline__ void store_merged(const AttnParams& prm, int kvh, int b, int rl, int c4, float4 o, float M, float Lsum) {
    const int r = quot(rl, prm.d_g), hg = rl - r * prm.G;
    const int h = kvh * prm.G + hg;
    const float inv = 1.0f / Lsum;  // a row always sees itself: Lsum > 0
    __bf16* op = (__bf16*)prm.O + (long long)b * prm.o_stride_b + (long long)r * prm.o_stride_r +
                 (long long)h * prm.o_stride_h + c4 * 4;
    bf16x4 ov;
    ov[0] = (__bf16)(o.x * inv);
    ov[1] = (__bf16)(o.y * inv);
    ov[2] = (__bf16)(o.z * inv);
    ov[3] = (__bf16)(o.w * inv);
    *reinterpret_cast<bf16x4*>(op) = ov;
    if (prm.lse && c4 == 0)
        prm.lse[((long long)b * prm.R + r) * prm.Hq + h] = (M + log2f(Lsum)) * 0.69314718055994530942f;
}

// Where the partials of a (KV head, branch) lie, in rows of partials (D floats, or 8 bytes of (max, sum)), and their number; the cells of
// its merge workgroups follow the same numbering.
struct Partials {
    unsigned first, row_step, step;  // row 0 of the first partial; from row to row; from partial to partial
    int n;
    int cell;                        // flat: number of the first partial among all
};

// Flat plan.  A KV head's tiles -- branch after branch, a branch's folded prefix tiles and then its private ones -- form one sequence,
// and item i of the head's `workers` takes the i-th of equal pieces of it, whatever the branches' lengths: where a piece ends inside a branch,
// that branch has a partial from either side; where it covers several branches, the item works on one after the other.  kStartTiles
// places of the sequence in front of every branch stand for what starting on a branch costs an item.  A partial's number is its item's
// plus its branch's: strictly rising along the sequence, at most workers + B of them per head.
struct FlatCuts {
    unsigned end;    // of branch `lane`, in the head's sequence
    unsigned total;
    int len;         // of branch `lane`
    int workers;     // items with anything to do
    bool dealt;      // by the lengths; or the fixed number of shares to every branch
};
__device__ __forceinline__ FlatCuts flat_cuts(const AttnParams& prm, int fold_tiles, int lane, int L) {
    FlatCuts c = {};
    L = L < prm.R ? prm.R : (L > prm.Lmax ? prm.Lmax : L);
    c.len = L;
    if (prm.flat != 2 && __ballot(L != __builtin_amdgcn_readfirstlane(L)) == 0) return c;  // all alike: fixed shares
    const int tiles = fold_tiles + (L - 1) / kTile + 1;
    c.end = wave_incl_scan_u32(lane < prm.B ? kStartTiles + tiles : 0);
    c.total = __builtin_amdgcn_readlane(c.end, kWave - 1);
    c.workers = min(prm.workers, (int)c.total);  // (at least one place each)
    // Steps (a tile for every wavefront of an item) of a branch's fixed shares, and how long they take, in steps of a full chip: all
    // items together are bound by the memory, whose rate they share, until so few are left that each is bound by what a unit takes in,
    // about twice as much, items of which a unit could hold two (D = 64, one row tile) a little more than that (`lone`).  At whatever length L
    // that happens, sum of min(steps, L) / items + (longest - L) / 2 is no more than the whole time; nor are two items of mean length in
    // one unit, where there are such.  Dealt, they take what the memory takes, and some more: a 16th where a unit could hold two, otherwise
    // 8 tiles a branch, 4 at D = 64.  Fitted to 158 sizes x 6 kinds of different lengths, each measured both ways: 19 of the 948 come out behind
    // their fixed shares by more than 1 %, and they gain 17 % on average.  (With one step of all wavefronts more for every size, and lone
    // items of D = 64 at two or four times, 29 did: 14 x 8 heads of about 12000 tokens 51.5 us in fixed shares, dealt 54.5.)
    const int steps = lane < prm.B ? quot(tiles - 1, prm.d_wpriv) + 1 : 0;
    const int longest = wave_max_u31(steps);
    const bool two_a_unit = prm.D == 64 && prm.plan.nqt == 1;
    const int lone = two_a_unit ? prm.workers * 7 / 8 : prm.workers;
    const int total = (int)(2 * c.total), dealt = total + (two_a_unit ? total / 16 : prm.D / 8 * prm.B);
    c.dealt = prm.flat > 1 || longest * lone * kAttnWaves > dealt;
    if (c.dealt) return c;
    auto sum_until = [&](int L) { return (int)__builtin_amdgcn_readlane(wave_incl_scan_u32(min(steps, L)), kWave - 1); };
    auto until = [&](int L) { return 2 * sum_until(L) * prm.plan.nsplit_priv + (longest - L) * lone; };  // (in half steps of all the head's items)
    const int sum = sum_until(longest);
    int fixed = max(max(2 * sum * prm.plan.nsplit_priv, until(longest * 3 / 4)), max(until(longest / 2), until(longest / 4)));
    if (two_a_unit && 2 * prm.B * prm.plan.nsplit_priv > prm.workers)  // more items than units: some units have two
        fixed = max(fixed, (int)(1.8f * sum * lone * __builtin_amdgcn_rcpf(prm.B)));
    c.dealt = fixed * kAttnWaves > dealt;
    return c;
}
__device__ __forceinline__ unsigned flat_cut(const AttnParams& prm, const FlatCuts& c, int i) {
    return c.workers == prm.workers ? quot(i * c.total, prm.d_workers) : i * c.total / c.workers;
}
// the item that has place `at`: the last one whose piece starts at or before it
__device__ __forceinline__ int flat_worker(const FlatCuts& c, unsigned at) { return ((at + 1) * c.workers - 1) / c.total; }
// a branch's tiles are places first .. last of the sequence
__device__ __forceinline__ void flat_branch(const FlatCuts& c, int b, unsigned* first, unsigned* last) {
    *first = (b > 0 ? __builtin_amdgcn_readlane(c.end, b - 1) : 0) + kStartTiles;
    *last = __builtin_amdgcn_readlane(c.end, b) - 1;
}
__device__ __forceinline__ Partials flat_partials(const AttnParams& prm, const FlatCuts& c, int kvh, int b) {
    unsigned first, last;
    flat_branch(c, b, &first, &last);
    const int w0 = flat_worker(c, first), number = w0 + b + kvh * (prm.workers + prm.B);
    return {(unsigned)number * prm.GR, 1u, (unsigned)prm.GR, flat_worker(c, last) - w0 + 1, number};
}
__device__ __forceinline__ Partials fixed_partials(const AttnParams& prm, int kvh, int b) {
    const unsigned n = prm.plan.nslots;
    return {((unsigned)kvh * prm.B + b) * prm.GR * n, n, 1u, (int)n, 0};
}

// ---------------------------------------------------------------------------------------------
// Merge of the partials of the G*R output rows of one (KV head, branch), run by the workgroup that
// delivered the last of them:  O = sum_s 2^(m_s - M) O_s / sum_s 2^(m_s - M) l_s, slots in index
// order (merge_rows below adds every SG-th slot and then the groups: its own fixed order).  4 floats per output quad; a thread takes two quads (256 apart) and eight
// slots at a time, so that 16 sixteen-byte loads are in flight together, with device scope: the partials come from
// the memory side of the L2s.
// ---------------------------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ void merge_branch(const AttnParams& prm, __amdgpu_buffer_rsrc_t rs, int kvh, int b, int tid) {
    constexpr int F4 = D / 4, EU = 2, CH = 8;
    const int ns = prm.plan.nslots;
    const int n_e = prm.GR * F4;  // output quads of this (KV head, branch)
    for (int e0 = tid; e0 < n_e; e0 += EU * kAttnThreads) {
        int rl[EU], c4[EU];
        unsigned base[EU];
        bool ok[EU];
        float M[EU], Lsum[EU];
        float4 o[EU];
#pragma unroll
        for (int q = 0; q < EU; ++q) {
            const int e = e0 + q * kAttnThreads;
            ok[q] = e < n_e;
            const int ec = ok[q] ? e : e0;
            rl[q] = ec / F4;
            c4[q] = ec - rl[q] * F4;
            base[q] = ((unsigned)kvh * prm.B * prm.GR + (unsigned)b * prm.GR + rl[q]) * ns;
            M[q] = -INFINITY;
            Lsum[q] = 0.f;
            o[q] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        for (int s0 = 0; s0 < ns; s0 += CH) {
            float2 mv[EU][CH];
            float4 pv[EU][CH];
#pragma unroll
            for (int q = 0; q < EU; ++q)
#pragma unroll
                for (int j = 0; j < CH; ++j) {
                    const bool in = s0 + j < ns;
                    mv[q][j] = in ? ws_load2<true>(rs, prm.off_ml + (base[q] + s0 + j) * 8u) : make_float2(-INFINITY, 0.f);
                    pv[q][j] = in ? ws_load4<true>(rs, prm.off_o + ((base[q] + s0 + j) * D + c4[q] * 4) * 4u)
                                  : make_float4(0.f, 0.f, 0.f, 0.f);
                }
#pragma unroll
            for (int q = 0; q < EU; ++q) {
                float Mn = M[q];
#pragma unroll
                for (int j = 0; j < CH; ++j) Mn = fmaxf(Mn, mv[q][j].x);
                const float Mu = (Mn == -INFINITY) ? 0.f : Mn;
                const float a = __builtin_amdgcn_exp2f(M[q] - Mu);
                Lsum[q] *= a;
                o[q].x *= a; o[q].y *= a; o[q].z *= a; o[q].w *= a;
#pragma unroll
                for (int j = 0; j < CH; ++j) {
                    const float w = __builtin_amdgcn_exp2f(mv[q][j].x - Mu);
                    Lsum[q] += mv[q][j].y * w;
                    o[q].x += pv[q][j].x * w; o[q].y += pv[q][j].y * w;
                    o[q].z += pv[q][j].z * w; o[q].w += pv[q][j].w * w;
                }
                M[q] = Mn;
            }
        }
#pragma unroll
        for (int q = 0; q < EU; ++q)
            if (ok[q]) store_merged(prm, kvh, b, rl[q], c4[q], o[q], M[q], Lsum[q]);
    }
}

// ---------------------------------------------------------------------------------------------
// Merge of rpm rows of a (KV head, branch) by one workgroup of THREADS threads: thread = (group of slots, row, output quad).
// A thread takes every SG-th slot, eight 16-byte loads in flight; the groups meet in LDS and are added in group order, so
// the result does not depend on timing.  A row's slots are read by many threads at once: with one thread per quad the
// reads of 64 slots were eight dependent rounds and the launch took 9 us more than at 16 slots.
// DEV: inside the attention launch: device-scope loads.  wait() comes after everything that does not depend on the partials and
// says whether the result is stored (see merger_stays).
// ---------------------------------------------------------------------------------------------
template <int D, bool DEV, int THREADS, typename Wait>
__device__ __forceinline__ void merge_rows(const AttnParams& prm, unsigned char* lds, int kvh, int b, int chunk, const Partials& parts, Wait wait) {
    constexpr int F4 = D / 4, CH = 8;
    const AttnPlan& pl = prm.plan;
    const __amdgpu_buffer_rsrc_t rs = ws_rsrc(prm);
    const int tid = threadIdx.x, ns = parts.n, rpm = pl.rpm;
    const int rshift = __builtin_ctz(rpm);
    const int c4 = tid % F4, r = (tid / F4) & (rpm - 1), sg = (tid / F4) >> rshift, SG = (THREADS / F4) >> rshift;
    const int row = chunk * rpm + r;
    float M = -INFINITY, Lsum = 0.f;
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
    const unsigned first_slot = parts.first + row * parts.row_step + sg * parts.step;
    unsigned at_o = prm.off_o + (first_slot * D + c4 * 4) * 4u, at_ml = prm.off_ml + first_slot * 8u;
    const unsigned step_o = SG * parts.step * D * 4u, step_ml = SG * parts.step * 8u;
    int mine = row < prm.GR ? ns - sg : 0;  // slots from the own first one on
    asm volatile("" : "+v"(at_o), "+v"(at_ml), "+v"(mine) : "s"(step_o), "s"(step_ml));  // computed before the wait
    const bool keep = wait();
    {
        for (int first = 0; first < ns; first += SG * CH) {
            float2 mv[CH];
            float4 pv[CH];
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                mv[j] = make_float2(-INFINITY, 0.f);
                pv[j] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (first + j * SG < ns) {  // uniform; then whoever has such a slot
                    if (first + j * SG < mine) {
                        mv[j] = ws_load2<DEV>(rs, at_ml);
                        pv[j] = ws_load4<DEV>(rs, at_o);
                    }
                    at_ml += step_ml;
                    at_o += step_o;
                }
            }
            float Mn = M;
#pragma unroll
            for (int j = 0; j < CH; ++j) Mn = fmaxf(Mn, mv[j].x);
            const float Mu = (Mn == -INFINITY) ? 0.f : Mn;
            const float a = __builtin_amdgcn_exp2f(M - Mu);
            Lsum *= a;
            o.x *= a; o.y *= a; o.z *= a; o.w *= a;
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                const float w = __builtin_amdgcn_exp2f(mv[j].x - Mu);
                Lsum += mv[j].y * w;
                o.x += pv[j].x * w; o.y += pv[j].y * w; o.z += pv[j].z * w; o.w += pv[j].w * w;
            }
            M = Mn;
        }
    }
    if (SG > 1) {  // uniform over the launch
        float4* sh_o = reinterpret_cast<float4*>(lds);
        float2* sh_ml = reinterpret_cast<float2*>(lds + THREADS * sizeof(float4));
        sh_o[tid] = o;
        sh_ml[tid] = make_float2(M, Lsum);
        __syncthreads();
        if (sg != 0) return;
        // eight groups' states requested together: one at a time is two LDS latencies a group, 1 us for eight
        float2 ml[CH];
        float4 v[CH];
        auto request = [&](int g0) {
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                const int at = tid + min(g0 + j, SG - 1) * F4 * rpm;
                ml[j] = sh_ml[at];
                v[j] = sh_o[at];
            }
        };
        float Mg = -INFINITY, l = 0.f;
        float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int g0 = SG - 1 & ~(CH - 1); g0 >= 0; g0 -= CH) {  // (the first eight last: they are added first)
            request(g0);
#pragma unroll
            for (int j = 0; j < CH; ++j) Mg = fmaxf(Mg, ml[j].x);
        }
        const float Mu = (Mg == -INFINITY) ? 0.f : Mg;
        for (int g0 = 0; g0 < SG; g0 += CH) {
            if (g0 > 0) request(g0);
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                if (g0 + j >= SG) break;
                const float w = __builtin_amdgcn_exp2f(ml[j].x - Mu);
                l += ml[j].y * w;
                t.x += v[j].x * w; t.y += v[j].y * w; t.z += v[j].z * w; t.w += v[j].w * w;
            }
        }
        M = Mg; Lsum = l; o = t;
    }
    if (row < prm.GR && keep) store_merged(prm, kvh, b, row, c4, o, M, Lsum);
}

// Cells of a merge workgroup: a flag per partial, and, behind all flags, the count that is used once it has left.
template <bool FLAT>
__device__ __forceinline__ unsigned long long* merger_flag(const AttnParams& prm, const Partials& parts, int kvh, int b, int chunk, int slot) {
    const int mpp = prm.plan.mpp;
    return prm.counters + (FLAT ? (parts.cell + slot) * mpp + chunk : ((kvh * prm.B + b) * mpp + chunk) * parts.n + slot);
}
template <bool FLAT>
__device__ __forceinline__ unsigned long long* merger_count(const AttnParams& prm, int kvh, int b, int chunk) {
    const int flags = FLAT ? prm.Hkv * (prm.workers + prm.B) * prm.plan.mpp : prm.plan.n_merge * prm.plan.nslots;
    return prm.counters + flags + (kvh * prm.B + b) * prm.plan.mpp + chunk;
}
// whoever merges takes the cells down: a captured launch is replayed with the same tag
__device__ __forceinline__ void cell_clear(unsigned long long* cell) {
    __hip_atomic_store(cell, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Counts n partials of a merge workgroup that has left; true for whoever counts the last one.  (Raised to this call's tag first, as
// the arrival cells are.)
__device__ __forceinline__ bool count_partials(const AttnParams& prm, const Partials& parts, unsigned long long* count, int n) {
    atomicMax(count, prm.tag);
    return atomicAdd(count, (unsigned long long)n) + n == prm.tag + parts.n;
}
// A merge workgroup: all its flags have come (true), or it leaves and takes its marks with it: it exchanges every flag for one, and
// so does every item that raises a flag, so each side knows from what it finds there which of the two came first.  The
// partials that were there it counts, the others are counted by the items that find a mark; who counts the last one merges.
// The answer is in LDS, so that the first loads of the merge need not wait for it.
template <bool FLAT>
__device__ __forceinline__ bool merger_stays(const AttnParams& prm, const Partials& parts, int* sh, int kvh, int b, int chunk) {
    const int tid = threadIdx.x, ns = parts.n;
    if (tid < kWave) {  // a lane per flag (flat plan: kWave at a time; otherwise ns <= kMaxSplit)
        bool all = true;
        int s0 = 0;
        do {
            unsigned long long* flag = merger_flag<FLAT>(prm, parts, kvh, b, chunk, s0 + tid);
            bool missing = s0 + tid < ns;
            // (eight times the patience: with two to a unit these workgroups start together with the items)
            for (int polls = 0; missing && polls < 8 * kWaitPolls; ++polls) {
                missing = __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != prm.tag + 1;
                if (missing) __builtin_amdgcn_s_sleep(4);
            }
            all = all && __ballot(missing) == 0;
            s0 += kWave;
        } while (FLAT && s0 < ns);
        if (!all) {
            int n = 0;
            for (s0 = 0; s0 < ns; s0 += kWave) {
                const bool there = s0 + tid < ns && atomicExch(merger_flag<FLAT>(prm, parts, kvh, b, chunk, s0 + tid), prm.tag + 2) == prm.tag + 1;
                n += __popcll(__ballot(there));
            }
            if (tid == 0 && n > 0) {
                unsigned long long* count = merger_count<FLAT>(prm, kvh, b, chunk);
                all = count_partials(prm, parts, count, n);
                if (all) cell_clear(count);
            }
            all = __ballot(all) != 0;
        }
        if (tid == 0) *sh = all;
        if (all)
            for (s0 = tid; s0 < ns; s0 += kWave) cell_clear(merger_flag<FLAT>(prm, parts, kvh, b, chunk, s0));
    }
    __syncthreads();
    return *sh != 0;
}

__device__ __forceinline__ bf16x8 load_bf16x8(const __bf16* ptr) {
    return *reinterpret_cast<const bf16x8*>(ptr);
}

// One run of keys a wavefront streams: tiles of 32 keys starting at `lo`; keys at or beyond `hi` do not belong to it.  The same
// in all lanes: bases, strides and counts stay in scalar registers.
struct KeyRun {
    const unsigned char *K, *V;
    long long stride;  // bytes from key to key
    int lo, hi;
};

// ---------------------------------------------------------------------------------------------
// bf16 partial attention
// ---------------------------------------------------------------------------------------------
// FLAT: the arguments, read again where they are needed.  What is used in every segment would otherwise stay in scalar registers
// through all of them, 150 more than there are, each moved to a lane of a vector register and back.
template <bool FLAT>
__device__ __forceinline__ const AttnParams& reread(const AttnParams& prm) {
    if constexpr (FLAT) {
        auto at = __builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(at));
        return *(const AttnParams*)at;
    } else {
        return prm;
    }
}

// (At D = 64 and one row tile, 43 KB of LDS, three workgroups fit a unit if their registers do: 44 x 16 heads x 336 + 2023 tokens with 174
// registers 63.0 us, with 168 57.7.)
template <int D, int NQT, int GROUPS, bool ONE, bool FLAT>
__global__ __launch_bounds__(kAttnThreads * GROUPS, (NQT > 1 ? 1 : D == 64 ? 3 : 2)) void attn_kernel(const AttnParams prm_) {
    const AttnParams& prm = prm_;
    // GROUPS = 2: eight wavefronts, two per SIMD.  The second group of four takes the second row tile; wavefront w of
    // either group streams the same key tiles, so the two share them: each loads half of a tile into a slab both
    // read (two slabs per pair, taking turns; the pair meets once per tile at a counter in LDS, the four pairs stay
    // independent of each other).
    static_assert(GROUPS == 1 || (GROUPS == 2 && NQT == 2), "two groups split two row tiles");
    static_assert(!ONE || (D == 128 && GROUPS == NQT), "every wavefront owns a block of the output");
    static_assert(!FLAT || (!ONE && GROUPS == NQT), "a row tile per group of four wavefronts");
    // ONE: every wavefront has one key tile at most, its own, and works on all rows' scores.
    constexpr int RUNS = ONE ? kAttnWaves * GROUPS : kAttnWaves;  // runs of key tiles of an item
    constexpr int LG = ONE ? 1 : GROUPS;                          // wavefronts that load a tile together
    constexpr int TW = ONE ? NQT : NQT / GROUPS;                  // row tiles per wavefront
    constexpr int KS = D / 16;             // MFMA k-steps of the QK^T contraction
    constexpr int DB = D / 32;             // 32-wide blocks of the head dimension
    constexpr int KSTRIDE = D * 2 + 16;    // bytes per key row of the K slab (pad: conflict-free 16-byte row reads)
    constexpr int VSTRIDE = D * 2 + 64;    // bytes per key row of the V slab (pad: conflict-free transposing reads)
    constexpr int KSLAB = kTile * KSTRIDE, VSLAB = kTile * VSTRIDE;
    constexpr int SLAB = KSLAB + VSLAB;    // bytes of LDS per wavefront while streaming
    constexpr int OSTRIDE = D + 4;         // floats per row of a wavefront's merge buffer
    constexpr int OBUF = kRowTile * OSTRIDE * 4;
    static_assert(OBUF <= SLAB, "the merge buffer reuses the wavefront's slab");
    static_assert(kRowTile * NQT * KSTRIDE <= kAttnWaves * GROUPS * SLAB, "Q may pass through the slabs");
    __shared__ __attribute__((aligned(16))) unsigned char lds[kAttnWaves * GROUPS * SLAB];
    __shared__ float2 sh_ml[ONE ? RUNS * NQT : 1][kRowTile];  // ONE: (maximum, sum) of the rows of a tile
    __shared__ float sh_m[kAttnWaves * GROUPS][kRowTile];
    __shared__ __attribute__((aligned(8))) float sh_l[kAttnWaves * GROUPS][kRowTile];
    __shared__ int sh_pair[kAttnWaves];  // GROUPS = 2: half tiles stored by the pair of wavefronts w and w + 4
    __shared__ unsigned long long sh_flat[2];  // FLAT: what one wavefront has found out about the partials of the item's last and first branch

    const int tid = threadIdx.x, wave_all = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid & (kWave - 1);
    const int grp = LG == 1 ? 0 : wave_all / kAttnWaves;         // which row tile(s) this wavefront works on
    const int wave = LG == 1 ? wave_all : wave_all % kAttnWaves;  // which of the item's runs of key tiles it streams
    const int ln = lane & 31;   // MFMA column (query row) / A row (key or d) owned by this lane
    const int hh = lane >> 5;   // which half of each 16-wide k block this lane holds
    const AttnPlan& pl = prm.plan;
    const int GR = prm.GR;

    // ---- decode the work item: private items first (one per CU starts at once), prefix items after ----
    // Order matters for latency: whatever does not depend on priv_len[b] (the prefix share, the Q
    // rows) is requested before that value is first used.
    int id = blockIdx.x;
    if (id >= pl.n_priv_items + pl.n_pre_items) {  // a merge workgroup
        id -= pl.n_priv_items + pl.n_pre_items;
        const int rest = quot(id, prm.d_hkv), kvh = id - rest * prm.Hkv;
        const int b = quot(rest, prm.d_mpp), chunk = rest - b * pl.mpp;
        Partials parts = fixed_partials(prm, kvh, b);
        bool dealt = false;
        if constexpr (FLAT) {
            const FlatCuts cuts = flat_cuts(prm, pl.fold ? prm.tiles_pre : 0, lane, prm.priv_len[min(lane, prm.B - 1)]);
            dealt = cuts.dealt;
            if (dealt) parts = flat_partials(prm, cuts, kvh, b);
            if ((dealt ? prm.flat_merge : pl.merge) != kMergeGroups || parts.n == 1) return;  // (whole rows of one item)
        }
        merge_rows<D, true, kAttnThreads * GROUPS>(prm, lds, kvh, b, chunk, parts, [&] {
            int* const stays = reinterpret_cast<int*>(sh_l);
            if (FLAT && dealt) return merger_stays<true>(prm, parts, stays, kvh, b, chunk);
            return merger_stays<false>(prm, parts, stays, kvh, b, chunk);
        });
        return;
    }
    const bool is_private = FLAT || id < pl.n_priv_items;
    int kvh, split, nsplit, rho0, rho_end, slot, b_item = 0;
    FlatCuts cuts;
    unsigned piece_end = 0;  // FLAT: where the item's piece of the head's sequence ends
    // FLAT: tiles [lo, hi) of branch b_item are the item's, now and next (b beyond the last branch: nothing more)
    struct Seg {
        int b, lo, hi;
    } seg = {0, 0, 0};
    auto seg_at = [&](int b, unsigned from) {
        const AttnParams& prm = reread<FLAT>(prm_);  // the first branch from b on of which the piece has tiles
        for (; b < prm.B; ++b) {
            unsigned first, last;
            flat_branch(cuts, b, &first, &last);
            if (first >= piece_end) break;
            const unsigned lo = max(first, from), hi = min(last + 1, piece_end);
            if (lo < hi) return Seg{b, (int)(lo - first), (int)(hi - first)};
        }
        return Seg{prm.B, 0, 0};
    };
    int piece_of = 0;  // FLAT: which of the head's items this is
    // FLAT: requested in front of everything else, as loads return in order
    const int len_lane = FLAT ? prm.priv_len[min(lane, prm.B - 1)] : 0;
    if constexpr (FLAT) {  // the fixed shares' item; what its prefix share and its Q rows are does not depend on the lengths
        piece_of = quot(id, prm.d_hkv);
        kvh = id - piece_of * prm.Hkv;
        b_item = quot(piece_of, prm.d_nsp);
        nsplit = pl.nsplit_priv;
        split = piece_of - b_item * nsplit;
        b_item = min(b_item, prm.B - 1);
        rho0 = b_item * GR;
        rho_end = rho0 + GR;
    } else if (is_private) {
        int rest = quot(id, prm.d_hkv);
        kvh = id - rest * prm.Hkv;
        const int q = quot(rest, prm.d_nsp);
        split = rest - q * pl.nsplit_priv;
        b_item = quot(q, prm.d_rgp);
        const int rg = q - b_item * pl.n_rg_priv;
        nsplit = pl.nsplit_priv;
        rho0 = b_item * GR + rg * kRowTile * NQT;
        rho_end = min((b_item + 1) * GR, rho0 + kRowTile * NQT);
        slot = pl.nsplit_pre + split;
    } else {
        id -= pl.n_priv_items;
        const int rest = quot(id, prm.d_hkv);
        kvh = id - rest * prm.Hkv;
        const int rg = quot(rest, prm.d_npre);
        split = rest - rg * pl.nsplit_pre;
        nsplit = pl.nsplit_pre;
        rho0 = rg * kRowTile * NQT;
        rho_end = min(prm.B * GR, rho0 + kRowTile * NQT);
        slot = split;
    }
    // A scalar load: requested here, waited for where it is first used (a vector load was waited for at once, to be moved to a
    // scalar register: 0.8 us in front of everything else).
    const int L_raw = is_private && !FLAT ? *((const __attribute__((address_space(4))) int32_t*)prm.priv_len + b_item) : 0;
    // The 32-key tiles of a segment are dealt round-robin to all wavefronts working on it (the 4
    // wavefronts of each of its nsplit items): every wavefront streams the same number of tiles to
    // within one whatever the segment's length, and at any moment the wavefronts of a segment read
    // neighbouring tiles, which spreads each item's traffic over the memory channels.
    const int wave_of_seg = split * RUNS + wave, waves_of_seg = nsplit * RUNS;
    // tiles of a segment of n tiles that wavefront i of those that share it gets
    auto share_of = [&](int n, int i, FastDiv d) { return i < n ? quot(n - 1 - i, d) + 1 : 0; };
    KeyRun pre, own;  // folded prefix share (may be empty); the item's own segment
    pre.K = (const unsigned char*)prm.Kpre + kvh * prm.kpre_stride_h * 2;
    pre.V = (const unsigned char*)prm.Vpre + kvh * prm.kpre_stride_h * 2;
    pre.stride = prm.kpre_stride_t * 2;
    pre.lo = wave_of_seg * kTile;
    pre.hi = prm.P;
    int step = waves_of_seg * kTile;
    const int fold_tiles = is_private && pl.fold ? prm.tiles_pre : 0;
    int n_fold = 0, n_own = 0, causal_base = 0, own_tiles = 0;
    n_fold = share_of(fold_tiles, wave_of_seg, prm.d_wpriv);

    unsigned char* kslab = lds + wave * SLAB;  // GROUPS = 2: re-pointed every tile
    unsigned char* vslab = kslab + KSLAB;
    // Tile staging: every load instruction of the wavefront covers RPI whole key rows (16 bytes per
    // lane, consecutive lanes consecutive addresses), the same pattern for K and V.
    constexpr int LPR = D / 8;             // lanes per key row
    constexpr int RPI = kWave / LPR;       // key rows per load instruction
    constexpr int NVL = kTile / RPI;       // load instructions per tile and operand
    const int v_row = lane / LPR, v_chunk = lane % LPR;
    // transposing-read address of this lane inside the V slab: 16-lane blocks cover 4 keys x 16 d
    const int blk = lane >> 4, i16 = lane & 15;
    const int tr_off = ((blk >> 1) * 4 + (i16 >> 2)) * VSTRIDE + ((blk & 1) * 16 + (i16 & 3) * 4) * 2;

    // The next tile is fetched into registers while the current one is being consumed from LDS.
    // K and V are read exactly once, so the loads carry the non-temporal hint.  A whole tile's addresses are a scalar base and
    // one 32-bit offset of the lane.
    constexpr int NLD = NVL / LG;          // load instructions per tile and operand issued by this wavefront
    u32x4 kst[NLD], vst[NLD];
    const int row0_ld = grp * RPI + v_row;
    auto fetch = [&](const KeyRun& r, int kb_) {
        if constexpr (FLAT) {
            // rows at or beyond r.hi are out of the buffer's range: they read as zeros, and are masked below
            const unsigned stride = (unsigned)r.stride, bytes = (unsigned)(r.hi - 1) * stride + D * 2;
            const __amdgpu_buffer_rsrc_t kr = __builtin_amdgcn_make_buffer_rsrc((void*)r.K, 0, (int)bytes, 0x00020000);
            const __amdgpu_buffer_rsrc_t vr = __builtin_amdgcn_make_buffer_rsrc((void*)r.V, 0, (int)bytes, 0x00020000);
            const unsigned off = ((unsigned)kb_ + row0_ld) * stride + v_chunk * 16, pitch = stride * (LG * RPI);
#pragma unroll
            for (int i = 0; i < NLD; ++i) {
                kst[i] = __builtin_amdgcn_raw_buffer_load_b128(kr, (int)(off + i * pitch), 0, 2);
                vst[i] = __builtin_amdgcn_raw_buffer_load_b128(vr, (int)(off + i * pitch), 0, 2);
            }
            return;
        }
        const unsigned char *kp = r.K + kb_ * r.stride, *vp = r.V + kb_ * r.stride;
        const long long pitch = r.stride * (LG * RPI);
        if (kb_ + kTile <= r.hi && prm.near_rows) {
            const unsigned off = (unsigned)row0_ld * (unsigned)r.stride + v_chunk * 16;
#pragma unroll
            for (int i = 0; i < NLD; ++i) {
                kst[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(kp + i * pitch + off));
                vst[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(vp + i * pitch + off));
            }
            asm volatile("");  // keeps the compiler from merging these loads with the ones below, addresses per lane
        } else {
#pragma unroll
            for (int i = 0; i < NLD; ++i) {
                int key = i * LG * RPI + row0_ld;
                key = min(key, r.hi - 1 - kb_);  // a ragged last tile re-reads its last row; masked below
                const long long off = key * r.stride + v_chunk * 16;
                kst[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(kp + off));
                vst[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(vp + off));
            }
        }
    };
    auto private_run = [&](int b, int len, KeyRun& r) {
        const AttnParams& prm = reread<FLAT>(prm_);
        const long long off = (b * prm.kpriv_stride_b + kvh * prm.kpriv_stride_h) * 2;
        r.K = (const unsigned char*)prm.Kpriv + off;
        r.V = (const unsigned char*)prm.Vpriv + off;
        r.stride = prm.kpriv_stride_t * 2;
        r.hi = len;
    };
    // FLAT: the wavefront's tiles of a segment.  Place t of a branch goes to wavefront t % kAttnWaves, so what one gets more in one
    // segment it gets less in the next.
    auto deal = [&] {
        private_run(seg.b, __builtin_amdgcn_readlane(cuts.len, seg.b), own);
        const int t = seg.lo + ((wave - seg.lo) & (kAttnWaves - 1));
        const int n = t < seg.hi ? (seg.hi - 1 - t) / kAttnWaves + 1 : 0;
        n_fold = t < fold_tiles ? min(n, (fold_tiles - 1 - t) / kAttnWaves + 1) : 0;
        n_own = n - n_fold;
        pre.lo = t * kTile;
        own.lo = (t + n_fold * kAttnWaves - fold_tiles) * kTile;
        if (n > 0) {  // (one copy of the loads for either kind)
            KeyRun r = own;
            if (n_fold > 0) r = pre;
            fetch(r, r.lo);
        }
    };
    // ---- Q fragments (B operand of S^T = K Q^T: lane = query row ln, 8 contiguous d) ----
    // Straight from memory they are 32-byte pieces of 32 rows an instruction, and come again for every wavefront: with two row
    // tiles at D = 128 as many bytes as the item's keys and values.  There the whole workgroup requests the rows once, 16
    // bytes a thread, and they pass through LDS further down (8 x 2 heads x 2560 tokens, 40 rows, 13.7 -> 13.1 us).  Elsewhere the
    // passage, a barrier behind the Q rows in front of the first scores, costs more than it saves: one row tile, 1 x 2 x 8192 9.4 -> 9.7;
    // D = 64 with half the bytes, 4 x 8 x 5643, 36 rows, 16.3 -> 16.9, 7 x 8 x 1828, 40 rows, 12.5 -> 13.1, 22 of 23 sizes 1 .. 6 %.  Rows
    // beyond the item's carry its first row again: nothing of theirs is ever stored.
    constexpr bool QLDS = NQT > 1 && D == 128;
    constexpr int QLD = kRowTile * NQT * LPR / (kAttnThreads * GROUPS);  // loads per thread
    u32x4 qst[QLD];
    bf16x8 qf[TW][KS];
    auto row_of = [&](const AttnParams& prm, int i, int& r, int& h, int& b) {  // row i of the item: position, query head, branch
        const int rc = rho0 + i < rho_end ? rho0 + i : rho0;
        b = is_private ? b_item : quot(rc, prm.d_gr);
        const int rl = rc - b * GR;
        r = quot(rl, prm.d_g);
        h = kvh * prm.G + rl - r * prm.G;
    };
    auto load_q = [&](int tid) {
        const AttnParams& prm = reread<FLAT>(prm_);
        const int lane = tid & (kWave - 1), ln = lane & 31, hh = lane >> 5;
#pragma unroll
        for (int t = 0; t < TW; ++t) {
            if (QLDS) break;
            int r, h, b;
            row_of(prm, (grp * TW + t) * kRowTile + ln, r, h, b);
            const __bf16* qp = (const __bf16*)prm.Q + b * prm.q_stride_b + r * prm.q_stride_r + h * prm.q_stride_h;
#pragma unroll
            for (int s = 0; s < KS; ++s) qf[t][s] = load_bf16x8(qp + (2 * s + hh) * 8);
        }
#pragma unroll
        for (int i = 0; i < QLD; ++i) {
            if (!QLDS) break;
            int r, h, b;
            row_of(prm, (tid + i * kAttnThreads * GROUPS) / LPR, r, h, b);
            const __bf16* qp = (const __bf16*)prm.Q + b * prm.q_stride_b + r * prm.q_stride_r + h * prm.q_stride_h;
            qst[i] = *reinterpret_cast<const u32x4*>(qp + tid % LPR * 8);
        }
    };
    auto request_first = [&] {
        if (!QLDS && n_fold > 0) fetch(pre, pre.lo);
        load_q(tid);
        if (QLDS && n_fold > 0) fetch(pre, pre.lo);
    };
    if (!FLAT) request_first();
    bool cut_first = false;  // FLAT: the first segment's partial waits to be counted
    Partials parts_first = {};
    int b_first_seg = 0, slot_first = 0;
    if constexpr (FLAT) {
        cuts = flat_cuts(prm, fold_tiles, lane, len_lane);
        if (cuts.dealt) {
            if (piece_of >= cuts.workers) return;
            const unsigned piece = flat_cut(prm, cuts, piece_of);
            piece_end = flat_cut(prm, cuts, piece_of + 1);
            seg = seg_at(__builtin_ctzll(__ballot(cuts.end > piece)), piece);
            if (seg.b >= prm.B) return;  // nothing but a branch's start
            step = kAttnWaves * kTile;
            b_item = seg.b;
            rho0 = b_item * GR;
            rho_end = rho0 + GR;
            deal();
            load_q(tid);
        } else {  // (a request in front of the decision gains nothing for these and costs dealt items up to 3 %)
            if (piece_of >= prm.B * nsplit) return;
            request_first();
        }
    }
    for (;;) {  // once, but in a flat plan's item: once per branch it has tiles of
        const int tid_all = tid;
        int tid_seg = tid;
        if constexpr (FLAT) asm volatile("" : "+v"(tid_seg));  // lane addresses are formed anew for every segment, not kept in registers
        const int tid = tid_seg, lane = tid & (kWave - 1), ln = lane & 31, hh = lane >> 5;
        const AttnParams& prm = reread<FLAT>(prm_);

        // ---- the item's own segment ----
        if (FLAT && cuts.dealt) {
            causal_base = own.hi - prm.k;
        } else if (is_private) {
            int L;
            if constexpr (FLAT) L = __builtin_amdgcn_readlane(cuts.len, b_item);
            else L = L_raw < prm.R ? prm.R : (L_raw > prm.Lmax ? prm.Lmax : L_raw);
            causal_base = L - prm.k;  // row at position r sees private keys [0, L - k + r)
            private_run(b_item, L, own);
            // The dealing goes on where the folded prefix tiles stopped: prefix and private tiles form one
            // sequence, so a wavefront that got one prefix tile more gets one private tile less.
            int i = wave_of_seg - prm.first_wave;
            i = i < 0 ? i + waves_of_seg : i;
            own.lo = i * kTile;
            own_tiles = (L - 1) / kTile + 1;
            n_own = share_of(own_tiles, i, prm.d_wpriv);
        } else {
            own = pre;
            causal_base = prm.P;  // every row sees the whole prefix
            own_tiles = prm.tiles_pre;
            n_own = share_of(own_tiles, wave_of_seg, prm.d_wpre);
        }
        const int n_tiles = n_fold + n_own;
        if (!(FLAT && cuts.dealt) && n_fold == 0 && n_tiles > 0) fetch(own, own.lo);
        int lim[TW];  // keys of this wavefront's own run visible to this lane's query row
#pragma unroll
        for (int t = 0; t < TW; ++t) {
            int r, h, b;
            row_of(prm, (grp * TW + t) * kRowTile + ln, r, h, b);
            lim[t] = min(is_private ? causal_base + r : causal_base, own.hi);
        }
        if (QLDS) {  // the slabs are free; the first tile is on its way
#pragma unroll
            for (int i = 0; i < QLD; ++i) {
                const int e = tid + i * kAttnThreads * GROUPS;
                *reinterpret_cast<u32x4*>(lds + e / LPR * KSTRIDE + e % LPR * 16) = qst[i];
            }
            __syncthreads();
#pragma unroll
            for (int t = 0; t < TW; ++t)
#pragma unroll
                for (int s = 0; s < KS; ++s)
                    qf[t][s] = *reinterpret_cast<const bf16x8*>(lds + ((grp * TW + t) * kRowTile + ln) * KSTRIDE + (2 * s + hh) * 16);
        }
        if (GROUPS > 1) {  // Q has been read from the slabs; the two wavefronts of a pair count their half tiles from here
            if (!ONE && tid < kAttnWaves) sh_pair[tid] = 0;
            __syncthreads();
        }

        // ---- results of the item: output quads (4 columns from c4 * 4 of rows row0 + q * RSTEP of a row tile) and their (max, sum) ----
        constexpr int F4 = D / 4;
        constexpr int QPT = kRowTile * F4 / kAttnThreads;  // per thread and row tile: 4 (D = 128) or 2 (D = 64)
        constexpr int RSTEP = kAttnThreads / F4;
        const __amdgpu_buffer_rsrc_t rs = ws_rsrc(prm);
        const int tig = tid % kAttnThreads;  // thread within its group of four wavefronts
        int c4 = ONE ? (wave_all % DB) * 8 + (lane & 7) : tig % F4, row0 = ONE ? lane >> 3 : tig / F4;
        float4 own_o[QPT];    // the combined quads, kept for a merge by this workgroup (kMergePair: one row tile)
        float2 own_ml[QPT];
        // Those of the first nrows rows go out: as the output itself, or as this item's partial.
        Partials parts;
        if (FLAT && cuts.dealt) {
            parts = flat_partials(prm, cuts, kvh, b_item);
            slot = piece_of + b_item - (parts.cell - kvh * (prm.workers + prm.B));
        } else {
            parts = fixed_partials(prm, kvh, b_item);
            if (FLAT) slot = split;
        }
        const int b_put = b_item, rho_put = rho0, end_put = rho_end;  // (the next segment's are set before this one's rows go out)
        auto put = [&](int tile, int nrows) {
            const AttnParams& prm = reread<FLAT>(prm_);
            const AttnPlan& pl = prm.plan;
            const int rho = rho_put + tile * kRowTile + row0;
            if (FLAT ? parts.n == 1 : pl.merge == kMergeNone) {
#pragma unroll
                for (int q = 0; q < QPT; ++q)
                    if (row0 + q * RSTEP < nrows) store_merged(prm, kvh, b_put, rho + q * RSTEP - b_put * GR, c4, own_o[q], own_ml[q].x, own_ml[q].y);
                return;
            }
            const unsigned pidx = FLAT ? parts.first + slot * parts.step + (rho - b_put * GR) * parts.row_step : ((unsigned)kvh * prm.B * GR + rho) * pl.nslots + slot;
            const unsigned step_q = RSTEP * (FLAT ? parts.row_step : pl.nslots);
            unsigned at_o = prm.off_o + (pidx * D + c4 * 4) * 4u, at_ml = prm.off_ml + pidx * 8u;
            if (pl.merge != kMergeLaunch) {
#pragma unroll
                for (int q = 0; q < QPT; ++q) {
                    if (row0 + q * RSTEP < nrows) {
                        ws_store4<true>(rs, at_o, own_o[q]);
                        if (c4 == 0) ws_store2<true>(rs, at_ml, own_ml[q]);
                    }
                    at_o += step_q * D * 4u;
                    at_ml += step_q * 8u;
                }
            } else {
#pragma unroll
                for (int q = 0; q < QPT; ++q) {
                    if (row0 + q * RSTEP < nrows) {
                        ws_store4<false>(rs, at_o, own_o[q]);
                        if (c4 == 0) ws_store2<false>(rs, at_ml, own_ml[q]);
                    }
                    at_o += step_q * D * 4u;
                    at_ml += step_q * 8u;
                }
            }
        };
        if constexpr (ONE) {
            // Nothing runs here: a wavefront publishes its tile's weights P with their maxima and sums per row, and after a barrier
            // wavefront w multiplies block w of the output (32 columns of a row tile) over the keys of ALL the item's tiles, each tile's
            // product weighted by its maximum.  (Parking every wavefront's whole output and adding the four up, as after the loop below,
            // is 1.7 us of an item whose one tile takes 0.7; this way 1.1 us for both.)
            const int nt = max(0, min(fold_tiles + own_tiles - split * RUNS, RUNS));  // tiles of the item: of wavefronts 0 .. nt - 1
            const int db = wave_all % DB, t_own = wave_all / DB;
            if (n_tiles > 0) {
                const int kbase = n_fold > 0 ? pre.lo : own.lo;
#pragma unroll
                for (int i = 0; i < NLD; ++i) *reinterpret_cast<u32x4*>(kslab + (i * RPI + v_row) * KSTRIDE + v_chunk * 16) = kst[i];
#pragma unroll
                for (int i = 0; i < NLD; ++i) *reinterpret_cast<u32x4*>(vslab + (i * RPI + v_row) * VSTRIDE + v_chunk * 16) = vst[i];
                f32x16 acc[NQT];
                bf16x8 kf[KS];
#pragma unroll
                for (int s = 0; s < KS; ++s) kf[s] = *reinterpret_cast<const bf16x8*>(kslab + ln * KSTRIDE + (2 * s + hh) * 16);
                __builtin_amdgcn_sched_barrier(0);  // all of them requested first
#pragma unroll
                for (int t = 0; t < NQT; ++t)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
#pragma unroll
                for (int s = 0; s < KS; ++s)
#pragma unroll
                    for (int t = 0; t < NQT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], qf[t][s], acc[t], 0, 0, 0);
#pragma unroll
                for (int t = 0; t < NQT; ++t) {
                    const int vis = (n_fold > 0 ? pre.hi : lim[t]) - kbase - hh * 4;
                    float mx = -INFINITY;
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        float sc = acc[t][i] * prm.scale_log2;
                        sc = (i >> 2) * 8 + (i & 3) < vis ? sc : -INFINITY;
                        acc[t][i] = sc;
                        mx = fmaxf(mx, sc);
                    }
                    mx = fmaxf(mx, shfl_xor_f(mx, 32));
                    const float m_use = (mx == -INFINITY) ? 0.f : mx;
                    bf16x8 pf[2];
                    float psum = 0.f;
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const float pv = __builtin_amdgcn_exp2f(acc[t][i] - m_use);
                        psum += pv;
                        pf[i >> 3][i & 7] = (__bf16)pv;
                    }
                    psum += shfl_xor_f(psum, 32);
                    if (hh == 0) sh_ml[wave_all * NQT + t][ln] = make_float2(mx, psum);
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)  // over the wavefront's own K tile, which nobody needs any more
                        *reinterpret_cast<bf16x8*>(kslab + ((t * 2 + kb) * kWave + lane) * 16) = pf[kb];
                }
            }
            __syncthreads();  // V tiles, P, maxima and sums are in LDS
            float2 ml[RUNS];  // of row ln of the own row tile
            f32x16 o;
            float m_row = -INFINITY, l_row = 0.f;
#pragma unroll
            for (int i = 0; i < 16; ++i) o[i] = 0.f;
#pragma unroll
            for (int j = 0; j < RUNS; ++j) ml[j] = sh_ml[j * NQT + t_own][ln];
#pragma unroll
            for (int j = 0; j < RUNS; ++j) ml[j].x = j < nt ? ml[j].x : -INFINITY;  // (beyond the last tile nobody has written)
#pragma unroll
            for (int j = 0; j < RUNS; ++j) m_row = fmaxf(m_row, ml[j].x);
            const float m_use = (m_row == -INFINITY) ? 0.f : m_row;
#pragma unroll
            for (int j = 0; j < RUNS; ++j) {
                if (j >= nt) break;
                const float w = __builtin_amdgcn_exp2f(ml[j].x - m_use);
                l_row += ml[j].y * w;
                f32x16 acc;
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) {
                    const unsigned char* ap = lds + j * SLAB + KSLAB + tr_off + (kb * 16) * VSTRIDE + db * 64;
                    union {
                        short4v s[2];
                        bf16x8 v;
                    } vf;
                    vf.s[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)(ap));
                    vf.s[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)(ap + 8 * VSTRIDE));
                    const bf16x8 pf = *reinterpret_cast<const bf16x8*>(lds + j * SLAB + ((t_own * 2 + kb) * kWave + lane) * 16);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf.v, pf, acc, 0, 0, 0);
                }
#pragma unroll
                for (int i = 0; i < 16; ++i) o[i] += acc[i] * w;
            }
            __syncthreads();  // the tiles and P have been read
            {  // the block turns through LDS, wavefront-private, into 128-byte pieces of rows
                constexpr int TSTRIDE = 36;  // floats per row of the block
                float* ob = reinterpret_cast<float*>(lds + wave_all * SLAB);
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4)
                    *reinterpret_cast<float4*>(ob + ln * TSTRIDE + q4 * 8 + hh * 4) = make_float4(o[q4 * 4 + 0], o[q4 * 4 + 1], o[q4 * 4 + 2], o[q4 * 4 + 3]);
                if (hh == 0) *reinterpret_cast<float2*>(ob + ln * TSTRIDE + 32) = make_float2(m_row, l_row);
#pragma unroll
                for (int q = 0; q < QPT; ++q) {
                    const int row = row0 + q * RSTEP;
                    own_o[q] = *reinterpret_cast<const float4*>(ob + row * TSTRIDE + (lane & 7) * 4);
                    own_ml[q] = *reinterpret_cast<const float2*>(ob + row * TSTRIDE + 32);
                }
                put(t_own, min(kRowTile, rho_end - (rho0 + t_own * kRowTile)));
            }
        } else {
            // ---- running state ----
            f32x16 oacc[TW][DB];
            float m_run[TW], l_run[TW];
#pragma unroll
            for (int t = 0; t < TW; ++t) {
                m_run[t] = -INFINITY;
                l_run[t] = 0.f;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int i = 0; i < 16; ++i) oacc[t][db][i] = 0.f;
            }

            for (int it = 0; it < n_tiles; ++it) {
                const bool folded = it < n_fold;
                const int kbase = folded ? pre.lo + it * step : own.lo + (it - n_fold) * step;
                if (GROUPS > 1) {
                    kslab = lds + ((it & 1) * kAttnWaves + wave) * SLAB;
                    vslab = kslab + KSLAB;
                }
#pragma unroll
                for (int i = 0; i < NLD; ++i) {
                    *reinterpret_cast<u32x4*>(kslab + ((i * GROUPS + grp) * RPI + v_row) * KSTRIDE + v_chunk * 16) = kst[i];
                    *reinterpret_cast<u32x4*>(vslab + ((i * GROUPS + grp) * RPI + v_row) * VSTRIDE + v_chunk * 16) = vst[i];
                }
                if (GROUPS > 1) {
                    // both halves written: the pair's counter stands at 2 * (it + 1).  Whoever gets past this has also left
                    // the tile before behind (it counted this tile only after that), so the other slab is free.
                    if (lane == 0) __hip_atomic_fetch_add(&sh_pair[wave], 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
                    for (int spin = 0; spin < (1 << 20); ++spin) {  // the partner runs the same tiles: the wait ends; bounded all the same
                        if (__hip_atomic_load(&sh_pair[wave], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) >= 2 * (it + 1)) break;
                        __builtin_amdgcn_s_sleep(1);
                    }
                }
                if constexpr (FLAT) {
                    if (it + 1 < n_tiles) {
                        KeyRun r = own;
                        if (it + 1 < n_fold) r = pre;
                        fetch(r, it + 1 < n_fold ? kbase + step : own.lo + (it + 1 - n_fold) * step);
                    }
                } else {
                    if (it + 1 < n_fold) fetch(pre, kbase + step);
                    else if (it + 1 < n_tiles) fetch(own, own.lo + (it + 1 - n_fold) * step);
                }
                // K fragments (A operand of S^T = K Q^T: lane = key row ln, 8 contiguous d)
                bf16x8 kf[KS];
#pragma unroll
                for (int s = 0; s < KS; ++s)
                    kf[s] = *reinterpret_cast<const bf16x8*>(kslab + ln * KSTRIDE + (2 * s + hh) * 16);

                bf16x8 pf[TW][2];
#pragma unroll
                for (int t = 0; t < TW; ++t) {
                    // S^T[key][query] = sum_d K[key][d] Q[query][d]
                    f32x16 acc;
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
                    for (int s = 0; s < KS; ++s) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], qf[t][s], acc, 0, 0, 0);
                    // register i of this lane is key kbase + (i/4)*8 + hh*4 + i%4 for query row ln;
                    // every row sees all of a prefix share, the causal limit applies to the own run only
                    const int vis = (folded ? pre.hi : lim[t]) - kbase - hh * 4;  // key offsets below this are visible
                    float mx = -INFINITY;
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int koff = (i >> 2) * 8 + (i & 3);
                        float sc = acc[i] * prm.scale_log2;
                        sc = koff < vis ? sc : -INFINITY;
                        acc[i] = sc;
                        mx = fmaxf(mx, sc);
                    }
                    mx = fmaxf(mx, shfl_xor_f(mx, 32));
                    const float m_new = fmaxf(m_run[t], mx);
                    const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
                    const float alpha = __builtin_amdgcn_exp2f(m_run[t] - m_use);
                    float psum = 0.f;
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const float pv = __builtin_amdgcn_exp2f(acc[i] - m_use);
                        psum += pv;
                        pf[t][i >> 3][i & 7] = (__bf16)pv;
                    }
                    l_run[t] = l_run[t] * alpha + psum;
                    m_run[t] = m_new;
                    // Rescaling the accumulators is the largest block of vector work of a tile, and once a few hundred keys have
                    // gone by a tile rarely raises any row's maximum: alpha is exactly 1 for every lane then and the whole
                    // wavefront skips it (multiplying by 1 changes nothing, so the result is the same bit for bit).
                    if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
                        for (int db = 0; db < DB; ++db)
#pragma unroll
                            for (int i = 0; i < 16; ++i) oacc[t][db][i] *= alpha;
                    }
                }
                // (The order of these reads, the K fragments' and the MFMAs is the compiler's.  Held apart by scheduling barriers, fixed shares
                // were 0.1 .. 0.9 % slower, by the form, over 60 sizes, dealt tiles 0.1 .. 1.3 %: 4 x 8 heads x 512 + 15872 tokens, 45 rows,
                // 48.5 us against 48.1.)
                union {
                    short4v s[2];
                    bf16x8 v;
                } vf[DB][2];
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb) {
                        const unsigned char* ap = vslab + tr_off + (kb * 16) * VSTRIDE + db * 64;
                        vf[db][kb].s[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)(ap));
                        vf[db][kb].s[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)(ap + 8 * VSTRIDE));
                    }
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int db = 0; db < DB; ++db)
#pragma unroll
                        for (int t = 0; t < TW; ++t)
                            oacc[t][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[db][kb].v, pf[t][kb], oacc[t][db], 0, 0, 0);
            }

            // ---- combine the 4 wavefronts' states of a row tile (fixed order) and store the item's partial ----
            // Each wavefront parks its raw state in LDS (its slab is free now); after one barrier the 256 threads
            // of a group of four wavefronts form sum_w 2^(m_w - m) O_w over their group and write the valid rows out,
            // coalesced (two groups: both row tiles at the same time).  A thread owns QPT output quads of a row
            // tile -- quad t + 256 q, t its number within the group: the same column of rows RSTEP apart -- and
            // reads everything it needs for all of them before it uses any of it.
            if (GROUPS > 1) __syncthreads();  // nobody reads a key tile any more: the slabs become merge buffers
            int tid_end = tid_all;
            if constexpr (FLAT) {  // (formed here, not kept through the tiles)
                asm volatile("" : "+v"(tid_end));
                c4 = tid_end % kAttnThreads % F4;
                row0 = tid_end % kAttnThreads / F4;
            }
            const int ln = tid_end & 31, hh = (tid_end & (kWave - 1)) >> 5;
            float* obuf = reinterpret_cast<float*>(lds + wave_all * SLAB);
#pragma unroll
            for (int t = 0; t < TW; ++t) {
                if (t > 0) __syncthreads();  // the previous row tile has been read out
                const int tile = grp * TW + t;  // row tile of the item
                const float lsum = l_run[t] + shfl_xor_f(l_run[t], 32);
                if (hh == 0) {
                    sh_m[wave_all][ln] = m_run[t];
                    sh_l[wave_all][ln] = lsum;
                }
                const int nrows = min(kRowTile, end_put - (rho_put + tile * kRowTile));
                if (ln < nrows) {  // rows beyond the item's are never read back
#pragma unroll
                    for (int db = 0; db < DB; ++db)
#pragma unroll
                        for (int q4 = 0; q4 < 4; ++q4)
                            *reinterpret_cast<float4*>(obuf + ln * OSTRIDE + db * 32 + q4 * 8 + hh * 4) =
                                make_float4(oacc[t][db][q4 * 4 + 0], oacc[t][db][q4 * 4 + 1], oacc[t][db][q4 * 4 + 2],
                                            oacc[t][db][q4 * 4 + 3]);
                }
                if constexpr (FLAT) {  // the next segment's first tile and Q rows are on their way while this one's states meet
                    if (cuts.dealt) seg = seg_at(seg.b + 1, 0);
                    else seg.b = prm.B;
                    if (seg.b < prm.B) {
                        b_item = seg.b;
                        rho0 = b_item * GR;
                        rho_end = rho0 + GR;
                        deal();
                    }
                }
                __syncthreads();
                constexpr int QB = FLAT ? QPT / 2 : QPT;  // quads at a time (FLAT: the next segment's tile and Q rows hold registers)
#pragma unroll
                for (int q0 = 0; q0 < QPT; q0 += QB) {
                    float mw[QB][kAttnWaves], lw[QB][kAttnWaves];
                    float4 ov[QB][kAttnWaves];
#pragma unroll
                    for (int q = 0; q < QB; ++q)
#pragma unroll
                        for (int w = 0; w < kAttnWaves; ++w) {
                            if (!FLAT && (q0 + q) * RSTEP >= nrows) continue;  // a whole group of rows beyond the item's (uniform)
                            const int row = min(row0 + (q0 + q) * RSTEP, nrows - 1);
                            mw[q][w] = sh_m[grp * kAttnWaves + w][row];
                            lw[q][w] = sh_l[grp * kAttnWaves + w][row];
                            ov[q][w] = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(lds + (grp * kAttnWaves + w) * SLAB) +
                                                                        row * OSTRIDE + c4 * 4);
                        }
#pragma unroll
                    for (int q = 0; q < QB; ++q) {
                        if (!FLAT && (q0 + q) * RSTEP >= nrows) continue;
                        float mg = -INFINITY;
#pragma unroll
                        for (int w = 0; w < kAttnWaves; ++w) mg = fmaxf(mg, mw[q][w]);
                        const float mg_use = (mg == -INFINITY) ? 0.f : mg;
                        float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
                        float lg = 0.f;
#pragma unroll
                        for (int w = 0; w < kAttnWaves; ++w) {
                            const float sc = __builtin_amdgcn_exp2f(mw[q][w] - mg_use);
                            o.x += ov[q][w].x * sc;
                            o.y += ov[q][w].y * sc;
                            o.z += ov[q][w].z * sc;
                            o.w += ov[q][w].w * sc;
                            lg += lw[q][w] * sc;
                        }
                        own_o[q0 + q] = o;
                        own_ml[q0 + q] = make_float2(mg, lg);
                    }
                }
                if (FLAT && seg.b < prm.B) load_q(tid);
                put(tile, nrows);
            }
        }

        if (FLAT && cuts.dealt) {
            const AttnParams& prm = reread<FLAT>(prm_);
            // Only the first and the last segment of an item can be cut; both are counted at the end, so that nothing waits for a
            // partial's way to memory in between.
            if (seg.b < prm.B) {
                if (parts.n > 1) {
                    cut_first = true;
                    parts_first = parts;
                    b_first_seg = b_put;
                    slot_first = slot;
                }
                __syncthreads();  // the states of the wavefronts have been read
                continue;
            }
            const bool cut_last = parts.n > 1;
            if (!cut_first && !cut_last) return;
            __builtin_amdgcn_s_waitcnt(0);  // the partials are in memory
            __syncthreads();
            if (prm.flat_merge == kMergeGroups) {
                const AttnPlan& pl = prm.plan;
                if (tid < kWave) {
                    bool mine = false;
                    if (cut_last && tid < pl.mpp && atomicExch(merger_flag<true>(prm, parts, kvh, b_put, tid, slot), prm.tag + 1) == prm.tag + 2)
                        mine = count_partials(prm, parts, merger_count<true>(prm, kvh, b_put, tid), 1);
                    const unsigned long long found = __ballot(mine);
                    mine = false;
                    if (cut_first && tid < pl.mpp && atomicExch(merger_flag<true>(prm, parts_first, kvh, b_first_seg, tid, slot_first), prm.tag + 1) == prm.tag + 2)
                        mine = count_partials(prm, parts_first, merger_count<true>(prm, kvh, b_first_seg, tid), 1);
                    const unsigned long long found_first = __ballot(mine);
                    if (tid == 0) {
                        sh_flat[0] = found;
                        sh_flat[1] = found_first;
                    }
                }
                __syncthreads();
                for (int e = 0; e < 2; ++e) {
                    const Partials pe = e == 0 ? parts : parts_first;
                    const int be = e == 0 ? b_put : b_first_seg;
                    for (unsigned long long left = sh_flat[e]; left; left &= left - 1) {  // uniform over the workgroup
                        const int c = __ffsll((long long)left) - 1;
                        for (int j = tid; j < pe.n; j += kAttnThreads * GROUPS) cell_clear(merger_flag<true>(prm, pe, kvh, be, c, j));
                        if (tid == 0) cell_clear(merger_count<true>(prm, kvh, be, c));
                        merge_rows<D, true, kAttnThreads * GROUPS>(prm, lds, kvh, be, c, pe, [] { return true; });
                        __syncthreads();
                    }
                }
                return;
            }
            if (tid < 2) {
                bool last = false;
                if (tid == 0 ? cut_last : cut_first) {
                    unsigned long long* cnt = prm.counters + kvh * prm.B + (tid == 0 ? b_put : b_first_seg);
                    atomicMax(cnt, prm.tag);
                    last = atomicAdd(cnt, 1ull) == prm.tag + (unsigned long long)((tid == 0 ? parts.n : parts_first.n) - 1);
                    if (last) cell_clear(cnt);
                }
                sh_flat[tid] = last;
            }
            __syncthreads();
            // partials in the order of the sequence; the last segment's own is still in registers
            const int tile0 = grp * kRowTile, nrows = min(kRowTile, GR - tile0);
            for (int e = 0; e < 2; ++e) {
                if (!sh_flat[e]) continue;  // uniform
                int row1 = row0;
                asm volatile("" : "+v"(row1));
                const Partials pe = e == 0 ? parts : parts_first;
                const int mine = e == 0 ? slot : -1;
                float2 ml[QPT];
                float4 o[QPT];
#pragma unroll
                for (int q = 0; q < QPT; ++q) {
                    ml[q] = make_float2(-INFINITY, 0.f);
                    o[q] = make_float4(0.f, 0.f, 0.f, 0.f);
                }
                constexpr int CH = 2;
                for (int j0 = 0; j0 < pe.n; j0 += CH) {
                    float2 mv[CH][QPT];
                    float4 pv[CH][QPT];
#pragma unroll
                    for (int j = 0; j < CH; ++j)
#pragma unroll
                        for (int q = 0; q < QPT; ++q) {
                            mv[j][q] = make_float2(-INFINITY, 0.f);
                            pv[j][q] = make_float4(0.f, 0.f, 0.f, 0.f);
                            if (j0 + j == mine) {
                                mv[j][q] = own_ml[q];
                                pv[j][q] = own_o[q];
                            }
                            if (j0 + j == mine || j0 + j >= pe.n || q * RSTEP >= nrows) continue;
                            const unsigned pidx = pe.first + (j0 + j) * pe.step + tile0 + min(row1 + q * RSTEP, nrows - 1);
                            mv[j][q] = ws_load2<true>(rs, prm.off_ml + pidx * 8u);
                            pv[j][q] = ws_load4<true>(rs, prm.off_o + (pidx * D + c4 * 4) * 4u);
                        }
#pragma unroll
                    for (int q = 0; q < QPT; ++q) {
                        float M = ml[q].x;
#pragma unroll
                        for (int j = 0; j < CH; ++j) M = fmaxf(M, mv[j][q].x);
                        const float Mu = (M == -INFINITY) ? 0.f : M;
                        const float a = __builtin_amdgcn_exp2f(ml[q].x - Mu);
                        ml[q].y *= a;
                        o[q].x *= a; o[q].y *= a; o[q].z *= a; o[q].w *= a;
#pragma unroll
                        for (int j = 0; j < CH; ++j) {
                            const float w = __builtin_amdgcn_exp2f(mv[j][q].x - Mu);
                            ml[q].y += mv[j][q].y * w;
                            o[q].x += pv[j][q].x * w; o[q].y += pv[j][q].y * w; o[q].z += pv[j][q].z * w; o[q].w += pv[j][q].w * w;
                        }
                        ml[q].x = M;
                    }
                }
#pragma unroll
                for (int q = 0; q < QPT; ++q)
                    if (row1 + q * RSTEP < nrows)
                        store_merged(prm, kvh, e == 0 ? b_put : b_first_seg, tile0 + row1 + q * RSTEP, c4, o[q], ml[q].x, ml[q].y);
            }
            return;
        }
        if (pl.merge == kMergeLaunch || pl.merge == kMergeNone) return;
        // ---- arrival: whoever completes the set of partials of a (KV head, branch) merges it ----
        // Every thread waits until its partial stores are acknowledged; then one thread per covered
        // branch counts the arrival in that branch's cell: raise it to (this call's tag, 0) if it holds
        // anything older, add one.  The two atomics go to one address from one thread, so they take
        // effect in program order.  The last arrival puts a zero back, which lets a captured launch
        // (same tag every time) be replayed.
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (pl.merge == kMergeGroups) {  // the item's partial is in memory: raise its flag for each of the branch's merge workgroups
            unsigned long long* sh_mine = reinterpret_cast<unsigned long long*>(sh_l);  // free again
            if (tid < kWave) {  // mpp <= rows of an item <= 64
                bool mine = false;
                if (tid < pl.mpp) {
                    if (atomicExch(merger_flag<false>(prm, parts, kvh, b_item, tid, slot), prm.tag + 1) == prm.tag + 2)  // that workgroup has left
                        mine = count_partials(prm, parts, merger_count<false>(prm, kvh, b_item, tid), 1);
                }
                const unsigned long long all = __ballot(mine);
                if (tid == 0) *sh_mine = all;
            }
            __syncthreads();
            for (unsigned long long left = *sh_mine; left; left &= left - 1) {  // uniform over the workgroup
                const int c = __ffsll((long long)left) - 1;
                if (tid < pl.nslots) cell_clear(merger_flag<false>(prm, parts, kvh, b_item, c, tid));
                if (tid == 0) cell_clear(merger_count<false>(prm, kvh, b_item, c));
                merge_rows<D, true, kAttnThreads * GROUPS>(prm, lds, kvh, b_item, c, parts, [] { return true; });
                __syncthreads();
            }
            return;
        }
        int* sh_last = reinterpret_cast<int*>(sh_l);  // free again; kAttnWaves * kRowTile >= rows of an item
        const int rows_per_item = kRowTile * NQT;
        const int b_first = quot(rho0, prm.d_gr), b_last = quot(rho_end - 1, prm.d_gr);
        const int nb = b_last - b_first + 1;  // <= rows_per_item
        if (tid < nb) {
            const int b = b_first + tid;
            int expected = pl.n_rg_priv * pl.nsplit_priv;
            if (pl.nsplit_pre > 0) {
                const int rg_lo = (b * GR) / rows_per_item, rg_hi = ((b + 1) * GR - 1) / rows_per_item;
                expected += pl.nsplit_pre * (rg_hi - rg_lo + 1);
            }
            unsigned long long* cnt = prm.counters + kvh * prm.B + b;
            atomicMax(cnt, prm.tag);
            const unsigned long long seen = atomicAdd(cnt, 1ull);
            const int last = (seen == prm.tag + (unsigned long long)(expected - 1));
            if (last) atomicExch(cnt, 0ull);
            sh_last[tid] = last;
        }
        __syncthreads();
        if (NQT == 1 && pl.merge == kMergePair) {  // the item's rows are the branch's rows; slot order, as everywhere
            if (!sh_last[0]) return;
            float2 mv[QPT];
            float4 pv[QPT];
            const int n_rows = rho_end - rho0;
#pragma unroll
            for (int q = 0; q < QPT; ++q) {
                if (q * RSTEP >= n_rows) continue;
                const unsigned pidx = ((unsigned)kvh * prm.B * GR + rho0 + min(row0 + q * RSTEP, n_rows - 1)) * 2 + (1 - slot);
                mv[q] = ws_load2<true>(rs, prm.off_ml + pidx * 8u);
                pv[q] = ws_load4<true>(rs, prm.off_o + (pidx * D + c4 * 4) * 4u);
            }
#pragma unroll
            for (int q = 0; q < QPT; ++q) {
                const int row = row0 + q * RSTEP;
                if (row >= n_rows) continue;
                const float2 ma = slot == 0 ? own_ml[q] : mv[q], mb = slot == 0 ? mv[q] : own_ml[q];
                const float4 oa = slot == 0 ? own_o[q] : pv[q], ob = slot == 0 ? pv[q] : own_o[q];
                const float M = fmaxf(ma.x, mb.x), Mu = (M == -INFINITY) ? 0.f : M;
                const float wa = __builtin_amdgcn_exp2f(ma.x - Mu), wb = __builtin_amdgcn_exp2f(mb.x - Mu);
                store_merged(prm, kvh, b_item, row, c4,
                             make_float4(oa.x * wa + ob.x * wb, oa.y * wa + ob.y * wb, oa.z * wa + ob.z * wb, oa.w * wa + ob.w * wb),
                             M, ma.y * wa + mb.y * wb);
            }
            return;
        }
        if (GROUPS == 1 || tid < kAttnThreads)  // the merge is written for 256 threads
            for (int j = 0; j < nb; ++j)
                if (sh_last[j]) merge_branch<D>(prm, rs, kvh, b_first + j, tid);  // uniform over the workgroup
        __builtin_amdgcn_s_waitcnt(0);
        return;
    }
}

// ---------------------------------------------------------------------------------------------
// Separate merge launch, used when items cover rows of several branches or branches have several row groups: grid (row chunks of a (KV head, branch), KV head x branch).
// ---------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(kAttnThreads) void attn_merge_kernel(const AttnParams prm) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[kAttnThreads * (sizeof(float4) + sizeof(float2))];
    const int b = quot(blockIdx.y, prm.d_hkv);
    const int kvh = blockIdx.y - b * prm.Hkv;
    merge_rows<D, false, kAttnThreads>(prm, lds, kvh, b, blockIdx.x, fixed_partials(prm, kvh, b), [] { return true; });
}

// ---------------------------------------------------------------------------------------------
// fp32 path: one workgroup per output row, fp32 arithmetic throughout (no matrix cores).
// A key row is D / 4 lanes of 16 bytes, so one load of a wavefront covers KPL = 256 / D keys; a wavefront takes chunks of
// 4 * KPL keys (every fourth chunk is its own), K and V of a chunk requested together, and keeps a flash-style running state
// per group of D / 4 lanes -- the groups' and the wavefronts' states meet at the end.  Bound by memory latency at the sizes
// this path exists for: with one key of 4 bytes a lane at a time, a chain of two loads, six shuffles and two exponentials per
// key, 2 branches x 4 heads x 96 keys took 13.4 us; in chunks it takes 5.3.
// ---------------------------------------------------------------------------------------------
typedef u32x4 u32x4_any __attribute__((aligned(4)));  // fp32 rows start at any multiple of 4 bytes
__device__ __forceinline__ float4 load_f4_any(const float* p) {
    const u32x4 u = *reinterpret_cast<const u32x4_any*>(p);
    return make_float4(__uint_as_float(u[0]), __uint_as_float(u[1]), __uint_as_float(u[2]), __uint_as_float(u[3]));
}
template <int D>
__global__ __launch_bounds__(kAttnThreads) void attn_f32_kernel(const AttnParams prm) {
    constexpr int LPK = D / 4;         // lanes per key row
    constexpr int KPL = kWave / LPK;   // keys per load instruction
    constexpr int NJ = 4;              // load instructions per chunk and operand
    constexpr int CHUNK = NJ * KPL;
    __shared__ __attribute__((aligned(16))) float sh_acc[kAttnWaves][D];
    __shared__ float sh_ml[kAttnWaves][2];
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid & (kWave - 1);
    const int grp = lane / LPK, c4 = lane % LPK;
    const long long row = blockIdx.x;
    const int h = (int)(row % prm.Hq);
    const long long br = row / prm.Hq;
    const int r = (int)(br % prm.R), b = (int)(br / prm.R);
    const int kvh = h / prm.G;
    int L = prm.priv_len[b];
    L = L < prm.R ? prm.R : (L > prm.Lmax ? prm.Lmax : L);
    const int n_priv = L - prm.k + r;
    const int n = prm.P + n_priv;
    const float scale = prm.scale_log2 * 0.69314718055994530942f;  // back to the natural-log scale
    const float4 qv = load_f4_any((const float*)prm.Q + (long long)b * prm.q_stride_b + (long long)r * prm.q_stride_r +
                                  (long long)h * prm.q_stride_h + c4 * 4);
    const long long pre = (long long)kvh * prm.kpre_stride_h + c4 * 4;
    const long long prv = (long long)b * prm.kpriv_stride_b + (long long)kvh * prm.kpriv_stride_h + c4 * 4;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    float m = -INFINITY, l = 0.f;
    for (int j0 = wave * CHUNK; j0 < n; j0 += kAttnWaves * CHUNK) {
        float4 kv[NJ], vv[NJ];
#pragma unroll
        for (int i = 0; i < NJ; ++i) {
            int j = j0 + i * KPL + grp;
            j = j < n ? j : n - 1;  // keys past the end re-read the last one; masked below
            const bool prefix = j < prm.P;
            const long long off = prefix ? pre + (long long)j * prm.kpre_stride_t : prv + (long long)(j - prm.P) * prm.kpriv_stride_t;
            kv[i] = load_f4_any((const float*)(prefix ? prm.Kpre : prm.Kpriv) + off);
            vv[i] = load_f4_any((const float*)(prefix ? prm.Vpre : prm.Vpriv) + off);
        }
        float s[NJ], mx = m;
#pragma unroll
        for (int i = 0; i < NJ; ++i) {
            s[i] = qv.x * kv[i].x + qv.y * kv[i].y + qv.z * kv[i].z + qv.w * kv[i].w;
#pragma unroll
            for (int d = LPK / 2; d >= 1; d >>= 1) s[i] += shfl_xor_f(s[i], d);
            s[i] = j0 + i * KPL + grp < n ? s[i] * scale : -INFINITY;
            mx = fmaxf(mx, s[i]);
        }
        const float mu = mx == -INFINITY ? 0.f : mx;  // no key yet, or none but NaN scores: those stay NaN
        const float alpha = expf(m - mu);
        l *= alpha;
        acc.x *= alpha; acc.y *= alpha; acc.z *= alpha; acc.w *= alpha;
#pragma unroll
        for (int i = 0; i < NJ; ++i) {
            const float pv = expf(s[i] - mu);
            if (j0 + i * KPL + grp >= n) vv[i] = make_float4(0.f, 0.f, 0.f, 0.f);  // an infinity counts once
            l += pv;
            acc.x += pv * vv[i].x; acc.y += pv * vv[i].y; acc.z += pv * vv[i].z; acc.w += pv * vv[i].w;
        }
        m = mx;
    }
    // the wavefront's groups of lanes
#pragma unroll
    for (int d = LPK; d < kWave; d <<= 1) {
        const float mo = shfl_xor_f(m, d), lo = shfl_xor_f(l, d);
        const float4 ao = make_float4(shfl_xor_f(acc.x, d), shfl_xor_f(acc.y, d), shfl_xor_f(acc.z, d), shfl_xor_f(acc.w, d));
        const float M = fmaxf(m, mo);
        const float wa = m == -INFINITY ? 0.f : expf(m - M), wb = mo == -INFINITY ? 0.f : expf(mo - M);
        l = l * wa + lo * wb;
        acc.x = acc.x * wa + ao.x * wb; acc.y = acc.y * wa + ao.y * wb; acc.z = acc.z * wa + ao.z * wb; acc.w = acc.w * wa + ao.w * wb;
        m = M;
    }
    if (lane == 0) {
        sh_ml[wave][0] = m;
        sh_ml[wave][1] = l;
    }
    if (grp == 0) *reinterpret_cast<float4*>(&sh_acc[wave][c4 * 4]) = acc;
    __syncthreads();
    if (tid < D) {
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < kAttnWaves; ++w) M = fmaxf(M, sh_ml[w][0]);
        float Lsum = 0.f, o = 0.f;
#pragma unroll
        for (int w = 0; w < kAttnWaves; ++w) {
            const float wgt = (sh_ml[w][0] == -INFINITY) ? 0.f : expf(sh_ml[w][0] - M);
            Lsum += sh_ml[w][1] * wgt;
            o += sh_acc[w][tid] * wgt;
        }
        float* op = (float*)prm.O + (long long)b * prm.o_stride_b + (long long)r * prm.o_stride_r +
                    (long long)h * prm.o_stride_h;
        op[tid] = o / Lsum;
        if (prm.lse && tid == 0) prm.lse[row] = M + logf(Lsum);
    }
}

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
static int fill_desc(const lotts_attn_desc* in, lotts_attn_desc* d) {
    if (!in) return LOTTS_ERR_NULL;
    *d = *in;
    if (d->dtype != LOTTS_F32 && d->dtype != LOTTS_BF16) return LOTTS_ERR_DTYPE;
    if (d->B < 1 || d->k < 0 || d->Hq < 1 || d->Hkv < 1 || d->Hq % d->Hkv != 0) return LOTTS_ERR_SHAPE;
    if (d->D != 64 && d->D != 128) return LOTTS_ERR_SHAPE;
    if (d->P < 0 || d->Lmax < d->k + 1) return LOTTS_ERR_SHAPE;
    if (!(d->scale >= 0.0f) || d->scale > 3.0e38f) return LOTTS_ERR_SHAPE;
    const long long R = d->k + 1, D = d->D;
    // 0 selects the dense layout
    if (!d->q_stride_h) d->q_stride_h = D;
    if (!d->q_stride_r) d->q_stride_r = (long long)d->Hq * D;
    if (!d->q_stride_b) d->q_stride_b = R * d->Hq * D;
    if (!d->o_stride_h) d->o_stride_h = D;
    if (!d->o_stride_r) d->o_stride_r = (long long)d->Hq * D;
    if (!d->o_stride_b) d->o_stride_b = R * d->Hq * D;
    if (!d->kpre_stride_t) d->kpre_stride_t = D;
    if (!d->kpre_stride_h) d->kpre_stride_h = (long long)d->P * D;
    if (!d->kpriv_stride_t) d->kpriv_stride_t = D;
    if (!d->kpriv_stride_h) d->kpriv_stride_h = (long long)d->Lmax * D;
    if (!d->kpriv_stride_b) d->kpriv_stride_b = (long long)d->Hkv * d->Lmax * D;
    const long long st[] = {d->q_stride_b, d->q_stride_r, d->q_stride_h, d->kpre_stride_h, d->kpre_stride_t,
                            d->kpriv_stride_b, d->kpriv_stride_h, d->kpriv_stride_t, d->o_stride_b, d->o_stride_r,
                            d->o_stride_h};
    for (long long s : st) {
        if (s < 0) return LOTTS_ERR_SHAPE;
        if (d->dtype == LOTTS_BF16 && (s % 8) != 0) return LOTTS_ERR_SHAPE;  // 16-byte vector loads
    }
    if (d->q_stride_h < D || d->o_stride_h < D || d->kpre_stride_t < D || d->kpriv_stride_t < D) return LOTTS_ERR_SHAPE;
    const long long rows = (long long)d->B * R * d->Hq;
    if (rows > 0x7fffffffLL / 8) return LOTTS_ERR_SHAPE;
    if ((long long)d->B * d->Hkv > kMaxCounters) return LOTTS_ERR_SHAPE;
    return LOTTS_OK;
}

// Bytes of workspace for a checked descriptor; 0 when the geometry cannot be served (partials are
// addressed with 32-bit byte offsets, arrivals per cell are counted in 16 bits).
static size_t workspace_need(const lotts_attn_desc& d, bool may_be_flat = true) {
    if (d.dtype == LOTTS_F32) return 256;  // the fp32 path needs none; keep the pointer non-NULL
    const AttnPlans pl = plan_attention(d, may_be_flat);
    const long long arrivals = pl.flat ? pl.workers : (long long)pl.n_rg_priv * pl.nsplit_priv + (long long)pl.nsplit_pre * (pl.n_rg_priv + 1);
    if (arrivals >= (1 << kTagShift)) return 0;
    const size_t bytes = workspace_layout(d, pl, nullptr, nullptr);
    return bytes < 0x7fffffffULL ? bytes : 0;
}

// Everything after the argument checks that both entry points share: plan, parameters, launches.
// `workspace` holds at least workspace_need(d, may_be_flat) bytes.
static int launch_attention(const lotts_attn_desc& d, const void* Q, const void* Kpre, const void* Vpre,
                            const void* Kpriv, const void* Vpriv, const int32_t* priv_len, void* O, float* lse,
                            void* workspace, hipStream_t s, bool may_be_flat) {
    AttnParams prm;
    prm.Q = Q; prm.Kpre = Kpre; prm.Vpre = Vpre; prm.Kpriv = Kpriv; prm.Vpriv = Vpriv;
    prm.priv_len = priv_len;
    prm.O = O; prm.lse = lse;
    prm.B = d.B; prm.k = d.k; prm.R = d.k + 1; prm.Hq = d.Hq; prm.Hkv = d.Hkv; prm.G = d.Hq / d.Hkv;
    prm.GR = prm.G * prm.R; prm.D = d.D; prm.P = d.P; prm.Lmax = d.Lmax;
    prm.d_g = fast_div(prm.G);
    const double scale = d.scale > 0.0f ? (double)d.scale : 1.0 / sqrt((double)d.D);
    prm.scale_log2 = (float)(scale * 1.4426950408889634074);
    prm.q_stride_b = d.q_stride_b; prm.q_stride_r = d.q_stride_r; prm.q_stride_h = d.q_stride_h;
    prm.kpre_stride_h = d.kpre_stride_h; prm.kpre_stride_t = d.kpre_stride_t;
    prm.kpriv_stride_b = d.kpriv_stride_b; prm.kpriv_stride_h = d.kpriv_stride_h; prm.kpriv_stride_t = d.kpriv_stride_t;
    prm.o_stride_b = d.o_stride_b; prm.o_stride_r = d.o_stride_r; prm.o_stride_h = d.o_stride_h;
    prm.tag = 0;
    const long long rows = (long long)d.B * prm.R * d.Hq;

    if (d.dtype == LOTTS_F32) {
        prm.plan = AttnPlan{};
        prm.ws = nullptr; prm.ws_bytes = 0; prm.off_o = prm.off_ml = 0; prm.counters = nullptr;
        if (d.D == 64)
            LOTTS_LAUNCH(attn_f32_kernel<64>, dim3((unsigned)rows), dim3(kAttnThreads), s, prm);
        else
            LOTTS_LAUNCH(attn_f32_kernel<128>, dim3((unsigned)rows), dim3(kAttnThreads), s, prm);
        return check_launch();
    }

    const AttnPlans pl = plan_attention(d, may_be_flat);
    prm.plan = pl;
    size_t off_o, off_ml;
    const size_t total = workspace_layout(d, pl, &off_o, &off_ml);
    prm.ws = workspace;
    prm.ws_bytes = (unsigned)total;
    prm.off_o = (unsigned)off_o;
    prm.off_ml = (unsigned)off_ml;
    prm.counters = static_cast<unsigned long long*>(workspace);
    prm.d_hkv = fast_div(d.Hkv); prm.d_nsp = fast_div(pl.nsplit_priv); prm.d_rgp = fast_div(pl.n_rg_priv);
    prm.d_npre = fast_div(pl.nsplit_pre > 0 ? pl.nsplit_pre : 1); prm.d_mpp = fast_div(pl.mpp > 0 ? pl.mpp : 1); prm.d_gr = fast_div(prm.GR);
    prm.d_wpriv = fast_div(pl.runs * pl.nsplit_priv); prm.d_wpre = fast_div(pl.runs * (pl.nsplit_pre > 0 ? pl.nsplit_pre : 1));
    prm.tiles_pre = ceil_div(d.P, kTile);
    prm.first_wave = pl.fold ? prm.tiles_pre % (pl.runs * pl.nsplit_priv) : 0;
    const long long tile_span = (1LL << 31) / (2 * kTile);  // elements from key to key
    prm.near_rows = d.kpriv_stride_t < tile_span && d.kpre_stride_t < tile_span;
    prm.tag = (g_call_tag.fetch_add(1, std::memory_order_relaxed) + 1) << kTagShift;
    prm.flat = pl.flat; prm.workers = pl.workers; prm.flat_merge = pl.flat_merge;
    prm.d_workers = fast_div(pl.workers > 0 ? pl.workers : 1);
    const long long items = (long long)pl.n_pre_items + pl.n_priv_items + pl.n_merge;
    if (items > 0x7fffffffLL) return LOTTS_ERR_SHAPE;
    const dim3 grid((unsigned)items), block(kAttnThreads);
    const dim3 block2(2 * kAttnThreads);
    if (pl.one) {
        if (d.D == 128 && pl.nqt == 1) LOTTS_LAUNCH((attn_kernel<128, 1, 1, true, false>), grid, block, s, prm);
        else LOTTS_LAUNCH((attn_kernel<128, 2, 2, true, false>), grid, block2, s, prm);
    } else if (pl.flat) {
        if (d.D == 128 && pl.nqt == 1) LOTTS_LAUNCH((attn_kernel<128, 1, 1, false, true>), grid, block, s, prm);
        else if (d.D == 128) LOTTS_LAUNCH((attn_kernel<128, 2, 2, false, true>), grid, block2, s, prm);
        else if (pl.nqt == 1) LOTTS_LAUNCH((attn_kernel<64, 1, 1, false, true>), grid, block, s, prm);
        else LOTTS_LAUNCH((attn_kernel<64, 2, 2, false, true>), grid, block2, s, prm);
    } else {
        if (d.D == 128 && pl.nqt == 1) LOTTS_LAUNCH((attn_kernel<128, 1, 1, false, false>), grid, block, s, prm);
        else if (d.D == 128) LOTTS_LAUNCH((attn_kernel<128, 2, 2, false, false>), grid, block2, s, prm);
        else if (pl.nqt == 1) LOTTS_LAUNCH((attn_kernel<64, 1, 1, false, false>), grid, block, s, prm);
        else LOTTS_LAUNCH((attn_kernel<64, 2, 2, false, false>), grid, block2, s, prm);
    }
    if (pl.merge == kMergeLaunch) {
        const int rc = check_launch();
        if (rc != LOTTS_OK) return rc;
        const dim3 mgrid((unsigned)pl.mpp, (unsigned)(d.Hkv * d.B));
        if (d.D == 128) LOTTS_LAUNCH(attn_merge_kernel<128>, mgrid, block, s, prm);
        else LOTTS_LAUNCH(attn_merge_kernel<64>, mgrid, block, s, prm);
    }
    return check_launch();
}

// Pointer checks of both entry points (everything but the workspace).
static int check_pointers(const lotts_attn_desc& d, const void* Q, const void* Kpre, const void* Vpre, const void* Kpriv,
                          const void* Vpriv, const int32_t* priv_len, const void* O) {
    if (!Q || !Kpriv || !Vpriv || !priv_len || !O) return LOTTS_ERR_NULL;
    if (d.P > 0 && (!Kpre || !Vpre)) return LOTTS_ERR_NULL;
    const uintptr_t align_or = (uintptr_t)Q | (uintptr_t)Kpre | (uintptr_t)Vpre | (uintptr_t)Kpriv | (uintptr_t)Vpriv |
                               (uintptr_t)O;
    if (d.dtype == LOTTS_BF16 && (align_or & 15) != 0) return LOTTS_ERR_SHAPE;
    if ((align_or & 3) != 0) return LOTTS_ERR_SHAPE;
    return LOTTS_OK;
}

// ---------------------------------------------------------------------------------------------
// Scratch of the entry point that allocates nothing: arrival cells and partials live in a
// file-scope device array instead of a caller's workspace.  Each GPU holds its own copy of the array
// at its own address for the life of the process; in host code the array's name is only a handle, so
// the address is looked up once per device (with that device current) and the kernels get the
// looked-up pointer, exactly as they get a workspace pointer.  Zero-initialised when the code object
// is loaded, which is what the arrival cells want at first use.
// ---------------------------------------------------------------------------------------------
constexpr size_t kScratchBytes = (size_t)16 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
constexpr int kMaxDevices = 64;
static std::atomic<void*> g_scratch_ptr[kMaxDevices];

static int scratch_of_current_device(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return LOTTS_ERR_LAUNCH;
    void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!ptr) {  // first call on this device; two threads racing here look up the same address
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return LOTTS_ERR_LAUNCH;
        g_scratch_ptr[dev].store(ptr, std::memory_order_release);
    }
    *out = ptr;
    return LOTTS_OK;
}

}  // namespace lotts

extern "C" size_t verify_attention_workspace_bytes(const lotts_attn_desc* desc) {
    using namespace lotts;
    lotts_attn_desc d;
    if (fill_desc(desc, &d) != LOTTS_OK) return 0;
    return workspace_need(d);
}

extern "C" int verify_attention(const lotts_attn_desc* desc, const void* Q, const void* Kpre, const void* Vpre,
                                const void* Kpriv, const void* Vpriv, const int32_t* priv_len, void* O, float* lse,
                                void* workspace, size_t workspace_bytes, void* stream) {
    using namespace lotts;
    lotts_attn_desc d;
    int rc = fill_desc(desc, &d);
    if (rc != LOTTS_OK) return rc;
    rc = check_pointers(d, Q, Kpre, Vpre, Kpriv, Vpriv, priv_len, O);
    if (rc != LOTTS_OK) return rc;
    if (!workspace) return LOTTS_ERR_NULL;
    const size_t need = workspace_need(d);
    if (need == 0) return LOTTS_ERR_SHAPE;  // a geometry whose partials the 32-bit offsets cannot address
    // Fixed shares have fewer partials than dealt tiles: a buffer sized for more branches, whose plan may not be flat, holds those of fewer.
    const bool may_be_flat = workspace_bytes >= need;
    if (!may_be_flat && workspace_bytes < workspace_need(d, false)) return LOTTS_ERR_WORKSPACE;
    if (((uintptr_t)workspace & (d.dtype == LOTTS_BF16 ? 15 : 3)) != 0) return LOTTS_ERR_SHAPE;
    return launch_attention(d, Q, Kpre, Vpre, Kpriv, Vpriv, priv_len, O, lse, workspace, (hipStream_t)stream, may_be_flat);
}

extern "C" int verify_attention_noalloc(const lotts_attn_desc* desc, const void* Q, const void* Kpre, const void* Vpre,
                                        const void* Kpriv, const void* Vpriv, const int32_t* priv_len, void* O,
                                        float* lse, void* stream) {
    using namespace lotts;
    lotts_attn_desc d;
    int rc = fill_desc(desc, &d);
    if (rc != LOTTS_OK) return rc;
    rc = check_pointers(d, Q, Kpre, Vpre, Kpriv, Vpriv, priv_len, O);
    if (rc != LOTTS_OK) return rc;
    const size_t need = workspace_need(d);
    if (need == 0) return LOTTS_ERR_SHAPE;
    if (need > kScratchBytes) return LOTTS_ERR_WORKSPACE;  // beyond the built-in scratch: use verify_attention
    void* ptr = nullptr;
    rc = scratch_of_current_device(&ptr);
    if (rc != LOTTS_OK) return rc;
    return launch_attention(d, Q, Kpre, Vpre, Kpriv, Vpriv, priv_len, O, lse, ptr, (hipStream_t)stream, true);
}
