// lsm_compact: single-pass k-way merge of sorted runs (paper section 2.2, compaction).
//
// Kernels, on one stream:
//   init_kernel       clears the per-call scratch (tile status words) and writes the
//                     first and last partition rows (where the runs are searched directly: done by
//                     the partition launch instead; an input of one tile needs neither).
//   partition         multi-sequence selection over the k runs for every interior tile
//                     boundary.  For target rank r it finds the key x with the largest
//                     L(x) = sum_j |{e in run j : e.key < x}| that is still <= r, and stores
//                     the k lower bounds.  Boundaries are therefore key-aligned (all versions
//                     of a key fall into the same tile) and tile sizes are within k of the
//                     nominal size.  One run: multiples of the spacing (partition_one_kernel).  Two
//                     runs: bisection on the merge path (partition_two_*).
//                     Inputs of up to 512 tiles take sample keys as boundaries instead of exact
//                     ranks (partition_ranked_kernel: tile sizes vary, within the capacity).
//                     Larger ones search the runs, one wave per boundary (partition_kernel,
//                     partition_many_kernel), most of them between rows that are ranked first
//                     (partition_rows_kernel, partition_between_kernel).  Long inputs of more than 16 runs
//                     first bracket every boundary, a group of lanes each, on a copy of every
//                     32nd key (sample_kernel, sample_rank_kernel, sample_fine_kernel) and search
//                     the runs only inside the brackets (bracket_partition_kernel).
//   merge_short_kernel  inputs of up to a tile per compute unit (below: what it does differently).
//   merge_kernel      one workgroup per tile: every thread loads its share of the tile's entries
//                     into registers, 16-byte surrogates (14 key bytes + index) are merged in LDS
//                     by ceil(log2 k) rounds of stable two-way merge-path merges, the newest
//                     version of every key is marked, the rest (and winning tombstones when the
//                     output is the last level) dropped, survivors are counted with a block
//                     prefix sum, the tile's output offset comes from a decoupled look-back over
//                     the tile status words, and the survivors leave through an LDS stage with
//                     contiguous 16-byte stores.  Every input byte is read once and every
//                     surviving byte written once.
#include <hip/hip_runtime.h>

#include <string.h>

#include <mutex>
#include <type_traits>

#include "lsm_common.h"

namespace lsm {

constexpr int kMergeThreads = 512;
constexpr int kMergeItems = 4;
constexpr int kTileCap = kMergeThreads * kMergeItems;  // entries per tile
constexpr int kRoundItems = 4;                         // outputs per thread in a merge round
// Largest boundary spacing in merged rank for k runs: a tile is at most k - 1 entries longer than this (keys are unique
// inside a run, so the boundary key's rank is less than k short of its target), which is the tile capacity.
__host__ __device__ inline uint64_t tile_nominal(uint32_t k) { return (uint64_t)kTileCap - k; }
// An input of fewer tiles than the chip has compute units is cut into shorter ones: a tile is a serial chain (load, merge
// rounds, look-back, store) on one compute unit, and with fewer entries every step of it has less to move.
// Long tiles throughout against this: 4 x 16,384 entries 37.8 -> 36.2 us, a write buffer of 100,001 128.5 -> 122.6, 96
// driver flushes 3.59 -> 3.22 ms.  256 as the shortest is within 4 % of it, 960 up to 2 us slower for three runs or more.
constexpr uint64_t kFillTiles = 256;
constexpr uint64_t kMinSpacing = 512;
// Up to a tile for every compute unit the tile is merged by merge_short_kernel: with one workgroup on a compute unit what counts is
// the chain of dependent steps, not how much the unit gets done, and one thread per entry has the shorter chain.  Both forms, us a call:
// 2 runs of 4,000 entries in all 15.2 / 13.5, 60,000 17.9 / 14.7, 300,000 24.0 / 21.4, 500,000 27.6 / 27.1; 8 runs, 4,000 23.8 /
// 18.5, 100,000 27.3 / 21.9; 24 runs, 100,000 35.2 / 31.1.  More tiles take turns, and merge_kernel gets more of them done.
constexpr int kShortThreads = 1024;
constexpr int kShortItems = kTileCap / kShortThreads;
static_assert(kShortTiles == kFillTiles, "a tile per compute unit");
// `jobs` compactions in the launch: each may have a tile that is not full.
inline uint32_t fill_spacing(uint64_t total, uint32_t jobs = 1) {
    const uint64_t tiles = kFillTiles - (jobs < kFillTiles / 4 ? jobs - 1 : 0), even = (total + tiles - 1) / tiles;
    if (even < kMinSpacing) return (uint32_t)kMinSpacing;
    return even < (uint64_t)kTileCap ? (uint32_t)even : (uint32_t)kTileCap;
}
__host__ __device__ inline uint32_t tile_spacing(uint32_t fill, uint32_t k) { return fill < (uint32_t)tile_nominal(k) ? fill : (uint32_t)tile_nominal(k); }
// Boundaries at ranked samples (three runs or more, see ranked_row): the inputs that 512 tiles hold, two on every compute unit.
// They have 512 entries at least; more tiles than that would run in turns, and the work of the launch grows with the samples,
// which get denser as a tile's mean size comes closer to its capacity: beyond kMostSamples the other searches are as fast
// (partition and merge, sampled against the window search: 16 runs, 600k entries 55 / 77 us with 10,300 samples, 750k 70 / 79
// with 19,700, 900k 130 / 83 with 47,000; 64 runs of 300k in all 64 / 57 us with 23,000; 48 runs 40 / 57 with 16,700).
constexpr uint64_t kRankedTiles = 512;
// No more than a tile for every compute unit where they have up to kShortMean entries in the mean: 512 / 256 tiles, 200k entries, 4
// runs 26.4 / 23.3 us, 8 runs 29.8 / 27.5, 24 runs 39.6 / 33.8; 300k 28.7 / 28.1, 31.9 / 30.2, 43.2 / 44.4; 400k 30.1 / 29.7, 33.8 /
// 36.7, 48.4 / 92 (samples would be too many).  A tile of more than kShortThreads entries gives its threads two each, and every later
// tile waits for it: samples are dense enough that there is none, if kShortSamples do.  4,000 entries, 8 / 16 / 24 runs, any tile up to the
// capacity 17.7 / 24.3 / 26.0 us, none so long 16.6 / 18.7 / 20.2.  With 16,384 samples the partition loses what the tiles gain
// (130k, 16 runs 28.6 -> 26.9, but 200k 29.3 -> 40.1).
constexpr uint64_t kShortMean = 1280;
constexpr uint64_t kShortSamples = 6144;
constexpr uint64_t kMostSamples = 20480;
constexpr uint32_t kMinStride = 8;
// Samples from one ranked sample to the next (sampled partition): ranked rows + boundaries between them, 16 x 4M entries 51 + 124
// us with 128, 25 + 132 with 256; 24 x 1M 21 + 92 and 12 + 100; 4 x 4M 8.7 + 34 and 6.7 + 33.
constexpr uint32_t kRowStride = 256;
constexpr uint64_t kSampleStride = 32;  // one key in 32 is copied for the sampled partition
// How the boundaries of three runs or more are found where ranked samples are too many.
//   A wave per boundary over the whole runs (partition_kernel): up to four runs, below kSampledMinTiles tiles; more than kFewRuns runs, below that.
//   Rows first (partition_rows_kernel, partition_between_kernel): some entries of every run are ranked in all runs, and a boundary's wave searches
//     between two of these rows.  Up to kRowsRuns runs of any length, up to kFewRuns below kSampledMinTiles tiles.
//   On a copy of every 32nd key (sample_kernel and the three after it): what is left.
// Whole calls, us; mixed runs, runs one after the other, runs in turns of 100 entries, the same keys in every run.
//   A wave per boundary / rows: 4 runs, 2M entries 87 86 93 74 / 86 75 93 71, 5M 187 174 193 153 / 183 158 186 142; 8 runs, 1M 68 70 79 60 / 64 49 68 56, 4M
//   168 169 174 149 / 167 138 167 142; 16 runs, 2M 124 145 154 117 / 115 86 119 108, 8M 374 368 407 390 / 339 277 344 347; 24 runs, 1M 105 155 158 95 /
//   95 64 148 81, 4M 232 274 310 245 / 225 171 289 233.
//   Samples / rows: 4 runs, 50M 1632 1532 1633 1228 / 1618 1456 1608 1231; 8 runs, 32M 1163 1069 1180 920 / 1142 971 1139 951; 16 runs, 16M 667 655
//   787 630 / 636 527 659 661, 67M 2546 2359 2775 2501 / 2496 2146 2449 2585, and the same at 80M and 120M; 8 runs of 200M in all 6611 6217 6764 5473 /
//   6519 5974 6644 5577; 3 runs of 400M within 1 %.  But 17 runs, 10M 505 473 637 466 / 516 399 545 508, 24 runs, 16M 759 715 964 764 / 791 614 886 831: two
//   lanes per run instead of four.
constexpr uint64_t kSampledMinTiles = 2048;
constexpr uint32_t kRowsRuns = 16;
constexpr uint64_t kRowsMost = (1ull << 32) - (1ull << 20);  // positions in 32 bits
// Entries from row to row.  With fewer, more samples are ranked, with more, more is left between them.  1,024 / 2,048 / 4,096 / 8,192 / 16,384, mixed
// and in turns: 5 runs, 1.2M entries 78 78 / 86 79 / 83 82 / 84 82 / -; 16 runs, 1.5M 103 106 / 102 107 / 101 133 / 101 132 / -, 3M 176 177 / 163 164 / 156
// 182 / 155 177 / -, 8M 388 410 / 365 370 / 348 398 / 340 373 / 342 355, 40M 1723 1706 / 1621 1581 / 1550 1571 / 1551 1516 / 1512 1456; 4 runs, 16M 577 572 / 551
// 549 / 541 535 / 547 537 / 549 539, 40M 1386 1381 / 1323 1336 / 1302 1284 / 1313 1301 / 1282 1338.
inline uint32_t row_entries(uint64_t total, uint32_t k) {
    if (total < 1500000) return 1024;
    if (total < 2500000) return 2048;
    return total < 8000000 ? 4096 : k <= 4 ? 8192 : 16384;
}
constexpr uint32_t kSpinLimit = 1u << 22;              // polls of one look-back window before giving up

struct Header {  // first 256 bytes of the workspace
    uint32_t unused;
    uint32_t validate_status;
    uint64_t reserved[31];
};
static_assert(kRoundItems == 4, "the register merge network is written for four outputs");
static_assert(sizeof(Header) == 256, "header is 256 bytes");

// A bare 32-byte key: one sample of a run.
struct SampleKey {
    uint4 q[2];
};

struct SampleTable {
    SampleKey* ptr[LSM_MAX_RUNS];
    uint64_t m[LSM_MAX_RUNS];  // samples of run j = ceil(n[j] / kSampleStride)
};

struct Workspace {
    uint64_t n_tiles;
    Header* hdr;
    uint64_t* status;   // [n_tiles]
    uint64_t* splits;   // [(n_tiles + 1) * k]; the sampled partition first keeps its ranked rows there
    uint64_t* ywin;     // [2 * (n_tiles - 1) * k] sample-space brackets of every boundary; or, in the room of these and the samples, ranked rows and their sums
    SampleTable st;
    uint4* clear;       // zeroed by the partition launch for a later kernel of the caller
    uint64_t clear_n;
    uint64_t* fresh;    // kShortTiles status words of the caller's own, zeroed by the partition launch (may be null)
    uint32_t spacing;   // boundary spacing of the direct partition (batch form: to be capped by tile_spacing for each job)
    uint32_t stride, per_tile, samples;  // entries from sample to sample, samples from boundary to boundary, in all (single form; see ranked_row)
};

__host__ __device__ inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

__global__ void init_kernel(RunTable rt, Workspace ws, uint64_t n_tiles, uint64_t* n_out) {
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    if (i == 0) {
        ws.hdr->validate_status = 0;
        if (n_tiles == 0) *n_out = 0;
    }
    for (uint64_t t = i; t < n_tiles; t += stride) ws.status[t] = 0;
    if (i < rt.k) {
        ws.splits[i] = 0;
        ws.splits[n_tiles * rt.k + i] = run_len(rt, (uint32_t)i);
    }
}

// ---------------------------------------------------------------------------------------
// Partition: a group of G lanes (G = smallest power of two >= k) works on one selection
// problem, lane j of the group owns sequence j, and a wave handles 64/G problems at once.
// For a target rank r the problem is: among the records still inside [lo_j, hi_j) of every
// sequence, find the key x with the largest L(x) = sum_j |{e in sequence j : e.key < x}| that
// is still <= r, and return the k lower bounds of x.  Each step takes a record of the widest
// range as pivot, every lane finds the pivot's lower bound in its own range, and the sum over
// the group decides which side of the pivot survives.  The pivot always leaves its range and
// the widest range at least halves every third step, so the loop ends after at most
// 3 * k * log2(longest sequence) steps whatever the input.
//
// The ranges need not be cuts of one key: it is enough that lo_j <= (the answer's lower bound
// in j) <= hi_j and that the answer itself lies inside its own sequence's range.  Lower bounds
// are then clamped into the ranges, which never changes on which side of r a sum falls.
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ uint64_t group_sum_u64(uint64_t v, int group) {
    for (int off = group >> 1; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}
__device__ __forceinline__ uint64_t group_max_u64(uint64_t v, int group) {
    for (int off = group >> 1; off > 0; off >>= 1) {
        uint64_t o = __shfl_xor(v, off, kWave);
        v = o > v ? o : v;
    }
    return v;
}

constexpr int kTailKeys = 4;        // ranges this short are finished from registers
constexpr int kTailKeysCached = 2;  // the same for searches on the cached sample arrays

// One step's bookkeeping once every lane has its lower bound lb (and whether the record there equals the pivot).
__device__ __forceinline__ void select_update(uint64_t& lo, uint64_t& hi, uint64_t& best, const uint64_t lb, const bool eq,
                                              const uint64_t mid, const bool is_src, const bool active, const bool own,
                                              const uint64_t r, const int group) {
    const uint64_t total = group_sum_u64(own ? lb : 0, group);
    if (!active) return;
    // on sorted input the pivot's own lane has lb == mid; the clamps only matter for inputs that
    // break the precondition, where they still shrink the widest range
    const uint64_t ub = lb + (eq ? 1 : 0);
    if (total <= r) {
        best = lb;
        lo = (is_src && ub < mid + 1) ? mid + 1 : ub;
    } else {
        hi = (is_src && lb > mid) ? mid : lb;
    }
}

template <bool kCached, typename E>
__device__ __forceinline__ uint64_t select_split(const E* run, uint64_t lo, uint64_t hi, const uint64_t r, const bool own,
                                                 const int member, const int group, const int group_base) {
    uint64_t best = lo;
    // on the cached sample arrays a shorter tail keeps the kernel at 64 registers (8 waves per SIMD), worth more there
    constexpr int kTail = kCached ? kTailKeysCached : kTailKeys;
    // phase 1: pivots and lower bounds from memory, until every range of the group is at most kTail long
    for (uint32_t iter = 0;; iter++) {
        const uint64_t width = hi - lo;
        const uint64_t widest = group_max_u64((width << 6) | (uint64_t)member, group);
        const bool active = (widest >> 6) > (uint64_t)kTail;
        if (__ballot(active) == 0) break;
        const int src = (int)(widest & 63);
        // bisection steps take the roundest position of the middle quarter when the records are in HBM
        // (a position other searches read too), the plain middle when they are cached
        uint64_t mid = lo + (width >> 1);
        if (!kCached && width) mid = tree_mid(lo + ((3 * width) >> 3), lo + ((5 * width) >> 3) + 1);
        if (iter % 3 != 2) {
            // interpolation steps: the candidates are the merged ranks [sum lo, sum hi); aim the pivot at
            // the same fraction of the widest range as a target rank is of that interval.  The target
            // is r minus, then r plus, a margin of the order of the estimate's standard deviation (the
            // square root of the interval: one such on the cached sample arrays, a quarter where every probe
            // is an HBM access and a missed bracket costs less than a wide one - both measured), so that two
            // steps bracket x from both sides.  Every third step is a bisection step, which keeps the worst
            // case logarithmic.
            const uint64_t rank_lo = group_sum_u64(own ? lo : 0, group), rank_hi = group_sum_u64(own ? hi : 0, group);
            uint64_t span = rank_hi - rank_lo, ahead = r > rank_lo ? r - rank_lo : 0;
            const uint64_t margin = span ? (1ull << ((64 - __builtin_clzll(span)) >> 1)) >> (kCached ? 0 : 2) : 0;
            if (iter % 3 == 0) ahead = ahead > margin ? ahead - margin : 0;
            else ahead += margin;
            if (ahead > span) ahead = span;
            const int shift = span >> 31 ? 64 - __builtin_clzll(span) - 31 : 0;
            span >>= shift;
            ahead >>= shift;
            uint64_t frac = span ? (ahead << 32) / span : 0;  // 32.32 fixed point in [0, 1]
            if (frac > 0xFFFFFFFFull) frac = 0xFFFFFFFFull;
            if (rank_hi - rank_lo >= 256 && width > 0 && width <= 0xFFFFFFFFull) {  // few candidates left: plain bisection
                mid = lo + ((width * frac) >> 32);
                if (mid >= hi) mid = hi - 1;
                // the roundest position within 1/16 of the range around the aim: likely read before, or again later
                const uint64_t slack = width >> 4;
                if (!kCached) mid = tree_mid(mid - lo > slack ? mid - slack : lo, hi - mid > slack + 1 ? mid + slack + 1 : hi);
            }
        }
        Key pivot = {{0, 0, 0, 0}};
        if (active && member == src) pivot = load_key(run + mid);
        for (int w = 0; w < 4; w++) pivot.w[w] = __shfl(pivot.w[w], group_base + src, kWave);
        uint64_t lb = lo;
        bool eq = false;
        if (own && active) lb = kCached ? lower_bound_eq4(run, lo, hi, pivot, eq) : lower_bound_eq(run, lo, hi, pivot, eq);
        select_update(lo, hi, best, lb, eq, mid, member == src, active, own, r, group);
    }
    // phase 2: the same steps on the at most kTail keys per range that are left, held in registers
    const uint64_t base = lo;
    const int cnt = (int)(hi - lo);  // <= kTail
    Key kk[kTail];
    for (int i = 0; i < kTail; i++) kk[i] = i < cnt ? load_key(run + base + i) : Key{{0, 0, 0, 0}};
    for (;;) {
        const uint64_t width = hi - lo;
        const uint64_t widest = group_max_u64((width << 6) | (uint64_t)member, group);
        const bool active = (widest >> 6) != 0;
        if (__ballot(active) == 0) break;
        const int src = (int)(widest & 63);
        const uint64_t mid = lo + (width >> 1);
        const int at = (int)(mid - base);
        Key pivot = kk[0];
        for (int i = 1; i < kTail; i++)
            if (at == i) pivot = kk[i];
        for (int w = 0; w < 4; w++) pivot.w[w] = __shfl(pivot.w[w], group_base + src, kWave);
        uint64_t lb = base;
        for (int i = 0; i < kTail; i++) lb += (i < cnt && key_less(kk[i], pivot)) ? 1 : 0;
        lb = lb < lo ? lo : (lb > hi ? hi : lb);
        bool eq = false;
        for (int i = 0; i < kTail; i++) eq = eq || (lb < hi && lb == base + i && key_equal(kk[i], pivot));
        select_update(lo, hi, best, lb, eq, mid, member == src, active, own, r, group);
    }
    return best;
}

// Two runs: the boundary of merged rank r by bisection on the merge path - how many entries of `a` are among the first r
// of the merged order (equal keys: a's first) - with two independent reads per step, then moved back by one entry when
// the two versions of a key would fall on either side of it.  Same result as select_split (the lower bounds of the key x
// with the largest L(x) <= r) in log2 of the shorter run's length dependent steps instead of a pivoting selection.
__device__ __forceinline__ void split_two(const lsm_entry_t* a, const uint64_t na, const lsm_entry_t* b, const uint64_t nb, const uint64_t r,
                                          uint64_t& ia, uint64_t& ib) {
    const uint64_t d = r < na + nb ? r : na + nb;
    uint64_t lo = d > nb ? d - nb : 0, hi = d < na ? d : na;  // the count lies in [lo, hi]
    while (lo < hi) {
        const uint64_t mid = lo + (hi - lo + 1) / 2;  // lo < mid <= hi, so d - mid < nb
        // mid entries of a fit among the first d iff a[mid - 1] does not come after b[d - mid]
        if (!key_less(load_key(b + (d - mid)), load_key(a + mid - 1))) lo = mid;
        else hi = mid - 1;
    }
    ia = lo;
    ib = d - lo;
    // a's version of a key just before the boundary and b's just after it: the key starts one entry earlier
    if (ia > 0 && ib < nb && key_equal(load_key(a + ia - 1), load_key(b + ib))) ia--;
}

// ---------------------------------------------------------------------------------------
// The same selection by one wave per boundary, for inputs of up to a few thousand boundaries: there the pivoting above
// is bound by its chain of some ninety dependent reads (4 x 16,384 entries: 68 us; 8 x 500,000: 178 us).
// The window [lo_j, hi_j) of run j is kept by the lanes with lane % group == j, so all of the wave's 64 / group groups
// know all windows.  A round reads `m` evenly spaced records of every window at once (one round trip) into LDS.  A
// record P with y_j records of window j below it has a lower bound there between xmin_j and xmax_j (the neighbouring
// records' positions), so Lmin(P) <= L(P) <= Lmax(P): if Lmax <= r, P is not above the answer and every lo_j moves up to
// its xmin_j; if Lmin > r, every hi_j moves down to its xmax_j.  Every step in LDS tries one record per group, evenly
// spaced in the window with the most records left, until the records that are left are in doubt; the next round reads
// the windows that remain more finely.  Once no window is longer than m all bounds are exact.
// Usually some three gaps per run remain of a window.  Where the runs' keys lie so that less than half of the
// candidates goes, one pivot is placed exactly (searched in the runs themselves), which halves the widest window.
// More than 32 runs (kMany): a round has eight records per run and a step one pivot.  Runs that cover different keys then
// cost a step each where the widest window was the first of many as wide, and a round each where a window's ends were not
// among its records (a run beyond the answer was known only to within a gap).  The pivot's window is therefore any of those
// within a quarter of the widest, by a hash of its number and the step, and a window's first and last records are read.  64
// runs of 65,536 entries in all: one after the other 381 -> 96 us, in turns of 100 entries 415 -> 178, mixed 78 -> 66 (the
// constant group).  With fewer runs, where a step tries several pivots and a round reads more of a window, the ends cost
// mixed runs up to 9 % and are left out.
// ---------------------------------------------------------------------------------------
// Sum / max over aligned groups of 1, 2, 4, ... 64 lanes; every lane of the wave must call.  Up to 16 lanes by DPP.
template <typename Op>
__device__ __forceinline__ uint32_t group_reduce(uint32_t v, int group, Op op) {
    if (group > 1) v = op(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true));    // lane ^ 1
    if (group > 2) v = op(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true));    // lane ^ 2
    if (group > 4) v = op(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, true));   // mirrored inside 8 lanes
    if (group > 8) v = op(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xF, 0xF, true));   // mirrored inside 16 lanes
    if (group > 16) v = op(v, (uint32_t)__shfl_xor((int)v, 16, kWave));
    if (group > 32) v = op(v, (uint32_t)__shfl_xor((int)v, 32, kWave));
    return v;
}
__device__ __forceinline__ uint32_t group_sum_u32(uint32_t v, int group) {
    return group_reduce(v, group, [](uint32_t a, uint32_t b) { return a + b; });
}
__device__ __forceinline__ uint32_t group_max_u32(uint32_t v, int group) {
    return group_reduce(v, group, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
}

constexpr uint32_t kFewRuns = 32;
constexpr int kGapBits = 9;  // fractional bits of a distance between records
static_assert(kSampledMinTiles * kTileCap <= (1ull << (32 - kGapBits)), "positions of more than kFewRuns runs in 32 bits");

template <int kPerLane>  // records a lane reads per round
struct WindowShared {
    ulonglong2 lo[kWave * kPerLane + kWave];  // key bytes 0..15 of record i of window j at j * (m + 1) + i: lists start in different banks
    ulonglong2 hi[kWave * kPerLane + kWave];  // key bytes 16..31
};

// The lower bound in run j = lane % group of the key with the largest L <= r, which lies in [lo, hi].  The whole wave calls; lanes without
// a run pass lo = hi = 0.  Fewer than 2^32 entries in all.
template <int kPerLane, bool kMany>
__device__ __forceinline__ uint32_t window_split(WindowShared<kPerLane>& s, const lsm_entry_t* run, uint32_t lo, uint32_t hi, const uint32_t r,
                                                 const int group_log_any) {
    const int group_log = kMany ? 6 : group_log_any;
    const int lane = threadIdx.x & (kWave - 1), group = 1 << group_log;
    const uint32_t j = lane & (group - 1), g = (uint32_t)lane >> group_log;
    const int groups_log = 6 - group_log;
    const uint32_t groups = 1u << groups_log, m = groups * kPerLane;
    ulonglong2* const my_lo = s.lo + j * (m + 1);
    ulonglong2* const my_hi = s.hi + j * (m + 1);
    uint32_t turn = 0;
    for (;;) {
        const uint32_t width = hi - lo;
        const bool exact = __ballot(width > m) == 0;
        const uint32_t count = width < m ? width : m;
        // record i of the window
        const uint32_t gap = width <= m ? 1 << (kMany ? kGapBits : 0) : (kMany ? ((width - 1) << kGapBits) / (m - 1) : width / m);
        const uint32_t first = lo + (!kMany && width > m ? gap >> 1 : 0);
        auto position = [&](uint32_t i) {
            if (kMany) return i + 1 < count ? lo + ((i * gap) >> kGapBits) : hi - 1;
            return first + i * gap;
        };
        __syncthreads();  // one wave: the last round's reads are done
        {
            uint4 a[kPerLane], b[kPerLane];
#pragma unroll
            for (int c = 0; c < kPerLane; c++) {
                const uint32_t i = g + c * groups;
                if (i < count) {
                    const uint4* e = reinterpret_cast<const uint4*>(run + position(i));
                    a[c] = load_global_u4(e);
                    b[c] = load_global_u4(e + 1);
                }
            }
#pragma unroll
            for (int c = 0; c < kPerLane; c++) {
                const uint32_t i = g + c * groups;
                if (i < count) {
                    const Key key = key_from_raw(a[c], b[c]);
                    my_lo[i] = make_ulonglong2(key.w[0], key.w[1]);
                    my_hi[i] = make_ulonglong2(key.w[2], key.w[3]);
                }
            }
        }
        __syncthreads();
        uint32_t left = 0, right = count;         // records of this window that are not settled
        uint32_t next_lo = lo, next_hi = hi;
        for (;; turn++) {
            const uint32_t open = right - left;
            uint32_t order = open;
            if (kMany && open != 0) {  // length to two bits behind the first, a hash: distinct windows in a different order every step
                const uint32_t bits = 32 - __builtin_clz(open);
                order = (((bits << 2) | (((open << 2) >> (bits - 1)) & 3)) << 6) | (((j + turn) * 0x9E3779B1u) >> 26);
            }
            const uint32_t chosen = (uint32_t)__builtin_amdgcn_readfirstlane((int)group_max_u32((order << 6) | j, group));
            const uint32_t jw = chosen & 63, w = kMany ? (uint32_t)__builtin_amdgcn_readlane((int)open, (int)jw) : chosen >> 6;
            if (w == 0) break;
            const uint32_t from = (uint32_t)__builtin_amdgcn_readlane((int)left, (int)jw);
            const uint32_t at_w = from + (w >= groups ? ((2 * g + 1) * w) >> (groups_log + 1) : (g < w ? g : w - 1));
            const ulonglong2 plo = s.lo[jw * (m + 1) + at_w], phi = s.hi[jw * (m + 1) + at_w];
            const bool own = j == jw;
            uint32_t y = left, end = right;
            bool same = own;  // record y is the pivot's key: a version of it in another run, or the pivot itself
            if (own) y = end = at_w;
            while (y < end) {
                const uint32_t mid = (y + end) >> 1;
                const ulonglong2 a = my_lo[mid];
                bool less = (a.x < plo.x) | ((a.x == plo.x) & (a.y < plo.y)), equal = false;
                if ((a.x == plo.x) & (a.y == plo.y)) {
                    const ulonglong2 b = my_hi[mid];
                    less = (b.x < phi.x) | ((b.x == phi.x) & (b.y < phi.y));
                    equal = (b.x == phi.x) & (b.y == phi.y);
                }
                y = less ? mid + 1 : y;
                end = less ? end : mid;
                same = less ? same : equal;
            }
            const uint32_t xmax = own || y < count ? position(y) : hi;
            const uint32_t xmin = own ? xmax : (y > 0 ? position(y - 1) + 1 : lo);
            const uint64_t below = __ballot(group_sum_u32(xmax, group) <= r), above = __ballot(group_sum_u32(xmin, group) > r);
            if ((below | above) == 0) break;  // all in doubt
            // the groups' records ascend: the last one that is not above the answer, the first one that is
            if (below != 0) {
                const int src = ((63 - __builtin_clzll(below)) & ~(group - 1)) | (int)j;
                left = (uint32_t)__shfl((int)(y + (same ? 1 : 0)), src, kWave);
                next_lo = (uint32_t)__shfl((int)xmin, src, kWave);
            }
            if (above != 0) {
                const int src = (__builtin_ctzll(above) & ~(group - 1)) | (int)j;
                right = (uint32_t)__shfl((int)y, src, kWave);
                next_hi = (uint32_t)__shfl((int)xmax, src, kWave);
            }
            right = right < left ? left : right;  // crossed bounds, here and below: only inputs that break the precondition
        }
        if (exact) return next_lo;
        next_hi = next_hi < next_lo ? next_lo : next_hi;
        const bool slow = group_sum_u32(next_hi - next_lo, group) > group_sum_u32(hi - lo, group) / 2;
        lo = next_lo;
        hi = next_hi;
        if (__builtin_amdgcn_readfirstlane(slow ? 1 : 0)) {
            const uint32_t len_w = group_max_u32(hi - lo, group);
            const int src = (int)__builtin_ctzll(__ballot(hi - lo == len_w));
            const uint32_t mid = (uint32_t)__shfl((int)(lo + len_w / 2), src, kWave);
            const lsm_entry_t* run_w = reinterpret_cast<const lsm_entry_t*>(__shfl(reinterpret_cast<uint64_t>(run), src, kWave));
            if (len_w > 1) {  // true: some window was longer than m
                const Key pivot = load_key(run_w + mid);
                bool eq;
                uint32_t lb = (uint32_t)lower_bound_eq4(run, lo, hi, pivot, eq);
                if (lane == src || (int)j == (src & (group - 1))) lb = mid;
                if (group_sum_u32(lb, group) <= r) lo = lb;
                else hi = lb;
            }
        }
    }
}

// split_two by a whole wave (all lanes get the result): 64 counts of [lo, hi] are tried together, so a step leaves a
// 64th of the range.
__device__ __forceinline__ void split_two_wave(const lsm_entry_t* a, const uint64_t na, const lsm_entry_t* b, const uint64_t nb, const uint64_t r,
                                               uint64_t& ia, uint64_t& ib) {
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint64_t d = r < na + nb ? r : na + nb;
    uint64_t lo = d > nb ? d - nb : 0, hi = d < na ? d : na;
    while (lo < hi) {
        const uint64_t w = hi - lo;
        auto tried = [&](uint64_t l) { return lo + ((l + 1) * w + kWave - 1) / kWave; };  // ascending, the last is hi
        const uint64_t mid = tried(lane);
        const bool fits = !key_less(load_key(b + (d - mid)), load_key(a + mid - 1));  // mid entries of a are among the first d: true up to the count
        const uint32_t n = __popcll(__ballot(fits));
        const uint64_t new_lo = n > 0 ? tried(n - 1) : lo, new_hi = n < (uint32_t)kWave ? tried(n) - 1 : hi;
        lo = new_lo;
        hi = new_hi;
    }
    ia = lo;
    ib = d - lo;
    if (ia > 0 && ib < nb && key_equal(load_key(a + ia - 1), load_key(b + ib))) ia--;
}

// ---------------------------------------------------------------------------------------
// Boundaries at sample keys, for small inputs of three runs or more: one launch in which every boundary is found without the
// others.  Every `stride`-th entry of every run is a sample.  A wave takes one sample c and counts the samples before it in
// every run (equal keys: those of lower runs count as before it), 64 / group lanes per run, each step one evenly spaced record
// per lane.  The sum t is c's place in the order of all samples, known without sorting them, and distinct for every sample:
// the samples with t = per_tile * row are the boundaries, and their waves go on to the lower bounds of c in the entries
// between two samples.  Tile sizes vary, but a tile holds per_tile samples, and less than `stride` entries of a run before
// its first one: at most (per_tile + k - 1) * stride entries, which the host keeps within the capacity.
// What bounds it: four or five dependent reads.  The window search below, three rounds of reads and some fifteen dependent
// searches in LDS, against this one: 4 x 16,384 entries 16.5 -> 4.5 us, 24 x 2,730 44 -> 7.3, 8 x 37,500 24.5 -> 6.5, 16 runs of
// 8,000 entries one after the other 39.8 -> 4.7; tiles of uneven size cost the merge up to 2 us of it (4 x 16,384: 17.4 -> 18.1).
// len: run lengths; upper: what the launch counts samples by (the same, or an upper bound: samples beyond a run's end come last, and
// their rows are the runs' ends).  kApart: a run's second sample is at `offset`
// (no more than stride) and the others follow from there; sums gets the sum of every row.
// ---------------------------------------------------------------------------------------
constexpr uint32_t kDies = 8;
__host__ __device__ inline uint32_t sample_apart(uint32_t i, uint32_t offset, uint32_t stride) { return i > 0 ? offset + (i - 1) * stride : 0; }
__host__ __device__ inline uint32_t samples_apart(uint32_t n, uint32_t offset, uint32_t stride) { return (n > 0) + (n > offset ? (n - offset + stride - 1) / stride : 0); }
template <typename E, bool kApart = false>  // E: entries, or bare keys
__device__ __forceinline__ void ranked_row(const E* run, const uint32_t len, const uint32_t upper, const uint32_t p, const uint32_t k,
                                            const int group_log, const uint32_t stride, const uint32_t per_tile, uint64_t* splits,
                                            const uint32_t offset = 0, uint32_t* sums = nullptr) {
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const int lanes_log = 6 - group_log;
    const uint32_t lanes = 1u << lanes_log, member = lane >> lanes_log, part = lane & (lanes - 1), shift = member << lanes_log;
    const uint64_t lanes_mask = lanes == (uint32_t)kWave ? ~0ull : (1ull << lanes) - 1;
    const bool head = part == 0 && member < k;
    auto samples_of = [&](uint32_t n) { return kApart ? samples_apart(n, offset, stride) : (n + stride - 1) / stride; };
    const uint32_t real = samples_of(len), launched = samples_of(upper);
    // which run the sample belongs to: samples are numbered run by run; kApart: the first eighth of each run's, and so on, an eighth for a die
    const uint32_t die = kApart ? p % kDies : 0, nth = kApart ? p / kDies : p;
    const uint32_t begin = kApart ? (uint32_t)((uint64_t)launched * die / kDies) : 0;
    const uint32_t mine = kApart ? (uint32_t)((uint64_t)launched * (die + 1) / kDies) - begin : launched;
    const uint32_t upto = wave_scan_u32(head ? mine : 0);
    const uint32_t own = (uint32_t)__popcll(__ballot(head && upto <= nth));
    if (kApart && own >= k) return;  // the eighths are not all of the same size
    const int own_lane = (int)(own << lanes_log);
    const uint32_t index = nth - (uint32_t)__shfl((int)(upto - mine - begin), own_lane, kWave);
    const uint32_t own_real = (uint32_t)__shfl((int)real, own_lane, kWave);
    uint32_t t, lo = 0, hi = 0;
    Key key = {{0, 0, 0, 0}};
    if (index < own_real) {
        const E* own_run = reinterpret_cast<const E*>(__shfl(reinterpret_cast<uint64_t>(run), own_lane, kWave));
        const uint32_t own_offset = kApart ? (uint32_t)__shfl((int)offset, own_lane, kWave) : 0;
        const uint32_t own_at = kApart ? sample_apart(index, own_offset, stride) : index * stride;
        const uint4* e = reinterpret_cast<const uint4*>(own_run + own_at);
        const uint4 k0 = load_global_u4(e), k1 = load_global_u4(e + 1);
        key = key_from_raw(k0, k1);
        // first record in [lo, hi) of those that place() gives that is not before the key
        auto search = [&](auto place, bool equal_is_before) {
            while (__ballot(lo < hi) != 0) {
                const uint32_t w = hi - lo;
                auto tried = [&](uint32_t m) { return lo + (((2 * m + 1) * w) >> (lanes_log + 1)); };  // ascending with m, below hi
                bool before = false;
                if (lo < hi) {
                    const uint4* q = reinterpret_cast<const uint4*>(run + place(tried(part)));
                    const uint4 q0 = load_global_u4(q), q1 = load_global_u4(q + 1);
                    const Key other = key_from_raw(q0, q1);
                    before = equal_is_before ? !key_less(key, other) : key_less(other, key);
                }
                const uint32_t n = (uint32_t)__popcll((__ballot(before) >> shift) & lanes_mask);  // the first n are before
                if (lo < hi) {
                    const uint32_t new_lo = n > 0 ? tried(n - 1) + 1 : lo, new_hi = n < lanes ? tried(n) : hi;
                    lo = new_lo;
                    hi = new_hi < new_lo ? new_lo : new_hi;  // only runs that are not sorted
                }
            }
        };
        lo = member == own ? index : 0;
        hi = member == own ? index : (member < k ? real : 0);
        auto sample_at = [&](uint32_t i) { return kApart ? sample_apart(i, offset, stride) : i * stride; };
        search([&](uint32_t i) { return kApart ? (uint64_t)sample_apart(i, offset, stride) : (uint64_t)i * stride; }, member < own);
        t = wave_scan_u32(head ? lo : 0);
        t = (uint32_t)__builtin_amdgcn_readlane((int)t, kWave - 1);
        if (t % per_tile != 0) return;
        // the lower bound: after the last sample before the key, or that sample if its key is the same
        hi = min(sample_at(lo), len);
        lo = lo > 0 ? sample_at(lo - 1) : 0;
        if (member == own) lo = hi = own_at;
        search([](uint32_t i) { return (uint64_t)i; }, false);
    } else {  // beyond the run's end
        const uint32_t surplus = wave_scan_u32(head ? launched - real : 0), all = wave_scan_u32(head ? real : 0);
        t = (uint32_t)__builtin_amdgcn_readlane((int)all, kWave - 1) + (uint32_t)__shfl((int)(surplus - (launched - real)), own_lane, kWave) + index - own_real;
        if (t % per_tile != 0) return;
        lo = len;
    }
    const uint32_t row = t / per_tile;
    if (head && row > 0) splits[(uint64_t)row * k + member] = lo;
    if (kApart) {
        const uint32_t sum = wave_scan_u32(head ? lo : 0);
        if (lane == kWave - 1) sums[row] = row > 0 ? sum : 0;
    }
}

// The boundaries that a workgroup works on, as a number in ascending order of the boundaries.  Workgroups go to the eight dies in
// turn; with this a die gets one contiguous eighth of the boundaries, and neighbours, whose searches end in the same records, share an
// L2.
__device__ __forceinline__ uint32_t near_block() {
    const uint32_t die = blockIdx.x % kDies, each = gridDim.x / kDies, more = gridDim.x % kDies;  // the first `more` dies get one more
    return die * each + min(die, more) + blockIdx.x / kDies;
}

// Lane bookkeeping shared by the partition kernels: which problem and which sequence a lane has.
struct GroupLane {
    int member, group_base;
    uint64_t slot;
};
__device__ __forceinline__ GroupLane group_lane(int group) {
    const int lane = threadIdx.x & (kWave - 1);
    GroupLane g;
    g.member = lane & (group - 1);
    g.group_base = lane - g.member;
    const uint64_t wave_id = (uint64_t)near_block() * (blockDim.x / kWave) + threadIdx.x / kWave;
    g.slot = wave_id * (uint64_t)(kWave / group) + (uint64_t)(lane / group);
    return g;
}

// Search over whole runs, one launch (where rows come first, in the first launch).
// kInit: the launch also clears the tile status words and writes the first and last split rows, which saves the
// separate init launch (a small compaction is then two launches: this one and the merge).
template <bool kInit>
__device__ __forceinline__ void partition_init(const RunTable& rt, const Workspace& ws, uint64_t n_tiles) {
    if (!kInit) return;
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t t = i; t < n_tiles; t += stride) ws.status[t] = 0;
    for (uint64_t c = i; c < ws.clear_n; c += stride) ws.clear[c] = make_uint4(0, 0, 0, 0);
    if (ws.fresh != nullptr)
        for (uint64_t t = i; t < kShortTiles; t += stride) ws.fresh[t] = 0;
    if (i < rt.k) {
        ws.splits[i] = 0;
        ws.splits[n_tiles * rt.k + i] = run_len(rt, (uint32_t)i);
    }
}

// two runs (every merge of a leveled tree): one wave per boundary up to kTwoWaves boundaries, then one lane, whose search
// reads a thirtieth of the records but takes log2 instead of log64 of the shorter run in dependent steps (10 boundaries of
// 3,600 + 36,000 entries: 7.7 us with one lane each, about 4 with a wave; 10,000 of 2M + 20M: 21 us with one lane)
constexpr uint64_t kTwoWaves = 1024;
template <bool kInit>
__global__ void __launch_bounds__(kWave) partition_two_wave_kernel(RunTable rt, Workspace ws, uint64_t n_tiles) {
    partition_init<kInit>(rt, ws, n_tiles);
    const uint64_t b = blockIdx.x + 1;
    uint64_t ia, ib;
    split_two_wave(rt.ptr[0], run_len(rt, 0), rt.ptr[1], run_len(rt, 1), b * ws.spacing, ia, ib);
    if (threadIdx.x == 0) {
        ws.splits[b * 2 + 0] = ia;
        ws.splits[b * 2 + 1] = ib;
    }
}
constexpr int kTwoThreads = 64;
template <bool kInit>
__global__ void __launch_bounds__(kTwoThreads) partition_two_kernel(RunTable rt, Workspace ws, uint64_t n_tiles) {
    partition_init<kInit>(rt, ws, n_tiles);
    const uint64_t b = (uint64_t)blockIdx.x * kTwoThreads + threadIdx.x + 1;
    if (b >= n_tiles) return;
    uint64_t ia, ib;
    split_two(rt.ptr[0], run_len(rt, 0), rt.ptr[1], run_len(rt, 1), b * ws.spacing, ia, ib);
    ws.splits[b * 2 + 0] = ia;
    ws.splits[b * 2 + 1] = ib;
}

// one run (a level that is rewritten without its tombstones): nothing to search.  Whole calls, us, on copied samples / a wave per boundary / so:
// 5M entries 200 / 164 / 136, 20M 595 / 618 / 518; 1M, where a wave per boundary was the rule, 39.8 / 35.1.
template <bool kInit>
__global__ void __launch_bounds__(kTwoThreads) partition_one_kernel(RunTable rt, Workspace ws, uint64_t n_tiles) {
    partition_init<kInit>(rt, ws, n_tiles);
    const uint64_t b = (uint64_t)blockIdx.x * kTwoThreads + threadIdx.x + 1, at = b * ws.spacing, n = run_len(rt, 0);
    if (b < n_tiles) ws.splits[b] = at < n ? at : n;
}

// other run counts: one wave per boundary
template <bool kInit, int kPerLane, bool kMany>
__global__ void __launch_bounds__(kWave) partition_kernel(RunTable rt, Workspace ws, uint64_t n_tiles, int group_log) {
    __shared__ WindowShared<kPerLane> s;
    partition_init<kInit>(rt, ws, n_tiles);
    const uint32_t b = near_block() + 1, lane = threadIdx.x, j = lane & ((1u << group_log) - 1);
    const bool own = j < rt.k;
    const uint32_t best = window_split<kPerLane, kMany>(s, own ? rt.ptr[j] : nullptr, 0, own ? (uint32_t)run_len(rt, j) : 0, b * ws.spacing, group_log);
    if (lane < rt.k) ws.splits[(uint64_t)b * rt.k + lane] = best;
}
template <bool kInit>
__global__ void __launch_bounds__(kWave) partition_ranked_kernel(RunTable rt, Workspace ws, uint64_t n_tiles, int group_log) {
    partition_init<kInit>(rt, ws, n_tiles);
    const uint32_t member = (threadIdx.x & (kWave - 1)) >> (6 - group_log);
    const bool mine = member < rt.k;
    ranked_row(mine ? rt.ptr[member] : nullptr, mine ? (uint32_t)run_len(rt, member) : 0, mine ? (uint32_t)rt.n[member] : 0, blockIdx.x, rt.k, group_log,
                ws.stride, ws.per_tile, ws.splits);
}
// Boundaries between rows, two launches.  partition_rows_kernel: the lower bounds of every row_entries-th entry of every run in all runs, in order
// of the entries' keys, a wave each (ranked_row).  partition_between_kernel: a boundary lies between the last row that is not beyond its rank and
// the next, some row_entries entries of all runs together, where window_split has two rounds left instead of five.  Run j's second sample is
// (j + 1) / k of row_entries into it: with samples at the same places of all runs, the rows of runs that advance together (the same keys in every
// run, or runs that take turns) come k at a time, and k * row_entries entries lie between them (24 runs in turns of 100 entries, 1M in all 195
// us, so 150; the same keys in 16 runs, 25M 1040 and 985).
// A die ranks an eighth of every run's samples: their searches read the same lines where runs cover the same keys (12 runs of 6M entries in all 272.7 us
// with an eighth of all samples, run by run, for a die, 270.0 so; 16 runs, 3M 162.6 and 158.7).
// Row t has c_j samples of run j before it, t in all, so L is no more than row_entries * t, and no less than the sum of offset_j + row_entries *
// (c_j - 2), row_entries * (t - 3/2 k).  Bound by the lines that both fetch (a record is 128 bytes of traffic, its neighbour aside).
__device__ __forceinline__ uint32_t* row_sums(const Workspace& ws, uint32_t n_rows, uint32_t k) { return reinterpret_cast<uint32_t*>(ws.ywin + (uint64_t)n_rows * k); }
__host__ __device__ inline uint32_t row_offset(uint32_t j, uint32_t k, uint32_t row_entries) { return (j + 1) * row_entries / k; }
template <bool kInit>
__global__ void __launch_bounds__(kWave) partition_rows_kernel(RunTable rt, Workspace ws, uint64_t n_tiles, uint32_t n_rows, uint32_t row_entries, int group_log) {
    partition_init<kInit>(rt, ws, n_tiles);
    const uint32_t member = (threadIdx.x & (kWave - 1)) >> (6 - group_log);
    const bool mine = member < rt.k;
    ranked_row<lsm_entry_t, true>(mine ? rt.ptr[member] : nullptr, mine ? (uint32_t)run_len(rt, member) : 0, mine ? (uint32_t)rt.n[member] : 0, blockIdx.x, rt.k,
                                  group_log, row_entries, 1, ws.ywin, mine ? row_offset(member, rt.k, row_entries) : 0, row_sums(ws, n_rows, rt.k));
}
template <int kPerLane>
__global__ void __launch_bounds__(kWave) partition_between_kernel(RunTable rt, Workspace ws, uint32_t n_rows, uint32_t row_entries, int group_log) {
    __shared__ WindowShared<kPerLane> s;
    const uint32_t b = near_block() + 1, lane = threadIdx.x, j = lane & ((1u << group_log) - 1);
    const bool own = j < rt.k;
    const uint32_t len = own ? (uint32_t)run_len(rt, j) : 0, r = b * ws.spacing;
    auto row = [&](uint32_t t) { return own && t > 0 ? (t < n_rows ? min((uint32_t)ws.ywin[(uint64_t)t * rt.k + j], len) : len) : 0; };  // inputs that are not sorted may leave a row unwritten
    // the last row that is not beyond r: one of 3/2 k + 2, and the first of them is not beyond it
    static_assert(kFewRuns * 3 / 2 + 2 <= kWave, "a row per lane");
    const uint32_t first = min(r / row_entries, n_rows - 1);
    const uint32_t sum = first + lane < n_rows ? row_sums(ws, n_rows, rt.k)[first + lane] : ~0u;
    const uint32_t at = first + (uint32_t)__popcll(__ballot(sum <= r) & ~1ull);
    const uint32_t lo = row(at), hi = row(at + 1);
    const uint32_t best = window_split<kPerLane, false>(s, own ? rt.ptr[j] : nullptr, lo, max(lo, hi), r, group_log);
    if (lane < rt.k) ws.splits[(uint64_t)b * rt.k + lane] = best;
}
// With many runs and many tiles the records that the waves' rounds read are more than the memory takes (a round of 64 runs is
// 512 lines of 128 bytes): beyond kWindowPieces pieces of tiles in runs the pivoting selection, whose searches share their
// first records, is the faster one for mixed runs.  Windows / pivoting: 64 runs, 2M entries 210 / 221 us, 2.5M 258 / 237,
// 3.9M 573 / 343; 48 runs, 2.5M 233 / 241, 3.2M 320 / 282, 3.9M 354 / 327; 33 runs, 3.9M 312 / 326.  (Runs one after the
// other the other way round, 64 runs of 3.9M 267 / 565: not what a tree's levels look like.)
constexpr uint64_t kWindowPieces = 65536;
template <bool kInit>
__global__ void __launch_bounds__(kWave) partition_many_kernel(RunTable rt, Workspace ws, uint64_t n_tiles) {
    partition_init<kInit>(rt, ws, n_tiles);
    const uint32_t b = near_block() + 1, lane = threadIdx.x;
    const bool own = lane < rt.k;
    const uint64_t best = select_split<false>(own ? rt.ptr[lane] : nullptr, 0, own ? run_len(rt, lane) : 0, b * (uint64_t)ws.spacing, own, (int)lane, kWave, 0);
    if (own) ws.splits[(uint64_t)b * rt.k + lane] = best;
}

static int log2_ceil(uint32_t k) {
    int log = 0;
    while ((1u << log) < k) log++;
    return log;
}
// Records a lane reads per round of the window search: 256 records in all for up to 16 runs, 512 beyond (16 or 8 per run).
static int records_per_lane(int group_log) { return group_log <= 4 ? 4 : 8; }

// ---------------------------------------------------------------------------------------
// Sampled partition, for large inputs of many runs.  Searching the runs directly costs tens of scattered
// 64-byte reads per boundary and run, which is HBM traffic of the order of the merge itself.
// Instead every kSampleStride-th key of each run is copied into a compact array (1/64 of the
// input bytes: it stays in the last-level cache), the selection is done on the samples, and the
// runs themselves are only searched inside the few dozen entries the samples leave open.
//
// With s = kSampleStride, a key P that has y_j samples below it in run j has x_j entries below
// it with s * (y_j - 1) < x_j <= s * y_j, so for Y = sum y_j:  s * (Y - k) < L(P) <= s * Y.
//   lower bracket: the sample key with the largest Y <= floor(r / s) has L <= r, so it is <= x;
//   upper bracket: the sample key with the largest Y <= ceil(r / s) + 2k - 1 has, if a larger sample
//                  exists at all, Y >= ceil(r / s) + k and therefore L > r: it is > x.
// The answer's lower bound in run j then lies in [s * (ylo_j - 1) + 1, s * yhi_j] (clamped to the run).
// The sample-space problems start from ranked samples (ranked_row above): every kRowStride-th sample of every run, its lower bounds
// in all runs' samples, in order.  With s2 = kRowStride, row t has s2 * (t - k) <= Y <= s2 * t, so the answer for a target Y lies
// between row floor(Y / s2) and row floor(Y / s2) + 1 + k.  (Every 16th boundary searched over whole sample arrays instead was a
// chain of some ninety dependent reads, 70 us for 16 x 4M entries and 52 for 4 x 4M, where the rows take 25 and 7.)
// ---------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) sample_kernel(RunTable rt, SampleTable st) {
    const uint32_t j = blockIdx.y;
    const uint4* src = reinterpret_cast<const uint4*>(rt.ptr[j]);
    uint4* dst = reinterpret_cast<uint4*>(st.ptr[j]);
    const uint64_t n16 = st.m[j] * 2, stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride)
        dst[i] = src[(i >> 1) * (kSampleStride * 4) + (i & 1)];  // 4 uint4 per entry; two lanes copy one key
}

__device__ __forceinline__ uint64_t sample_target(uint64_t b, int side, uint32_t k) {
    const uint64_t r = b * tile_nominal(k);
    return side ? (r + kSampleStride - 1) / kSampleStride + 2ull * k - 1 : r / kSampleStride;
}

// the ranked rows: one wave per ranked sample, all of them boundaries of the sample arrays
__global__ void __launch_bounds__(kWave) sample_rank_kernel(Workspace ws, uint32_t k, int group_log) {
    const uint32_t member = threadIdx.x >> (6 - group_log);
    const bool mine = member < k;
    const uint32_t m = mine ? (uint32_t)ws.st.m[member] : 0;
    ranked_row(mine ? ws.st.ptr[member] : nullptr, m, m, blockIdx.x, k, group_log, kRowStride, 1, ws.splits);
}

// problem p = 2 * (b - 1) + side for boundary b, between the ranked rows that enclose its target
__global__ void __launch_bounds__(256) sample_fine_kernel(Workspace ws, uint32_t k, uint64_t n_tiles, uint64_t n_rows, int group) {
    const GroupLane g = group_lane(group);
    const uint64_t b = g.slot / 2 + 1;
    const int side = (int)(g.slot & 1);
    const bool own = b < n_tiles && g.member < (int)k;
    const SampleKey* run = own ? ws.st.ptr[g.member] : nullptr;
    const uint64_t target = sample_target(b, side, k);
    uint64_t lo = 0, hi = 0;
    if (own) {
        const uint64_t row = target / kRowStride, from = row < n_rows ? row : n_rows - 1, above = row + 1 + k;
        lo = ws.splits[from * k + g.member];
        hi = above < n_rows ? ws.splits[above * k + g.member] : ws.st.m[g.member];
        if (hi > ws.st.m[g.member]) hi = ws.st.m[g.member];  // only inputs that break the precondition
        if (lo > hi) lo = hi;
    }
    const uint64_t best = select_split<true>(run, lo, hi, target, own, g.member, group, g.group_base);
    if (own) ws.ywin[g.slot * k + g.member] = best;
}

// the boundary itself, searched inside the brackets
__global__ void __launch_bounds__(256) bracket_partition_kernel(RunTable rt, Workspace ws, uint64_t n_tiles, int group) {
    const GroupLane g = group_lane(group);
    const uint64_t b = g.slot + 1;
    const bool own = b < n_tiles && g.member < (int)rt.k;
    const uint64_t r = b * tile_nominal(rt.k);
    const lsm_entry_t* run = own ? rt.ptr[g.member] : nullptr;
    uint64_t lo = 0, hi = 0, yhi = 0;
    if (own) {
        const uint64_t n = rt.n[g.member];
        const uint64_t ylo = ws.ywin[(2 * (b - 1)) * rt.k + g.member];
        yhi = ws.ywin[(2 * (b - 1) + 1) * rt.k + g.member];
        lo = ylo ? (ylo - 1) * kSampleStride + 1 : 0;
        hi = yhi * kSampleStride;
        if (hi > n) hi = n;
    }
    // no sample above the upper target: the upper bracket proves nothing, search to the end of the runs
    const uint64_t y_total = group_sum_u64(own ? yhi : 0, group);
    if (own && y_total < (r + kSampleStride - 1) / kSampleStride + rt.k) hi = rt.n[g.member];
    if (lo > hi) lo = hi;  // only inputs that break the precondition
    const uint64_t best = select_split<false>(run, lo, hi, r, own, g.member, group, g.group_base);
    if (own) ws.splits[b * rt.k + g.member] = best;
}

// ---------------------------------------------------------------------------------------
// Tile merge.
//
// Every thread owns kMergeItems entries of the tile and keeps their 64 bytes in registers
// from the load to the final store.  What moves through LDS during the merge rounds is one
// 16-byte "surrogate" per entry: the first 14 key bytes (as a 112-bit big-endian number) and
// the entry's tile-local index in the low 16 bits.  Surrogates are merged with stable
// two-way merge-path merges (the left list = lower run indices wins ties).  Afterwards each
// merged position gets the rest of its key (bytes 14..31), its seqno and its type, so that
// neighbours can be compared exactly.  Equal surrogates with different key tails mean the
// 14-byte order was not enough: a short group of such positions is put in key order in place
// (one thread, insertion sort by the tail), and a tile with a longer group is redone by the
// exact path below (ranks by binary search over the tile's pieces with full 32-byte compares).
// ---------------------------------------------------------------------------------------
enum : uint8_t { kFlagEq = 1, kFlagFullEq = 2 };
constexpr uint32_t kNoSlot = 0xFFFF;          // of an entry that does not survive
constexpr int kRepairMax = 32;                // longest prefix-tie group one thread puts in key order
constexpr int kStageEntries = kTileCap / 2;  // output staging: 64 bytes per survivor, two passes at most

struct TileHead {  // what the whole workgroup knows of its tile
    uint32_t seg[LSM_MAX_RUNS + 1];  // start of each run's piece in tile-local index space
    uint64_t lo[LSM_MAX_RUNS];       // first entry of each run's piece
    const lsm_entry_t* run[LSM_MAX_RUNS];  // copy of the run pointers (indexed per lane)
    uint32_t tile;                   // number of the tile inside its compaction (what the look-back counts in)
    uint32_t n;
    uint32_t failed;
    uint64_t base;
    // batched compactions only: what the single form takes from its kernel arguments
    uint32_t k, flags, job_tiles, fence_stride;
    lsm_entry_t* out;
    uint64_t* n_out;
    uint64_t* status;
    uint4* fence_out;
    uint64_t* key_hashes;
    uint64_t epoch;  // of the status words, in its place
};

struct MergeShared : TileHead {
    uint4 buf[2][kTileCap];          // surrogate ping-pong; then 2 x uint4 of key tail/seqno/type per position; then output staging
    uint16_t rank[kTileCap];         // tile-local entry index -> merged position
    alignas(8) uint16_t prefix[kTileCap];  // survivors before this merged position, kNoSlot if its entry does not survive
    alignas(4) uint8_t flag[kTileCap + 8];  // per merged position: kFlagEq | kFlagFullEq; on the exact path: 1 = survives
    uint32_t wave_count[kMergeThreads / kWave];
    uint32_t inexact;                // some position has an equal surrogate but a different key tail
};

// The tile kernel has three forms.  Single: one compaction, tile = workgroup, pieces from the split table.
// Range: one tile per key range of a tree - the pieces are the parts of the runs inside the range, found by the
// tile itself, and the survivors go to a fixed slot of the result (no look-back).  Batch: many independent
// compactions in one launch - the workgroup looks up its job, and everything the single form takes from kernel
// arguments comes from the job's descriptor.
enum : int { kModeSingle = 0, kModeRange = 1, kModeBatch = 2 };

constexpr uint32_t kHashesBehind = 0x80000000u;
struct JobDesc {       // one compaction of a batch (device memory, written by the host)
    uint32_t first_tile;   // number of its first tile in the launch
    uint32_t first_wave;   // number of its first wave in the partition launch
    uint32_t run_off;      // where its runs start in the run pointer / length arrays
    uint16_t stride, per_tile;  // entries from sample to sample, samples from boundary to boundary; stride 0: exact ranks, a wave per tile
    uint64_t splits_off;   // where its split table starts (in 64-bit words)
    lsm_entry_t* out;
    uint64_t* n_out;
    uint4* fence_out;      // optional fence index of the job's output
    uint32_t n_tiles, k, flags, fence_stride;
    uint4* clear;          // optional memory the partition launch zeroes for a later kernel
    uint32_t clear_n;      // 16-byte words of it; with kHashesBehind the merge puts the keys' filter hashes behind them
    uint32_t waves;        // of the partition launch
};
static_assert(sizeof(JobDesc) == 80, "descriptor layout");
static_assert(kMostClearWords <= kHashesBehind, "the words of a span leave the bit free");

struct ModeArgs {
    // single form: optional filter hashes of the output's keys (kExtras = 2)
    uint64_t* key_hashes;
    // range form
    const uint8_t* lo_keys;   // [n_tiles x 32]
    const uint8_t* hi_keys;
    uint32_t* counts;         // [n_tiles]
    uint32_t max_entries;     // slot pitch of the result
    // batch form
    const uint32_t* tile_job;             // [n_tiles] job of every tile
    const JobDesc* jobs;
    const lsm_entry_t* const* run_ptr;    // runs of all jobs
    const uint64_t* run_n;
};

struct Sur {  // hi = key bytes 0..7, lo = key bytes 8..13 << 16 | index
    uint64_t hi, lo;
};
__device__ __forceinline__ Sur sur_load(const uint4* p) {
    uint4 v = *p;
    Sur r;
    r.hi = ((uint64_t)v.y << 32) | v.x;
    r.lo = ((uint64_t)v.w << 32) | v.z;
    return r;
}
__device__ __forceinline__ void sur_store(uint4* p, const Sur& v) {
    *p = make_uint4((uint32_t)v.hi, (uint32_t)(v.hi >> 32), (uint32_t)v.lo, (uint32_t)(v.lo >> 32));
}
// Where the record of position p sits in the 16-byte-per-position LDS arrays.  Threads own four consecutive
// positions, so lane t of a wave reads or writes position 4t + i: without this every second lane would
// fall on the same banks (64-byte stride).  The swap inside each group of four spreads eight lanes over all banks.
__device__ __forceinline__ uint32_t sw(uint32_t p) { return p ^ ((p >> 3) & 3); }

// a < b as 128-bit numbers (key bits, then index)
__device__ __forceinline__ bool sur_less(const Sur& a, const Sur& b) { return a.hi < b.hi || (a.hi == b.hi && a.lo < b.lo); }
// afterwards a < b
__device__ __forceinline__ void sur_order(Sur& a, Sur& b) {
    const bool swap = sur_less(b, a);
    const Sur t = a;
    a.hi = swap ? b.hi : a.hi;
    a.lo = swap ? b.lo : a.lo;
    b.hi = swap ? t.hi : b.hi;
    b.lo = swap ? t.lo : b.lo;
}
__device__ __forceinline__ bool sur_same_key(const Sur& a, const Sur& b) { return a.hi == b.hi && ((a.lo ^ b.lo) >> 16) == 0; }

// Last j < k with seg[j] <= e (empty pieces share an offset with their successor).  Branch-free;
// top_step = largest power of two below k (0 for k = 1).
__device__ __forceinline__ uint32_t piece_of(const uint32_t* seg, uint32_t k, uint32_t top_step, uint32_t e) {
    uint32_t j = 0;
    for (uint32_t step = top_step; step > 0; step >>= 1) {
        const uint32_t c = j + step;
        const uint32_t v = seg[min(c, k - 1)];
        j = ((c < k) & (v <= e)) ? c : j;
    }
    return j;
}

// Publish this tile's survivor count and return the number of survivors in all earlier tiles
// (decoupled look-back).  Called by wave 0 only, all 64 lanes.  Earlier tiles are earlier
// workgroups, which have started (or finished) by the time this one runs, and will publish; the
// wait is bounded anyway, and a tile that gives up publishes kStFailed, which propagates forward.
__device__ uint64_t lookback(uint64_t* status, uint64_t tile, uint64_t count, bool self_failed, bool* failed) {
    const int lane = threadIdx.x & (kWave - 1);
    *failed = self_failed;
    if (self_failed) {
        if (lane == 0) __hip_atomic_store(&status[tile], kStFailed << kStShift, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return 0;
    }
    if (tile == 0) {
        if (lane == 0) __hip_atomic_store(&status[0], (kStPrefix << kStShift) | count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return 0;
    }
    if (lane == 0) __hip_atomic_store(&status[tile], (kStAggregate << kStShift) | count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint64_t base = 0;
    int64_t top = (int64_t)tile - 1;  // lane l looks at tile top - l
    bool bad = false;
    for (;;) {
        int64_t t = top - lane;
        uint64_t st = kStPrefix << kStShift;  // tiles before tile 0: an empty prefix
        uint32_t spins = 0;
        for (;;) {
            if (t >= 0) st = __hip_atomic_load(&status[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            bool ready = (st >> kStShift) != kStEmpty;
            if (__ballot(!ready) == 0) break;
            if (++spins > kSpinLimit) {
                bad = true;
                break;
            }
            __builtin_amdgcn_s_sleep(2);
        }
        if (bad) break;
        uint64_t state = st >> kStShift;
        if (__ballot(state == kStFailed) != 0) {
            bad = true;
            break;
        }
        uint64_t pmask = __ballot(state == kStPrefix);
        int first = pmask ? __ffsll((unsigned long long)pmask) - 1 : kWave - 1;  // nearest tile with a full prefix
        base += wave_sum_u64(lane <= first ? (st & kStValueMask) : 0);
        if (pmask) break;
        top -= kWave;
    }
    *failed = bad;
    uint64_t word = bad ? (kStFailed << kStShift) : ((kStPrefix << kStShift) | (base + count));
    if (lane == 0) __hip_atomic_store(&status[tile], word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return base;
}

// order of two entries with the same 14-byte key prefix by the rest of the key, from their info words
__device__ __forceinline__ bool tail_less(const uint4 a0, const uint4 a1, const uint4 b0, const uint4 b1) {
    const uint32_t ta = ((a0.z >> 8) & 0xFF) << 8 | ((a0.z >> 16) & 0xFF), tb = ((b0.z >> 8) & 0xFF) << 8 | ((b0.z >> 16) & 0xFF);
    if (ta != tb) return ta < tb;  // key bytes 14, 15
    const uint64_t a2 = __builtin_bswap64(((uint64_t)a1.y << 32) | a1.x), b2 = __builtin_bswap64(((uint64_t)b1.y << 32) | b1.x);
    if (a2 != b2) return a2 < b2;  // key bytes 16..23
    return __builtin_bswap64(((uint64_t)a1.w << 32) | a1.z) < __builtin_bswap64(((uint64_t)b1.w << 32) | b1.z);
}

// Where key range `t` starts and ends in every run: bounds[2 j] and bounds[2 j + 1] = lower bounds of its two keys in run j.
// The threads of the workgroup are shared evenly by the 2 k searches, 32 lanes each at most, and every step reads one
// record per lane, evenly spaced in what is left: a chain of five reads in a run of four million entries with 32 lanes, ten
// with the four lanes that 64 runs leave.  The two searches of a run read the same records until they part.  (One lane per
// run, bisection for the start and doubling steps for the end, was a chain of some thirty reads and most of the kernel's
// time: 500 ranges of a 4M-entry tree took 21.9 us, now 15.5; 2,000 of a 20M-entry tree 92.7, now 53.0; one range of 50,000
// entries 14.3, now 10.1.)
__device__ __forceinline__ void range_bounds(const RunTable& rt, const ModeArgs& ma, const uint64_t t, uint64_t* bounds) {
    uint32_t lanes_log = 5;
    while ((uint32_t)kMergeThreads >> lanes_log < 2 * rt.k) lanes_log--;
    const uint32_t lanes = 1u << lanes_log, member = threadIdx.x & (lanes - 1), problem = threadIdx.x >> lanes_log;
    const bool own = problem < 2 * rt.k;
    const lsm_entry_t* run = own ? rt.ptr[problem >> 1] : nullptr;
    uint64_t lo = 0, hi = own ? rt.n[problem >> 1] : 0;  // the bound lies in [lo, hi]
    const Key key = load_key(((problem & 1) ? ma.hi_keys : ma.lo_keys) + t * LSM_KEY_BYTES);
    const uint32_t shift = threadIdx.x & (kWave - 1) & ~(lanes - 1);
    while (__ballot(lo < hi) != 0) {
        const uint64_t w = hi - lo;
        auto tried = [&](uint32_t m) { return lo + (((2 * (uint64_t)m + 1) * w) >> (lanes_log + 1)); };  // ascending with m, below hi
        bool less = false;
        if (lo < hi) {
            const uint4* e = reinterpret_cast<const uint4*>(run + tried(member));
            const uint4 k0 = load_global_u4(e), k1 = load_global_u4(e + 1);
            less = key_less(key_from_raw(k0, k1), key);
        }
        const uint32_t n = (uint32_t)__popcll((__ballot(less) >> shift) & ((1ull << lanes) - 1));  // the first n records are less
        if (lo < hi) {
            const uint64_t new_lo = n > 0 ? tried(n - 1) + 1 : lo, new_hi = n < lanes ? tried(n) : hi;
            lo = new_lo;
            hi = new_hi < new_lo ? new_lo : new_hi;  // only runs that are not sorted
        }
    }
    if (own && member == 0) bounds[problem] = lo;
}

// The tile's k pieces; called by wave 0 only.  Tile number = workgroup number: the look-back below waits only for
// tiles with smaller numbers, and workgroups are handed to the compute units in ascending order, so the
// tiles waited for are resident or done.  (A ticket taken with an atomic would make that independent
// of the dispatch order, but it costs a second dependent memory round trip before the first load: the
// tickets come back in a different order than the workgroup numbers for 99 % of the tiles.)  The waits
// are bounded in any case.
template <int kMode>
__device__ __forceinline__ void tile_pieces(TileHead& s, const RunTable& rt, const Workspace& ws, const uint64_t n_tiles, const ModeArgs& ma, const uint64_t* bounds) {
    const int lane = threadIdx.x & (kWave - 1);
    __builtin_amdgcn_s_setprio(3);  // the other waves wait for this one: let it issue first
    uint64_t t = blockIdx.x;        // tile number inside its compaction
    uint32_t kk = rt.k;
    uint64_t a = 0, b = 0, len = ~0ull;
    if (kMode == kModeSingle) {
        if (lane < (int)kk) {
            if (n_tiles == 1) {  // one tile is the whole input: launched on its own, without a split table
                b = run_len(rt, lane);
            } else {
                a = ws.splits[t * kk + lane];
                b = ws.splits[(t + 1) * kk + lane];
                if (ws.stride != 0) len = run_len(rt, lane);  // exact ranks write every row, within the runs
            }
            s.run[lane] = rt.ptr[lane];
        }
    } else if (kMode == kModeRange) {
        // the part of every run inside [lo_key, hi_key)
        const Key lo_key = load_key(ma.lo_keys + t * LSM_KEY_BYTES), hi_key = load_key(ma.hi_keys + t * LSM_KEY_BYTES);
        if (lane < (int)kk) {
            a = bounds[2 * lane];
            b = key_less(lo_key, hi_key) ? bounds[2 * lane + 1] : a;
            s.run[lane] = rt.ptr[lane];
        }
    } else {
        const JobDesc d = ma.jobs[ma.tile_job[t]];  // the same words for every lane
        kk = d.k;
        t -= d.first_tile;
        if (lane < (int)kk) {
            a = ws.splits[d.splits_off + t * kk + lane];
            b = ws.splits[d.splits_off + (t + 1) * kk + lane];
            s.run[lane] = ma.run_ptr[d.run_off + lane];
            if (d.stride != 0) len = ma.run_n[d.run_off + lane];
        }
        if (lane == 0) {
            s.k = kk;
            s.flags = d.flags;
            s.job_tiles = d.n_tiles;
            s.out = d.out;
            s.n_out = d.n_out;
            s.status = ws.status + d.first_tile;
            s.fence_out = d.fence_out;
            s.fence_stride = d.fence_stride;
            s.key_hashes = d.clear_n & kHashesBehind ? reinterpret_cast<uint64_t*>(d.clear + (d.clear_n & ~kHashesBehind)) : nullptr;
        }
    }
    const bool mine = lane < (int)kk;
    // piece lengths -> offsets (inclusive scan over the lanes); only inputs that break the precondition can make a row
    // pair inconsistent, or leave a row of the sampled ranks unwritten
    // (a key range may simply hold more than a tile: reported as an overflow of that range)
    const bool bad = mine && (b < a || b > len || b - a > (uint64_t)kTileCap);
    uint32_t incl = (mine && !bad) ? (uint32_t)(b - a) : 0;
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t v = __shfl_up(incl, off, kWave);
        if (lane >= off) incl += v;
    }
    const uint32_t total = __shfl(incl, kWave - 1, kWave);
    const bool ok = __ballot(bad) == 0 && total <= (uint32_t)kTileCap;
    if (mine) {
        s.lo[lane] = a;
        s.seg[lane + 1] = ok ? incl : 0;
    }
    if (lane == 0) {
        s.seg[0] = 0;
        s.tile = (uint32_t)t;
        s.n = ok ? total : 0;
        s.failed = ok ? 0 : 1;
    }
    __builtin_amdgcn_s_setprio(0);
}

// A tile from its loaded entries to the merged positions, kItems entries a thread (see merge_short_kernel): at[i] = position of entry
// tid + i * kThreads among the tile's entries in the order (key, run); the bits of the survivors are set in alive[], which is zero, as is
// deep.  mem: 4 * kCap pieces.  All threads of the workgroup.
template <int kItems, int kThreads, int kCap, int kHeld>
__device__ __forceinline__ void short_rank(const TileHead& s, uint4* const mem, uint32_t* const alive, uint32_t& deep, const uint4 (&ent)[kHeld][4],
                                           const uint32_t (&piece)[kHeld], uint32_t (&at)[kHeld], const uint32_t n, const uint32_t k, const uint32_t flags) {
    const uint32_t tid = threadIdx.x;
    uint4* const tails = mem + 2 * kCap;  // by entry: key bytes 16..31
    uint4* const infos = mem + 3 * kCap;  // by entry: seqno, type | key bytes 14..15 << 8
    Sur sur[kItems];
#pragma unroll
    for (int i = 0; i < kItems; i++) {
        const uint32_t e = tid + i * kThreads;
        at[i] = e;
        const Key key = key_from_raw(ent[i][0], ent[i][1]);
        sur[i].hi = key.w[0];
        sur[i].lo = (key.w[1] & ~0xFFFFull) | e;
        if (e < n) {
            sur_store(&mem[e], sur[i]);
            tails[e] = ent[i][1];
            infos[e] = make_uint4(ent[i][2].x, ent[i][2].y, (ent[i][2].z & 0xFF) | (ent[i][0].w & 0xFFFF0000u) >> 8, 0);
        }
    }
    __syncthreads();
    // ---- merge rounds: an entry's place in the merged list is its place in its own list and the number of smaller ones in the
    //      other list of the pair
    uint4* in = mem;
    uint4* dst = mem + kCap;
    for (uint32_t width = 1; width < k; width <<= 1) {
        uint32_t lo[kItems], hi[kItems], from[kItems];
#pragma unroll
        for (int i = 0; i < kItems; i++) {
            const uint32_t j = piece[i], first = j & ~(width - 1), other = first ^ width;  // lists of `width` runs
            const uint32_t begin = s.seg[min(other, k)], end = s.seg[min(other + width, k)];
            const bool valid = tid + i * kThreads < n;
            lo[i] = from[i] = begin;
            hi[i] = valid ? end : begin;
        }
        bool go = true;
        while (go) {
            go = false;
#pragma unroll
            for (int i = 0; i < kItems; i++) {
                if (lo[i] < hi[i]) {
                    const uint32_t mid = (lo[i] + hi[i]) >> 1;
                    const bool less = sur_less(sur_load(&in[mid]), sur[i]);
                    lo[i] = less ? mid + 1 : lo[i];
                    hi[i] = less ? hi[i] : mid;
                    go = go || lo[i] < hi[i];
                }
            }
        }
#pragma unroll
        for (int i = 0; i < kItems; i++) {
            const uint32_t below = lo[i] - from[i];
            const bool right = (piece[i] & width) != 0;  // at[] counts the whole of the other list, which lies before this one
            at[i] += right ? below - (s.seg[piece[i] & ~(width - 1)] - from[i]) : below;
            if (tid + i * kThreads < n) sur_store(&dst[at[i]], sur[i]);
        }
        __syncthreads();
        uint4* const t = in;
        in = dst, dst = t;
    }
    // ---- neighbours with the same 14 bytes: the rest of the key orders them, the newest version of a key survives
    bool win[kItems];
#pragma unroll
    for (int i = 0; i < kItems; i++) {
        const uint32_t e = tid + i * kThreads, p = at[i];
        win[i] = e < n;
        if (!win[i]) continue;
        const Sur me = sur[i];
        const uint4 my_info = make_uint4(ent[i][2].x, ent[i][2].y, (ent[i][2].z & 0xFF) | (ent[i][0].w & 0xFFFF0000u) >> 8, 0), my_tail = ent[i][1];
        const uint64_t seq = ((uint64_t)my_info.y << 32) | my_info.x;
        uint32_t left = 0, right = 0, before = 0;
        auto meet = [&](const uint32_t other) {
            const uint4 info = infos[other], tail = tails[other];
            const bool same = ((info.z ^ my_info.z) >> 8) == 0 && tail.x == my_tail.x && tail.y == my_tail.y && tail.z == my_tail.z && tail.w == my_tail.w;
            if (same) {
                const uint64_t its = ((uint64_t)info.y << 32) | info.x;
                if (its > seq || (its == seq && other < e)) win[i] = false;
                before += other < e;
            } else {
                before += tail_less(info, tail, my_info, my_tail);
            }
        };
        Sur l = sur_load(&in[p > 0 ? p - 1 : 0]), r = sur_load(&in[min(p + 1, n - 1)]);  // both at once: most entries have no such neighbour
        while (left < p && sur_same_key(l, me) && left <= (uint32_t)kRepairMax) {
            meet((uint32_t)l.lo & 0xFFFF);
            left++;
            l = sur_load(&in[p > left ? p - left - 1 : 0]);
        }
        while (p + right + 1 < n && sur_same_key(r, me) && right <= (uint32_t)kRepairMax) {
            meet((uint32_t)r.lo & 0xFFFF);
            right++;
            r = sur_load(&in[min(p + right + 1, n - 1)]);
        }
        if (left + right >= (uint32_t)kRepairMax) deep = 1;
        at[i] = p - left + before;
        if ((flags & LSM_BOTTOMMOST) && (ent[i][2].z & 0xFF) == LSM_TOMBSTONE) win[i] = false;
    }
#pragma unroll
    for (int i = 0; i < kItems; i++)
        if (win[i]) atomicOr(&alive[at[i] >> 5], 1u << (at[i] & 31));
    __syncthreads();
    if (deep == 0) return;
    // ---- exact path, as in merge_kernel: binary search over the tile's other pieces with full 32-byte compares
    __syncthreads();
    uint4* const heads = mem;  // by entry: key bytes 0..15
#pragma unroll
    for (int i = 0; i < kItems; i++)
        if (tid + i * kThreads < n) heads[tid + i * kThreads] = ent[i][0];
    if (tid < kCap / 32) alive[tid] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kItems; i++) {
        const uint32_t e = tid + i * kThreads, j = piece[i];
        if (e >= n) continue;
        const Key x = key_from_raw(ent[i][0], ent[i][1]);
        const uint64_t seq = ((uint64_t)ent[i][2].y << 32) | ent[i][2].x;
        uint32_t p = e - s.seg[j];
        bool wins = true;
        for (uint32_t j2 = 0; j2 < k; j2++) {
            if (j2 == j) continue;
            const uint32_t first = s.seg[j2], last = s.seg[j2 + 1];
            uint32_t lb = first, ub = last;
            while (lb < ub) {
                const uint32_t mid = (lb + ub) >> 1;
                if (entry_key_less(&heads[mid], &tails[mid], x)) lb = mid + 1;
                else ub = mid;
            }
            p += lb - first;
            if (lb < last && key_equal(key_from_raw(heads[lb], tails[lb]), x)) {
                const uint64_t other = ((uint64_t)infos[lb].y << 32) | infos[lb].x;
                if (other > seq || (other == seq && j2 < j)) wins = false;
                if (j2 < j) p++;
            }
        }
        if (wins && (flags & LSM_BOTTOMMOST) && (ent[i][2].z & 0xFF) == LSM_TOMBSTONE) wins = false;
        at[i] = p;
        if (wins) atomicOr(&alive[p >> 5], 1u << (p & 31));
    }
    __syncthreads();
}

// two workgroups per compute unit = four waves per SIMD: at most 128 vector registers.
// kExtras: what else the output pass does (compiled out otherwise).  1: rewrites value pointers and / or writes the fence
// index; 2: also writes the filter hash of every survivor's key.
template <int kExtras, int kMode>
__global__ void __launch_bounds__(kMergeThreads) __attribute__((amdgpu_waves_per_eu(4, 4))) merge_kernel(RunTable rt, Workspace ws, uint64_t n_tiles, uint32_t flags_arg,
                                                               lsm_entry_t* out_arg, uint64_t* n_out_arg, const uint64_t* remap_base,
                                                               uint32_t remap_files, uint4* fence_out_arg, uint32_t fence_stride_arg, ModeArgs ma) {
    __shared__ MergeShared s;
    // staging of the survivors' filter hashes (kExtras = 2): the first half lives in s.rank, which is dead by then
    __shared__ uint64_t hash_stage_upper[kExtras == 2 ? kStageEntries / 2 : 1];
    static_assert(sizeof(s.rank) == sizeof(uint64_t) * (kStageEntries / 2), "s.rank holds half a pass of hashes");
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = tid / kWave;

    uint64_t* const bounds = reinterpret_cast<uint64_t*>(s.buf[0]);  // range form: free until the entries are loaded
    if (kMode == kModeRange) {
        range_bounds(rt, ma, blockIdx.x, bounds);
        __syncthreads();
    }

    uint32_t* const alive = reinterpret_cast<uint32_t*>(s.rank);  // range form
    if (wave == 0) {
        if (lane == 0) s.inexact = 0;
        tile_pieces<kMode>(s, rt, ws, n_tiles, ma, bounds);
    } else if (kMode == kModeRange && wave == 1) {
        alive[lane] = 0;
    }
    __syncthreads();
    const uint64_t tile = s.tile;
    if (blockIdx.x >= n_tiles) return;  // cannot happen: the grid has exactly n_tiles workgroups
    const uint32_t n = s.n;
    const uint32_t k = kMode == kModeBatch ? s.k : rt.k;
    const uint32_t flags = kMode == kModeBatch ? s.flags : flags_arg;
    lsm_entry_t* const out = kMode == kModeBatch ? s.out : out_arg;
    uint64_t* const n_out = kMode == kModeBatch ? s.n_out : n_out_arg;
    const uint64_t last_tile = kMode == kModeBatch ? (uint64_t)s.job_tiles - 1 : n_tiles - 1;
    uint4* const fence_out = kMode == kModeBatch ? s.fence_out : fence_out_arg;
    const uint32_t fence_stride = kMode == kModeBatch ? s.fence_stride : fence_stride_arg;
    const auto key_hashes = [&] { return kMode == kModeBatch ? s.key_hashes : ma.key_hashes; };  // read where it is used: no register to spare
    const uint32_t top_step = k > 1 ? 1u << (31 - __builtin_clz(k - 1)) : 0;

    if (kMode == kModeRange && n <= (uint32_t)kMergeThreads) {
        // ---- a range of no more entries than threads, as nearly all are: one entry per thread, as in merge_short_kernel, and stored from
        //      registers: 500 ranges of a 4M-entry tree 15.3 -> 11.1 us, 2,000 of a 20M-entry tree 51.6 -> 35.9, one of 50,000 entries the same
        uint4 ent[1][4];
        uint32_t piece[1], at[1];
        const uint32_t e = (uint32_t)tid < n ? tid : 0;
        piece[0] = piece_of(s.seg, k, top_step, e);
        const uint4* const src = reinterpret_cast<const uint4*>(s.run[piece[0]] + s.lo[piece[0]] + (e - s.seg[piece[0]]));
#pragma unroll
        for (int part = 0; part < 4; part++) {
            ent[0][part] = make_uint4(0, 0, 0, 0);
            if ((uint32_t)tid < n) ent[0][part] = load_global_u4(src + part);
        }
        short_rank<1, kMergeThreads, kMergeThreads>(s, s.buf[0], alive, s.inexact, ent, piece, at, n, k, flags);
        constexpr uint32_t kWords = kMergeThreads / 32;
        const uint32_t bits = (uint32_t)lane < kWords ? alive[lane] : 0, incl = wave_scan_u32(__popc(bits));
        const uint32_t total = __shfl(incl, kWave - 1, kWave);
        const uint32_t word = at[0] >> 5, bit = at[0] & 31, b = __shfl(bits, word & (kWords - 1), kWave);
        const uint32_t slot = __shfl(incl - __popc(bits), word & (kWords - 1), kWave) + __popc(b & ((1u << bit) - 1));
        const bool failed = s.failed != 0 || total > ma.max_entries;
        if (tid == 0) ma.counts[tile] = failed ? ~0u : total;
        if (!failed && (uint32_t)tid < n && ((b >> bit) & 1) != 0) {
            uint4* const dst = reinterpret_cast<uint4*>(out + tile * (uint64_t)ma.max_entries + slot);
#pragma unroll
            for (int part = 0; part < 4; part++) dst[part] = ent[0][part];
        }
        return;
    }

    // ---- load: entry e = tid + i * kMergeThreads stays in this thread's registers until it is stored
    // the few instructions of a memory phase should not queue behind the other workgroup's merge arithmetic
    __builtin_amdgcn_s_setprio(2);
    uint4 ent[kMergeItems][4];
    uint32_t pos[kMergeItems];  // merged position of the entry
    {
        // all addresses first, then all loads, so that the loads of one thread are in flight together
        // (threads without an entry re-read entry 0 and never use it; an unusable tile has n = 0)
        const uint4* src[kMergeItems];
#pragma unroll
        for (int i = 0; i < kMergeItems; i++) {
            const uint32_t e = tid + i * kMergeThreads;
            const uint32_t ee = e < n ? e : 0;
            const uint32_t j = piece_of(s.seg, k, top_step, ee);
            src[i] = reinterpret_cast<const uint4*>(s.run[j] + s.lo[j] + (ee - s.seg[j]));
            pos[i] = 0;
        }
        if (n > 0) {
#pragma unroll
            for (int i = 0; i < kMergeItems; i++)
#pragma unroll
                for (int part = 0; part < 4; part++) ent[i][part] = load_global_u4(src[i] + part);
        } else {
#pragma unroll
            for (int i = 0; i < kMergeItems; i++)
#pragma unroll
                for (int part = 0; part < 4; part++) ent[i][part] = make_uint4(0, 0, 0, 0);
        }
    }
#pragma unroll
    for (int i = 0; i < kMergeItems; i++) {
        const uint32_t e = tid + i * kMergeThreads;
        if (e < n) {
            Key kk = key_from_raw(ent[i][0], ent[i][1]);
            Sur v;
            v.hi = kk.w[0];
            v.lo = (kk.w[1] & ~0xFFFFull) | e;
            sur_store(&s.buf[0][sw(e)], v);
        }
    }
    if (tid == 0) s.flag[n] = 0;
    __builtin_amdgcn_s_setprio(0);
    __syncthreads();

    // ---- merge rounds: lists of `width` runs each are merged pairwise.  Surrogates are compared as whole
    //      128-bit numbers: the index in the low bits grows with the run number, so the order is the stable one
    //      (equal keys: lower run first) and all values are distinct.  Thread t produces outputs
    //      [4t, 4t + 4): a co-rank search finds where they start in the two lists, then the next four of each
    //      list are read at once and merged in registers (half-cleaner + two exchange stages), so the only
    //      dependent LDS reads of a round are those of the search.
    const uint32_t j_first = piece_of(s.seg, k, top_step, min((uint32_t)(tid * kRoundItems), n ? n - 1 : 0));
    int cur = 0;
    for (uint32_t width = 1; width < k; width <<= 1) {
        const uint4* in = s.buf[cur];
        uint4* dst = s.buf[cur ^ 1];
        uint32_t o = tid * kRoundItems, j = j_first;
        const uint32_t o_end = min(o + (uint32_t)kRoundItems, n);
        while (o < o_end) {
            // the pair of lists whose output range contains position o (o lies in piece j)
            const uint32_t ra = (j / (2 * width)) * 2 * width, rb = min(ra + width, k), rc = min(ra + 2 * width, k);
            const uint32_t sa = s.seg[ra], sb = s.seg[rb], sc = s.seg[rc];
            const uint32_t len_a = sb - sa, len_b = sc - sb;
            const uint32_t stop = min(o_end, sc);
            // co-rank of diagonal d: how many of the first d outputs come from the left list
            const uint32_t d = o - sa;
            uint32_t lo = d > len_b ? d - len_b : 0, hi = min(d, len_a);
            while (lo < hi) {
                const uint32_t mid = (lo + hi) >> 1;
                if (sur_less(sur_load(&in[sw(sa + mid)]), sur_load(&in[sw(sb + (d - 1 - mid))]))) lo = mid + 1;
                else hi = mid;
            }
            const uint32_t a = lo, b = d - lo;
            Sur x[kRoundItems], y[kRoundItems];
#pragma unroll
            for (int i = 0; i < kRoundItems; i++) {
                x[i] = sur_load(&in[sw(min(sa + a + i, (uint32_t)kTileCap - 1))]);
                y[i] = sur_load(&in[sw(min(sb + b + i, (uint32_t)kTileCap - 1))]);
                if (a + i >= len_a) x[i].hi = x[i].lo = ~0ull;  // past the end of a list: larger than any surrogate
                if (b + i >= len_b) y[i].hi = y[i].lo = ~0ull;
            }
            // the four smallest of x[0..3], y[0..3] in order
            Sur c[kRoundItems];
#pragma unroll
            for (int i = 0; i < kRoundItems; i++) c[i] = sur_less(x[i], y[kRoundItems - 1 - i]) ? x[i] : y[kRoundItems - 1 - i];
            sur_order(c[0], c[2]);
            sur_order(c[1], c[3]);
            sur_order(c[0], c[1]);
            sur_order(c[2], c[3]);
#pragma unroll
            for (int i = 0; i < kRoundItems; i++)
                if (o + i < stop) sur_store(&dst[sw(o + i)], c[i]);
            o = stop;
            for (j = rc; j + 1 < k && s.seg[j + 1] <= o; j++) {}  // piece of the next position (skips empty pieces)
        }
        __syncthreads();
        cur ^= 1;
    }

    // ---- merged position p <-> entry index; does p repeat the 14-byte key prefix of p-1?
    {
        const uint4* fin = s.buf[cur];
        const uint32_t o0 = tid * kMergeItems;
        if (o0 < n) {
            Sur prev = sur_load(&fin[sw(o0 > 0 ? o0 - 1 : 0)]);
            for (uint32_t o = o0; o < min(o0 + (uint32_t)kMergeItems, n); o++) {
                Sur v = sur_load(&fin[sw(o)]);
                s.flag[o] = (o > 0 && sur_same_key(prev, v)) ? kFlagEq : 0;
                s.rank[v.lo & 0xFFFF] = (uint16_t)o;
                prev = v;
            }
        }
    }
    __syncthreads();

    // ---- every owner posts key bytes 14..31, seqno and type of its entries at their merged positions
    uint4* info0 = s.buf[0];  // {seqno lo, seqno hi, type | key bytes 14..15 << 8, entry index} of the entry at a position
    uint4* info1 = s.buf[1];  // its key bytes 16..31
#pragma unroll
    for (int i = 0; i < kMergeItems; i++) {
        const uint32_t e = tid + i * kMergeThreads;
        if (e < n) {
            const uint32_t p = s.rank[e];
            pos[i] = p;
            info0[sw(p)] = make_uint4(ent[i][2].x, ent[i][2].y, (ent[i][2].z & 0xFF) | (ent[i][0].w & 0xFFFF0000u) >> 8, e);
            info1[sw(p)] = ent[i][1];
        }
    }
    __syncthreads();

    // ---- exact equality with the previous position; a differing tail under an equal prefix makes the tile inexact.
    //      A thread's four positions are neighbours, so the words of positions o0-1 .. o0+3 that some comparison
    //      needs are all requested before the first compare.
    {
        const uint32_t o0 = tid * kMergeItems;
        if (o0 < n) {
            const uint32_t f = *reinterpret_cast<const uint32_t*>(&s.flag[o0]);
            bool eq[kMergeItems + 1];
#pragma unroll
            for (int i = 0; i < kMergeItems; i++) eq[i] = o0 + i < n && ((f >> (8 * i)) & kFlagEq) != 0;
            eq[kMergeItems] = false;
            uint32_t z[kMergeItems + 1];
            uint4 t[kMergeItems + 1];  // [i] = position o0 + i - 1
#pragma unroll
            for (int i = 0; i <= kMergeItems; i++) {
                const bool need = (i > 0 && eq[i - 1]) || eq[i];  // compared as a position or as a predecessor
                z[i] = 0;
                t[i] = make_uint4(0, 0, 0, 0);
                if (need) {
                    z[i] = info0[sw(o0 + i - 1)].z;
                    t[i] = info1[sw(o0 + i - 1)];
                }
            }
            uint32_t g = f;
            bool inexact = false;
#pragma unroll
            for (int i = 0; i < kMergeItems; i++) {
                if (eq[i]) {
                    const bool same = ((z[i + 1] ^ z[i]) >> 8) == 0 && t[i + 1].x == t[i].x && t[i + 1].y == t[i].y &&
                                      t[i + 1].z == t[i].z && t[i + 1].w == t[i].w;
                    g |= same ? (uint32_t)kFlagFullEq << (8 * i) : 0;
                    inexact = inexact || !same;
                }
            }
            if (g != f) *reinterpret_cast<uint32_t*>(&s.flag[o0]) = g;
            if (inexact) s.inexact = 1;
        }
    }
    __syncthreads();

    if (s.inexact != 0) {
        // ---- repair: positions that share the 14-byte prefix but not the whole key stand in run order, not in
        //      key order.  The thread whose share holds the first position of such a group sorts the group by the
        //      rest of the key (stable, so equal keys keep their run order); a group too long for one thread
        //      sends the whole tile to the exact path instead.
        const uint32_t o0 = tid * kMergeItems;
        for (uint32_t o = o0; o < min(o0 + (uint32_t)kMergeItems, n); o++) {
            if ((s.flag[o] & kFlagEq) != 0 || (s.flag[o + 1] & kFlagEq) == 0) continue;  // flag[n] is 0
            uint32_t end = o + 1;
            bool broken = false;
            for (; s.flag[end] & kFlagEq; end++) broken = broken || (s.flag[end] & kFlagFullEq) == 0;
            if (!broken) continue;
            if (end - o > (uint32_t)kRepairMax) {
                s.inexact = 2;
                continue;
            }
            for (uint32_t a = o + 1; a < end; a++) {
                const uint4 x0 = info0[sw(a)], x1 = info1[sw(a)];
                uint32_t b = a;
                for (; b > o && tail_less(x0, x1, info0[sw(b - 1)], info1[sw(b - 1)]); b--) {
                    info0[sw(b)] = info0[sw(b - 1)];
                    info1[sw(b)] = info1[sw(b - 1)];
                }
                info0[sw(b)] = x0;
                info1[sw(b)] = x1;
            }
            s.rank[info0[sw(o)].w] = (uint16_t)o;
            for (uint32_t a = o + 1; a < end; a++) {
                const bool same = !tail_less(info0[sw(a - 1)], info1[sw(a - 1)], info0[sw(a)], info1[sw(a)]);  // sorted: not less = equal
                s.flag[a] = same ? (kFlagEq | kFlagFullEq) : kFlagEq;
                s.rank[info0[sw(a)].w] = (uint16_t)a;
            }
        }
        __syncthreads();
        if (s.inexact == 1) {
#pragma unroll
            for (int i = 0; i < kMergeItems; i++) {
                const uint32_t e = tid + i * kMergeThreads;
                if (e < n) pos[i] = s.rank[e];
            }
        }
    }

    uint32_t survive = 0;  // bit i: the entry at this thread's position i is an output entry
    if (s.inexact != 2) {
        // ---- survivors: newest version of each key (largest seqno, ties to the earlier = lower run),
        //      minus winning tombstones when the output is the last level.  Groups of equal keys are short and
        //      mostly lie inside a thread's four positions: those are settled from registers, and only a
        //      group that crosses into a neighbour's share is followed through LDS.
        const uint32_t o0 = tid * kMergeItems;
        if (o0 < n) {
            const uint32_t f = *reinterpret_cast<const uint32_t*>(&s.flag[o0]);
            const bool more = o0 + kMergeItems < n && (s.flag[o0 + kMergeItems] & kFlagFullEq) != 0;  // the group goes on to the right
            bool fe[kMergeItems];
            uint64_t seq[kMergeItems];
            uint32_t type[kMergeItems];
#pragma unroll
            for (int i = 0; i < kMergeItems; i++) {
                const bool valid = o0 + i < n;
                const uint4 me = info0[sw(valid ? o0 + i : o0)];
                fe[i] = valid && ((f >> (8 * i)) & kFlagFullEq) != 0;
                seq[i] = ((uint64_t)me.y << 32) | me.x;
                type[i] = me.z & 0xFF;
            }
#pragma unroll
            for (int i = 0; i < kMergeItems; i++) {
                bool win = true, chain = true;
#pragma unroll
                for (int q = i; q >= 1; q--) {  // earlier members of the group
                    chain = chain && fe[q];
                    if (chain && seq[q - 1] >= seq[i]) win = false;
                }
                if (chain && fe[0])
                    for (uint32_t p = o0; s.flag[p] & kFlagFullEq; p--) {  // flag[0] never has the bit
                        const uint4 v = info0[sw(p - 1)];
                        if ((((uint64_t)v.y << 32) | v.x) >= seq[i]) win = false;
                    }
                chain = true;
#pragma unroll
                for (int q = i + 1; q < kMergeItems; q++) {  // later members
                    chain = chain && fe[q];
                    if (chain && seq[q] > seq[i]) win = false;
                }
                if (chain && more)
                    for (uint32_t p = o0 + kMergeItems; s.flag[p] & kFlagFullEq; p++) {  // flag[n] is 0
                        const uint4 v = info0[sw(p)];
                        if ((((uint64_t)v.y << 32) | v.x) > seq[i]) win = false;
                    }
                if (win && (flags & LSM_BOTTOMMOST) && type[i] == LSM_TOMBSTONE) win = false;
                if (win && o0 + i < n) survive |= 1u << i;
            }
        }
    } else {
        // ---- exact path: merged position and winner of every entry by binary search over the
        //      tile's other pieces with full 32-byte compares, order (key, run index).  The keys
        //      are staged in LDS in entry order (the info arrays are not needed any more), so only
        //      the seqno of an equal key in another piece is read from global memory.
        __syncthreads();
        uint4* klo = s.buf[0];  // key bytes 0..15 of entry e
        uint4* khi = s.buf[1];  // key bytes 16..31
#pragma unroll
        for (int i = 0; i < kMergeItems; i++) {
            const uint32_t e = tid + i * kMergeThreads;
            if (e < n) {
                klo[e] = ent[i][0];
                khi[e] = ent[i][1];
            }
        }
        for (uint32_t o = tid; o <= n; o += kMergeThreads) s.flag[o] = 0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kMergeItems; i++) {
            const uint32_t e = tid + i * kMergeThreads;
            if (e < n) {
                const uint32_t j = piece_of(s.seg, k, top_step, e);
                const Key x = key_from_raw(ent[i][0], ent[i][1]);
                const uint64_t seq = ((uint64_t)ent[i][2].y << 32) | ent[i][2].x;
                uint32_t p = e - s.seg[j];
                bool win = true;
                for (uint32_t j2 = 0; j2 < k; j2++) {
                    if (j2 == j) continue;
                    const uint32_t first = s.seg[j2], last = s.seg[j2 + 1];
                    uint32_t lb = first, ub = last;
                    while (lb < ub) {
                        const uint32_t mid = (lb + ub) >> 1;
                        if (entry_key_less(&klo[mid], &khi[mid], x)) lb = mid + 1;
                        else ub = mid;
                    }
                    p += lb - first;
                    if (lb < last && key_equal(key_from_raw(klo[lb], khi[lb]), x)) {
                        const uint64_t other = s.run[j2][s.lo[j2] + (lb - first)].seqno;
                        if (other > seq || (other == seq && j2 < j)) win = false;
                        if (j2 < j) p++;
                    }
                }
                if (win && (flags & LSM_BOTTOMMOST) && (ent[i][2].z & 0xFF) == LSM_TOMBSTONE) win = false;
                pos[i] = p;
                if (win) s.flag[p] = 1;
            }
        }
        __syncthreads();
        if (tid * kMergeItems < n) {
            const uint32_t f = *reinterpret_cast<const uint32_t*>(&s.flag[tid * kMergeItems]);
#pragma unroll
            for (int i = 0; i < kMergeItems; i++) survive |= tid * kMergeItems + i < n ? ((f >> (8 * i)) & 1) << i : 0;
        }
    }

    // ---- survivors before each merged position (block-wide exclusive prefix sum in position order)
    uint32_t total = 0;
    {
        const uint32_t mine = __popc(survive), incl = wave_scan_u32(mine);
        if (lane == kWave - 1) s.wave_count[wave] = incl;
        __syncthreads();
        uint32_t before = incl - mine;
#pragma unroll
        for (int w = 0; w < kMergeThreads / kWave; w++) {
            const uint32_t c = s.wave_count[w];
            before += w < wave ? c : 0;
            total += c;
        }
        uint32_t slot[kMergeItems];
#pragma unroll
        for (int i = 0; i < kMergeItems; i++) {
            slot[i] = (survive >> i) & 1 ? before : kNoSlot;
            before += (survive >> i) & 1;
        }
        *reinterpret_cast<uint2*>(&s.prefix[tid * kMergeItems]) = make_uint2(slot[0] | slot[1] << 16, slot[2] | slot[3] << 16);
    }

    __syncthreads();  // prefix[] complete, last reads of info[] done: the staging area is free

    // ---- output offset of this tile: wave 0 looks back while the other waves already stage their survivors
    if (wave == 0) {
        __builtin_amdgcn_s_setprio(3);  // the stores of the whole tile wait for this wave
        bool failed;
        uint64_t base;
        if (kMode == kModeRange) {
            // a range has its own slot of max_entries entries; one that holds more (or more than a tile) is reported
            base = tile * (uint64_t)ma.max_entries;
            failed = s.failed != 0 || total > ma.max_entries;
            if (lane == 0) ma.counts[tile] = failed ? ~0u : total;
        } else {
            base = lookback(kMode == kModeBatch ? s.status : ws.status, tile, total, s.failed != 0, &failed);
        }
        if (lane == 0) {
            s.base = base;
            if (failed) s.failed = 1;
        }
    }

    // ---- survivors leave through an LDS stage so that the global stores are contiguous; the four
    //      16-byte parts of a slot are rotated by the slot number to spread them over the banks
    uint4* stage = &s.buf[0][0];
    __builtin_amdgcn_s_setprio(2);  // output is a memory phase again
    uint64_t base = 0;
    uint32_t first = 0;
    do {
#pragma unroll
        for (int i = 0; i < kMergeItems; i++) {
            const uint32_t e = tid + i * kMergeThreads;
            const uint32_t at = e < n ? s.prefix[pos[i]] : kNoSlot;
            if (at != kNoSlot) {
                // pointer rewrite for merged tensor files (paper section 3.4): vptr = base[file] + offset
                if (kExtras && first == 0 && remap_files != 0 && (ent[i][2].z & 0xFF) == LSM_PUT && ent[i][3].y < remap_files) {
                    const uint64_t v = remap_base[ent[i][3].y] + ent[i][3].x;
                    ent[i][3].x = (uint32_t)v;
                    ent[i][3].y = (uint32_t)(v >> 32);
                }
                const uint32_t slot = at - first;  // wraps for slots before this pass
                if (slot < (uint32_t)kStageEntries) {
#pragma unroll
                    for (int part = 0; part < 4; part++) stage[slot * 4 + (part ^ (slot & 3))] = ent[i][part];
                    // the filter hash of the survivor's key travels with it (paper section 2.2: a new run gets its Bloom
                    // filter; the filter is then built from these 8-byte values, not from the run)
                    if (kExtras == 2 && key_hashes() != nullptr) {
                        const uint64_t h = bloom_key_hash(key_from_raw(ent[i][0], ent[i][1]));
                        if (slot < (uint32_t)kStageEntries / 2) reinterpret_cast<uint64_t*>(s.rank)[slot] = h;
                        else hash_stage_upper[slot - kStageEntries / 2] = h;
                    }
                }
            }
        }
        __syncthreads();
        if (first == 0) {
            const bool failed = s.failed != 0;
            base = s.base;
            if (kMode != kModeRange && tile == last_tile && tid == 0) *n_out = failed ? ~0ull : base + total;
            if (failed) return;
        }
        // Nontemporal: whole lines leave the L2 at once and take no place from the lines that other tiles are loading (each is
        // asked for four times, 16 bytes at a time).  2M + 20M entries 675 -> 635 us, 4.4 TB/s; 16 x 4M 2648 -> 2508, 8 x 500k with
        // fences and hashes 338 -> 325; inputs of a few tiles are the same.  Nontemporal loads instead lose (2M + 20M 800 us): a
        // line is gone before its other three quarters are asked for.  So do loads of whole lines by four lanes (660, 2540), which
        // cost a transposition in registers, and reading the tile 256 to 1,024 further on ahead (737 to 823, 2725 to 2930).
        const uint32_t count = min(total - first, (uint32_t)kStageEntries);
        uint4* dst = reinterpret_cast<uint4*>(out + base + first);
        for (uint32_t c = tid; c < count * 4; c += kMergeThreads) {
            const uint32_t part = (c ^ (c >> 2)) & 3;  // which 16 bytes of the entry stage[c] holds
            store_streaming_u4(&dst[(c & ~3u) | part], stage[c]);
        }
        if (kExtras && fence_out != nullptr) {
            // fence index of the new run: the key of every fence_stride-th output entry.  The first one of this pass is the only
            // division: one per output entry, and flags read byte by byte for the prefix sum above, cost the merge of 2M + 20M
            // entries 29 us of 704
            const uint64_t fence = (base + first + fence_stride - 1) / fence_stride;
            const uint64_t skip = fence * fence_stride - (base + first);  // entries before it
            for (uint64_t q = tid; skip + (q >> 1) * fence_stride < count; q += kMergeThreads) {
                const uint32_t slot = (uint32_t)(skip + (q >> 1) * fence_stride), part = q & 1;
                fence_out[fence * 2 + q] = stage[slot * 4 + (part ^ (slot & 3))];
            }
        }
        if (kExtras == 2 && key_hashes() != nullptr) {
            for (uint32_t c = tid; c < count; c += kMergeThreads)
                key_hashes()[base + first + c] = c < (uint32_t)kStageEntries / 2 ? reinterpret_cast<const uint64_t*>(s.rank)[c]
                                                                                  : hash_stage_upper[c - kStageEntries / 2];
        }
        first += kStageEntries;
        if (first < total) __syncthreads();  // the stage is reused
    } while (first < total);
}

// ---------------------------------------------------------------------------------------
// Tile merge where there is a compute unit for every tile: the time of a call is one tile's chain of dependent steps.
//   - One thread per entry (two in tiles of more than kShortThreads).  It finds the entry's place in a merge round by one binary search
//     in the other list of the pair and keeps surrogate and place in registers, so nothing is read back: 1.2 us a round of 512 entries,
//     where merge_kernel, four outputs a thread, has two waves at work and takes 2.0.
//   - Key tails, seqnos and types lie in LDS by entry from the load on.  An entry looks at its two neighbours in the final order, and
//     only where one has the same 14 bytes goes on to the group's other members: order by the rest of the key, newest version and
//     survival come out at once, without the passes that post them by position, compare, repair and count (1.1 us, 3.9 there).  A group longer
//     than kRepairMax sends the tile to the exact path, as there.
//   - Survivors are bits by position; every wave adds up the 64 words for itself.
//   - The look-back asks for all earlier tiles' words at once.
// LDS: 130 KB, one workgroup on a compute unit.  Whole kernel, 128 tiles of 512 entries of four runs 17.0 -> 11.4 us; one tile of a driver's merge 11.0 -> 8.6.
// What is left of the 11.4: pieces 1.3, load 1.2, rounds 2.4, neighbours 1.4, look-back 2.6 (two trips through the
// memory-side cache, and the spread of the tiles), stage and store 1.1.
// ---------------------------------------------------------------------------------------
constexpr int kShortWindows = (int)((kShortTiles + kWave - 1) / kWave);

struct ShortShared : TileHead {
    uint4 mem[4 * kTileCap];          // surrogate ping-pong, key tails, seqno / type by entry index; then output staging
    uint32_t alive[kTileCap / 32];    // bit p: the entry at merged position p is an output entry
    uint32_t deep;                    // some prefix-tie group is long
};

// lookback for tiles with no more than kShortTiles - 1 before them: all their status words are asked for at once.
__device__ uint64_t lookback_few(uint64_t* status, const uint64_t epoch, const uint32_t tile, const uint64_t count, const bool self_failed, bool* failed) {
    const int lane = threadIdx.x & (kWave - 1);
    *failed = self_failed;
    auto publish = [&](uint64_t state, uint64_t value) {
        if (lane == 0) __hip_atomic_store(&status[tile], (state << kStShift) | epoch | value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    if (self_failed || tile == 0) {
        publish(self_failed ? kStFailed : kStPrefix, self_failed ? 0 : count);
        return 0;
    }
    publish(kStAggregate, count);
    uint64_t base = 0;
    bool bad = false;
    for (uint32_t spins = 0;; spins++) {
        uint64_t st[kShortWindows];  // lane l, window w: tile - 1 - 64 w - l
#pragma unroll
        for (int w = 0; w < kShortWindows; w++) {
            const int t = (int)tile - 1 - w * kWave - lane;
            st[w] = kStPrefix << kStShift;  // tiles before tile 0: an empty prefix
            if (t >= 0) {
                st[w] = __hip_atomic_load(&status[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (((st[w] ^ epoch) >> kStEpochShift) & (kStEpochs - 1)) st[w] = kStEmpty;  // of an earlier call
            }
        }
        bool ready = true, open = true;  // open: no prefix nearer than window w
        base = 0;
#pragma unroll
        for (int w = 0; w < kShortWindows; w++) {
            const uint64_t state = st[w] >> kStShift, pmask = __ballot(state == kStPrefix);
            const int first = pmask ? __ffsll((unsigned long long)pmask) - 1 : kWave - 1;  // nearest tile with a full prefix
            if (open) {
                ready = ready && __ballot(lane <= first && state == kStEmpty) == 0;
                bad = bad || __ballot(lane <= first && state == kStFailed) != 0;
                base += lane <= first ? st[w] & kStValueMask : 0;
            }
            open = open && pmask == 0;
        }
        if (ready || bad) break;
        bad = spins >= kSpinLimit;
        if (bad) break;
        __builtin_amdgcn_s_sleep(1);
    }
    base = wave_sum_u64(base);
    *failed = bad;
    publish(bad ? kStFailed : kStPrefix, bad ? 0 : base + count);
    return base;
}

// From the tile's pieces on; s.alive and s.deep are zero.
template <int kExtras>
__device__ __forceinline__ void short_tile(ShortShared& s, uint64_t* hash_stage, const uint64_t* remap_base, const uint32_t remap_files) {
    const uint32_t tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    const uint32_t n = s.n, tile = s.tile;
    const uint32_t k = s.k, flags = s.flags;
    const uint32_t top_step = k > 1 ? 1u << (31 - __builtin_clz(k - 1)) : 0;
    uint4 ent[kShortItems][4];
    uint32_t piece[kShortItems], at[kShortItems];
    {
        const uint4* src[kShortItems];
#pragma unroll
        for (int i = 0; i < kShortItems; i++) {
            const uint32_t e = tid + i * kShortThreads, ee = e < n ? e : 0;
            piece[i] = piece_of(s.seg, k, top_step, ee);
            src[i] = reinterpret_cast<const uint4*>(s.run[piece[i]] + s.lo[piece[i]] + (ee - s.seg[piece[i]]));
        }
#pragma unroll
        for (int i = 0; i < kShortItems; i++)
#pragma unroll
            for (int part = 0; part < 4; part++) {
                ent[i][part] = make_uint4(0, 0, 0, 0);
                if (tid + i * kShortThreads < n) ent[i][part] = load_global_u4(src[i] + part);
            }
    }
    if (n <= (uint32_t)kShortThreads) short_rank<1, kShortThreads, kTileCap>(s, s.mem, s.alive, s.deep, ent, piece, at, n, k, flags);
    else short_rank<kShortItems, kShortThreads, kTileCap>(s, s.mem, s.alive, s.deep, ent, piece, at, n, k, flags);

    // ---- survivors before each position, by every wave for itself; s.alive is complete
    const uint32_t bits = s.alive[lane], incl = wave_scan_u32(__popc(bits));
    const uint32_t total = __shfl(incl, kWave - 1, kWave), before = incl - __popc(bits);
    uint32_t slot[kShortItems];
#pragma unroll
    for (int i = 0; i < kShortItems; i++) {
        const bool mine = tid + i * kShortThreads < n;
        const uint32_t word = mine ? at[i] >> 5 : 0, bit = at[i] & 31;
        const uint32_t b = __shfl(bits, word, kWave), r = __shfl(before, word, kWave) + __popc(b & ((1u << bit) - 1));
        slot[i] = mine && ((b >> bit) & 1) ? r : kNoSlot;
    }

    // ---- output offset of this tile: wave 0 looks back while the other waves stage their survivors
    if (wave == 0) {
        __builtin_amdgcn_s_setprio(3);
        bool failed;
        const uint64_t base = lookback_few(s.status, s.epoch, tile, total, s.failed != 0, &failed);
        if (lane == 0) {
            s.base = base;
            if (failed) s.failed = 1;
        }
    }
    uint4* const stage = s.mem;
    uint64_t* const key_hashes = s.key_hashes;
#pragma unroll
    for (int i = 0; i < kShortItems; i++) {
        if (slot[i] == kNoSlot) continue;
        if (kExtras && remap_files != 0 && (ent[i][2].z & 0xFF) == LSM_PUT && ent[i][3].y < remap_files) {
            const uint64_t v = remap_base[ent[i][3].y] + ent[i][3].x;
            ent[i][3].x = (uint32_t)v;
            ent[i][3].y = (uint32_t)(v >> 32);
        }
#pragma unroll
        for (int part = 0; part < 4; part++) stage[slot[i] * 4 + (part ^ (slot[i] & 3))] = ent[i][part];
        if (kExtras == 2 && key_hashes != nullptr) hash_stage[slot[i]] = bloom_key_hash(key_from_raw(ent[i][0], ent[i][1]));
    }
    __syncthreads();
    const bool failed = s.failed != 0;
    const uint64_t base = s.base;
    if (tile == s.job_tiles - 1 && tid == 0) *s.n_out = failed ? ~0ull : base + total;
    if (failed) return;
    uint4* const dst = reinterpret_cast<uint4*>(s.out + base);
    for (uint32_t c = tid; c < total * 4; c += kShortThreads) {
        const uint32_t part = (c ^ (c >> 2)) & 3;
        store_streaming_u4(&dst[(c & ~3u) | part], stage[c]);
    }
    uint4* const fence_out = s.fence_out;
    if (kExtras && fence_out != nullptr) {
        const uint32_t fence_stride = s.fence_stride;
        const uint64_t fence = (base + fence_stride - 1) / fence_stride, skip = fence * fence_stride - base;
        for (uint64_t q = tid; skip + (q >> 1) * fence_stride < total; q += kShortThreads) {
            const uint32_t at_slot = (uint32_t)(skip + (q >> 1) * fence_stride), part = q & 1;
            fence_out[fence * 2 + q] = stage[at_slot * 4 + (part ^ (at_slot & 3))];
        }
    }
    if (kExtras == 2 && key_hashes != nullptr)
        for (uint32_t c = tid; c < total; c += kShortThreads) key_hashes[base + c] = hash_stage[c];
}

template <int kExtras, int kMode>
__global__ void __launch_bounds__(kShortThreads) merge_short_kernel(RunTable rt, Workspace ws, uint64_t n_tiles, uint32_t flags, lsm_entry_t* out,
                                                                   uint64_t* n_out, const uint64_t* remap_base, uint32_t remap_files,
                                                                   uint4* fence_out, uint32_t fence_stride, ModeArgs ma) {
    static_assert(kMode == kModeSingle || kMode == kModeBatch, "ranges have tiles of their own");
    __shared__ ShortShared s;
    __shared__ uint64_t hash_stage[kExtras == 2 ? kTileCap : 1];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    if (wave == 0) {
        if (kMode == kModeSingle && lane == 0) {
            s.k = rt.k;
            s.flags = flags;
            s.job_tiles = (uint32_t)n_tiles;
            s.out = out;
            s.n_out = n_out;
            s.status = ws.status;
            s.fence_out = fence_out;
            s.fence_stride = fence_stride;
            s.key_hashes = ma.key_hashes;
        }
        if (lane == 0) s.epoch = 0;
        tile_pieces<kMode>(s, rt, ws, n_tiles, ma, nullptr);
    } else if (wave == 1) {
        s.alive[lane] = 0;
    } else if (wave == 2 && lane == 0) {
        s.deep = 0;
    }
    static_assert(kTileCap / 32 == kWave, "a wave holds the survivors' bits");
    __syncthreads();
    short_tile<kExtras>(s, hash_stage, remap_base, remap_files);
}

// Compactions of one or two runs each in a single launch, where the caller keeps status words of its own (see ClearSpan): every workgroup
// finds the two boundaries of its tile itself, a wave each, and nothing has to be zeroed or written for it beforehand.
// A launch less is 4 us on the GPU, and the two searches cost the tile two (96 driver flushes 2564 -> 2291 us).
template <uint32_t kJobs, uint32_t kRuns>
struct WholeTable {
    JobDesc jobs[kJobs];
    const lsm_entry_t* run_ptr[kRuns];
    uint64_t run_n[kRuns];
    uint64_t* status;
    uint64_t epoch;  // in its place
    uint32_t n_jobs, spacing;
};
template <int kExtras, uint32_t kJobs, uint32_t kRuns>
__global__ void __launch_bounds__(kShortThreads) merge_whole_kernel(WholeTable<kJobs, kRuns> table) {
    __shared__ ShortShared s;
    __shared__ uint64_t hash_stage[kExtras == 2 ? kTileCap : 1];
    __shared__ uint64_t rows[2][2];  // where the tile starts and ends in the two runs
    const uint32_t tid = threadIdx.x;
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    uint32_t job = 0;
    if (kJobs > 1)
        for (uint32_t q = 1; q < table.n_jobs; q++) job = table.jobs[q].first_tile <= blockIdx.x ? q : job;
    const JobDesc& d = table.jobs[job];
    const uint32_t tile = blockIdx.x - d.first_tile;
    const lsm_entry_t *a = table.run_ptr[d.run_off], *b = d.k > 1 ? table.run_ptr[d.run_off + 1] : a;
    const uint64_t na = table.run_n[d.run_off], nb = d.k > 1 ? table.run_n[d.run_off + 1] : 0;
    if (wave < 2) {
        const uint32_t row = tile + wave;
        uint64_t ia = 0, ib = 0;
        if (row >= d.n_tiles) ia = na, ib = nb;
        else if (row > 0) split_two_wave(a, na, b, nb, row * (uint64_t)tile_spacing(table.spacing, d.k), ia, ib);
        if (lane == 0) rows[wave][0] = ia, rows[wave][1] = ib;
    } else if (wave == 2) {
        s.alive[lane] = 0;
        if (lane == 0) {
            s.deep = 0;
            s.tile = tile;
            s.k = d.k;
            s.flags = d.flags;
            s.job_tiles = d.n_tiles;
            s.out = d.out;
            s.n_out = d.n_out;
            s.status = table.status + d.first_tile;
            s.epoch = table.epoch;
            s.fence_out = d.fence_out;
            s.fence_stride = d.fence_stride;
            s.key_hashes = d.clear_n & kHashesBehind ? reinterpret_cast<uint64_t*>(d.clear + (d.clear_n & ~kHashesBehind)) : nullptr;
            s.run[0] = a;
            s.run[1] = b;
        }
    } else {  // what a later kernel needs zeroed
        constexpr uint32_t kOthers = kShortThreads - 3 * kWave;
        for (uint32_t c = tile * kOthers + tid - 3 * kWave; c < (d.clear_n & ~kHashesBehind); c += d.n_tiles * kOthers) d.clear[c] = make_uint4(0, 0, 0, 0);
    }
    __syncthreads();
    if (tid == 0) {
        const uint64_t len_a = rows[1][0] - rows[0][0], len_b = rows[1][1] - rows[0][1];
        // only inputs that break the precondition can make a pair of rows inconsistent
        const bool ok = rows[0][0] <= rows[1][0] && rows[0][1] <= rows[1][1] && len_a + len_b <= (uint64_t)kTileCap && len_a <= (uint64_t)kTileCap;
        s.lo[0] = rows[0][0];
        s.lo[1] = rows[0][1];
        s.seg[0] = 0;
        s.seg[1] = ok ? (uint32_t)len_a : 0;
        s.seg[2] = ok ? (uint32_t)(len_a + len_b) : 0;
        s.n = s.seg[2];
        s.failed = ok ? 0 : 1;
    }
    __syncthreads();
    short_tile<kExtras>(s, hash_stage, nullptr, 0);
}

// ---------------------------------------------------------------------------------------
// Partition of a batch of independent compactions.  A job of boundaries at ranked samples has a wave per sample (ranked_row),
// any other one a wave per tile, the wave of tile t > 0 searching boundary t over the job's whole runs (the jobs of a batch are
// small).  A job's first wave also writes the first (all zero) and the last (run lengths) row of its split table; its waves
// together write the job number and clear the status word of each of its tiles.
// ---------------------------------------------------------------------------------------
// A batch that is small enough travels as a kernel argument (kInline): the partition's waves take their job from there,
// and the jobs' first ones put the descriptors where the merge kernel looks for them.  (Copying the table first
// was a transfer of 4 us before the first kernel, and a wait of the host for the previous one.)
constexpr uint32_t kInlineJobs = 20, kInlineRuns = 56;
struct BatchInline {
    JobDesc jobs[kInlineJobs];
    const lsm_entry_t* run_ptr[kInlineRuns];
    uint64_t run_n[kInlineRuns];
};
constexpr uint32_t kWholeRuns = 2 * kInlineJobs;
static_assert(kWholeRuns <= kInlineRuns, "the runs of a table of pairs");
static_assert(sizeof(BatchInline) <= 2560, "fits the argument segment of a launch beside the rest");

template <int kPerLane, bool kMany, bool kInline>
__global__ void __launch_bounds__(kWave) partition_batch_kernel(Workspace ws, ModeArgs ma, int group_log, uint32_t n_jobs, BatchInline table) {
    __shared__ WindowShared<kPerLane> s;
    const JobDesc* const jobs = kInline ? table.jobs : ma.jobs;
    uint32_t job = 0;
    if (kInline) {
        for (uint32_t q = 1; q < n_jobs; q++) job = jobs[q].first_wave <= blockIdx.x ? q : job;
    } else {
        for (uint32_t left = n_jobs - 1; left > 0;) {  // last job whose first wave is not beyond this one
            const uint32_t half = (left + 1) / 2, at = job + half;
            if (jobs[at].first_wave <= blockIdx.x) job = at, left -= half;
            else left = half - 1;
        }
    }
    const JobDesc d = jobs[job];
    const lsm_entry_t* const* run_ptr = kInline ? table.run_ptr : ma.run_ptr;
    const uint64_t* run_n = kInline ? table.run_n : ma.run_n;
    const uint32_t lane = threadIdx.x, w = blockIdx.x - d.first_wave, waves = d.waves;
    if (kInline && w == 0) {
        if (lane == 0) const_cast<JobDesc*>(ma.jobs)[job] = d;
        if (lane < d.k) const_cast<const lsm_entry_t**>(ma.run_ptr)[d.run_off + lane] = run_ptr[d.run_off + lane];
        if (lane < d.k) const_cast<uint64_t*>(ma.run_n)[d.run_off + lane] = run_n[d.run_off + lane];
    }
    for (uint64_t c = w * (uint64_t)kWave + lane; c < (d.clear_n & ~kHashesBehind); c += (uint64_t)waves * kWave) d.clear[c] = make_uint4(0, 0, 0, 0);
    if (ws.fresh != nullptr && blockIdx.x == 0)
        for (uint32_t t = lane; t < kShortTiles; t += kWave) ws.fresh[t] = 0;
    for (uint32_t t = w * kWave + lane; t < d.n_tiles; t += waves * kWave) {
        const_cast<uint32_t*>(ma.tile_job)[d.first_tile + t] = job;
        ws.status[d.first_tile + t] = 0;
    }
    uint64_t* const rows = ws.splits + d.splits_off;
    if (w == 0 && lane < d.k) {
        rows[lane] = 0;
        rows[(uint64_t)d.n_tiles * d.k + lane] = run_n[d.run_off + lane];
    }
    if (d.stride != 0) {
        const int log = 32 - __builtin_clz(d.k - 1);
        const uint32_t member = lane >> (6 - log);
        const bool mine = member < d.k;
        const uint32_t len = mine ? (uint32_t)run_n[d.run_off + member] : 0;
        ranked_row(mine ? run_ptr[d.run_off + member] : nullptr, len, len, w, d.k, log, d.stride, d.per_tile, rows);
        return;
    }
    if (w == 0) return;  // the boundary of tile w
    if (d.k == 2) {
        uint64_t ia, ib;
        split_two_wave(run_ptr[d.run_off], run_n[d.run_off], run_ptr[d.run_off + 1], run_n[d.run_off + 1], w * (uint64_t)tile_spacing(ws.spacing, 2), ia, ib);
        if (lane < 2) rows[w * 2 + lane] = lane == 0 ? ia : ib;
        return;
    }
    const uint32_t j = lane & ((1u << group_log) - 1);
    const bool own = j < d.k;
    const uint32_t best = window_split<kPerLane, kMany>(s, own ? run_ptr[d.run_off + j] : nullptr, 0, own ? (uint32_t)run_n[d.run_off + j] : 0,
                                                        w * tile_spacing(ws.spacing, d.k), group_log);
    if (lane < d.k) rows[w * d.k + lane] = best;
}

// ---------------------------------------------------------------------------------------
// Optional input check (LSM_VALIDATE): every run strictly ascending, type bytes valid.
// ---------------------------------------------------------------------------------------
__global__ void validate_kernel(RunTable rt, Workspace ws) {
    const uint32_t j = blockIdx.y;
    const lsm_entry_t* run = rt.ptr[j];
    const uint64_t n = rt.n[j];
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    uint32_t bad = 0;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        if (run[i].type > LSM_TOMBSTONE) bad |= 2;
        if (i + 1 < n && !key_less(load_key(run + i), load_key(run + i + 1))) bad |= 1;
    }
    if (bad) atomicOr(&ws.hdr->validate_status, bad);
}

// Spacing of one compaction: an input that fits a tile stays one (a single launch).
static uint32_t single_spacing(uint64_t total, uint32_t k) {
    return total <= tile_nominal(k) ? (uint32_t)tile_nominal(k) : tile_spacing(fill_spacing(total), k);
}
static uint64_t tiles_for(uint64_t total, uint32_t spacing) { return (total + spacing - 1) / spacing; }
// How a compaction is cut into tiles: at merged ranks `spacing` apart, or (stride != 0) at ranked samples.
struct Cut {
    uint32_t spacing = 0;
    uint64_t tiles = 0;
    uint32_t stride = 0, per_tile = 0, samples = 0;
};
// `all`: entries of everything in the same launch, this compaction's among them.
static Cut cut_runs(const uint64_t* run_lens, uint32_t k, uint32_t spacing, uint64_t all) {
    uint64_t total = 0;
    for (uint32_t j = 0; j < k; j++) total += run_lens[j];
    Cut exact;
    exact.spacing = spacing;
    exact.tiles = tiles_for(total, spacing);
    const uint64_t few = (all + kShortTiles - 1) / kShortTiles;
    const uint64_t even = few <= kShortMean ? few : (all + kRankedTiles - 1) / kRankedTiles;
    const uint64_t mean = even < kMinSpacing ? kMinSpacing : even;
    if (k < 3 || exact.tiles < 2 || mean >= (uint64_t)kTileCap) return exact;
    const uint64_t most_tiles = tiles_for(total, (uint32_t)mean);
    // the densest samples that the tile capacity asks for, and four to a tile for even sizes; where the samples are few enough, so
    // dense that no tile has more than an entry for each thread of the short form
    for (const uint32_t cap : {(uint32_t)kShortThreads, (uint32_t)kTileCap}) {
        if (mean + (k - 1) * kMinStride > cap) continue;
        const uint64_t most_samples = (cap == (uint32_t)kTileCap ? kMostSamples : kShortSamples) * total / all;
        Cut cut = exact;
        cut.stride = (uint32_t)(cap - mean) / (k - 1);
        if (cut.stride > mean / 4) cut.stride = (uint32_t)mean / 4;
        for (; cut.stride >= kMinStride; cut.stride -= (cut.stride + 15) / 16) {
            uint64_t samples = 0;
            for (uint32_t j = 0; j < k; j++) samples += (run_lens[j] + cut.stride - 1) / cut.stride;
            if (samples > most_samples + k) break;
            cut.samples = (uint32_t)samples;
            cut.per_tile = (uint32_t)((samples + most_tiles - 1) / most_tiles);
            cut.tiles = (samples + cut.per_tile - 1) / cut.per_tile;
            if ((cut.per_tile + k - 1) * cut.stride <= cap) return cut;
        }
    }
    return exact;
}

// Lays the workspace out; with base == nullptr it only measures.  Returns the bytes used.
static size_t carve(void* base, const uint64_t* run_lens, uint32_t k, Workspace* ws) {
    uint64_t total = 0;
    for (uint32_t j = 0; j < k; j++) total += run_lens[j];
    const Cut cut = cut_runs(run_lens, k, single_spacing(total, k), total);
    const uint64_t n_tiles = tiles_for(total, cut.spacing);
    char* p = static_cast<char*>(base);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char* at = p ? p + off : nullptr;
        off += align256(bytes);
        return at;
    };
    Workspace w;
    w.hdr = reinterpret_cast<Header*>(take(sizeof(Header)));
    w.status = reinterpret_cast<uint64_t*>(take(n_tiles * sizeof(uint64_t)));
    w.splits = reinterpret_cast<uint64_t*>(take((n_tiles + 1) * (uint64_t)k * sizeof(uint64_t)));
    w.ywin = reinterpret_cast<uint64_t*>(take(2 * (n_tiles ? n_tiles - 1 : 0) * (uint64_t)k * sizeof(uint64_t)));
    for (uint32_t j = 0; j < LSM_MAX_RUNS; j++) {
        w.st.m[j] = j < k ? (run_lens[j] + kSampleStride - 1) / kSampleStride : 0;
        w.st.ptr[j] = j < k ? reinterpret_cast<SampleKey*>(take(w.st.m[j] * sizeof(SampleKey))) : nullptr;
    }
    w.n_tiles = n_tiles;
    if (cut.stride != 0) {  // may be more tiles, but without the samples' copies: a fraction of the space above
        const size_t all = off;
        off = 0;
        w.hdr = reinterpret_cast<Header*>(take(sizeof(Header)));
        w.status = reinterpret_cast<uint64_t*>(take(cut.tiles * sizeof(uint64_t)));
        w.splits = reinterpret_cast<uint64_t*>(take((cut.tiles + 1) * (uint64_t)k * sizeof(uint64_t)));
        w.n_tiles = cut.tiles;
        if (off < all) off = all;
    }
    w.clear = nullptr;
    w.clear_n = 0;
    w.fresh = nullptr;
    w.spacing = cut.spacing;
    w.stride = cut.stride;
    w.per_tile = cut.per_tile;
    w.samples = cut.samples;
    if (ws) *ws = w;
    return off;
}

}  // namespace lsm

extern "C" size_t lsm_compact_workspace_bytes(const uint64_t* run_lens, uint32_t n_runs) {
    if (run_lens == nullptr || n_runs == 0 || n_runs > LSM_MAX_RUNS) return 0;
    return lsm::carve(nullptr, run_lens, n_runs, nullptr);
}

extern "C" int lsm_compact(const lsm_run_t* runs, uint32_t n_runs, uint32_t flags, const lsm_out_t* out, void* workspace,
                           size_t workspace_bytes, void* stream) {
    return lsm_compact_timed(runs, n_runs, flags, out, workspace, workspace_bytes, stream, nullptr);
}

extern "C" int lsm_compact_timed(const lsm_run_t* runs, uint32_t n_runs, uint32_t flags, const lsm_out_t* out, void* workspace,
                                 size_t workspace_bytes, void* stream_v, const lsm_compact_events_t* ev) {
    return lsm_compact_remap(runs, n_runs, flags, out, workspace, workspace_bytes, stream_v, nullptr, ev);
}

namespace lsm {

// Enqueues the kernels of one compaction.  rt.n are the run lengths the launch sizes are taken from.
static int launch_compaction(const RunTable& rt, uint32_t flags, const lsm_out_t* out, void* workspace, hipStream_t stream,
                             const uint64_t* remap_base, uint32_t remap_files, const lsm_compact_events_t* ev, const ClearSpan& clear = ClearSpan(),
                             bool* cleared = nullptr) {
    const uint32_t n_runs = rt.k;
    uint64_t total = 0;
    for (uint32_t j = 0; j < n_runs; j++) total += rt.n[j];
    if (tiles_for(total, single_spacing(total, n_runs)) >= (1ull << 31)) return LSM_ERR_BAD_ARG;
    Workspace ws;
    carve(workspace, rt.n, n_runs, &ws);
    const uint64_t n_tiles = ws.n_tiles;

    // how the boundaries are found: see kSampledMinTiles
    bool rows = n_runs > 2 && ws.stride == 0 && rt.n_dev == nullptr && total < kRowsMost &&
                (n_runs <= kRowsRuns ? n_tiles >= (n_runs <= 4 ? kSampledMinTiles : 2) : n_runs <= kFewRuns && n_tiles < kSampledMinTiles);
    const uint32_t row_step = row_entries(total, n_runs);
    uint32_t n_rows = 0, row_blocks = 0;
    for (uint32_t j = 0; rows && j < n_runs; j++) {
        const uint32_t samples = samples_apart((uint32_t)rt.n[j], row_offset(j, n_runs, row_step), row_step);
        n_rows += samples;
        row_blocks += (samples + kDies - 1) / kDies * kDies;  // an eighth may be one longer than another
    }
    const char* const rows_end = reinterpret_cast<const char*>(ws.st.ptr[n_runs - 1] + ws.st.m[n_runs - 1]);  // of the room that they share with what copied samples need
    rows = rows && n_rows != 0 && n_rows <= (uint64_t)(rows_end - reinterpret_cast<const char*>(ws.ywin)) / ((n_runs + 1) * sizeof(uint64_t));
    // everything but copied samples: where the input is not validated, the first launch of the partition does the clearing as well
    const bool direct = n_tiles > 1 && (n_tiles < kSampledMinTiles || n_runs <= kRowsRuns);
    const bool fused_init = (direct || n_tiles == 1) && !(flags & LSM_VALIDATE);  // one tile needs neither status word nor split rows
    auto build_filter = [&](const ClearSpan& span) {  // right behind the merge, if it is asked for
        if (ws.clear_n == 0 || span.filter_bits == 0) return (int)LSM_OK;
        const bool hashed = span.filter != nullptr;
        const CountedFilter filter = {out->entries, total, ws.status + n_tiles - 1, hashed ? span.filter : span.p, span.filter_bits, hashed ? span.p : nullptr};
        if (build_filters_counted(&filter, 1, stream) != LSM_OK) return (int)LSM_ERR_HIP;
        span.filter_built = true;
        return (int)LSM_OK;
    };
    if (clear.bytes != 0 && direct && fused_init) {
        ws.clear = static_cast<uint4*>(clear.p);
        ws.clear_n = clear.bytes / 16;
        *cleared = true;
    }
    const uint32_t fence_stride = out->fence_keys ? out->fence_stride : 1u;
    if (clear.status != nullptr && clear.epoch == 0 && direct && fused_init) {
        ws.fresh = clear.status;
        clear.status_zeroed = true;
    }
    if (clear.status != nullptr && clear.epoch != 0 && n_runs <= 2 && n_tiles > 1 && n_tiles <= kShortTiles && fused_init && remap_files == 0 && !ev && !rt.n_dev) {
        WholeTable<1, 2> table = {};
        table.jobs[0] = JobDesc{0, 0, 0, 0, 0, 0, out->entries, out->n_out, reinterpret_cast<uint4*>(out->fence_keys), (uint32_t)n_tiles, n_runs, flags,
                                fence_stride, ws.clear, (uint32_t)ws.clear_n, 0};
        if (clear.filter != nullptr) table.jobs[0].clear_n |= kHashesBehind;
        for (uint32_t j = 0; j < n_runs; j++) table.run_ptr[j] = rt.ptr[j], table.run_n[j] = rt.n[j];
        table.status = ws.status = clear.status;
        table.epoch = (uint64_t)clear.epoch << kStEpochShift;
        table.n_jobs = 1;
        table.spacing = ws.spacing;
        const dim3 grid((uint32_t)n_tiles), threads(kShortThreads);
        if (clear.filter != nullptr) hipLaunchKernelGGL((merge_whole_kernel<2, 1, 2>), grid, threads, 0, stream, table);
        else hipLaunchKernelGGL((merge_whole_kernel<1, 1, 2>), grid, threads, 0, stream, table);
        if (hipGetLastError() != hipSuccess) return LSM_ERR_HIP;
        return build_filter(clear);
    }
    if (!fused_init) {
        uint32_t init_blocks = (uint32_t)((n_tiles + 255) / 256);
        if (init_blocks == 0) init_blocks = 1;
        if (init_blocks > 1024) init_blocks = 1024;
        hipLaunchKernelGGL(init_kernel, dim3(init_blocks), dim3(256), 0, stream, rt, ws, n_tiles, out->n_out);
    }

    if (flags & LSM_VALIDATE) {
        hipLaunchKernelGGL(validate_kernel, dim3(256, n_runs), dim3(256), 0, stream, rt, ws);
        uint32_t vs = 0;
        if (hipMemcpyAsync(&vs, &ws.hdr->validate_status, sizeof(vs), hipMemcpyDeviceToHost, stream) != hipSuccess)
            return LSM_ERR_HIP;
        if (hipStreamSynchronize(stream) != hipSuccess) return LSM_ERR_HIP;
        if (vs & 1) return LSM_ERR_UNSORTED;
        if (vs & 2) return LSM_ERR_BAD_ENTRY;
    }
    if (ev && ev->before_partition && hipEventRecord(static_cast<hipEvent_t>(ev->before_partition), stream) != hipSuccess)
        return LSM_ERR_HIP;
    if (n_tiles > 1) {
        int group = 1;
        while (group < (int)n_runs) group <<= 1;
        const uint64_t per_block = (uint64_t)(256 / kWave) * (kWave / group);  // selection problems per workgroup
        auto blocks = [&](uint64_t problems) { return dim3((uint32_t)((problems + per_block - 1) / per_block)); };
        if (direct) {
            const int group_log = log2_ceil(n_runs);
            const dim3 waves((uint32_t)(n_tiles - 1));
            auto launch = [&](auto init) {
                constexpr bool kInit = decltype(init)::value;
                const dim3 lanes((uint32_t)((n_tiles - 1 + kTwoThreads - 1) / kTwoThreads));
                if (n_runs == 1)
                    hipLaunchKernelGGL(partition_one_kernel<kInit>, lanes, dim3(kTwoThreads), 0, stream, rt, ws, n_tiles);
                else if (n_runs == 2 && n_tiles <= kTwoWaves)
                    hipLaunchKernelGGL(partition_two_wave_kernel<kInit>, waves, dim3(kWave), 0, stream, rt, ws, n_tiles);
                else if (n_runs == 2)
                    hipLaunchKernelGGL(partition_two_kernel<kInit>, lanes, dim3(kTwoThreads), 0, stream, rt, ws, n_tiles);
                else if (ws.stride != 0)
                    hipLaunchKernelGGL(partition_ranked_kernel<kInit>, dim3(ws.samples), dim3(kWave), 0, stream, rt, ws, n_tiles, group_log);
                else if (rows) {
                    hipLaunchKernelGGL(partition_rows_kernel<kInit>, dim3(row_blocks), dim3(kWave), 0, stream, rt, ws, n_tiles, n_rows, row_step, group_log);
                    if (records_per_lane(group_log) == 4)
                        hipLaunchKernelGGL(partition_between_kernel<4>, waves, dim3(kWave), 0, stream, rt, ws, n_rows, row_step, group_log);
                    else
                        hipLaunchKernelGGL(partition_between_kernel<8>, waves, dim3(kWave), 0, stream, rt, ws, n_rows, row_step, group_log);
                } else if (n_runs <= kRowsRuns && n_tiles < kSampledMinTiles)
                    hipLaunchKernelGGL((partition_kernel<kInit, 4, false>), waves, dim3(kWave), 0, stream, rt, ws, n_tiles, group_log);
                else if (n_runs > kFewRuns && n_tiles * n_runs <= kWindowPieces)
                    hipLaunchKernelGGL((partition_kernel<kInit, 8, true>), waves, dim3(kWave), 0, stream, rt, ws, n_tiles, group_log);
                else
                    hipLaunchKernelGGL(partition_many_kernel<kInit>, waves, dim3(kWave), 0, stream, rt, ws, n_tiles);
            };
            if (fused_init) launch(std::true_type{});
            else launch(std::false_type{});
        } else {
            uint64_t m_max = 0, n_rows = 0;  // fewer rows than tiles: a row stands for kRowStride * kSampleStride entries
            for (uint32_t j = 0; j < n_runs; j++) {
                m_max = ws.st.m[j] > m_max ? ws.st.m[j] : m_max;
                n_rows += (ws.st.m[j] + kRowStride - 1) / kRowStride;
            }
            uint64_t sample_blocks = (2 * m_max + 255) / 256;
            if (sample_blocks > 4096) sample_blocks = 4096;
            hipLaunchKernelGGL(sample_kernel, dim3((uint32_t)sample_blocks, n_runs), dim3(256), 0, stream, rt, ws.st);
            hipLaunchKernelGGL(sample_rank_kernel, dim3((uint32_t)n_rows), dim3(kWave), 0, stream, ws, n_runs, log2_ceil(n_runs));
            hipLaunchKernelGGL(sample_fine_kernel, blocks(2 * (n_tiles - 1)), dim3(256), 0, stream, ws, n_runs, n_tiles, n_rows, group);
            hipLaunchKernelGGL(bracket_partition_kernel, blocks(n_tiles - 1), dim3(256), 0, stream, rt, ws, n_tiles, group);
        }
    }
    if (ev && ev->before_merge && hipEventRecord(static_cast<hipEvent_t>(ev->before_merge), stream) != hipSuccess)
        return LSM_ERR_HIP;
    if (n_tiles > 0) {
        uint4* const fence_out = reinterpret_cast<uint4*>(out->fence_keys);
        ModeArgs extras = {};
        extras.key_hashes = out->key_hashes != nullptr ? out->key_hashes : ws.clear_n != 0 ? clear.hashes() : nullptr;
        auto launch = [&](auto extras_value) {
            constexpr int kExtras = decltype(extras_value)::value;
            if (n_tiles <= kShortTiles)
                hipLaunchKernelGGL((merge_short_kernel<kExtras, kModeSingle>), dim3((uint32_t)n_tiles), dim3(kShortThreads), 0, stream, rt, ws, n_tiles, flags,
                                   out->entries, out->n_out, remap_base, remap_files, fence_out, fence_stride, extras);
            else
                hipLaunchKernelGGL((merge_kernel<kExtras, kModeSingle>), dim3((uint32_t)n_tiles), dim3(kMergeThreads), 0, stream, rt, ws, n_tiles, flags,
                                   out->entries, out->n_out, remap_base, remap_files, fence_out, fence_stride, extras);
        };
        if (extras.key_hashes != nullptr) launch(std::integral_constant<int, 2>{});
        else if (remap_files != 0 || fence_out != nullptr) launch(std::integral_constant<int, 1>{});
        else launch(std::integral_constant<int, 0>{});
    }
    if (ev && ev->after_merge && hipEventRecord(static_cast<hipEvent_t>(ev->after_merge), stream) != hipSuccess)
        return LSM_ERR_HIP;
    if (hipGetLastError() != hipSuccess) return LSM_ERR_HIP;
    if (build_filter(clear) != LSM_OK) return LSM_ERR_HIP;
    if (flags & LSM_VALIDATE) {
        uint64_t n = 0;
        if (hipMemcpyAsync(&n, out->n_out, sizeof(n), hipMemcpyDeviceToHost, stream) != hipSuccess) return LSM_ERR_HIP;
        if (hipStreamSynchronize(stream) != hipSuccess) return LSM_ERR_HIP;
        if (n == ~0ull) return LSM_ERR_INTERNAL;
    }
    return LSM_OK;
}

int compact_device_lengths(const lsm_entry_t* const* ptr, const uint64_t* n_upper, const uint64_t* n_dev, uint32_t k, uint32_t flags,
                           const lsm_out_t* out, void* workspace, size_t workspace_bytes, hipStream_t stream) {
    if (k == 0 || k > LSM_MAX_RUNS || (flags & LSM_VALIDATE)) return LSM_ERR_BAD_ARG;
    if (workspace == nullptr || workspace_bytes < lsm_compact_workspace_bytes(n_upper, k)) return LSM_ERR_WORKSPACE;
    RunTable rt;
    rt.k = k;
    rt.n_dev = n_dev;
    uint64_t total = 0;
    for (uint32_t j = 0; j < LSM_MAX_RUNS; j++) {
        rt.ptr[j] = j < k ? ptr[j] : nullptr;
        rt.n[j] = j < k ? n_upper[j] : 0;
        total += rt.n[j];
    }
    // with lengths that are only bounds the sampled partition would copy samples from beyond the runs' ends
    if (tiles_for(total, single_spacing(total, k)) >= kSampledMinTiles) return LSM_ERR_BAD_ARG;
    return launch_compaction(rt, flags, out, workspace, stream, nullptr, 0, nullptr);
}

}  // namespace lsm

namespace lsm {
// The checks of a compaction's arguments, and its launch.
static int checked_compaction(const lsm_run_t* runs, uint32_t n_runs, uint32_t flags, const lsm_out_t* out, void* workspace, size_t workspace_bytes,
                              hipStream_t stream, const lsm_remap_t* remap, const lsm_compact_events_t* ev, const ClearSpan& clear, bool* cleared) {
    if (remap != nullptr && remap->n_files != 0 && remap->base == nullptr) return LSM_ERR_NULL;
    const uint64_t* remap_base = remap ? remap->base : nullptr;
    const uint32_t remap_files = remap ? remap->n_files : 0;
    if (runs == nullptr || out == nullptr || out->n_out == nullptr) return LSM_ERR_NULL;
    if (n_runs == 0 || n_runs > LSM_MAX_RUNS) return LSM_ERR_BAD_ARG;
    RunTable rt;
    rt.k = n_runs;
    rt.n_dev = nullptr;
    uint64_t total = 0;
    for (uint32_t j = 0; j < LSM_MAX_RUNS; j++) {
        rt.ptr[j] = nullptr;
        rt.n[j] = 0;
    }
    for (uint32_t j = 0; j < n_runs; j++) {
        if (runs[j].n > 0 && runs[j].entries == nullptr) return LSM_ERR_NULL;
        if ((reinterpret_cast<uintptr_t>(runs[j].entries) & 63) != 0) return LSM_ERR_BAD_ARG;
        rt.ptr[j] = runs[j].entries;
        rt.n[j] = runs[j].n;
        total += runs[j].n;
    }
    if (total > 0 && out->entries == nullptr) return LSM_ERR_NULL;
    if ((reinterpret_cast<uintptr_t>(out->entries) & 63) != 0) return LSM_ERR_BAD_ARG;
    if (out->capacity < total) return LSM_ERR_CAPACITY;
    if (out->fence_keys != nullptr && (out->fence_stride == 0 || (reinterpret_cast<uintptr_t>(out->fence_keys) & 15) != 0))
        return LSM_ERR_BAD_ARG;
    if ((reinterpret_cast<uintptr_t>(out->key_hashes) & 7) != 0) return LSM_ERR_BAD_ARG;
    if (workspace == nullptr || (reinterpret_cast<uintptr_t>(workspace) & 255) != 0 ||
        workspace_bytes < lsm_compact_workspace_bytes(rt.n, n_runs))
        return LSM_ERR_WORKSPACE;
    return launch_compaction(rt, flags, out, workspace, stream, remap_base, remap_files, ev, clear, cleared);
}

int compact_clearing(const lsm_run_t* runs, uint32_t n_runs, uint32_t flags, const lsm_out_t* out, void* workspace, size_t workspace_bytes,
                     const ClearSpan& clear, bool* cleared, hipStream_t stream) {
    *cleared = false;
    return checked_compaction(runs, n_runs, flags, out, workspace, workspace_bytes, stream, nullptr, nullptr, clear, cleared);
}
}  // namespace lsm

extern "C" int lsm_compact_remap(const lsm_run_t* runs, uint32_t n_runs, uint32_t flags, const lsm_out_t* out, void* workspace,
                                 size_t workspace_bytes, void* stream, const lsm_remap_t* remap, const lsm_compact_events_t* ev) {
    return lsm::checked_compaction(runs, n_runs, flags, out, workspace, workspace_bytes, static_cast<hipStream_t>(stream), remap, ev, lsm::ClearSpan(),
                                   nullptr);
}

// ---------------------------------------------------------------------------------------
// lsm_range_scan: the live content of many key ranges of a tree, one tile per range.
// ---------------------------------------------------------------------------------------
extern "C" int lsm_range_scan(const lsm_ranges_t* ranges, const lsm_tree_t* tree, const lsm_range_out_t* out, void* stream_v) {
    using namespace lsm;
    if (ranges == nullptr || tree == nullptr || out == nullptr) return LSM_ERR_NULL;
    if (ranges->max_entries == 0 || ranges->max_entries > LSM_RANGE_MAX_ENTRIES || tree->n_runs > LSM_MAX_RUNS) return LSM_ERR_BAD_ARG;
    if (ranges->n_ranges == 0) return LSM_OK;
    if (ranges->lo_keys == nullptr || ranges->hi_keys == nullptr || out->entries == nullptr || out->counts == nullptr) return LSM_ERR_NULL;
    if (((reinterpret_cast<uintptr_t>(ranges->lo_keys) | reinterpret_cast<uintptr_t>(ranges->hi_keys)) & 15) != 0 ||
        (reinterpret_cast<uintptr_t>(out->entries) & 63) != 0)
        return LSM_ERR_BAD_ARG;
    if (tree->n_runs > 0 && tree->runs == nullptr) return LSM_ERR_NULL;
    RunTable rt;
    rt.k = tree->n_runs ? tree->n_runs : 1;  // a tree without runs: one empty run
    rt.n_dev = nullptr;
    for (uint32_t j = 0; j < LSM_MAX_RUNS; j++) {
        rt.ptr[j] = nullptr;
        rt.n[j] = 0;
    }
    for (uint32_t j = 0; j < tree->n_runs; j++) {
        const lsm_run_t& r = tree->runs[j].run;
        if (r.n > 0 && r.entries == nullptr) return LSM_ERR_NULL;
        if ((reinterpret_cast<uintptr_t>(r.entries) & 63) != 0) return LSM_ERR_BAD_ARG;
        rt.ptr[j] = r.entries;
        rt.n[j] = r.n;
    }
    ModeArgs ma = {};
    ma.lo_keys = ranges->lo_keys;
    ma.hi_keys = ranges->hi_keys;
    ma.counts = out->counts;
    ma.max_entries = ranges->max_entries;
    Workspace ws = {};
    hipLaunchKernelGGL((merge_kernel<0, kModeRange>), dim3(ranges->n_ranges), dim3(kMergeThreads), 0, static_cast<hipStream_t>(stream_v), rt, ws,
                       (uint64_t)ranges->n_ranges, (uint32_t)LSM_BOTTOMMOST, out->entries, (uint64_t*)nullptr, (const uint64_t*)nullptr, 0u,
                       (uint4*)nullptr, 1u, ma);
    return hipGetLastError() == hipSuccess ? LSM_OK : LSM_ERR_HIP;
}

// ---------------------------------------------------------------------------------------
// lsm_compact_batch: many independent small compactions in two launches.
// Workspace: tile status words | split tables of all jobs | the table the host builds (job of every tile, job
// descriptors, run pointers, run lengths).
// ---------------------------------------------------------------------------------------
namespace lsm {
struct BatchLayout {
    uint64_t tiles, split_words, runs;
    size_t status, splits, tile_job, jobs, run_ptr, run_n, total;
    uint64_t all;  // entries
    uint32_t k_max, spacing;
};
// Pinned host memory for the job table of one thread, with an event that tells when the last copy out of it is done.
struct BatchStaging {
    unsigned char* mem = nullptr;
    size_t capacity = 0;
    hipEvent_t copied = nullptr;
    bool pending = false;

    unsigned char* acquire(size_t bytes) {
        if (pending && hipEventSynchronize(copied) != hipSuccess) return nullptr;
        pending = false;
        if (copied == nullptr && hipEventCreateWithFlags(&copied, hipEventDisableTiming) != hipSuccess) return nullptr;
        if (bytes > capacity) {
            if (mem != nullptr) (void)hipHostFree(mem);
            mem = nullptr;
            capacity = 0;
            const size_t want = bytes < (1u << 16) ? (1u << 16) : bytes + bytes / 2;
            void* p = nullptr;
            if (hipHostMalloc(&p, want, hipHostMallocDefault) != hipSuccess) return nullptr;
            mem = static_cast<unsigned char*>(p);
            capacity = want;
        }
        return mem;
    }
    bool copy_enqueued(hipStream_t stream) {
        if (hipEventRecord(copied, stream) != hipSuccess) return false;
        pending = true;
        return true;
    }
    // no destructor: at thread or process exit the HIP runtime may already be gone; the memory goes with the process
};

static int batch_layout(const lsm_compact_job_t* jobs, uint32_t n_jobs, BatchLayout* l) {
    l->tiles = l->split_words = l->runs = 0;
    l->k_max = 1;
    l->all = 0;
    for (uint32_t j = 0; j < n_jobs; j++) {
        if (jobs[j].runs == nullptr || jobs[j].n_runs > LSM_MAX_RUNS) continue;  // refused below
        for (uint32_t r = 0; r < jobs[j].n_runs; r++) l->all += jobs[j].runs[r].n;
    }
    l->spacing = fill_spacing(l->all, n_jobs);
    for (uint32_t j = 0; j < n_jobs; j++) {
        const lsm_compact_job_t& job = jobs[j];
        if (job.runs == nullptr) return LSM_ERR_NULL;
        if (job.n_runs == 0 || job.n_runs > LSM_MAX_RUNS || (job.flags & LSM_VALIDATE)) return LSM_ERR_BAD_ARG;
        if (job.out.fence_keys != nullptr && (job.out.fence_stride == 0 || (reinterpret_cast<uintptr_t>(job.out.fence_keys) & 15) != 0))
            return LSM_ERR_BAD_ARG;
        if (job.out.key_hashes != nullptr) return LSM_ERR_BAD_ARG;  // filters of a batch: lsm_build_bloom_batch
        uint64_t total = 0, lens[LSM_MAX_RUNS];
        for (uint32_t r = 0; r < job.n_runs; r++) total += lens[r] = job.runs[r].n;
        const uint32_t spacing = tile_spacing(l->spacing, job.n_runs);
        if (tiles_for(total, spacing) >= kSampledMinTiles) return LSM_ERR_BAD_ARG;  // a large compaction: lsm_compact
        uint64_t nt = cut_runs(lens, job.n_runs, spacing, l->all).tiles;
        if (nt == 0) nt = 1;  // an empty job keeps one (empty) tile, which writes its count
        l->tiles += nt;
        l->split_words += (nt + 1) * job.n_runs;
        l->runs += job.n_runs;
        if (job.n_runs > l->k_max) l->k_max = job.n_runs;
    }
    if (l->tiles >= (1ull << 31)) return LSM_ERR_BAD_ARG;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += align256(bytes);
        return at;
    };
    l->status = take(l->tiles * sizeof(uint64_t));
    l->splits = take(l->split_words * sizeof(uint64_t));
    l->tile_job = take(l->tiles * sizeof(uint32_t));
    l->jobs = take((size_t)n_jobs * sizeof(JobDesc));  // from here on: written by the host, one copy
    l->run_ptr = take(l->runs * sizeof(void*));
    l->run_n = take(l->runs * sizeof(uint64_t));
    l->total = off;
    return LSM_OK;
}
}  // namespace lsm

extern "C" size_t lsm_compact_batch_workspace_bytes(const lsm_compact_job_t* jobs, uint32_t n_jobs) {
    lsm::BatchLayout l;
    if (jobs == nullptr || n_jobs == 0 || lsm::batch_layout(jobs, n_jobs, &l) != LSM_OK) return 0;
    return l.total;
}

namespace lsm {
int compact_batch_clearing(const lsm_compact_job_t* jobs, uint32_t n_jobs, void* workspace, size_t workspace_bytes, const ClearSpan* clear, hipStream_t stream) {
    BatchLayout l;
    const int rc = batch_layout(jobs, n_jobs, &l);
    if (rc != LSM_OK) return rc;
    for (uint32_t j = 0; j < n_jobs; j++) {
        const lsm_compact_job_t& job = jobs[j];
        uint64_t total = 0;
        for (uint32_t r = 0; r < job.n_runs; r++) {
            if (job.runs[r].n > 0 && job.runs[r].entries == nullptr) return LSM_ERR_NULL;
            if ((reinterpret_cast<uintptr_t>(job.runs[r].entries) & 63) != 0) return LSM_ERR_BAD_ARG;
            total += job.runs[r].n;
        }
        if (job.out.n_out == nullptr || (total > 0 && job.out.entries == nullptr)) return LSM_ERR_NULL;
        if ((reinterpret_cast<uintptr_t>(job.out.entries) & 63) != 0) return LSM_ERR_BAD_ARG;
        if (job.out.capacity < total) return LSM_ERR_CAPACITY;
    }
    if (workspace == nullptr || (reinterpret_cast<uintptr_t>(workspace) & 255) != 0 || workspace_bytes < l.total) return LSM_ERR_WORKSPACE;
    const bool fits_inline = n_jobs <= kInlineJobs && l.runs <= kInlineRuns;
    BatchInline table = {};
    JobDesc* desc = table.jobs;
    const lsm_entry_t** run_ptr = table.run_ptr;
    uint64_t* run_n = table.run_n;
    // a larger table is built in pinned host memory kept per thread (so the copy below really is asynchronous) and
    // is not written again before the copy of the previous call from this thread has finished
    static thread_local BatchStaging staging;
    const size_t table_bytes = l.total - l.jobs;
    unsigned char* copied = nullptr;
    if (!fits_inline) {
        copied = staging.acquire(table_bytes);
        if (copied == nullptr) return LSM_ERR_HIP;
        memset(copied, 0, table_bytes);
        desc = reinterpret_cast<JobDesc*>(copied);
        run_ptr = reinterpret_cast<const lsm_entry_t**>(copied + (l.run_ptr - l.jobs));
        run_n = reinterpret_cast<uint64_t*>(copied + (l.run_n - l.jobs));
    }
    uint64_t tile = 0, wave = 0, split_word = 0, run = 0;
    bool any_fences = false, any_hashes = false;
    for (uint32_t j = 0; j < n_jobs; j++) {
        const lsm_compact_job_t& job = jobs[j];
        for (uint32_t r = 0; r < job.n_runs; r++) {
            run_ptr[run + r] = job.runs[r].entries;
            run_n[run + r] = job.runs[r].n;
        }
        const Cut cut = cut_runs(run_n + run, job.n_runs, tile_spacing(l.spacing, job.n_runs), l.all);
        const uint64_t nt = cut.tiles ? cut.tiles : 1;
        JobDesc& d = desc[j];
        d.first_tile = (uint32_t)tile;
        d.first_wave = (uint32_t)wave;
        d.waves = cut.stride != 0 ? cut.samples : (uint32_t)nt;
        d.stride = (uint16_t)cut.stride;
        d.per_tile = (uint16_t)cut.per_tile;
        d.run_off = (uint32_t)run;
        d.splits_off = split_word;
        d.out = job.out.entries;
        d.n_out = job.out.n_out;
        d.fence_out = reinterpret_cast<uint4*>(job.out.fence_keys);
        d.fence_stride = job.out.fence_keys ? job.out.fence_stride : 1u;
        any_fences = any_fences || job.out.fence_keys != nullptr;
        d.n_tiles = (uint32_t)nt;
        d.k = job.n_runs;
        d.flags = job.flags;
        d.clear = clear ? static_cast<uint4*>(clear[j].p) : nullptr;
        d.clear_n = clear ? (uint32_t)(clear[j].bytes / 16) : 0;
        if (clear && clear[j].filter != nullptr) d.clear_n |= kHashesBehind, any_hashes = true;
        tile += nt;
        wave += d.waves;
        split_word += (nt + 1) * job.n_runs;
        run += job.n_runs;
    }
    char* base = static_cast<char*>(workspace);
    if (!fits_inline) {
        if (hipMemcpyAsync(base + l.jobs, copied, table_bytes, hipMemcpyHostToDevice, stream) != hipSuccess) return LSM_ERR_HIP;
        if (!staging.copy_enqueued(stream)) return LSM_ERR_HIP;
    }
    Workspace ws = {};
    ws.status = reinterpret_cast<uint64_t*>(base + l.status);
    ws.splits = reinterpret_cast<uint64_t*>(base + l.splits);
    ws.spacing = l.spacing;
    ModeArgs ma = {};
    ma.tile_job = reinterpret_cast<const uint32_t*>(base + l.tile_job);
    ma.jobs = reinterpret_cast<const JobDesc*>(base + l.jobs);
    ma.run_ptr = reinterpret_cast<const lsm_entry_t* const*>(base + l.run_ptr);
    ma.run_n = reinterpret_cast<const uint64_t*>(base + l.run_n);
    if (clear != nullptr && clear[0].status != nullptr && clear[0].epoch == 0) {
        ws.fresh = clear[0].status;
        clear[0].status_zeroed = true;
    }
    const bool whole = clear != nullptr && clear[0].status != nullptr && clear[0].epoch != 0 && fits_inline && l.k_max <= 2 && tile <= kShortTiles;
    const int group_log = log2_ceil(l.k_max);
    const dim3 waves((uint32_t)wave), threads(kWave);
    auto launch = [&](auto inline_table) {
        constexpr bool kInline = decltype(inline_table)::value;
        if (records_per_lane(group_log) == 4) hipLaunchKernelGGL((partition_batch_kernel<4, false, kInline>), waves, threads, 0, stream, ws, ma, group_log, n_jobs, table);
        else if (l.k_max <= kFewRuns) hipLaunchKernelGGL((partition_batch_kernel<8, false, kInline>), waves, threads, 0, stream, ws, ma, group_log, n_jobs, table);
        else hipLaunchKernelGGL((partition_batch_kernel<8, true, kInline>), waves, threads, 0, stream, ws, ma, group_log, n_jobs, table);
    };
    if (whole) {
        WholeTable<kInlineJobs, kWholeRuns> one = {};
        memcpy(one.jobs, table.jobs, sizeof(one.jobs));
        memcpy(one.run_ptr, table.run_ptr, sizeof(one.run_ptr));
        memcpy(one.run_n, table.run_n, sizeof(one.run_n));
        one.status = ws.status = clear[0].status;
        one.epoch = (uint64_t)clear[0].epoch << kStEpochShift;
        one.n_jobs = n_jobs;
        one.spacing = l.spacing;
        if (any_hashes) hipLaunchKernelGGL((merge_whole_kernel<2, kInlineJobs, kWholeRuns>), dim3((uint32_t)tile), dim3(kShortThreads), 0, stream, one);
        else hipLaunchKernelGGL((merge_whole_kernel<1, kInlineJobs, kWholeRuns>), dim3((uint32_t)tile), dim3(kShortThreads), 0, stream, one);
    } else if (fits_inline) {
        launch(std::true_type{});
    } else {
        launch(std::false_type{});
    }
    RunTable rt = {};
    rt.k = 1;
    auto launch_merge = [&](auto extras_value) {
        constexpr int kExtras = decltype(extras_value)::value;
        if (tile <= kShortTiles)
            hipLaunchKernelGGL((merge_short_kernel<kExtras, kModeBatch>), dim3((uint32_t)tile), dim3(kShortThreads), 0, stream, rt, ws, tile, 0u,
                               (lsm_entry_t*)nullptr, (uint64_t*)nullptr, (const uint64_t*)nullptr, 0u, (uint4*)nullptr, 1u, ma);
        else
            hipLaunchKernelGGL((merge_kernel<kExtras, kModeBatch>), dim3((uint32_t)tile), dim3(kMergeThreads), 0, stream, rt, ws, tile, 0u,
                               (lsm_entry_t*)nullptr, (uint64_t*)nullptr, (const uint64_t*)nullptr, 0u, (uint4*)nullptr, 1u, ma);
    };
    // any_fences: the form that also writes fence indices (a job without one has a null pointer in its descriptor)
    if (!whole && any_hashes) launch_merge(std::integral_constant<int, 2>{});
    else if (!whole && any_fences) launch_merge(std::integral_constant<int, 1>{});
    else if (!whole) launch_merge(std::integral_constant<int, 0>{});
    if (hipGetLastError() != hipSuccess) return LSM_ERR_HIP;
    for (uint32_t j = 0; clear != nullptr && j < n_jobs;) {
        CountedFilter filters[kInlineJobs];
        const uint32_t first = j;
        uint32_t count = 0;
        for (; j < n_jobs && count < kInlineJobs; j++) {
            const JobDesc& d = desc[j];
            if (d.clear_n == 0 || clear[j].filter_bits == 0) continue;
            const bool hashed = clear[j].filter != nullptr;
            uint64_t total = 0;
            for (uint32_t r = 0; r < d.k; r++) total += run_n[d.run_off + r];
            filters[count++] = CountedFilter{d.out, total, ws.status + d.first_tile + d.n_tiles - 1, hashed ? clear[j].filter : clear[j].p, clear[j].filter_bits, hashed ? clear[j].p : nullptr};
        }
        if (count != 0 && build_filters_counted(filters, count, stream) != LSM_OK) return LSM_ERR_HIP;
        for (uint32_t q = first; q < j; q++) clear[q].filter_built = desc[q].clear_n != 0 && clear[q].filter_bits != 0;
    }
    return LSM_OK;
}
}  // namespace lsm

extern "C" int lsm_compact_batch(const lsm_compact_job_t* jobs, uint32_t n_jobs, void* workspace, size_t workspace_bytes, void* stream) {
    if (n_jobs == 0) return LSM_OK;
    if (jobs == nullptr) return LSM_ERR_NULL;
    return lsm::compact_batch_clearing(jobs, n_jobs, workspace, workspace_bytes, nullptr, static_cast<hipStream_t>(stream));
}

// ---------------------------------------------------------------------------------------
// lsm_compact_static: the same compaction for callers that cannot allocate device memory.  The workspace is a
// file-scope device array; each GPU holds its own copy at its own address, looked up once per device.
// ---------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[LSM_STATIC_SCRATCH_BYTES];

namespace lsm {
constexpr int kMaxDevices = 64;
static std::mutex g_scratch_lock;
static void* g_scratch_ptr[kMaxDevices];  // device address of `scratch` on device d, once known

// Device address of this GPU's copy of `scratch` (the array's name itself is only a host-side handle).
static int scratch_address(void** ptr) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return LSM_ERR_HIP;
    std::lock_guard<std::mutex> hold(g_scratch_lock);
    if (g_scratch_ptr[dev] == nullptr) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return LSM_ERR_HIP;
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return LSM_OK;
}
}  // namespace lsm

extern "C" int lsm_compact_static(const lsm_run_t* runs, uint32_t n_runs, uint32_t flags, const lsm_out_t* out, void* stream) {
    if (runs == nullptr) return LSM_ERR_NULL;
    if (n_runs == 0 || n_runs > LSM_MAX_RUNS) return LSM_ERR_BAD_ARG;
    if (flags & LSM_VALIDATE) return LSM_ERR_BAD_ARG;  // validation copies a status word to the host and waits
    uint64_t lens[LSM_MAX_RUNS];
    for (uint32_t j = 0; j < n_runs; j++) lens[j] = runs[j].n;
    if (lsm_compact_workspace_bytes(lens, n_runs) > (size_t)LSM_STATIC_SCRATCH_BYTES) return LSM_ERR_STATIC_LIMIT;
    void* ws = nullptr;
    const int rc = lsm::scratch_address(&ws);
    if (rc != LSM_OK) return rc;
    // every word of the scratch that a call reads is written by that call's own kernels first (the tile status words are
    // cleared before the merge), so what the previous call left behind does not matter
    return lsm_compact_remap(runs, n_runs, flags, out, ws, LSM_STATIC_SCRATCH_BYTES, stream, nullptr, nullptr);
}
