// lsm_flush_buffer: the write buffer as a sorted run (paper section 2.2: the in-memory buffer is flushed as a
// sorted run).  Total order of the buffer's entries: key ascending, then newest first (larger seqno; equal seqnos: the
// one written later); an entry survives unless its predecessor in that order has the same key.
//
// Up to kFlushDirect entries: by counting, in two launches without a clearing pass or global atomics (one launch up to
// kSmallEntries, flush_small_kernel).
//   flush_rank_kernel   the number of entries that precede entry i in the total order (its rank), and whether i is
//                       shadowed, by comparing it with every other entry;
//   flush_place_kernel  an entry that is not shadowed goes to position rank - |{shadowed j : rank_j < rank_i}|, from a
//                       bitmap of the shadowed ranks that every workgroup makes for itself in LDS.
// A larger buffer is cut into segments of 2,048 or 4,096 entries in write order, every segment is sorted by one workgroup
// (flush_sort_kernel), and the sorted segments are merged by the compaction kernels (the segment written last is the
// newest run, so that among equal sequence numbers the later write wins there as well).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "lsm_common.h"

namespace lsm {

__device__ __forceinline__ int key_cmp(const Key& a, const Key& b) {
    for (int w = 0; w < 4; w++)
        if (a.w[w] != b.w[w]) return a.w[w] < b.w[w] ? -1 : 1;
    return 0;
}

constexpr uint32_t kShadowed = 0x80000000u;  // flag in a packed rank

// The first 16 key bytes as a 128-bit number, lowest word first.
__device__ __forceinline__ uint4 key_head(const uint4 q) {
    return make_uint4(__builtin_bswap32(q.w), __builtin_bswap32(q.z), __builtin_bswap32(q.y), __builtin_bswap32(q.x));
}
// Adds to rank how many of the four numbers o[] are below `head`, all as 128-bit numbers; diff[i] is zero only if o[i] is equal to
// it.  One subtraction with borrow each, where the compiler makes three 64-bit compares and two selects of the same (64-bit
// compares take twice the time of these).  The four chains are interleaved: a vector instruction may read a carry that another
// one has written only two instructions later.
__device__ __forceinline__ void count_less(const uint4 (&o)[4], const uint4 head, uint32_t& rank, uint32_t (&diff)[4]) {
    uint32_t a0, a1, a2, a3, b0, b1, b2, b3, c0, c1, c2, c3, d0, d1, d2, d3;
    uint64_t ca, cb, cc, cd;  // borrows
    asm("v_sub_co_u32_e64 %[a0], %[ca], %[ax], %[hx]\n\tv_sub_co_u32_e64 %[b0], %[cb], %[bx], %[hx]\n\t"
        "v_sub_co_u32_e64 %[c0], %[cc], %[cx], %[hx]\n\tv_sub_co_u32_e64 %[d0], %[cd], %[dx], %[hx]\n\t"
        "v_subb_co_u32_e64 %[a1], %[ca], %[ay], %[hy], %[ca]\n\tv_subb_co_u32_e64 %[b1], %[cb], %[by], %[hy], %[cb]\n\t"
        "v_subb_co_u32_e64 %[c1], %[cc], %[cy], %[hy], %[cc]\n\tv_subb_co_u32_e64 %[d1], %[cd], %[dy], %[hy], %[cd]\n\t"
        "v_subb_co_u32_e64 %[a2], %[ca], %[az], %[hz], %[ca]\n\tv_subb_co_u32_e64 %[b2], %[cb], %[bz], %[hz], %[cb]\n\t"
        "v_subb_co_u32_e64 %[c2], %[cc], %[cz], %[hz], %[cc]\n\tv_subb_co_u32_e64 %[d2], %[cd], %[dz], %[hz], %[cd]\n\t"
        "v_subb_co_u32_e64 %[a3], %[ca], %[aw], %[hw], %[ca]\n\tv_subb_co_u32_e64 %[b3], %[cb], %[bw], %[hw], %[cb]\n\t"
        "v_subb_co_u32_e64 %[c3], %[cc], %[cw], %[hw], %[cc]\n\tv_subb_co_u32_e64 %[d3], %[cd], %[dw], %[hw], %[cd]\n\t"
        "v_addc_co_u32_e64 %[rank], %[ca], 0, %[rank], %[ca]\n\tv_addc_co_u32_e64 %[rank], %[cb], 0, %[rank], %[cb]\n\t"
        "v_addc_co_u32_e64 %[rank], %[cc], 0, %[rank], %[cc]\n\tv_addc_co_u32_e64 %[rank], %[cd], 0, %[rank], %[cd]\n\ts_nop 1"
        : [a0] "=&v"(a0), [a1] "=&v"(a1), [a2] "=&v"(a2), [a3] "=&v"(a3), [b0] "=&v"(b0), [b1] "=&v"(b1), [b2] "=&v"(b2), [b3] "=&v"(b3),
          [c0] "=&v"(c0), [c1] "=&v"(c1), [c2] "=&v"(c2), [c3] "=&v"(c3), [d0] "=&v"(d0), [d1] "=&v"(d1), [d2] "=&v"(d2), [d3] "=&v"(d3),
          [ca] "=&s"(ca), [cb] "=&s"(cb), [cc] "=&s"(cc), [cd] "=&s"(cd), [rank] "+v"(rank)
        : [ax] "v"(o[0].x), [ay] "v"(o[0].y), [az] "v"(o[0].z), [aw] "v"(o[0].w), [bx] "v"(o[1].x), [by] "v"(o[1].y), [bz] "v"(o[1].z), [bw] "v"(o[1].w),
          [cx] "v"(o[2].x), [cy] "v"(o[2].y), [cz] "v"(o[2].z), [cw] "v"(o[2].w), [dx] "v"(o[3].x), [dy] "v"(o[3].y), [dz] "v"(o[3].z), [dw] "v"(o[3].w),
          [hx] "v"(head.x), [hy] "v"(head.y), [hz] "v"(head.z), [hw] "v"(head.w));
    diff[0] = a0 | a1 | a2 | a3;
    diff[1] = b0 | b1 | b2 | b3;
    diff[2] = c0 | c1 | c2 | c3;
    diff[3] = d0 | d1 | d2 | d3;
}

// Ranks one entry against `count` others, of which this thread takes every `slices`-th: heads[c] = the first 16 bytes of entry
// base + c's key, padded with all ones to a multiple of 4 * slices.  The rest of a key and the seqno are read from the
// buffer on a 16-byte tie only: an entry with itself, versions of a key.
__device__ __forceinline__ void rank_against(const uint4* heads, const uint32_t base, const uint32_t count, const uint32_t slice, const uint32_t slices,
                                             const lsm_entry_t* buffer, const uint32_t n, const uint32_t i, const uint4 head, const Key& key,
                                             const uint64_t seq, uint32_t& rank, bool& shadowed) {
    for (uint32_t c = slice; c < count; c += 4 * slices) {
        uint4 o[4];
        uint32_t diff[4];
#pragma unroll
        for (int a = 0; a < 4; a++) o[a] = heads[c + a * slices];
        count_less(o, head, rank, diff);
        if (min(min(diff[0], diff[1]), min(diff[2], diff[3])) == 0) {
#pragma unroll
            for (int a = 0; a < 4; a++) {
                const uint32_t e = base + c + a * slices;
                if (diff[a] != 0 || e == i || e >= n) continue;
                const lsm_entry_t* other = buffer + e;
                const int cmp = key_cmp(load_key(other), key);
                const bool newer = cmp == 0 && (other->seqno > seq || (other->seqno == seq && e > i));
                shadowed = shadowed || newer;
                rank += (cmp < 0 || newer) ? 1 : 0;
            }
        }
    }
}

// n^2 compares of 16-byte key halves.  A workgroup ranks only kRankEntries entries, so that a buffer of a few thousand
// is hundreds of workgroups (one thread per entry left 15 workgroups with 3,600 serial compares each: 387 us for this
// step on 3,600 entries): 16 lanes hold 16 entries, and the 64 groups of 16 lanes share the other entries out, which are
// staged in LDS (the lanes of a wave read four records at a time).  Bound by the instructions of the compares, eight a pair (15.9 -> 11.5 us
// for 3,600 entries since they are a subtraction with borrow), and by the chain of steps of a workgroup: with 512 threads, 32 groups, a call
// of 3,600 entries takes 14.3 us, with 1,024 13.4; 4,096 15.4 and 14.1; 8,192 31.3 and 30.0; up to 1,500 the same.
constexpr int kRankThreads = 1024;
constexpr int kRankEntries = 16;
constexpr int kRankTile = 2048;  // records staged at a time
__global__ void __launch_bounds__(kRankThreads) flush_rank_kernel(const lsm_entry_t* buffer, uint32_t n, uint32_t* packed) {
    constexpr uint32_t kSlices = kRankThreads / kRankEntries;
    static_assert(kRankTile % (4 * kSlices) == 0 && kRankTile % kRankThreads == 0, "padding of the staged records");
    __shared__ uint4 tile[kRankTile];
    __shared__ uint32_t part[kRankThreads / kWave][kRankEntries];
    const uint32_t i = blockIdx.x * kRankEntries + threadIdx.x % kRankEntries;
    const uint32_t slice = threadIdx.x / kRankEntries;
    const lsm_entry_t* me = buffer + (i < n ? i : 0);
    const Key key = load_key(me);
    const uint4 head = key_head(*reinterpret_cast<const uint4*>(me));
    const uint64_t seq = me->seqno;
    uint32_t rank = 0;
    bool shadowed = false;
    for (uint32_t t0 = 0; t0 < n; t0 += kRankTile) {
        const uint32_t count = min((uint32_t)kRankTile, n - t0);
        __syncthreads();
        uint4 q[kRankTile / kRankThreads];
#pragma unroll
        for (int a = 0; a < kRankTile / kRankThreads; a++) {
            const uint32_t c = threadIdx.x + a * kRankThreads;
            q[a] = make_uint4(~0u, ~0u, ~0u, ~0u);
            if (c < count) q[a] = *reinterpret_cast<const uint4*>(buffer + t0 + c);
        }
#pragma unroll
        for (int a = 0; a < kRankTile / kRankThreads; a++) tile[threadIdx.x + a * kRankThreads] = key_head(q[a]);
        __syncthreads();
        rank_against(tile, t0, count, slice, kSlices, buffer, n, i, head, key, seq, rank, shadowed);
    }
    // both results of the 64 slices in one word: the sums stay below 2^16 (rank) and 2^7 (slices that saw a newer version)
    uint32_t v = rank | (shadowed ? 1u << 16 : 0u);
    v += __shfl_xor(v, 16, kWave);
    v += __shfl_xor(v, 32, kWave);
    if ((threadIdx.x & (kWave - 1)) < kRankEntries) part[threadIdx.x / kWave][threadIdx.x % kRankEntries] = v;
    __syncthreads();
    if (threadIdx.x < kRankEntries && i < n) {
        v = 0;
        for (int w = 0; w < kRankThreads / kWave; w++) v += part[w][threadIdx.x];
        packed[i] = (v & 0xFFFF) | ((v >> 16) != 0 ? kShadowed : 0u);
    }
}

// A buffer of up to kSmallEntries entries in one launch of one workgroup: eight threads rank an entry, the shadowed ranks are a bitmap
// in LDS, four threads copy an entry.  Such calls are bound by the host, which the second launch costs 2.5 us; 256 entries
// would be longer on the GPU than in two launches (8.9 us with four threads an entry, against 7.1).
constexpr uint32_t kSmallEntries = 128;
constexpr int kSmallThreads = 1024;
__global__ void __launch_bounds__(kSmallThreads) flush_small_kernel(const lsm_entry_t* buffer, uint32_t n, lsm_entry_t* out, uint64_t* n_out,
                                                                   uint4* fence_out, uint32_t fence_stride) {
    constexpr uint32_t kSlices = kSmallThreads / kSmallEntries;
    static_assert(kSmallEntries % (4 * kSlices) == 0, "padding of the records");
    __shared__ uint4 heads[kSmallEntries];
    __shared__ uint32_t packed[kSlices][kSmallEntries];  // by slice; the first row becomes the result
    __shared__ uint32_t bits[kSmallEntries / 32];        // bit r: the entry of rank r is shadowed
    const uint32_t tid = threadIdx.x;
    const uint32_t copied = tid / 4 < n ? tid / 4 : n;  // the entry that this thread copies a quarter of
    const uint4 part = copied < n ? reinterpret_cast<const uint4*>(buffer + copied)[tid & 3] : make_uint4(0, 0, 0, 0);
    if (tid < kSmallEntries) {
        uint4 q = make_uint4(~0u, ~0u, ~0u, ~0u);
        if (tid < n) q = *reinterpret_cast<const uint4*>(buffer + tid);
        heads[tid] = key_head(q);
    }
    if (tid < kSmallEntries / 32) bits[tid] = 0;
    const uint32_t i = tid % kSmallEntries, slice = tid / kSmallEntries;
    uint32_t rank = 0;
    bool shadowed = false;
    __syncthreads();
    if (i < n) {
        const Key key = load_key(buffer + i);
        rank_against(heads, 0, n, slice, kSlices, buffer, n, i, heads[i], key, buffer[i].seqno, rank, shadowed);
    }
    packed[slice][i] = rank | (shadowed ? 1u << 16 : 0u);
    __syncthreads();
    if (tid < n) {
        uint32_t v = 0;
        for (uint32_t g = 0; g < kSlices; g++) v += packed[g][tid];
        v = (v & 0xFFFF) | ((v >> 16) != 0 ? kShadowed : 0u);
        packed[0][tid] = v;
        if (v & kShadowed) atomicOr(&bits[(v & 0xFFFF) >> 5], 1u << (v & 31));
    }
    __syncthreads();
    const uint32_t p = copied < n ? packed[0][copied] : kShadowed;
    uint32_t before = 0, total = 0;
#pragma unroll
    for (uint32_t w = 0; w < kSmallEntries / 32; w++) {
        const uint32_t b = bits[w], c = __popc(b);
        total += c;
        before += w < (p & 0xFFFF) >> 5 ? c : (w == (p & 0xFFFF) >> 5 ? __popc(b & ((1u << (p & 31)) - 1)) : 0);
    }
    if (tid == 0) *n_out = n - total;
    if (p & kShadowed) return;
    const uint32_t at = p - before;
    reinterpret_cast<uint4*>(out + at)[tid & 3] = part;
    if (fence_out != nullptr && (tid & 3) < 2 && at % fence_stride == 0) fence_out[(at / fence_stride) * 2 + (tid & 3)] = part;
}

// Up to here ranks by comparing all pairs: 8,192 entries take 32 us, where sorting segments and merging them takes 50 us for
// 8,193 (three dependent launches).
constexpr uint64_t kFlushDirect = 8192;

// Four lanes per entry.  Every workgroup reads all packed ranks (at most 32 KB, from the L2).
constexpr int kPlaceThreads = 256;
static_assert(kFlushDirect == kPlaceThreads * 32, "one 32-bit word of the bitmap per thread");
__global__ void __launch_bounds__(kPlaceThreads) flush_place_kernel(const lsm_entry_t* buffer, uint32_t n, const uint32_t* packed,
                                                                   lsm_entry_t* out, uint64_t* n_out, uint4* fence_out, uint32_t fence_stride) {
    __shared__ uint32_t bits[kPlaceThreads];    // bit r: the entry of rank r is shadowed
    __shared__ uint32_t before[kPlaceThreads];  // shadowed ranks below the word
    __shared__ uint32_t wave_sum[kPlaceThreads / kWave];
    const int tid = threadIdx.x;
    bits[tid] = 0;
    __syncthreads();
    const uint32_t i = blockIdx.x * (kPlaceThreads / 4) + tid / 4;
    const uint32_t p = i < n ? packed[i] : kShadowed;
    const uint4 part = i < n ? reinterpret_cast<const uint4*>(buffer + i)[tid & 3] : make_uint4(0, 0, 0, 0);
    constexpr int kAhead = 8;  // ranks a thread reads before it looks at the first
    for (uint32_t e0 = tid; e0 < n; e0 += kAhead * kPlaceThreads) {
        uint32_t r[kAhead];
#pragma unroll
        for (int a = 0; a < kAhead; a++) r[a] = e0 + a * kPlaceThreads < n ? packed[e0 + a * kPlaceThreads] : 0;
#pragma unroll
        for (int a = 0; a < kAhead; a++)
            if (r[a] & kShadowed) atomicOr(&bits[(r[a] & ~kShadowed) >> 5], 1u << (r[a] & 31));
    }
    __syncthreads();
    const uint32_t count = __popc(bits[tid]);
    uint32_t incl = count;
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t v = __shfl_up(incl, off, kWave);
        if ((tid & (kWave - 1)) >= off) incl += v;
    }
    if ((tid & (kWave - 1)) == kWave - 1) wave_sum[tid / kWave] = incl;
    __syncthreads();
    uint32_t total = 0, lead = 0;
    for (int w = 0; w < kPlaceThreads / kWave; w++) {
        if (w < tid / kWave) lead += wave_sum[w];
        total += wave_sum[w];
    }
    before[tid] = lead + incl - count;
    __syncthreads();
    if (blockIdx.x == 0 && tid == 0) *n_out = n - total;
    if (p & kShadowed) return;
    const uint32_t at = p - before[p >> 5] - __popc(bits[p >> 5] & ((1u << (p & 31)) - 1));
    reinterpret_cast<uint4*>(out + at)[tid & 3] = part;
    if (fence_out != nullptr && (tid & 3) < 2 && at % fence_stride == 0) fence_out[(at / fence_stride) * 2 + (tid & 3)] = part;
}

// ---------------------------------------------------------------------------------------
// One workgroup sorts one segment.
// What moves through LDS is a 16-byte record per entry: the first 14 key bytes as a 112-bit number and, below, the
// entry's age (0 = written last), so records are distinct and versions of a key come in write order, newest write
// first.  Every thread sorts four consecutive records in registers and every wave its 256, by bitonic merges between lanes (data moves inside
// rows of 16 lanes by DPP, no LDS and no barrier); then log2(segment / 256) rounds of merge-path merges
// double the sorted lists, a thread producing four outputs per round from four records of either list (bitonic
// half-cleaner and merge network).  Positions whose 14 bytes equal a neighbour's (versions of a key, and keys that
// differ further on) are settled afterwards by the rest of the key, seqno and age: each by comparing itself with the whole
// group, or, where some group is long, by a merge sort of the whole segment that compares these.  Bound by LDS
// operations of one compute unit per segment; all pairs of a segment instead took 936 us for 100,001 entries, this 24
// (27 with merge-path rounds in LDS for lists of less than 256 as well): load 1, sort in waves 6, three rounds 5, ties 3, positions 1, output 3.5.  The entries themselves are
// read a second time for the output (they come from the L2).
// ---------------------------------------------------------------------------------------
// Short segments put more compute units to work (a segment is a serial chain on one), at the price of one merge round more and more
// runs to find boundaries in: 100,001 entries 47.3 + 7.7 + 25.9 us (sort, partition, merge) with segments of 4,096, 27.3 + 10.4 + 30.4
// with 2,048; segments of 1,024 (up to 65,536 entries) gain nothing more (50,000: 62.8 us in all, 60.2 with 1,024; 20,000: 55.1
// both).  Beyond 64 short ones, the most a merge takes, long segments.  Four records per thread: with eight, half as many waves,
// a segment of 4,096 takes 47.5 us instead of 41.8, of 2,048 37.7 instead of 27.5.
constexpr uint64_t kLongSegment = 4096, kShortSegment = 2048;
constexpr int kSortItems = 4;
constexpr uint64_t kMostShort = kShortSegment * LSM_MAX_RUNS;
static_assert(kLongSegment * LSM_MAX_RUNS >= LSM_MAX_BUFFER, "the segments of the largest buffer must fit one compaction");
// Groups are settled by comparing their positions one by one, a serial chain of LDS reads that grows with the square of the
// members (one group of 4,096: 10.6 ms a segment), unless four lanes in a row have nothing but positions that
// share their 14 bytes with the one before: the merge sort takes about as long as the first sort whatever the groups
// (8,193 versions of one key 128 us in all, 62 for distinct keys).  That is so for every group of 32 members and for none of 16.
// 100,001 entries in groups of about 10 / 20 / 64 members: 164 / 181 / 313 us one by one, 174 / 170 / 166 by the merge sort.
template <int kSortThreads>
struct SortShared {
    static constexpr uint32_t kFlushSegment = kSortThreads * kSortItems;
    uint4 buf[2][kFlushSegment];       // records, two sides; then the rest of the key and the seqno of tied positions
    uint16_t order[kFlushSegment];     // final position -> age
    uint16_t other[kFlushSegment];     // second side of the merge sort of tied positions
    uint32_t wave_count[kSortThreads / kWave];
    uint32_t deep;                     // some group is long
    alignas(4) uint8_t flag[kFlushSegment + 8];  // sorted position: 1 = same 14 bytes as the one before
    alignas(4) uint8_t lose[kFlushSegment];      // final position: 1 = shadowed
};

struct Rec {
    uint64_t hi, lo;
};
__device__ __forceinline__ Rec rec_load(const uint4* p) {
    const uint4 v = *p;
    return Rec{((uint64_t)v.y << 32) | v.x, ((uint64_t)v.w << 32) | v.z};
}
__device__ __forceinline__ void rec_store(uint4* p, const Rec& v) {
    *p = make_uint4((uint32_t)v.hi, (uint32_t)(v.hi >> 32), (uint32_t)v.lo, (uint32_t)(v.lo >> 32));
}
__device__ __forceinline__ bool rec_less(const Rec& a, const Rec& b) { return (a.hi < b.hi) | ((a.hi == b.hi) & (a.lo < b.lo)); }
__device__ __forceinline__ void rec_order(Rec& a, Rec& b) {
    const bool swap = rec_less(b, a);
    const Rec t = a;
    a.hi = swap ? b.hi : a.hi, a.lo = swap ? b.lo : a.lo;
    b.hi = swap ? t.hi : b.hi, b.lo = swap ? t.lo : b.lo;
}
// v of the lane whose number differs in the bits of kMask
template <int kMask>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
    auto dpp = [](uint32_t x, auto control) { return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, decltype(control)::value, 0xF, 0xF, true); };
    using std::integral_constant;
    if constexpr (kMask == 1) return dpp(v, integral_constant<int, 0xB1>{});            // quad_perm 1 0 3 2
    else if constexpr (kMask == 2) return dpp(v, integral_constant<int, 0x4E>{});       // quad_perm 2 3 0 1
    else if constexpr (kMask == 3) return dpp(v, integral_constant<int, 0x1B>{});       // quad_perm 3 2 1 0
    else if constexpr (kMask == 7) return dpp(v, integral_constant<int, 0x141>{});      // mirrored half row
    else if constexpr (kMask == 15) return dpp(v, integral_constant<int, 0x140>{});     // mirrored row
    else if constexpr (kMask == 8) return dpp(v, integral_constant<int, 0x128>{});      // row turned by eight
    else if constexpr (kMask == 4) return lane_xor<3>(lane_xor<7>(v));
    else return (uint32_t)__shfl_xor((int)v, kMask, kWave);
}
// One exchange between lanes: the lane with the lower number keeps the smaller record of each pair.  kMirror: record i meets the other
// lane's record 3 - i.
template <int kMask, bool kMirror>
__device__ __forceinline__ void lanes_order(Rec (&c)[4]) {
    constexpr int kTop = kMask >= 32 ? 32 : (kMask >= 16 ? 16 : (kMask >= 8 ? 8 : (kMask >= 4 ? 4 : (kMask >= 2 ? 2 : 1))));
    const bool upper = (threadIdx.x & kTop) != 0;
    Rec other[4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const Rec& x = c[kMirror ? 3 - i : i];
        other[i].hi = ((uint64_t)lane_xor<kMask>((uint32_t)(x.hi >> 32)) << 32) | lane_xor<kMask>((uint32_t)x.hi);
        other[i].lo = ((uint64_t)lane_xor<kMask>((uint32_t)(x.lo >> 32)) << 32) | lane_xor<kMask>((uint32_t)x.lo);
    }
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const bool take = rec_less(other[i], c[i]) != upper;
        c[i].hi = take ? other[i].hi : c[i].hi;
        c[i].lo = take ? other[i].lo : c[i].lo;
    }
}
// The wave's 256 records in ascending order, four per lane: lists of four, then bitonic merges of lists twice as long each time.
template <int kLanes>  // of a list
__device__ __forceinline__ void lanes_merge(Rec (&c)[4]) {
    lanes_order<2 * kLanes - 1, true>(c);  // the second list backwards
    if constexpr (kLanes >= 32) lanes_order<16, false>(c);
    if constexpr (kLanes >= 16) lanes_order<8, false>(c);
    if constexpr (kLanes >= 8) lanes_order<4, false>(c);
    if constexpr (kLanes >= 4) lanes_order<2, false>(c);
    if constexpr (kLanes >= 2) lanes_order<1, false>(c);
    rec_order(c[0], c[2]), rec_order(c[1], c[3]);
    rec_order(c[0], c[1]), rec_order(c[2], c[3]);
}
__device__ __forceinline__ void wave_sort(Rec (&c)[4]) {
    rec_order(c[0], c[1]), rec_order(c[2], c[3]);  // odd-even merge sort of four (Batcher): five exchanges
    rec_order(c[0], c[2]), rec_order(c[1], c[3]);
    rec_order(c[1], c[2]);
    lanes_merge<1>(c);
    lanes_merge<2>(c);
    lanes_merge<4>(c);
    lanes_merge<8>(c);
    lanes_merge<16>(c);
    lanes_merge<32>(c);
}
// where position p sits in the 16-byte arrays: threads own four consecutive positions (a stride of 64 bytes), so the positions of
// a group of four are permuted by the group's number
__device__ __forceinline__ uint32_t rec_at(uint32_t p) { return p ^ ((p >> 3) & (kSortItems - 1)); }

// What orders tied positions: their group (the group's first position, above key bytes 14..15), key bytes 16..31, then the
// newest version first.
struct Tied {
    uint32_t head, age;
    uint64_t k2, k3, seq;
};
__device__ __forceinline__ Tied tied_load(const uint4* info0, const uint4* info1, uint32_t p) {
    const uint4 a = info0[p], b = info1[p];
    return Tied{a.z, a.w, __builtin_bswap64(((uint64_t)b.y << 32) | b.x), __builtin_bswap64(((uint64_t)b.w << 32) | b.z), ((uint64_t)a.y << 32) | a.x};
}
__device__ __forceinline__ bool tied_same_key(const Tied& a, const Tied& b) { return (a.head == b.head) & (a.k2 == b.k2) & (a.k3 == b.k3); }
__device__ __forceinline__ bool tied_newer(const Tied& a, const Tied& b) { return a.seq > b.seq || (a.seq == b.seq && a.age < b.age); }
__device__ __forceinline__ bool tied_less(const Tied& a, const Tied& b) {
    if (a.head != b.head) return a.head < b.head;
    if (a.k2 != b.k2) return a.k2 < b.k2;
    if (a.k3 != b.k3) return a.k3 < b.k3;
    return tied_newer(a, b);
}

// Merge sort of all positions of the segment by tied_less, `len` of them in use: s.order[p] becomes the age of the p-th and
// s.lose[p] whether it is shadowed.  The whole workgroup calls; the info arrays are filled for every position.
template <int kSortThreads>
__device__ void flush_sort_tied(SortShared<kSortThreads>& s, const uint4* info0, const uint4* info1, const uint32_t len) {
    const uint32_t o = threadIdx.x * kSortItems;
    uint16_t *from = s.order, *to = s.other;
    for (uint32_t i = 0; i < (uint32_t)kSortItems; i++) {
        const Tied x = tied_load(info0, info1, o + i);
        uint32_t k = i;
        for (; k > 0 && tied_less(x, tied_load(info0, info1, from[o + k - 1])); k--) from[o + k] = from[o + k - 1];
        from[o + k] = (uint16_t)(o + i);
    }
    __syncthreads();
    for (uint32_t width = kSortItems; width < len; width <<= 1) {
        const uint32_t sa = o & ~(2 * width - 1), sb = sa + width, d = o - sa;
        uint32_t lo = d > width ? d - width : 0, hi = min(d, width);
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (tied_less(tied_load(info0, info1, from[sa + mid]), tied_load(info0, info1, from[sb + (d - 1 - mid)]))) lo = mid + 1;
            else hi = mid;
        }
        uint32_t a = lo, b = d - lo;
        Tied x = {}, y = {};
        if (a < width) x = tied_load(info0, info1, from[sa + a]);
        if (b < width) y = tied_load(info0, info1, from[sb + b]);
        for (uint32_t i = 0; i < (uint32_t)kSortItems; i++) {
            if (b >= width || (a < width && tied_less(x, y))) {
                to[o + i] = from[sa + a];
                if (++a < width) x = tied_load(info0, info1, from[sa + a]);
            } else {
                to[o + i] = from[sb + b];
                if (++b < width) y = tied_load(info0, info1, from[sb + b]);
            }
        }
        __syncthreads();
        uint16_t* const swap = from;
        from = to;
        to = swap;
    }
    uint16_t age[kSortItems];
    Tied prev = tied_load(info0, info1, from[o > 0 ? o - 1 : 0]);
#pragma unroll
    for (int i = 0; i < kSortItems; i++) {
        const Tied x = tied_load(info0, info1, from[o + i]);
        age[i] = (uint16_t)x.age;
        s.lose[o + i] = o + i > 0 && tied_same_key(prev, x) ? 1 : 0;
        prev = x;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kSortItems; i++) s.order[o + i] = age[i];
}

template <int kSortThreads>
__global__ void __launch_bounds__(kSortThreads) flush_sort_kernel(const lsm_entry_t* buffer, uint32_t n, lsm_entry_t* out, uint64_t* counts) {
    __shared__ SortShared<kSortThreads> s;
    constexpr uint32_t kFlushSegment = kSortThreads * kSortItems;
    static_assert(kSortItems == 4, "the sorting network is written for four");
    const uint32_t tid = threadIdx.x;
    // segments are numbered newest first, the order in which the merge takes them as runs
    const uint32_t seg = gridDim.x - 1 - blockIdx.x;
    const uint32_t first = seg * (uint32_t)kFlushSegment;
    const uint32_t len = min((uint32_t)kFlushSegment, n - first);
    const lsm_entry_t* src = buffer + first;

    if (tid == 0) s.deep = 0;
    // ---- records; age a = entry len - 1 - a of the segment.  Unused positions hold the largest value.
    const uint32_t o = tid * kSortItems;
    Rec c[kSortItems];
    {
        uint4 q[kSortItems];
#pragma unroll
        for (int i = 0; i < kSortItems; i++) q[i] = *reinterpret_cast<const uint4*>(src + min(o + i, len - 1));
#pragma unroll
        for (int i = 0; i < kSortItems; i++) {
            c[i].hi = __builtin_bswap64(((uint64_t)q[i].y << 32) | q[i].x);
            c[i].lo = (__builtin_bswap64(((uint64_t)q[i].w << 32) | q[i].z) & ~0xFFFFull) | (len - 1 - (o + i));
            if (o + i >= len) c[i].hi = c[i].lo = ~0ull;
        }
    }
    wave_sort(c);
#pragma unroll
    for (int i = 0; i < kSortItems; i++) rec_store(&s.buf[0][rec_at(o + i)], c[i]);
    __syncthreads();
    // ---- merge rounds
    uint32_t cur = 0;
    for (uint32_t width = kSortItems * kWave; width < len; width <<= 1) {
        const uint4* in = s.buf[cur];
        uint4* dst = s.buf[cur ^ 1];
        const uint32_t sa = o & ~(2 * width - 1), sb = sa + width, d = o - sa;  // both lists are `width` long (padding included)
        uint32_t lo = d > width ? d - width : 0, hi = min(d, width);
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (rec_less(rec_load(&in[rec_at(sa + mid)]), rec_load(&in[rec_at(sb + (d - 1 - mid))]))) lo = mid + 1;
            else hi = mid;
        }
        const uint32_t a = lo, b = d - lo;
#pragma unroll
        for (int i = 0; i < kSortItems; i++) {
            // the smallest half of two ascending lists: element i of one against the other's element as far from its end
            Rec x = {~0ull, ~0ull}, y = {~0ull, ~0ull};
            if (a + i < width) x = rec_load(&in[rec_at(sa + a + i)]);
            if (b + kSortItems - 1 - i < width) y = rec_load(&in[rec_at(sb + b + kSortItems - 1 - i)]);
            c[i] = rec_less(x, y) ? x : y;
        }
#pragma unroll
        for (int step = kSortItems / 2; step > 0; step >>= 1)
#pragma unroll
            for (int i = 0; i < kSortItems; i++)
                if ((i & step) == 0) rec_order(c[i], c[i + step]);
#pragma unroll
        for (int i = 0; i < kSortItems; i++) rec_store(&dst[rec_at(o + i)], c[i]);
        __syncthreads();
        cur ^= 1;
    }

    // ---- which positions share their 14 bytes with a neighbour?  c[] holds this thread's four sorted records.
    bool any = false, all = true;
    {
        Rec prev = c[0];
        if (o > 0) prev = rec_load(&s.buf[cur][rec_at(o - 1)]);
#pragma unroll
        for (int i = 0; i < kSortItems; i++) {
            const bool eq = o + i > 0 && o + i < len && prev.hi == c[i].hi && ((prev.lo ^ c[i].lo) >> 16) == 0;
            s.flag[o + i] = eq ? 1 : 0;
            s.lose[o + i] = 0;
            s.order[o + i] = (uint16_t)(c[i].lo & 0xFFFF);
            any = any || eq;
            all = all && eq;
            prev = c[i];
        }
    }
    const uint64_t full = __ballot(all);
    if ((full & full >> 1 & full >> 2 & full >> 3) != 0) s.deep = 1;
    if (tid == 0) s.flag[kFlushSegment] = 0;
    if (__syncthreads_or(any)) {
        const bool deep = s.deep != 0;
        uint32_t start[kSortItems] = {};
        if (deep) {  // where the group of every position starts: the last position without a flag up to it
            uint32_t last = 0;
#pragma unroll
            for (int i = 0; i < kSortItems; i++) last = s.flag[o + i] == 0 ? o + i : last;
            for (int off = 1; off < kWave; off <<= 1) {
                const uint32_t v = __shfl_up(last, off, kWave);
                if ((int)(tid & (kWave - 1)) >= off) last = max(last, v);
            }
            if ((tid & (kWave - 1)) == kWave - 1) s.wave_count[tid / kWave] = last;
            last = __shfl_up(last, 1, kWave);
            if ((tid & (kWave - 1)) == 0) last = 0;
            __syncthreads();
            for (uint32_t w = 0; w < tid / kWave; w++) last = max(last, s.wave_count[w]);
#pragma unroll
            for (int i = 0; i < kSortItems; i++) {
                last = s.flag[o + i] == 0 ? o + i : last;
                start[i] = last;
            }
        }
        // members of groups post the rest of their key, seqno and age at their sorted position
        uint4* info0 = s.buf[0];  // {seqno, group and key bytes 14..15, age}
        uint4* info1 = s.buf[1];  // key bytes 16..31
#pragma unroll
        for (int i = 0; i < kSortItems; i++) {
            const uint32_t p = o + i, age = (uint32_t)c[i].lo & 0xFFFF;
            if (p < len && (s.flag[p] | s.flag[p + 1]) != 0) {
                const uint4* e = reinterpret_cast<const uint4*>(src + (len - 1 - age));
                const uint4 k0 = e[0], meta = e[2];
                info0[p] = make_uint4(meta.x, meta.y, (start[i] << 16) | (__builtin_bswap32(k0.w) & 0xFFFF), age);
                info1[p] = e[1];
            } else if (deep) {
                info0[p] = make_uint4(0, 0, p << 16, age);
                info1[p] = make_uint4(0, 0, 0, 0);
            }
        }
        __syncthreads();
        if (deep) {
            flush_sort_tied(s, info0, info1, len);
        } else {
            for (uint32_t i = 0; i < (uint32_t)kSortItems; i++) {
                const uint32_t p = o + i;
                if (p >= len || (s.flag[p] | s.flag[p + 1]) == 0) continue;
                uint32_t first_member = p;
                while (s.flag[first_member] != 0) first_member--;  // flag[0] is 0
                const Tied a = tied_load(info0, info1, p);
                uint32_t rank = 0, q = first_member;
                bool shadowed = false;
                do {
                    if (q != p) {
                        const Tied b = tied_load(info0, info1, q);
                        const bool same = tied_same_key(a, b), newer = same && tied_newer(b, a);
                        const bool less = b.head != a.head ? b.head < a.head : (b.k2 != a.k2 ? b.k2 < a.k2 : b.k3 < a.k3);
                        shadowed = shadowed || newer;
                        rank += (same ? newer : less) ? 1 : 0;
                    }
                    q++;
                } while (s.flag[q] != 0);  // flag[len ..] is 0
                s.order[first_member + rank] = (uint16_t)a.age;
                s.lose[first_member + rank] = shadowed ? 1 : 0;
            }
        }
        __syncthreads();
    }

    // ---- positions of the survivors (block-wide prefix sum); order[] becomes output slot -> entry of the segment
    uint32_t keep = 0, mine[kSortItems];
#pragma unroll
    for (int i = 0; i < kSortItems; i++) {
        const uint32_t p = o + i;
        mine[i] = p < len && s.lose[p] == 0 ? len - 1 - s.order[p] : ~0u;
        keep += mine[i] != ~0u ? 1 : 0;
    }
    uint32_t incl = keep;
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t v = __shfl_up(incl, off, kWave);
        if ((int)(tid & (kWave - 1)) >= off) incl += v;
    }
    if ((tid & (kWave - 1)) == kWave - 1) s.wave_count[tid / kWave] = incl;
    __syncthreads();
    uint32_t slot = incl - keep, total = 0;
    for (uint32_t w = 0; w < kSortThreads / kWave; w++) {
        if (w < tid / kWave) slot += s.wave_count[w];
        total += s.wave_count[w];
    }
#pragma unroll
    for (int i = 0; i < kSortItems; i++)
        if (mine[i] != ~0u) s.order[slot++] = (uint16_t)mine[i];
    if (tid == 0) counts[blockIdx.x] = total;
    __syncthreads();
    // ---- output, four lanes per entry
    const uint4* from = reinterpret_cast<const uint4*>(src);
    uint4* to = reinterpret_cast<uint4*>(out + first);
    for (uint32_t x = tid; x < total * 4; x += kSortThreads) to[x] = from[(uint32_t)s.order[x >> 2] * 4 + (x & 3)];
}

__host__ inline size_t up256(size_t x) { return (x + 255) & ~size_t(255); }

// Workspace of the segmented path: sorted segments | segment counts | compaction workspace.
struct FlushLayout {
    size_t sorted, counts, compact, total;
    uint32_t segments;
    uint64_t segment;  // entries
    uint64_t upper[LSM_MAX_RUNS];  // entries per segment, newest segment first (the order the compaction takes them in)
};
static FlushLayout flush_layout(uint64_t n) {
    FlushLayout l;
    l.segment = n <= kMostShort ? kShortSegment : kLongSegment;
    l.segments = (uint32_t)((n + l.segment - 1) / l.segment);
    for (uint32_t j = 0; j < LSM_MAX_RUNS; j++) l.upper[j] = 0;
    for (uint32_t g = 0; g < l.segments; g++) {
        const uint64_t lo = g * l.segment;
        l.upper[l.segments - 1 - g] = (n - lo < l.segment) ? n - lo : l.segment;
    }
    l.sorted = 0;
    l.counts = up256(n * sizeof(lsm_entry_t));
    l.compact = l.counts + up256(LSM_MAX_RUNS * sizeof(uint64_t));
    l.total = l.compact + lsm_compact_workspace_bytes(l.upper, l.segments);
    return l;
}

}  // namespace lsm

extern "C" size_t lsm_flush_workspace_bytes(uint64_t n) {
    if (n > LSM_MAX_BUFFER) return 0;
    if (n <= lsm::kFlushDirect) return (size_t)n * sizeof(uint32_t);
    // never less than for a smaller buffer: more, shorter segments take more room to merge
    const size_t mine = lsm::flush_layout(n).total, shorter = lsm::flush_layout(n < lsm::kMostShort ? n : lsm::kMostShort).total;
    return mine > shorter ? mine : shorter;
}

extern "C" int lsm_flush_buffer(const lsm_entry_t* buffer, uint64_t n, const lsm_out_t* out, void* workspace, size_t workspace_bytes,
                                void* stream_v) {
    using namespace lsm;
    if (out == nullptr || out->n_out == nullptr) return LSM_ERR_NULL;
    if (n > 0 && (buffer == nullptr || out->entries == nullptr)) return LSM_ERR_NULL;
    if (n > LSM_MAX_BUFFER) return LSM_ERR_BAD_ARG;
    if ((reinterpret_cast<uintptr_t>(buffer) & 63) != 0 || (reinterpret_cast<uintptr_t>(out->entries) & 63) != 0) return LSM_ERR_BAD_ARG;
    if (out->fence_keys != nullptr && (out->fence_stride == 0 || (reinterpret_cast<uintptr_t>(out->fence_keys) & 15) != 0))
        return LSM_ERR_BAD_ARG;
    if (out->key_hashes != nullptr) return LSM_ERR_BAD_ARG;  // the filter of a flushed run: lsm_build_bloom
    if (out->capacity < n) return LSM_ERR_CAPACITY;
    const bool direct = n <= kFlushDirect;
    if (n > 0 && (workspace == nullptr || (reinterpret_cast<uintptr_t>(workspace) & (direct ? 3 : 255)) != 0 ||
                  workspace_bytes < lsm_flush_workspace_bytes(n)))
        return LSM_ERR_WORKSPACE;
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    uint4* fence_out = reinterpret_cast<uint4*>(out->fence_keys);
    const uint32_t fence_stride = out->fence_keys ? out->fence_stride : 1u;
    if (direct) {
        if (n > 0 && n <= kSmallEntries) {
            hipLaunchKernelGGL(flush_small_kernel, dim3(1), dim3(kSmallThreads), 0, stream, buffer, (uint32_t)n, out->entries, out->n_out, fence_out, fence_stride);
            return hipGetLastError() == hipSuccess ? LSM_OK : LSM_ERR_HIP;
        }
        uint32_t* packed = static_cast<uint32_t*>(workspace);
        const uint32_t per_block = kPlaceThreads / 4;
        if (n > 0)
            hipLaunchKernelGGL(flush_rank_kernel, dim3(((uint32_t)n + kRankEntries - 1) / kRankEntries), dim3(kRankThreads), 0, stream, buffer, (uint32_t)n, packed);
        hipLaunchKernelGGL(flush_place_kernel, dim3(n > 0 ? ((uint32_t)n + per_block - 1) / per_block : 1), dim3(kPlaceThreads), 0, stream, buffer,
                           (uint32_t)n, packed, out->entries, out->n_out, fence_out, fence_stride);
        return hipGetLastError() == hipSuccess ? LSM_OK : LSM_ERR_HIP;
    }
    // segments sorted on their own, into the workspace
    const FlushLayout l = flush_layout(n);
    char* base = static_cast<char*>(workspace);
    lsm_entry_t* sorted = reinterpret_cast<lsm_entry_t*>(base + l.sorted);
    uint64_t* counts = reinterpret_cast<uint64_t*>(base + l.counts);  // newest segment first
    auto sort = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, dim3(l.segments), dim3(threads), 0, stream, buffer, (uint32_t)n, sorted, counts);
    };
    if (l.segment == kShortSegment) sort(flush_sort_kernel<kShortSegment / kSortItems>, kShortSegment / kSortItems);
    else sort(flush_sort_kernel<kLongSegment / kSortItems>, kLongSegment / kSortItems);
    if (hipGetLastError() != hipSuccess) return LSM_ERR_HIP;
    // one merge of the sorted segments, the one written last first; their lengths stay on the device
    const lsm_entry_t* ptr[LSM_MAX_RUNS];
    for (uint32_t j = 0; j < l.segments; j++) ptr[j] = sorted + (uint64_t)(l.segments - 1 - j) * l.segment;
    return compact_device_lengths(ptr, l.upper, counts, l.segments, 0, out, base + l.compact, workspace_bytes - l.compact, stream);
}
