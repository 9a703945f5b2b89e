// Shared device-side definitions of the LSM key-index kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lsm_index.h"

namespace lsm {

constexpr int kWave = 64;

// A key as four big-endian-numeric words: comparing w[0], w[1], ... as unsigned integers is
// byte-string (memcmp) order of the 32 key bytes.
struct Key {
    uint64_t w[4];
};

__device__ __forceinline__ Key key_from_raw(uint4 lo, uint4 hi) {
    Key k;
    k.w[0] = __builtin_bswap64(((uint64_t)lo.y << 32) | lo.x);
    k.w[1] = __builtin_bswap64(((uint64_t)lo.w << 32) | lo.z);
    k.w[2] = __builtin_bswap64(((uint64_t)hi.y << 32) | hi.x);
    k.w[3] = __builtin_bswap64(((uint64_t)hi.w << 32) | hi.z);
    return k;
}

// Key of an entry (or of a 32-byte key record) in global or shared memory; p is 16-byte aligned.
__device__ __forceinline__ Key load_key(const void* p) {
    const uint4* q = reinterpret_cast<const uint4*>(p);
    return key_from_raw(q[0], q[1]);
}

__device__ __forceinline__ bool key_less(const Key& a, const Key& b) {
    if (a.w[0] != b.w[0]) return a.w[0] < b.w[0];
    if (a.w[1] != b.w[1]) return a.w[1] < b.w[1];
    if (a.w[2] != b.w[2]) return a.w[2] < b.w[2];
    return a.w[3] < b.w[3];
}

__device__ __forceinline__ bool key_equal(const Key& a, const Key& b) {
    return ((a.w[0] ^ b.w[0]) | (a.w[1] ^ b.w[1]) | (a.w[2] ^ b.w[2]) | (a.w[3] ^ b.w[3])) == 0;
}

// key < k for a key kept as two separate halves (bytes 0..15 at lo, bytes 16..31 at hi); the second
// half is read only when the first 16 bytes tie.
__device__ __forceinline__ bool entry_key_less(const uint4* lo, const uint4* hi, const Key& k) {
    const uint4 a = *lo;
    const uint64_t w0 = __builtin_bswap64(((uint64_t)a.y << 32) | a.x);
    const uint64_t w1 = __builtin_bswap64(((uint64_t)a.w << 32) | a.z);
    if (w0 != k.w[0]) return w0 < k.w[0];
    if (w1 != k.w[1]) return w1 < k.w[1];
    const uint4 b = *hi;
    const uint64_t w2 = __builtin_bswap64(((uint64_t)b.y << 32) | b.x);
    const uint64_t w3 = __builtin_bswap64(((uint64_t)b.w << 32) | b.z);
    if (w2 != k.w[2]) return w2 < k.w[2];
    return w3 < k.w[3];
}

// Three-way compare of a record's key with k (-1, 0, +1) given the record's first 16 key bytes;
// the second half is read only when those tie.
template <typename E>
__device__ __forceinline__ int entry_key_cmp(const E* e, const uint4 lo, const Key& k) {
    const uint64_t w0 = __builtin_bswap64(((uint64_t)lo.y << 32) | lo.x);
    const uint64_t w1 = __builtin_bswap64(((uint64_t)lo.w << 32) | lo.z);
    if (w0 != k.w[0]) return w0 < k.w[0] ? -1 : 1;
    if (w1 != k.w[1]) return w1 < k.w[1] ? -1 : 1;
    const uint4 hi = reinterpret_cast<const uint4*>(e)[1];
    const uint64_t w2 = __builtin_bswap64(((uint64_t)hi.y << 32) | hi.x);
    const uint64_t w3 = __builtin_bswap64(((uint64_t)hi.w << 32) | hi.z);
    if (w2 != k.w[2]) return w2 < k.w[2] ? -1 : 1;
    if (w3 != k.w[3]) return w3 < k.w[3] ? -1 : 1;
    return 0;
}

// The probe position of a search step in [lo, hi), lo < hi: the index with the most trailing zero
// bits.  Positions then form one fixed search tree over the whole array whatever range a search
// starts from, so searches for nearby keys - and repeated searches in a shrinking range - read the
// same few records (the ancestors of the answer) instead of a fresh set of midpoints each time.
__device__ __forceinline__ uint64_t tree_mid(uint64_t lo, uint64_t hi) {
    const uint64_t last = hi - 1, diff = lo ^ last;
    if (diff == 0) return lo;
    const int top = 63 - __builtin_clzll(diff);  // highest bit in which lo and last differ: set in last, clear in lo
    return last & ~((1ull << top) - 1);
}

// Number of records of run[lo, hi) whose key is < k, plus lo (global memory), by bisection along
// the fixed tree.  eq tells whether the record at the result lies inside
// [lo, hi) and has exactly the key k.
template <typename E>
__device__ __forceinline__ uint64_t lower_bound_eq(const E* run, uint64_t lo, uint64_t hi, const Key& k, bool& eq,
                                                   const bool fresh = true) {
    if (fresh) eq = false;  // always describes the record at the current hi
    while (lo < hi) {
        const uint64_t mid = tree_mid(lo, hi);
        const int c = entry_key_cmp(run + mid, *reinterpret_cast<const uint4*>(run + mid), k);
        if (c < 0) lo = mid + 1;
        else hi = mid, eq = c == 0;
    }
    return lo;
}

// The same result by four-way steps at the quartiles of the range (three records read together per
// step): half the dependent round trips for half as many reads again.  For arrays that stay in cache,
// where the round trips are what costs.
template <typename E>
__device__ __forceinline__ uint64_t lower_bound_eq4(const E* run, uint64_t lo, uint64_t hi, const Key& k, bool& eq) {
    eq = false;  // always describes the record at the current hi
    while (hi - lo >= 3) {
        const uint64_t w = hi - lo;
        const uint64_t m1 = lo + (w >> 2), m2 = lo + (w >> 1), m3 = lo + ((3 * w) >> 2);  // lo <= m1 < m2 < m3 < hi
        const uint4 a1 = *reinterpret_cast<const uint4*>(run + m1);
        const uint4 a2 = *reinterpret_cast<const uint4*>(run + m2);
        const uint4 a3 = *reinterpret_cast<const uint4*>(run + m3);
        const int c1 = entry_key_cmp(run + m1, a1, k), c2 = entry_key_cmp(run + m2, a2, k), c3 = entry_key_cmp(run + m3, a3, k);
        if (c3 < 0) {
            lo = m3 + 1;
        } else if (c2 < 0) {
            lo = m2 + 1, hi = m3, eq = c3 == 0;
        } else if (c1 < 0) {
            lo = m1 + 1, hi = m2, eq = c2 == 0;
        } else {
            hi = m1, eq = c1 == 0;
        }
    }
    return lower_bound_eq(run, lo, hi, k, eq, false);  // at most two records left; eq carries over
}

// Sum / max over the 64 lanes of a wave; every lane must call.
__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) {
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}
__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v) {
    for (int off = kWave / 2; off > 0; off >>= 1) {
        uint64_t o = __shfl_xor(v, off, kWave);
        v = o > v ? o : v;
    }
    return v;
}

// Inclusive prefix sum over the lanes of a wave: shifts inside rows of 16 lanes (0 comes in at a row's start), then the sums
// of the rows below.
template <int kOff>
__device__ __forceinline__ uint32_t row_shift_up(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x110 | kOff, 0xF, 0xF, true);
}
__device__ __forceinline__ uint32_t wave_scan_u32(uint32_t v) {
    v += row_shift_up<1>(v);
    v += row_shift_up<2>(v);
    v += row_shift_up<4>(v);
    v += row_shift_up<8>(v);
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)v, 15), b = (uint32_t)__builtin_amdgcn_readlane((int)v, 31);
    const uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)v, 47);
    return v + (lane >= 16 ? a : 0) + (lane >= 32 ? b : 0) + (lane >= 48 ? c : 0);
}

// 16-byte load through a pointer that is known to be global memory (it went through LDS or a
// table, so the compiler cannot tell): a global instead of a flat load.
__device__ __forceinline__ uint4 load_global_u4(const uint4* p) { typedef uint32_t v4 __attribute__((ext_vector_type(4))); const v4 v = *(const __attribute__((address_space(1))) v4*)p; return make_uint4(v.x, v.y, v.z, v.w); }

// 16-byte store of output that does not displace what the L2 holds.  For what is more than the L2s take, or written where nothing on the chip reads it soon;
// merges of a few tiles use it as well, though a filter or the next merge may read their output at once: 4 x 16,384 entries 18.6 us with plain stores, 18.2
// so, write buffers of 100,001 57.4 and 56.7; a driver's flushes the same (96 of 3,600 entries 2.25 to 2.31 ms either way).
__device__ __forceinline__ void store_streaming_u4(uint4* p, const uint4 q) { typedef uint32_t v4 __attribute__((ext_vector_type(4))); const v4 v = {q.x, q.y, q.z, q.w}; __builtin_nontemporal_store(v, (__attribute__((address_space(1))) v4*)p); }

// Bloom filter addressing: the block of a key and the six bits it sets or tests there, as four 32-bit masks.
__device__ __forceinline__ uint64_t mix64(uint64_t x) {
    x ^= x >> 30;
    x *= 0xBF58476D1CE4E5B9ull;
    x ^= x >> 27;
    x *= 0x94D049BB133111EBull;
    x ^= x >> 31;
    return x;
}
// the hash h of a key; its top half picks the block
__device__ __forceinline__ uint64_t bloom_key_hash(const Key& k) {
    uint64_t h = 0x5EED251116138ull;
    for (int i = 0; i < 4; i++) h = mix64(h ^ k.w[i]);
    return h;
}
// the bit positions, seven bits each from the lowest up
__device__ __forceinline__ uint64_t bloom_bits(uint64_t h) { return mix64(h ^ 0x9E3779B97F4A7C15ull); }
__device__ __forceinline__ uint4 bloom_mask(uint64_t h) {
    const uint64_t g = bloom_bits(h);
    uint32_t m[4] = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 6; j++) {
        const uint32_t b = (uint32_t)(g >> (7 * j)) & 127;
#pragma unroll
        for (int w = 0; w < 4; w++) m[w] |= (b >> 5) == (uint32_t)w ? 1u << (b & 31) : 0u;
    }
    return make_uint4(m[0], m[1], m[2], m[3]);
}
__device__ __forceinline__ uint64_t bloom_hash(const Key& k, uint4& mask) {
    const uint64_t h = bloom_key_hash(k);
    mask = bloom_mask(h);
    return h;
}
__device__ __forceinline__ uint32_t bloom_block(uint64_t h, uint32_t n_blocks) { return (uint32_t)(((h >> 32) * (uint64_t)n_blocks) >> 32); }
__device__ __forceinline__ bool bloom_excludes(const uint4 w, const uint4 mask) {
    return (((w.x & mask.x) ^ mask.x) | ((w.y & mask.y) ^ mask.y) | ((w.z & mask.z) ^ mask.z) | ((w.w & mask.w) ^ mask.w)) != 0;
}

// Hash index of a run: 64-byte buckets of kIndexSlots slots.  Bytes 0..15: the slots' 16-bit tag fields (low 15 bits
// = tag; bit 15 of the first field = more keys fall into the bucket than it has slots); bytes 16..47: the slots' 32-bit
// positions, all ones = empty slot; bytes 48..63: zero.
constexpr uint32_t kIndexSlots = 8;
constexpr uint32_t kIndexNoEntry = 0xFFFFFFFFu;
constexpr uint32_t kIndexTagMask = 0x7FFFu;
__host__ __device__ inline uint64_t index_buckets(uint64_t n) { return n ? (n + 3) / 4 : 1; }

// Tile status word of a compaction: top two bits = state, then 20 bits that say which call has written it (0 where the call's first
// launch has zeroed the words), low 42 bits = value.  The last tile's holds the number of output entries.
constexpr uint64_t kStEmpty = 0, kStAggregate = 1, kStPrefix = 2, kStFailed = 3;
#ifndef LSM_STATUS_EPOCH_BITS
#define LSM_STATUS_EPOCH_BITS 20  // fewer where a test wants to see them used up
#endif
constexpr int kStShift = 62, kStEpochShift = 42, kStEpochBits = LSM_STATUS_EPOCH_BITS;
constexpr uint64_t kStValueMask = (1ull << kStEpochShift) - 1;
constexpr uint32_t kStEpochs = 1u << kStEpochBits;

// Run descriptors passed to kernels by value.
struct RunTable {
    const lsm_entry_t* ptr[LSM_MAX_RUNS];
    uint64_t n[LSM_MAX_RUNS];  // run lengths; upper bounds when n_dev is given
    const uint64_t* n_dev;     // optional: the run lengths in device memory (written by an earlier kernel of the stream)
    uint32_t k;
};
__device__ __forceinline__ uint64_t run_len(const RunTable& rt, uint32_t j) { return rt.n_dev ? rt.n_dev[j] : rt.n[j]; }

// Calls between the parts of the library (arguments are checked by the caller).
constexpr uint64_t kShortTiles = 256;
constexpr uint64_t kMostClearWords = 1ull << 31;  // 16-byte words of a span: fewer than this (a bit of their number is taken, see kHashesBehind)
struct ClearSpan {  // device memory to be zeroed by a launch that is made anyway; 16-byte aligned
    void* p = nullptr;
    size_t bytes = 0;  // a multiple of 16
    // not 0: the span is for the Bloom filter of the compaction's output, which is to be built there as well, with so many bits
    // per key; filter_built says whether the launch for it has been made
    uint32_t filter_bits = 0;
    mutable bool filter_built = false;
    // Status words of the caller's own, kShortTiles of them.  epoch 0: unknown contents, zeroed by a launch that is made anyway if
    // there is one (status_zeroed says so).  Otherwise every word is zero or of a smaller epoch, and a merge of two runs that is short
    // enough is one launch.  (In a batch: those of its first job.)
    uint64_t* status = nullptr;
    uint32_t epoch = 0;
    mutable bool status_zeroed = false;
    void* filter = nullptr;  // not null: p is a FilterScratch, and the filter is built there from the keys' hashes, which the merge writes
    uint64_t* hashes() const { return filter != nullptr ? reinterpret_cast<uint64_t*>(static_cast<char*>(p) + bytes) : nullptr; }
};
// Filters of up to kSmallFilterBlocks blocks are built in a workgroup's LDS, longer ones behind a merge from the keys' hashes, which
// the merge writes: sorted by ranges of blocks, then every range in LDS.
constexpr uint32_t kSmallFilterBlocks = 8192;
constexpr uint64_t kSmallFilterKeys = 1u << 18;  // a longer run with so small a filter is not
inline bool small_filter(uint64_t n, uint64_t blocks) { return blocks <= kSmallFilterBlocks && n <= kSmallFilterKeys; }
// Memory for the latter: a cursor for each range, to be zeroed, right behind them the hashes, then [range][cap] hashes by range.
struct FilterScratch {
    uint32_t unit_log, n_ranges, cap;  // blocks of a range; hashes it has room for
    size_t zeroed, ranged, total;      // bytes
};
constexpr uint32_t kMostFilterRanges = 1024;
inline FilterScratch filter_scratch(uint64_t n, uint64_t blocks) {
    FilterScratch s;
    s.unit_log = 8;  // a range for three quarters of the compute units, or more, of up to 4,096 blocks (64 KiB)
    while (s.unit_log < 12 && (blocks >> (s.unit_log + 1)) >= 192) s.unit_log++;
    const uint64_t ranges = (blocks + (1u << s.unit_log) - 1) >> s.unit_log;
    s.n_ranges = ranges > kMostFilterRanges ? 0 : (uint32_t)ranges;  // 0: not built this way
    // eight standard deviations more than the mean; a range with more is built from all hashes
    const uint64_t mean = (uint64_t)((unsigned __int128)n * (1u << s.unit_log) / blocks) + 1, cap = mean + (uint64_t)(8 * __builtin_sqrt((double)mean)) + 32;
    s.cap = (uint32_t)(cap > n ? n : cap);
    s.zeroed = (s.n_ranges * 4 + 255) & ~size_t(255);
    s.ranged = (s.zeroed + n * 8 + 255) & ~size_t(255);
    s.total = s.ranged + (size_t)s.n_ranges * s.cap * 8;
    return s;
}
// lsm_compact and lsm_compact_batch that also zero a span (per job), and build a filter in it.  *cleared: whether lsm_compact had
// a launch to zero it in.
int compact_clearing(const lsm_run_t* runs, uint32_t n_runs, uint32_t flags, const lsm_out_t* out, void* workspace, size_t workspace_bytes,
                     const ClearSpan& clear, bool* cleared, hipStream_t stream);
int compact_batch_clearing(const lsm_compact_job_t* jobs, uint32_t n_jobs, void* workspace, size_t workspace_bytes, const ClearSpan* clear, hipStream_t stream);
struct IngestJob {  // a copy of a run with its fence index; clear_n 16-byte words are zeroed along with it
    const lsm_entry_t* from;
    lsm_entry_t* to;
    uint64_t n;
    void* fences;
    uint4* clear;
    uint64_t clear_n;
};
int ingest_runs(const IngestJob* jobs, uint32_t count, uint32_t fence_stride, hipStream_t stream);
// Sum of hit_len[0 .. n_req) and number of values above zero, written to stats[0] and stats[1] (pinned host memory);
// then stats[2] = ticket.
int probe_stats(const uint32_t* hit_len, uint32_t n_req, uint64_t* stats, uint64_t ticket, hipStream_t stream);
// lsm_build_bloom_batch; `cleared`: the filters are known to be all zero.
int build_filters(const lsm_run_t* runs, void* const* filters_out, const uint64_t* n_blocks, uint32_t n_runs, bool cleared, hipStream_t stream);
// Filters of runs whose lengths are on the device: a tile status word (the last of a compaction), and no more than `most`.  A run whose
// compaction failed gets none.
struct CountedFilter {
    const lsm_entry_t* entries;
    uint64_t most;
    const uint64_t* status;
    void* filter;
    uint32_t bits;
    void* scratch;  // not null: a FilterScratch with the keys' hashes; null: a small filter, on memory that is zero
};
int build_filters_counted(const CountedFilter* filters, uint32_t count, hipStream_t stream);
// Compaction of runs whose exact lengths are only known on the device (n_upper[j] >= n_dev[j]; launch sizes come from
// the upper bounds, surplus tiles stay empty).  Needs a workspace of lsm_compact_workspace_bytes(n_upper, k) bytes.
int compact_device_lengths(const lsm_entry_t* const* ptr, const uint64_t* n_upper, const uint64_t* n_dev, uint32_t k, uint32_t flags,
                           const lsm_out_t* out, void* workspace, size_t workspace_bytes, hipStream_t stream);

}  // namespace lsm
