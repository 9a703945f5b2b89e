// Sorting key hashes by where they land in a hashed structure (Bloom filter blocks, hash index buckets), so that the
// structure can be built range by range in on-chip memory instead of by read-modify-write operations on scattered
// words of HBM.  A hash's unit (filter block, index bucket) is ((h >> 32) * n_units) >> 32, which grows with the hash,
// so a range of consecutive units is a contiguous range of hash values.
//   clear     the range counters
//   count     every workgroup counts, in LDS, how many hashes of its chunk fall into each range and adds its counts to
//             the range totals (one global atomic per range and workgroup)
//   scatter   every workgroup counts its chunk again, reserves its share of each range with one returning atomic per
//             range, and copies each hash (or its position and what an index needs of it) to its range's part of the
//             workspace; where a range starts it adds up from the totals itself
// The order of the hashes inside a range is not defined.  Ranges and chunks are sized by the input, so that a few
// million hashes are work for the whole chip too: with 4,096 units per range and 65,536 hashes per workgroup throughout,
// 2.7M hashes were 42 workgroups and 83 ranges, 143 us for a filter and 138 us for an index.
// Up to kScanHashes hashes are not sorted at all: the workgroup of a range reads all of them (see the fill kernels).
#ifndef LSM_PARTITION_H
#define LSM_PARTITION_H

#include <hip/hip_runtime.h>

#include "lsm_common.h"

namespace lsm {

constexpr uint32_t kMaxRangeUnits = 4096;  // units (filter blocks, index buckets) per range
constexpr uint32_t kMinRangeUnits = 256;
constexpr uint32_t kMaxRanges = 8192;     // range counters of a workgroup (32 KiB of LDS)
constexpr uint32_t kMaxChunk = 65536;     // hashes per workgroup of the count and scatter passes
constexpr uint32_t kMinChunk = 4096;
constexpr uint64_t kScanHashes = 65536;   // 64 per thread of a range's workgroup: some 5 us, where four launches take 20
constexpr int kPartThreads = 1024;
constexpr int kPartAhead = 4;             // hashes a thread reads before it handles the first

// Units per range: a power of two that gives a range to most of the 256 compute units if there are enough units.
__host__ __device__ inline uint32_t range_units(uint64_t n_units) {
    uint32_t u = kMaxRangeUnits;
    while (u > kMinRangeUnits && (n_units + u - 1) / u < 192) u >>= 1;
    return u;
}

static __global__ void range_clear_kernel(uint32_t* counters, uint32_t count) {
    for (uint32_t b = blockIdx.x * blockDim.x + threadIdx.x; b < count; b += gridDim.x * blockDim.x) counters[b] = 0;
}

// f(i) for this thread's share of [first, last), kPartAhead values at a time: `load` fetches, `use` handles.
template <typename Load, typename Use>
__device__ __forceinline__ void part_for_each(uint64_t first, uint64_t last, Load load, Use use) {
    for (uint64_t i0 = first + threadIdx.x; i0 < last; i0 += (uint64_t)kPartAhead * kPartThreads) {
        decltype(load(i0)) v[kPartAhead];
#pragma unroll
        for (int a = 0; a < kPartAhead; a++) {
            const uint64_t i = i0 + (uint64_t)a * kPartThreads;
            v[a] = load(i < last ? i : i0);
        }
#pragma unroll
        for (int a = 0; a < kPartAhead; a++) {
            const uint64_t i = i0 + (uint64_t)a * kPartThreads;
            if (i < last) use(i, v[a]);
        }
    }
}

// Sum of totals[0 .. range), by the whole workgroup.
__device__ __forceinline__ uint32_t range_begin(const uint32_t* totals, uint32_t range) {
    __shared__ uint32_t wave_sum[kPartThreads / kWave];
    uint32_t v = 0;
    for (uint32_t r = threadIdx.x; r < range; r += kPartThreads) v += totals[r];
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    if ((threadIdx.x & (kWave - 1)) == 0) wave_sum[threadIdx.x / kWave] = v;
    __syncthreads();
    v = 0;
    for (int w = 0; w < kPartThreads / kWave; w++) v += wave_sum[w];
    return v;
}

// What is copied for hash i: the hash, or (kWithPos) what an index is built from, in as many bytes: position, unit inside the range, and
// the hash's low 15 bits.
constexpr int kPosTagBits = 15;
static_assert(kMaxRangeUnits <= 1u << (32 - kPosTagBits), "unit and tag in 32 bits");
__device__ __forceinline__ uint64_t pos_record(uint64_t h, uint32_t i, uint32_t unit_in_range) {
    return ((uint64_t)i << 32) | (unit_in_range << kPosTagBits) | ((uint32_t)h & ((1u << kPosTagBits) - 1));
}

// kScatter = false: count.  kScatter = true: count, reserve, copy.
template <bool kScatter, bool kWithPos>
__global__ void __launch_bounds__(kPartThreads) range_pass_kernel(const uint64_t* hashes, uint64_t n, uint32_t chunk, uint32_t n_units, uint32_t unit_log,
                                                                 uint32_t n_ranges, uint32_t* totals, uint32_t* cursors, uint64_t* ranged) {
    __shared__ uint32_t count[kMaxRanges];
    const uint64_t first = (uint64_t)blockIdx.x * chunk;
    const uint64_t last = first + chunk < n ? first + chunk : n;
    for (uint32_t b = threadIdx.x; b < n_ranges; b += kPartThreads) count[b] = 0;
    __syncthreads();
    auto load = [&](uint64_t i) { return hashes[i]; };
    part_for_each(first, last, load, [&](uint64_t, uint64_t h) { atomicAdd(&count[bloom_block(h, n_units) >> unit_log], 1u); });
    __syncthreads();
    if (!kScatter) {
        for (uint32_t b = threadIdx.x; b < n_ranges; b += kPartThreads)
            if (count[b]) atomicAdd(&totals[b], count[b]);
        return;
    }
    // where every range starts: exclusive prefix sum over the totals, a few consecutive ranges per thread
    __shared__ uint32_t wave_sum[kPartThreads / kWave];
    const uint32_t per = (n_ranges + kPartThreads - 1) / kPartThreads, r0 = threadIdx.x * per, r1 = min(n_ranges, r0 + per);
    uint32_t mine = 0;
    for (uint32_t r = r0; r < r1; r++) mine += totals[r];
    uint32_t incl = mine;
    const int lane = threadIdx.x & (kWave - 1);
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t o = __shfl_up(incl, off, kWave);
        if (lane >= off) incl += o;
    }
    if (lane == kWave - 1) wave_sum[threadIdx.x / kWave] = incl;
    __syncthreads();
    uint32_t before = incl - mine;
    for (uint32_t w = 0; w < threadIdx.x / kWave; w++) before += wave_sum[w];
    // count[r] becomes where this workgroup's next hash of range r goes (the workspace holds fewer than 2^32 hashes)
    for (uint32_t r = r0; r < r1; r++) {
        const uint32_t c = count[r];
        if (c) count[r] = before + atomicAdd(&cursors[r], c);
        before += totals[r];
    }
    __syncthreads();
    part_for_each(first, last, load, [&](uint64_t i, uint64_t h) {
        const uint32_t unit = bloom_block(h, n_units), at = atomicAdd(&count[unit >> unit_log], 1u);
        ranged[at] = kWithPos ? pos_record(h, (uint32_t)i, unit & ((1u << unit_log) - 1)) : h;
    });
}

// The same scatter for up to kStagedRanges ranges: a workgroup takes kItems hashes per thread, reads them once, keeps them in registers, puts
// them in order of their ranges in LDS, reserves its place in every range with one atomic, and stores them from there, neighbours next to each
// other, where the pass above stores them one by one all over the workspace.  Bound by a workgroup's chain (load 2 us, count, reserve 4, store) and the
// stores.  2.7M hashes 24.7 -> 16.4 us, with positions 25.5 -> 17.2; whole filter / index of 1M keys 27.8 -> 23.5 / 31.7 -> 26.0 us, 4M 55.0 -> 43.4 /
// 92.8 -> 60.6, 16M 182 -> 117 / 433 -> 236.
// kCapped: no totals are known, a range's part of `ranged` has room for `cap` hashes and what does not fit is left out (its cursor counts it all the same).
constexpr uint32_t kStagedRanges = 1024;
template <bool kWithPos, int kItems, bool kCapped>
__device__ __forceinline__ void staged_scatter(const uint64_t* hashes, const uint64_t n, const uint64_t first, const uint32_t n_units, const uint32_t unit_log,
                                               const uint32_t n_ranges, const uint32_t* totals, const uint32_t cap, uint32_t* cursors, uint64_t* ranged) {
    constexpr uint32_t kChunk = kItems * kPartThreads;
    __shared__ uint64_t stage[kChunk];
    __shared__ uint16_t range_of[kWithPos ? kChunk : 1];
    __shared__ uint32_t start[kStagedRanges], place[kStagedRanges];
    __shared__ uint32_t wave_sum[2][kPartThreads / kWave];
    static_assert(kStagedRanges <= kPartThreads && kChunk <= 65536, "a range per thread, places in 16 bits");
    const uint32_t tid = threadIdx.x, count = n - first < kChunk ? (uint32_t)(n - first) : kChunk;
    uint64_t h[kItems];
#pragma unroll
    for (int a = 0; a < kItems; a++) h[a] = tid + a * kPartThreads < count ? hashes[first + tid + a * kPartThreads] : 0;
    const uint32_t all = !kCapped && tid < n_ranges ? totals[tid] : 0;
    if (tid < kStagedRanges) start[tid] = 0;
    __syncthreads();
    uint32_t at[kItems];  // range << 16 | place among the workgroup's hashes of the range
#pragma unroll
    for (int a = 0; a < kItems; a++) {
        const uint32_t unit = bloom_block(h[a], n_units), r = unit >> unit_log;
        at[a] = r << 16;
        if (tid + a * kPartThreads < count) at[a] |= atomicAdd(&start[r], 1u);
        if (kWithPos) h[a] = pos_record(h[a], (uint32_t)(first + tid + a * kPartThreads), unit & ((1u << unit_log) - 1));
    }
    __syncthreads();
    const uint32_t mine = tid < n_ranges ? start[tid] : 0;
    uint32_t reserved = 0;
    if (mine != 0) reserved = atomicAdd(&cursors[tid], mine);
    const uint32_t incl = wave_scan_u32(mine), all_incl = kCapped ? 0 : wave_scan_u32(all);
    if ((tid & (kWave - 1)) == kWave - 1) wave_sum[0][tid / kWave] = incl, wave_sum[1][tid / kWave] = all_incl;
    __syncthreads();
    uint32_t before = incl - mine, all_before = all_incl - all;
    for (uint32_t w = 0; w < tid / kWave; w++) {
        before += wave_sum[0][w];
        if (!kCapped) all_before += wave_sum[1][w];
    }
    if (tid < n_ranges) start[tid] = before, place[tid] = all_before + reserved;
    __syncthreads();
#pragma unroll
    for (int a = 0; a < kItems; a++) {
        if (tid + a * kPartThreads >= count) continue;
        const uint32_t r = at[a] >> 16, to = start[r] + (at[a] & 0xFFFF);
        stage[to] = h[a];
        if (kWithPos) range_of[to] = (uint16_t)r;
    }
    __syncthreads();
    for (uint32_t i = tid; i < count; i += kPartThreads) {
        const uint64_t v = stage[i];
        const uint32_t r = kWithPos ? range_of[i] : bloom_block(v, n_units) >> unit_log, to = place[r] + (i - start[r]);
        if (!kCapped) ranged[to] = v;
        else if (to < cap) ranged[(uint64_t)r * cap + to] = v;
    }
}
template <bool kWithPos, int kItems>
__global__ void __launch_bounds__(kPartThreads) range_staged_kernel(const uint64_t* hashes, uint64_t n, uint32_t n_units, uint32_t unit_log, uint32_t n_ranges,
                                                                   const uint32_t* totals, uint32_t* cursors, uint64_t* ranged) {
    staged_scatter<kWithPos, kItems, false>(hashes, n, (uint64_t)blockIdx.x * (kItems * kPartThreads), n_units, unit_log, n_ranges, totals, 0, cursors, ranged);
}

// Workspace of a partition of n hashes into n_ranges ranges: totals, cursors, the hashes (or records) by range.
struct RangeLayout {
    uint32_t n_ranges, unit_log, chunk;
    bool scan;  // not sorted: the fill kernel reads the hashes themselves
    size_t totals, cursors, ranged, total;
};
inline RangeLayout range_layout(uint64_t n, uint64_t n_units, bool with_pos) {
    auto up = [](size_t x) { return (x + 255) & ~size_t(255); };
    RangeLayout l;
    const uint32_t units = range_units(n_units);
    l.unit_log = 31 - __builtin_clz(units);
    l.n_ranges = (uint32_t)((n_units + units - 1) / units);
    l.scan = n <= kScanHashes && l.n_ranges <= 1024;
    const uint64_t even = ((n + 255) / 256 + kPartThreads - 1) / kPartThreads * kPartThreads;  // a chunk for every compute unit
    l.chunk = (uint32_t)(even < kMinChunk ? kMinChunk : (even > kMaxChunk ? kMaxChunk : even));
    l.totals = 0;
    l.cursors = l.totals + up((size_t)l.n_ranges * 4);
    l.ranged = l.cursors + up((size_t)l.n_ranges * 4);
    l.total = l.ranged + up((size_t)n * (with_pos ? 16 : 8));  // 16: what callers have been told; the records of an index take half of it
    return l;
}
inline bool range_partition_applies(uint64_t n, uint64_t n_units) {
    return n_units > 0 && n < (1ull << 32) && (n_units + kMaxRangeUnits - 1) / kMaxRangeUnits <= kMaxRanges;
}

// Enqueues the passes (none for hashes that are not sorted).  `workspace` is laid out by range_layout.
template <bool kWithPos>
inline void launch_range_partition(const uint64_t* hashes, uint64_t n, uint64_t n_units, const RangeLayout& l, void* workspace, hipStream_t stream) {
    if (l.scan) return;
    char* base = static_cast<char*>(workspace);
    uint32_t* totals = reinterpret_cast<uint32_t*>(base + l.totals);
    uint32_t* cursors = reinterpret_cast<uint32_t*>(base + l.cursors);
    uint64_t* ranged = reinterpret_cast<uint64_t*>(base + l.ranged);
    const uint32_t chunks = (uint32_t)((n + l.chunk - 1) / l.chunk);
    const uint32_t counters = (uint32_t)((l.ranged - l.totals) / 4);
    hipLaunchKernelGGL(range_clear_kernel, dim3((counters + 255) / 256), dim3(256), 0, stream, totals, counters);
    if (chunks == 0) return;
    hipLaunchKernelGGL((range_pass_kernel<false, kWithPos>), dim3(chunks), dim3(kPartThreads), 0, stream, hashes, n, l.chunk, (uint32_t)n_units, l.unit_log,
                       l.n_ranges, totals, cursors, ranged);
    if (l.n_ranges <= kStagedRanges) {
        constexpr int kItems = kWithPos ? 6 : 8;  // two workgroups on a compute unit
        hipLaunchKernelGGL((range_staged_kernel<kWithPos, kItems>), dim3((uint32_t)((n + kItems * kPartThreads - 1) / (kItems * kPartThreads))), dim3(kPartThreads), 0,
                           stream, hashes, n, (uint32_t)n_units, l.unit_log, l.n_ranges, totals, cursors, ranged);
        return;
    }
    hipLaunchKernelGGL((range_pass_kernel<true, kWithPos>), dim3(chunks), dim3(kPartThreads), 0, stream, hashes, n, l.chunk, (uint32_t)n_units, l.unit_log,
                       l.n_ranges, totals, cursors, ranged);
}

}  // namespace lsm

#endif
