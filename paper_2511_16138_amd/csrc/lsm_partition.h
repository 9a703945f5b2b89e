// Sorting key hashes by where they land in a hashed structure (Bloom filter blocks, hash index buckets), so that the
// structure can be built range by range in on-chip memory instead of by read-modify-write operations on scattered
// words of HBM.  A hash's unit (filter block, index bucket) is ((h >> 32) * n_units) >> 32, which grows with the hash,
// so a range of consecutive units is a contiguous range of hash values.
//   clear     the range counters
//   count     every workgroup counts, in LDS, how many hashes of its chunk fall into each range and adds its counts to
//             the range totals (one global atomic per range and workgroup)
//   scatter   every workgroup counts its chunk again, reserves its share of each range with one returning atomic per
//             range, and copies each hash (with its position in the input, if asked) to its range's part of the
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

// kScatter = false: count.  kScatter = true: count, reserve, copy.  kWithPos: the copy of hash i is a 16-byte record
// {h, i, 0}: one store per hash (an 8-byte and a 4-byte store into two arrays took a fifth longer).
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
        const uint32_t at = atomicAdd(&count[bloom_block(h, n_units) >> unit_log], 1u);
        if (kWithPos) reinterpret_cast<uint4*>(ranged)[at] = make_uint4((uint32_t)h, (uint32_t)(h >> 32), (uint32_t)i, 0);  // one 16-byte record
        else ranged[at] = h;
    });
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
    l.total = l.ranged + up((size_t)n * (with_pos ? 16 : 8));
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
    hipLaunchKernelGGL((range_pass_kernel<true, kWithPos>), dim3(chunks), dim3(kPartThreads), 0, stream, hashes, n, l.chunk, (uint32_t)n_units, l.unit_log,
                       l.n_ranges, totals, cursors, ranged);
}

}  // namespace lsm

#endif
