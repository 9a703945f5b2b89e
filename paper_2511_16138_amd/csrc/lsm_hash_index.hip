// lsm_build_hash_index: hash index of a run.  Paper section 2.2 has a point lookup go through a Bloom filter and the
// in-memory fence pointers of a run; with the run in HBM the fence search is a dozen dependent reads.  This index
// answers "can the key be in this run, and where" with one 16-byte read (the tags of the key's bucket) and finds
// the entry with one more read of the same 64-byte line: it does the work of the filter (a key whose tag is not in
// its bucket is not in the run) and of the fence search.
//
// Format (also in the header, at lsm_hash_index_t): ceil(n / 4) buckets of 64 bytes with eight slots; a key with filter
// hash h belongs to bucket ((h >> 32) * n_buckets) >> 32 and has the 15-bit tag h & 0x7FFF.  Bytes 0..15 of a bucket
// are the slots' tag fields (16 bits each), bytes 16..47 the slots' positions in the run (32 bits each, all ones = empty
// slot), the rest is zero.  A bucket that more than eight keys fall into holds eight of them and has bit 15 of its
// first tag field set, which sends a lookup that finds nothing among the eight to the fence index.
//
// Build: the hashes and their positions are sorted by ranges of at most 4,096 buckets (lsm_partition.h); a workgroup per
// 1,024 buckets of a range hands out their slots with counters in LDS, assembles the buckets there, and writes every byte of
// them exactly once.
// Which keys of a crowded bucket are kept, and the order of the slots in a bucket, depend on the order the
// workgroup happens to see the hashes in: lookups give the same answers for every such table.
#include <hip/hip_runtime.h>

#include "lsm_common.h"
#include "lsm_partition.h"

namespace lsm {

// A workgroup per 1,024 buckets (64 KiB) of a range (blockIdx.y: which): they are assembled in LDS and leave with
// contiguous 16-byte stores: scattered 2- and 4-byte stores straight into the table cost 4.6 bytes of HBM writes per byte
// of table.  Every part reads the records of the whole range (they
// stay in the caches); records of 8 bytes instead of 16, 2.7M keys 22.5 -> 16.0 us.  kScan: the hashes are not sorted
// (`hashes` are all n of them, totals is not used), and the range picks its own.
constexpr uint32_t kFillBuckets = 1024;
template <bool kScan>
__global__ void __launch_bounds__(kPartThreads) index_fill_kernel(const uint64_t* hashes, const uint64_t* ranged, uint64_t n, const uint32_t* totals,
                                                                 uint32_t n_buckets, uint32_t unit_log, uint4* table) {
    __shared__ uint4 part[kFillBuckets * 4];  // the buckets of this pass
    __shared__ uint32_t count[kFillBuckets];
    const uint32_t range_first = blockIdx.x << unit_log, range_last = min(n_buckets, range_first + (1u << unit_log));
    uint64_t begin = 0, end = n;
    if (!kScan) {
        begin = range_begin(totals, blockIdx.x);
        end = begin + totals[blockIdx.x];
    }
    const uint32_t first_bucket = range_first + blockIdx.y * kFillBuckets;
    if (first_bucket >= range_last) return;
    const uint32_t buckets = min(range_last - first_bucket, kFillBuckets);
    // every bucket starts empty: tag fields 0, positions all ones, the rest 0
    for (uint32_t i = threadIdx.x; i < buckets * 4; i += kPartThreads) {
        const uint32_t fill = ((i & 3) == 1 || (i & 3) == 2) ? kIndexNoEntry : 0u;
        part[i] = make_uint4(fill, fill, fill, fill);
    }
    for (uint32_t b = threadIdx.x; b < buckets; b += kPartThreads) count[b] = 0;
    __syncthreads();
    uint16_t* tags = reinterpret_cast<uint16_t*>(part);
    uint32_t* words = reinterpret_cast<uint32_t*>(part);
    auto put = [&](uint32_t bucket, uint32_t tag, uint32_t position) {
        const uint32_t b = bucket - first_bucket;  // wraps for the buckets before these
        if (b >= buckets) return;
        const uint32_t k = atomicAdd(&count[b], 1u);
        if (k >= kIndexSlots) return;  // a crowded bucket keeps the first eight keys that arrive
        tags[b * 32 + k] = (uint16_t)tag;
        words[b * 16 + 4 + k] = position;
    };
    static_assert(kIndexTagMask == (1u << kPosTagBits) - 1, "a record holds the tag");
    if (kScan)
        part_for_each(begin, end, [&](uint64_t i) { return hashes[i]; },
                      [&](uint64_t i, uint64_t h) { put(bloom_block(h, n_buckets), (uint32_t)h & kIndexTagMask, (uint32_t)i); });
    else
        part_for_each(begin, end, [&](uint64_t i) { return ranged[i]; },
                      [&](uint64_t, uint64_t rec) { put(range_first + ((uint32_t)rec >> kPosTagBits), (uint32_t)rec & kIndexTagMask, (uint32_t)(rec >> 32)); });
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < buckets; b += kPartThreads)
        if (count[b] > kIndexSlots) tags[b * 32] |= 0x8000u;  // crowded
    __syncthreads();
    uint4* dst = table + (uint64_t)first_bucket * 4;
    for (uint32_t i = threadIdx.x; i < buckets * 4; i += kPartThreads) dst[i] = part[i];
}

}  // namespace lsm

extern "C" uint64_t lsm_hash_index_buckets(uint64_t n) { return lsm::index_buckets(n); }

extern "C" size_t lsm_hash_index_workspace_bytes(uint64_t n) {
    if (n >= 0xFFFFFFFFull || !lsm::range_partition_applies(n, lsm::index_buckets(n))) return 0;
    return lsm::range_layout(n, lsm::index_buckets(n), true).total;
}

extern "C" int lsm_build_hash_index(const uint64_t* hashes, uint64_t n, void* table_out, void* workspace, size_t workspace_bytes,
                                    void* stream_v) {
    using namespace lsm;
    if (table_out == nullptr || (n > 0 && hashes == nullptr)) return LSM_ERR_NULL;
    if ((reinterpret_cast<uintptr_t>(table_out) & 63) != 0 || (reinterpret_cast<uintptr_t>(hashes) & 7) != 0) return LSM_ERR_BAD_ARG;
    const uint64_t n_buckets = index_buckets(n);
    if (n >= 0xFFFFFFFFull || !range_partition_applies(n, n_buckets)) return LSM_ERR_BAD_ARG;  // positions are 32-bit, all ones = no entry
    const RangeLayout l = range_layout(n, n_buckets, true);
    if (workspace == nullptr || (reinterpret_cast<uintptr_t>(workspace) & 255) != 0 || workspace_bytes < l.total) return LSM_ERR_WORKSPACE;
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    launch_range_partition<true>(hashes, n, n_buckets, l, workspace, stream);
    char* base = static_cast<char*>(workspace);
    const uint64_t* ranged = reinterpret_cast<const uint64_t*>(base + l.ranged);
    const uint32_t* totals = reinterpret_cast<const uint32_t*>(base + l.totals);
    const uint32_t parts = ((1u << l.unit_log) + kFillBuckets - 1) / kFillBuckets;
    if (l.scan)
        hipLaunchKernelGGL(index_fill_kernel<true>, dim3(l.n_ranges, parts), dim3(kPartThreads), 0, stream, hashes, ranged, n, totals, (uint32_t)n_buckets, l.unit_log,
                           static_cast<uint4*>(table_out));
    else
        hipLaunchKernelGGL(index_fill_kernel<false>, dim3(l.n_ranges, parts), dim3(kPartThreads), 0, stream, hashes, ranged, n, totals, (uint32_t)n_buckets,
                           l.unit_log, static_cast<uint4*>(table_out));
    return hipGetLastError() == hipSuccess ? LSM_OK : LSM_ERR_HIP;
}
