// lsm_build_bloom and its forms: blocked Bloom filter of a run (paper section 2.2 names Bloom filters as the structure that
// lets a lookup skip a run; appendix B uses point lookups in "Probe").  A key sets six bits of one 16-byte block.  Bits only
// ever get set, so every way of building a filter gives the same bytes:
//   bloom_small_kernel    short runs: shares of the keys in LDS, one launch where the memory is zero or one share is all
//   bloom_insert_kernel   longer ones from the entries: one thread per key, two 64-bit atomics at most
//   bloom_fill_kernel     from the keys' hashes, sorted by range of blocks: built in LDS, written once
//   bloom_scatter_kernel, bloom_ranges_kernel   the same right behind a merge, lengths on the device, several runs per launch
#include <hip/hip_runtime.h>

#include <type_traits>

#include "lsm_common.h"
#include "lsm_partition.h"

namespace lsm {

__global__ void bloom_clear_kernel(uint4* blocks, uint64_t n_blocks) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_blocks; i += stride) blocks[i] = make_uint4(0, 0, 0, 0);
}

__global__ void bloom_insert_kernel(const lsm_entry_t* entries, uint64_t n, uint32_t* words, uint32_t n_blocks) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        uint4 mask;
        const uint32_t block = bloom_block(bloom_hash(load_key(entries + i), mask), n_blocks);
        // two 64-bit halves (little-endian: word 0 is the low half of the first)
        unsigned long long* w = reinterpret_cast<unsigned long long*>(words + (uint64_t)block * 4);
        const unsigned long long lo = ((unsigned long long)mask.y << 32) | mask.x, hi = ((unsigned long long)mask.w << 32) | mask.z;
        if (lo) atomicOr(w + 0, lo);
        if (hi) atomicOr(w + 1, hi);
    }
}

// The same two steps for up to kBloomBatch runs per launch (blockIdx.y = run), for the many small runs that a round of
// flushes into several trees produces.
constexpr uint32_t kBloomBatch = 64;
template <uint32_t kRuns>
struct BloomJobs {
    const lsm_entry_t* entries[kRuns];
    uint64_t n[kRuns];
    uint32_t* words[kRuns];
    uint32_t n_blocks[kRuns];
};

// What the kernels are told of the runs beside their jobs: nothing, or that the lengths in the jobs are upper bounds and the true
// ones are in device memory, in tile status words.
struct KnownLengths {
    __device__ __forceinline__ void look_up(uint32_t, uint64_t&, uint32_t&) const {}
};
template <uint32_t kRuns>
struct CountedLengths {
    const uint64_t* status[kRuns];
    uint32_t bits[kRuns];
    __device__ __forceinline__ void look_up(uint32_t run, uint64_t& n, uint32_t& n_blocks) const {
        const uint64_t word = *status[run], counted = word & kStValueMask;
        n = (word >> kStShift) != kStPrefix ? 0 : (counted < n ? counted : n);
        const uint32_t blocks = (uint32_t)((n * bits[run] + 127) / 128);  // as lsm_bloom_blocks
        n_blocks = blocks == 0 ? 1 : blocks;
    }
};

template <uint32_t kRuns>
__global__ void bloom_clear_batch_kernel(BloomJobs<kRuns> jobs) {
    uint4* blocks = reinterpret_cast<uint4*>(jobs.words[blockIdx.y]);
    const uint64_t n_blocks = jobs.n_blocks[blockIdx.y], stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_blocks; i += stride) blocks[i] = make_uint4(0, 0, 0, 0);
}

template <uint32_t kRuns>
__global__ void bloom_insert_batch_kernel(BloomJobs<kRuns> jobs) {
    const lsm_entry_t* entries = jobs.entries[blockIdx.y];
    uint32_t* words = jobs.words[blockIdx.y];
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t n = jobs.n[blockIdx.y];
    const uint32_t n_blocks = jobs.n_blocks[blockIdx.y];
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        uint4 mask;
        const uint32_t block = bloom_block(bloom_hash(load_key(entries + i), mask), n_blocks);
        unsigned long long* w = reinterpret_cast<unsigned long long*>(words + (uint64_t)block * 4);
        const unsigned long long lo = ((unsigned long long)mask.y << 32) | mask.x, hi = ((unsigned long long)mask.w << 32) | mask.z;
        if (lo) atomicOr(w + 0, lo);
        if (hi) atomicOr(w + 1, hi);
    }
}

// Sets the six bits of hash h in a filter block in LDS, one atomic per bit: putting them together as a mask first costs
// more vector instructions than the one or two atomics it saves.
__device__ __forceinline__ void bloom_set_lds(uint32_t* block, uint64_t h) {
    const uint64_t g = bloom_bits(h);
#pragma unroll
    for (int j = 0; j < 6; j++) {
        const uint32_t b = (uint32_t)(g >> (7 * j)) & 127;
        atomicOr(&block[b >> 5], 1u << (b & 31));
    }
}

// A filter of at most kSmallFilterBlocks blocks (128 KiB) is built in LDS, for the short runs of a tree's upper levels.
// blockIdx.y = run, blockIdx.x = a share of its keys, `ahead` keys per thread.  A run of one share is written out by its
// only workgroup; the shares of a longer one are combined by atomics in the order of the words (whole lines at a time and
// one per word, where an atomic per key goes to a line of its own: 16 x 30,000 keys took 39 us that way), on a
// filter that an earlier launch has cleared.  One workgroup for 36,000 keys took 22 us: it reads 2.3 MB.
constexpr int kBloomSmallThreads = 1024;
template <uint32_t kBlocks, int kAhead, uint32_t kRuns, typename Lengths>
__global__ void __launch_bounds__(kBloomSmallThreads) bloom_small_kernel(BloomJobs<kRuns> jobs, Lengths lengths) {
    __shared__ uint4 blocks[kBlocks];
    uint32_t* f = reinterpret_cast<uint32_t*>(blocks);
    uint64_t* words = reinterpret_cast<uint64_t*>(blocks);
    constexpr uint32_t kShare = kAhead * kBloomSmallThreads;
    const lsm_entry_t* entries = jobs.entries[blockIdx.y];
    const uint64_t first = (uint64_t)blockIdx.x * kShare;
    uint64_t n = jobs.n[blockIdx.y];
    uint32_t n_blocks = jobs.n_blocks[blockIdx.y];  // <= kBlocks (checked by the host)
    lengths.look_up(blockIdx.y, n, n_blocks);       // no more than that
    if (blockIdx.x > 0 && first >= n) return;       // a shorter run than the longest of the batch
    // all keys of a thread are read before the first is hashed
    Key key[kAhead];
#pragma unroll
    for (int a = 0; a < kAhead; a++) {
        const uint64_t i = first + threadIdx.x + (uint64_t)a * kBloomSmallThreads;
        if (i < n) key[a] = load_key(entries + i);
    }
    for (uint32_t w = threadIdx.x; w < n_blocks * 2; w += kBloomSmallThreads) words[w] = 0;
    __syncthreads();
#pragma unroll
    for (int a = 0; a < kAhead; a++) {
        if (first + threadIdx.x + (uint64_t)a * kBloomSmallThreads >= n) break;
        const uint64_t h = bloom_key_hash(key[a]);
        bloom_set_lds(f + (uint64_t)bloom_block(h, n_blocks) * 4, h);
    }
    __syncthreads();
    if (n <= kShare) {
        uint4* out = reinterpret_cast<uint4*>(jobs.words[blockIdx.y]);
        for (uint32_t b = threadIdx.x; b < n_blocks; b += kBloomSmallThreads) out[b] = blocks[b];
    } else {
        unsigned long long* out = reinterpret_cast<unsigned long long*>(jobs.words[blockIdx.y]);
        for (uint32_t w = threadIdx.x; w < n_blocks * 2; w += kBloomSmallThreads)
            if (words[w]) atomicOr(out + w, (unsigned long long)words[w]);
    }
}

// The runs of `jobs`, all with small filters; `cleared`: the filters are known to be all zero.  A thread hashes one key
// (hashing is some 800 cycles a key and wave: four per thread took 11 us where one takes 6), or two when one would be
// more than a workgroup of them for every compute unit (16 x 30,000 keys: 19 us against 22).  On memory that is not zero,
// shares are two launches, and up to kOneLaunch keys a workgroup takes a whole run: 2,500 keys 5.0 us against 7.0, 4,096 6.9
// against 7.0, 5,000 8.2 against 7.1.  Calls for many runs are bound by the host, which the second launch costs 2.5 us (one run
// of 5,000 keys 8.7 against 11.4, of 8,192 12.1 against 12.4).  Filters of runs whose lengths are on the device are built on
// cleared memory only.
template <uint32_t kRuns, typename Lengths>
static void launch_bloom_small(const BloomJobs<kRuns>& jobs, const Lengths& lengths, uint32_t count, bool cleared, hipStream_t stream) {
    constexpr int kMostAhead = !std::is_same<Lengths, KnownLengths>::value ? 2 : (kRuns == 1 ? 4 : 8);
    constexpr uint64_t kOneLaunch = (uint64_t)kMostAhead * kBloomSmallThreads;
    uint64_t most_keys = 0, all_keys = 0;
    uint32_t most_blocks = 0;
    for (uint32_t j = 0; j < count; j++) {
        most_keys = jobs.n[j] > most_keys ? jobs.n[j] : most_keys;
        most_blocks = jobs.n_blocks[j] > most_blocks ? jobs.n_blocks[j] : most_blocks;
        all_keys += jobs.n[j];
    }
    int ahead = all_keys > 256ull * kBloomSmallThreads || (most_keys > kBloomSmallThreads && most_keys <= 2 * kBloomSmallThreads) ? 2 : 1;
    if (!cleared && most_keys > 2 * kBloomSmallThreads && most_keys <= kOneLaunch) ahead = most_keys <= 4 * kBloomSmallThreads ? 4 : 8;
    const uint64_t share = ahead * (uint64_t)kBloomSmallThreads;
    const dim3 grid(most_keys ? (uint32_t)((most_keys + share - 1) / share) : 1, count), threads(kBloomSmallThreads);
    if (grid.x > 1 && !cleared) {
        if constexpr (kRuns == 1)
            hipLaunchKernelGGL(bloom_clear_kernel, dim3((most_blocks + 255) / 256), dim3(256), 0, stream, reinterpret_cast<uint4*>(jobs.words[0]), (uint64_t)most_blocks);
        else
            hipLaunchKernelGGL(bloom_clear_batch_kernel<kRuns>, dim3((most_blocks + 255) / 256, count), dim3(256), 0, stream, jobs);
    }
    auto launch = [&](auto blocks) {
        constexpr uint32_t kBlocks = decltype(blocks)::value;
        auto with = [&](auto keys) { hipLaunchKernelGGL((bloom_small_kernel<kBlocks, decltype(keys)::value, kRuns, Lengths>), grid, threads, 0, stream, jobs, lengths); };
        if (ahead == 1) with(std::integral_constant<int, 1>{});
        else if (ahead == 2) with(std::integral_constant<int, 2>{});
        else if (ahead == 4) with(std::integral_constant<int, kMostAhead < 4 ? kMostAhead : 4>{});
        else with(std::integral_constant<int, kMostAhead>{});
    };
    if (most_blocks > kSmallFilterBlocks / 2) launch(std::integral_constant<uint32_t, kSmallFilterBlocks>{});
    else launch(std::integral_constant<uint32_t, kSmallFilterBlocks / 2>{});
}

// ---------------------------------------------------------------------------------------
// Filter of a long run without global atomics.  The atomic build above is bound by the rate of read-modify-write
// operations on scattered 8-byte words (two per key); this one moves the keys' 8-byte hashes instead: they are sorted
// by ranges of consecutive filter blocks (at most 4,096 blocks = 64 KiB; the passes of lsm_partition.h), then one
// workgroup per range builds the range's part of the filter in LDS from its hashes and writes it out once.
// The order of the hashes inside a range does not matter: bits are only ever set.
// ---------------------------------------------------------------------------------------
__global__ void hash_keys_kernel(const lsm_entry_t* entries, uint64_t n, uint64_t* hashes) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) hashes[i] = bloom_key_hash(load_key(entries + i));
}

// one workgroup per range; kScan: `hashes` are all n hashes as they came (totals is not used), else they are sorted by range
template <bool kScan>
__global__ void __launch_bounds__(kPartThreads) bloom_fill_kernel(const uint64_t* hashes, uint64_t n, const uint32_t* totals, uint32_t n_blocks,
                                                                 uint32_t unit_log, uint4* filter) {
    __shared__ uint4 part[kMaxRangeUnits];
    uint32_t* f = reinterpret_cast<uint32_t*>(part);
    const uint32_t range = blockIdx.x, first_block = range << unit_log;
    const uint32_t blocks = min(1u << unit_log, n_blocks - first_block);
    for (uint32_t w = threadIdx.x; w < blocks * 4; w += kPartThreads) f[w] = 0;
    uint64_t begin = 0, end = n;
    if (!kScan) {
        begin = range_begin(totals, range);
        end = begin + totals[range];
    }
    __syncthreads();
    part_for_each(begin, end, [&](uint64_t i) { return hashes[i]; }, [&](uint64_t, uint64_t h) {
        const uint32_t block = bloom_block(h, n_blocks) - first_block;  // wraps for the blocks before the range
        if (kScan && block >= blocks) return;
        bloom_set_lds(f + block * 4, h);
    });
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < blocks; b += kPartThreads) filter[first_block + b] = part[b];
}

}  // namespace lsm

extern "C" size_t lsm_bloom_workspace_bytes(uint64_t n, uint64_t n_blocks) {
    if (!lsm::range_partition_applies(n, n_blocks)) return 0;
    return lsm::range_layout(n, n_blocks, false).total;
}

extern "C" int lsm_hash_keys(const lsm_run_t* run, uint64_t* hashes_out, void* stream_v) {
    using namespace lsm;
    if (run == nullptr) return LSM_ERR_NULL;
    if (run->n == 0) return LSM_OK;
    if (run->entries == nullptr || hashes_out == nullptr) return LSM_ERR_NULL;
    if ((reinterpret_cast<uintptr_t>(run->entries) & 63) != 0 || (reinterpret_cast<uintptr_t>(hashes_out) & 7) != 0) return LSM_ERR_BAD_ARG;
    uint64_t blocks = (run->n + 255) / 256;
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(hash_keys_kernel, dim3((uint32_t)blocks), dim3(256), 0, static_cast<hipStream_t>(stream_v), run->entries, run->n, hashes_out);
    return hipGetLastError() == hipSuccess ? LSM_OK : LSM_ERR_HIP;
}

extern "C" int lsm_build_bloom_hashed(const uint64_t* hashes, uint64_t n, void* filter_out, uint64_t n_blocks, void* workspace,
                                      size_t workspace_bytes, void* stream_v) {
    using namespace lsm;
    if (filter_out == nullptr || (n > 0 && hashes == nullptr)) return LSM_ERR_NULL;
    if (n_blocks == 0 || n_blocks >= (1ull << 32)) return LSM_ERR_BAD_ARG;
    if ((reinterpret_cast<uintptr_t>(filter_out) & 15) != 0 || (reinterpret_cast<uintptr_t>(hashes) & 7) != 0) return LSM_ERR_BAD_ARG;
    if (!range_partition_applies(n, n_blocks)) return LSM_ERR_BAD_ARG;
    const RangeLayout l = range_layout(n, n_blocks, false);
    if (workspace == nullptr || (reinterpret_cast<uintptr_t>(workspace) & 255) != 0 || workspace_bytes < l.total) return LSM_ERR_WORKSPACE;
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    launch_range_partition<false>(hashes, n, n_blocks, l, workspace, stream);
    char* base = static_cast<char*>(workspace);
    const uint32_t* totals = reinterpret_cast<const uint32_t*>(base + l.totals);
    if (l.scan)
        hipLaunchKernelGGL(bloom_fill_kernel<true>, dim3(l.n_ranges), dim3(kPartThreads), 0, stream, hashes, n, totals, (uint32_t)n_blocks, l.unit_log,
                           static_cast<uint4*>(filter_out));
    else
        hipLaunchKernelGGL(bloom_fill_kernel<false>, dim3(l.n_ranges), dim3(kPartThreads), 0, stream, reinterpret_cast<const uint64_t*>(base + l.ranged), n,
                           totals, (uint32_t)n_blocks, l.unit_log, static_cast<uint4*>(filter_out));
    return hipGetLastError() == hipSuccess ? LSM_OK : LSM_ERR_HIP;
}

extern "C" uint64_t lsm_bloom_blocks(uint64_t n, uint32_t bits_per_key) {
    if (bits_per_key == 0) return 0;
    const unsigned __int128 bits = (unsigned __int128)n * bits_per_key;
    const unsigned __int128 blocks = bits == 0 ? 1 : (bits + 127) / 128;
    return blocks >= ((unsigned __int128)1 << 32) ? 0 : (uint64_t)blocks;
}

extern "C" int lsm_build_bloom(const lsm_run_t* run, void* filter_out, uint64_t n_blocks, void* stream_v) {
    using namespace lsm;
    if (run == nullptr || filter_out == nullptr) return LSM_ERR_NULL;
    if (run->n > 0 && run->entries == nullptr) return LSM_ERR_NULL;
    if (n_blocks == 0 || n_blocks >= (1ull << 32)) return LSM_ERR_BAD_ARG;
    if ((reinterpret_cast<uintptr_t>(filter_out) & 15) != 0 || (reinterpret_cast<uintptr_t>(run->entries) & 63) != 0)
        return LSM_ERR_BAD_ARG;
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    if (n_blocks <= kSmallFilterBlocks && run->n <= kSmallFilterKeys) {
        BloomJobs<1> jobs = {};  // 28 bytes of arguments: the 1.8 KB of a batch cost the host 1 us per launch
        jobs.entries[0] = run->entries;
        jobs.n[0] = run->n;
        jobs.words[0] = static_cast<uint32_t*>(filter_out);
        jobs.n_blocks[0] = (uint32_t)n_blocks;
        launch_bloom_small(jobs, KnownLengths(), 1, false, stream);
        return hipGetLastError() == hipSuccess ? LSM_OK : LSM_ERR_HIP;
    }
    uint64_t clear_blocks = (n_blocks + 255) / 256;
    if (clear_blocks > 4096) clear_blocks = 4096;
    hipLaunchKernelGGL(bloom_clear_kernel, dim3((uint32_t)clear_blocks), dim3(256), 0, stream, static_cast<uint4*>(filter_out), n_blocks);
    if (run->n > 0) {
        uint64_t blocks = (run->n + 255) / 256;
        if (blocks > 16384) blocks = 16384;
        hipLaunchKernelGGL(bloom_insert_kernel, dim3((uint32_t)blocks), dim3(256), 0, stream, run->entries, run->n,
                           static_cast<uint32_t*>(filter_out), (uint32_t)n_blocks);
    }
    return hipGetLastError() == hipSuccess ? LSM_OK : LSM_ERR_HIP;
}

namespace lsm {
int build_filters(const lsm_run_t* runs, void* const* filters_out, const uint64_t* n_blocks, uint32_t n_runs, bool cleared, hipStream_t stream) {
    // a launch takes runs of one kind: small filters, or any
    for (int large = 0; large < 2; large++) {
        BloomJobs<kBloomBatch> jobs = {};
        uint32_t count = 0;
        uint64_t most_blocks = 1, most_entries = 0;
        for (uint32_t j = 0; j <= n_runs; j++) {
            if (count == kBloomBatch || (j == n_runs && count > 0)) {
                if (large == 0) {
                    launch_bloom_small(jobs, KnownLengths(), count, cleared, stream);
                } else {
                    uint64_t cx = (most_blocks + 255) / 256, ix = (most_entries + 255) / 256;
                    if (cx > 1024) cx = 1024;
                    if (ix > 4096) ix = 4096;
                    if (!cleared) hipLaunchKernelGGL(bloom_clear_batch_kernel<kBloomBatch>, dim3((uint32_t)cx, count), dim3(256), 0, stream, jobs);
                    if (most_entries > 0)
                        hipLaunchKernelGGL(bloom_insert_batch_kernel<kBloomBatch>, dim3((uint32_t)ix, count), dim3(256), 0, stream, jobs);
                }
                jobs = {};
                count = 0, most_blocks = 1, most_entries = 0;
            }
            if (j == n_runs) break;
            if ((n_blocks[j] > kSmallFilterBlocks || runs[j].n > kSmallFilterKeys) != (large == 1)) continue;
            jobs.entries[count] = runs[j].entries;
            jobs.n[count] = runs[j].n;
            jobs.words[count] = static_cast<uint32_t*>(filters_out[j]);
            jobs.n_blocks[count] = (uint32_t)n_blocks[j];
            most_blocks = n_blocks[j] > most_blocks ? n_blocks[j] : most_blocks;
            most_entries = runs[j].n > most_entries ? runs[j].n : most_entries;
            count++;
        }
    }
    return hipGetLastError() == hipSuccess ? LSM_OK : LSM_ERR_HIP;
}
}  // namespace lsm

// ---------------------------------------------------------------------------------------
// Filters of merged runs that are too long for one workgroup's LDS, built right behind the merge, whose output pass has written the
// keys' hashes: the hashes are sorted by range of blocks and every range is built in LDS, as in lsm_build_bloom_hashed, but the
// lengths are on the device, one launch takes several runs, and a range's part of the scratch memory has room for somewhat more hashes than
// fall into it, so that none of them has to be counted first.  The atomics of bloom_insert_batch_kernel, two per key on a line of its
// own, go to memory past the L2s: filters of 8 runs, 1M keys in all, 115 us, this 19 and 3 more in the merge; a run of 70,000 keys 11 either way, of
// 400,000 60 and 13.  (One launch in which every range's workgroup reads all hashes of its run and keeps its own:
// 39 us for the 8 runs, 21 for 70,000 keys.)
// ---------------------------------------------------------------------------------------
namespace lsm {
template <uint32_t kRuns>
struct HashedJobs {
    uint64_t most[kRuns];  // upper bounds of the lengths
    uint32_t* cursors[kRuns];
    const uint64_t* hashes[kRuns];
    uint64_t* ranged[kRuns];
    uint4* filter[kRuns];
    uint32_t unit_log[kRuns], cap[kRuns];
};

// Bound by the chain of a workgroup's steps (7 us for 10 workgroups, 11 for 130).
constexpr uint32_t kScatterItems = 8, kScatterChunk = kScatterItems * kPartThreads;
static_assert(kMostFilterRanges <= kStagedRanges, "as many as a workgroup scatters to");
template <uint32_t kRuns>
__global__ void __launch_bounds__(kPartThreads) bloom_scatter_kernel(HashedJobs<kRuns> jobs, CountedLengths<kRuns> lengths) {
    const uint32_t run = blockIdx.y, unit_log = jobs.unit_log[run];
    uint64_t n = jobs.most[run];
    uint32_t n_blocks = 1;
    lengths.look_up(run, n, n_blocks);
    const uint64_t first = (uint64_t)blockIdx.x * kScatterChunk;
    if (first >= n) return;
    staged_scatter<false, kScatterItems, true>(jobs.hashes[run], n, first, n_blocks, unit_log, ((n_blocks - 1) >> unit_log) + 1, nullptr, jobs.cap[run],
                                               jobs.cursors[run], jobs.ranged[run]);
}

// One workgroup per range.  A range with more hashes than it has room for is built from all of them.
template <uint32_t kRuns>
__global__ void __launch_bounds__(kPartThreads) bloom_ranges_kernel(HashedJobs<kRuns> jobs, CountedLengths<kRuns> lengths) {
    __shared__ uint4 part[kMaxRangeUnits];
    const uint32_t run = blockIdx.y, range = blockIdx.x, unit_log = jobs.unit_log[run], first_block = range << unit_log;
    uint64_t n = jobs.most[run];
    uint32_t n_blocks = 1;
    lengths.look_up(run, n, n_blocks);
    if (first_block >= n_blocks) return;
    const uint32_t blocks = min(1u << unit_log, n_blocks - first_block), held = n != 0 ? jobs.cursors[run][range] : 0;
    for (uint32_t b = threadIdx.x; b < blocks; b += kPartThreads) part[b] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    const bool all = held > jobs.cap[run];
    const uint64_t* const hashes = all ? jobs.hashes[run] : jobs.ranged[run] + (uint64_t)range * jobs.cap[run];
    part_for_each(0, all ? n : held, [&](uint64_t i) { return hashes[i]; }, [&](uint64_t, uint64_t h) {
        const uint32_t block = bloom_block(h, n_blocks) - first_block;  // wraps for the blocks before the range
        if (block < blocks) bloom_set_lds(reinterpret_cast<uint32_t*>(part + block), h);
    });
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < blocks; b += kPartThreads) jobs.filter[run][first_block + b] = part[b];
}

template <uint32_t kRuns>
static void launch_counted(const CountedFilter* filters, uint32_t count, hipStream_t stream) {
    // a launch takes filters of one kind: small ones, or those from hashes
    for (int large = 0; large < 2; large++) {
        BloomJobs<kRuns> jobs = {};
        HashedJobs<kRuns> hashed = {};
        CountedLengths<kRuns> lengths = {};
        uint32_t taken = 0, most_ranges = 0;
        uint64_t most = 0;
        for (uint32_t j = 0; j < count; j++) {
            const CountedFilter& f = filters[j];
            if ((f.scratch != nullptr) != (large == 1)) continue;
            const uint64_t blocks = lsm_bloom_blocks(f.most, f.bits);
            if (large == 1) {
                const FilterScratch at = filter_scratch(f.most, blocks);
                char* const base = static_cast<char*>(f.scratch);
                hashed.most[taken] = f.most;
                hashed.cursors[taken] = reinterpret_cast<uint32_t*>(base);
                hashed.hashes[taken] = reinterpret_cast<const uint64_t*>(base + at.zeroed);
                hashed.ranged[taken] = reinterpret_cast<uint64_t*>(base + at.ranged);
                hashed.filter[taken] = static_cast<uint4*>(f.filter);
                hashed.unit_log[taken] = at.unit_log;
                hashed.cap[taken] = at.cap;
                most_ranges = at.n_ranges > most_ranges ? at.n_ranges : most_ranges;
            } else {
                jobs.entries[taken] = f.entries;
                jobs.n[taken] = f.most;
                jobs.words[taken] = static_cast<uint32_t*>(f.filter);
                jobs.n_blocks[taken] = (uint32_t)blocks;
            }
            lengths.status[taken] = f.status;
            lengths.bits[taken] = f.bits;
            most = f.most > most ? f.most : most;
            taken++;
        }
        if (taken == 0) continue;
        if (large == 0) {
            launch_bloom_small(jobs, lengths, taken, true, stream);
        } else {
            hipLaunchKernelGGL(bloom_scatter_kernel<kRuns>, dim3((uint32_t)((most + kScatterChunk - 1) / kScatterChunk), taken), dim3(kPartThreads), 0, stream, hashed, lengths);
            hipLaunchKernelGGL(bloom_ranges_kernel<kRuns>, dim3(most_ranges, taken), dim3(kPartThreads), 0, stream, hashed, lengths);
        }
    }
}
int build_filters_counted(const CountedFilter* filters, uint32_t count, hipStream_t stream) {
    constexpr uint32_t kRuns = 16;  // a smaller argument block than that of a batch
    if (count == 1) launch_counted<1>(filters, 1, stream);
    else
        for (uint32_t j = 0; j < count; j += kRuns) launch_counted<kRuns>(filters + j, count - j < kRuns ? count - j : kRuns, stream);
    return hipGetLastError() == hipSuccess ? LSM_OK : LSM_ERR_HIP;
}
}  // namespace lsm

extern "C" int lsm_build_bloom_batch(const lsm_run_t* runs, void* const* filters_out, const uint64_t* n_blocks, uint32_t n_runs,
                                     void* stream_v) {
    using namespace lsm;
    if (n_runs == 0) return LSM_OK;
    if (runs == nullptr || filters_out == nullptr || n_blocks == nullptr) return LSM_ERR_NULL;
    for (uint32_t j = 0; j < n_runs; j++) {
        if (filters_out[j] == nullptr || (runs[j].n > 0 && runs[j].entries == nullptr)) return LSM_ERR_NULL;
        if (n_blocks[j] == 0 || n_blocks[j] >= (1ull << 32)) return LSM_ERR_BAD_ARG;
        if ((reinterpret_cast<uintptr_t>(filters_out[j]) & 15) != 0 || (reinterpret_cast<uintptr_t>(runs[j].entries) & 63) != 0)
            return LSM_ERR_BAD_ARG;
    }
    return build_filters(runs, filters_out, n_blocks, n_runs, false, static_cast<hipStream_t>(stream_v));
}
