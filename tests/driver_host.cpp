// The library's driver (lsm_driver.cpp) on the CPU: the calls it makes of the HIP runtime and of the library's kernels,
// answered by the checker in host memory.  What the driver decides - which runs are merged, what becomes of them when a
// call of it fails - can then be tested without a GPU, failures included.  Test infrastructure only.
//
// "Device" memory is filled with 0xAB, so that memory that was handed out but never written is seen.  Work is done when it
// is enqueued, which is one of the orders a stream allows, or, where a test asks for it, as late as one allows.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <utility>
#include <vector>

#include "lsm_common.h"
#include "lsm_index.h"

extern "C" {
uint64_t oracle_compact(const lsm_entry_t* const* runs, const uint64_t* lens, uint32_t n_runs, uint32_t flags, lsm_entry_t* out);
void oracle_build_fences(const lsm_entry_t* run, uint64_t n, uint32_t stride, uint8_t* fence_keys);
uint64_t oracle_bloom_blocks(uint64_t n, uint32_t bits_per_key);
void oracle_build_bloom(const lsm_entry_t* run, uint64_t n, uint8_t* filter, uint64_t n_blocks);
int oracle_bloom_may_contain(const uint8_t* filter, uint64_t n_blocks, const uint8_t* key);

// What a test sets and reads.  *_in: the call of that kind, counted from 1, that fails next (0 = none does).
int64_t host_malloc_in = 0;   // device memory runs out
int64_t host_kernel_in = 0;   // a kernel call is refused, nothing was launched
int64_t host_late_in = 0;     // a kernel call reports an error although its work is done
uint64_t host_mallocs = 0, host_kernels = 0;
uint64_t host_bytes = 0, host_largest = 0;  // of device memory: all that was asked for, and at once
uint32_t host_pinned_flags = ~0u;   // flags that every pinned allocation was made with
uint64_t host_dirty_filters = 0;    // filters built on memory that was promised to be zero and was not
uint64_t host_stale_words = 0;      // status words of a merge in one launch that were neither zero nor of an earlier call
uint64_t host_outside = 0;          // workspaces and scratch memory that reach beyond their block, or into each other
uint64_t host_zeroings = 0, host_whole_merges = 0, host_hashed_filters = 0;  // launches that zeroed status words, merges in one launch, filters built in scratch memory
int64_t host_slow_stats = 0;        // what a probe batch found is written when the stream is next asked or waited for, no earlier
int64_t host_slow_merges = 0;       // the same for merges and sorted write buffers; every time the stream is asked, one of them ends

void host_reset() {
    host_malloc_in = host_kernel_in = host_late_in = host_slow_stats = host_slow_merges = 0;
    host_mallocs = host_kernels = host_dirty_filters = host_bytes = host_largest = 0;
    host_stale_words = host_outside = host_zeroings = host_whole_merges = host_hashed_filters = 0;
    host_pinned_flags = ~0u;
}

// ---------------------------------------------------------------------------------------------------- HIP runtime
static std::map<char*, size_t> blocks_of_memory;
hipError_t hipMalloc(void** p, size_t bytes) {
    host_mallocs++;
    host_bytes += bytes;
    host_largest = std::max<uint64_t>(host_largest, bytes);
    if (host_malloc_in > 0 && --host_malloc_in == 0) return hipErrorOutOfMemory;
    if (bytes > size_t(1) << 32) return hipErrorOutOfMemory;  // a small device
    *p = std::aligned_alloc(256, (bytes + 255) / 256 * 256);
    std::memset(*p, 0xAB, (bytes + 255) / 256 * 256);
    blocks_of_memory[static_cast<char*>(*p)] = bytes;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    blocks_of_memory.erase(static_cast<char*>(p));
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned int flags) {
    host_pinned_flags &= flags;
    *p = std::malloc(bytes);
    return hipSuccess;
}
hipError_t hipHostFree(void* p) {
    std::free(p);
    return hipSuccess;
}
static std::deque<std::function<void()>> under_way;
static hipError_t step() {
    if (!under_way.empty()) {
        const std::function<void()> work = std::move(under_way.front());
        under_way.pop_front();
        work();
    }
    return under_way.empty() ? hipSuccess : hipErrorNotReady;
}
static hipError_t catch_up() {
    while (step() != hipSuccess) {}
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return catch_up(); }
hipError_t hipStreamQuery(hipStream_t) { return step(); }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t bytes, hipMemcpyKind, hipStream_t) {
    std::memcpy(dst, src, bytes);
    return hipSuccess;
}

// ---------------------------------------------------------------------------------------------------- kernels
static bool refused() {
    host_kernels++;
    return host_kernel_in > 0 && --host_kernel_in == 0;
}
// work of a kernel, behind what the stream still has to do
static void enqueue(int64_t slow, std::function<void()> work) {
    under_way.push_back(std::move(work));
    if (slow == 0) (void)catch_up();
}
static int done() { return host_late_in > 0 && --host_late_in == 0 ? LSM_ERR_HIP : LSM_OK; }

// Merges, one or a batch, with what the library does with the memory that the driver lends it: the workspace and a long filter's scratch memory are
// written all over, status words are zeroed by a call without an epoch, and written by a merge of one or two runs in one launch with one.
struct Lent {
    char* at;
    size_t bytes;
};
static void merge_all(const lsm_compact_job_t* jobs, uint32_t n_jobs, void* workspace, size_t workspace_bytes, const lsm::ClearSpan* clear) {
    struct Job {
        std::vector<const lsm_entry_t*> ptr;
        std::vector<uint64_t> len;
        uint64_t total = 0;
        uint32_t flags;
        lsm_out_t out;
        lsm::ClearSpan clear;
        Lent scratch{nullptr, 0};
    };
    std::vector<Job> work(n_jobs);
    bool pairs = true;
    for (uint32_t j = 0; j < n_jobs; j++) {
        Job& w = work[j];
        for (uint32_t r = 0; r < jobs[j].n_runs; r++) w.ptr.push_back(jobs[j].runs[r].entries), w.len.push_back(jobs[j].runs[r].n), w.total += jobs[j].runs[r].n;
        w.flags = jobs[j].flags, w.out = jobs[j].out;
        if (clear != nullptr) w.clear = clear[j];
        if (w.clear.filter != nullptr) w.scratch = Lent{static_cast<char*>(w.clear.p), lsm::filter_scratch(w.total, oracle_bloom_blocks(w.total, w.clear.filter_bits)).total};
        if (clear != nullptr && w.clear.bytes != 0 && w.clear.filter_bits != 0) clear[j].filter_built = true;
        pairs = pairs && jobs[j].n_runs <= 2;
    }
    const lsm::ClearSpan first = clear != nullptr ? clear[0] : lsm::ClearSpan();
    const bool zeroes = first.status != nullptr && first.epoch == 0, whole = first.status != nullptr && first.epoch != 0 && pairs;
    if (zeroes) first.status_zeroed = clear[0].status_zeroed = true;
    const Lent own{static_cast<char*>(workspace), workspace_bytes};
    enqueue(host_slow_merges, [=] {
        std::vector<Lent> lent = {own};
        if (first.status != nullptr) lent.push_back(Lent{reinterpret_cast<char*>(first.status), lsm::kShortTiles * sizeof(uint64_t)});
        for (const Job& w : work)
            if (w.scratch.bytes != 0) lent.push_back(w.scratch);
        for (size_t i = 0; i < lent.size(); i++) {
            auto block = blocks_of_memory.upper_bound(lent[i].at);
            const bool inside = block != blocks_of_memory.begin() && (--block, lent[i].at + lent[i].bytes <= block->first + block->second);
            if (!inside || reinterpret_cast<uintptr_t>(lent[i].at) % 256 != 0) host_outside++;
            for (size_t q = 0; q < i; q++)
                if (lent[i].at < lent[q].at + lent[q].bytes && lent[q].at < lent[i].at + lent[i].bytes) host_outside++;
        }
        if (zeroes) host_zeroings++, std::memset(first.status, 0, lsm::kShortTiles * sizeof(uint64_t));
        if (whole) {
            host_whole_merges++;
            for (uint64_t t = 0; t < lsm::kShortTiles; t++)
                if (first.status[t] != 0 && ((first.status[t] << 2) >> (lsm::kStEpochShift + 2)) >= first.epoch) host_stale_words++;  // unwritten memory is of a large one
            for (uint64_t t = 0; t < work.size() && t < lsm::kShortTiles; t++)
                first.status[t] = (lsm::kStPrefix << lsm::kStShift) | ((uint64_t)first.epoch << lsm::kStEpochShift) | work[t].total;
        }
        const bool ours = host_outside == 0;  // else a test has failed, and nothing is written there
        if (ours) std::memset(own.at, 0xCD, own.bytes);
        for (const Job& w : work) {
            if (ours && w.scratch.bytes != 0) std::memset(w.scratch.at, 0xCE, w.scratch.bytes);
            if (w.scratch.bytes == 0 && w.clear.bytes != 0) std::memset(w.clear.p, 0, w.clear.bytes);
            const uint64_t n = oracle_compact(w.ptr.data(), w.len.data(), (uint32_t)w.ptr.size(), w.flags, w.out.entries);
            if (w.out.fence_keys != nullptr) oracle_build_fences(w.out.entries, n, w.out.fence_stride, static_cast<uint8_t*>(w.out.fence_keys));
            if (w.clear.bytes != 0 && w.clear.filter_bits != 0) {
                host_hashed_filters += w.clear.filter != nullptr;
                uint8_t* const filter = static_cast<uint8_t*>(w.clear.filter != nullptr ? w.clear.filter : w.clear.p);
                if (n != 0) oracle_build_bloom(w.out.entries, n, filter, oracle_bloom_blocks(n, w.clear.filter_bits));
            }
            *w.out.n_out = n;
        }
    });
}

size_t lsm_compact_workspace_bytes(const uint64_t* lens, uint32_t n_runs) {
    if (n_runs > LSM_MAX_RUNS) return 0;
    size_t bytes = 1024;
    for (uint32_t r = 0; r < n_runs; r++) bytes += (lens[r] * 64 + 255) / 256 * 256;
    return bytes;
}
size_t lsm_compact_batch_workspace_bytes(const lsm_compact_job_t* jobs, uint32_t n_jobs) {
    for (uint32_t j = 0; j < n_jobs; j++)
        if (jobs[j].n_runs > LSM_MAX_RUNS) return 0;
    size_t bytes = 1024 * n_jobs;
    for (uint32_t j = 0; j < n_jobs; j++)
        for (uint32_t r = 0; r < jobs[j].n_runs; r++) bytes += (jobs[j].runs[r].n * 64 + 255) / 256 * 256;
    return bytes;
}
size_t lsm_flush_workspace_bytes(uint64_t n) { return 4 * n; }
int lsm_flush_buffer(const lsm_entry_t* buffer, uint64_t n, const lsm_out_t* out_at, void*, size_t, void*) {
    if (refused()) return LSM_ERR_HIP;
    enqueue(host_slow_merges, [=, out = *out_at] {
        std::vector<lsm_entry_t> v(buffer, buffer + n);
        std::reverse(v.begin(), v.end());
        std::stable_sort(v.begin(), v.end(), [](const lsm_entry_t& a, const lsm_entry_t& b) {
            const int c = std::memcmp(a.key, b.key, LSM_KEY_BYTES);
            return c != 0 ? c < 0 : a.seqno > b.seqno;
        });
        uint64_t m = 0;
        for (uint64_t i = 0; i < n; i++)
            if (i == 0 || std::memcmp(v[i].key, v[i - 1].key, LSM_KEY_BYTES) != 0) out.entries[m++] = v[i];
        if (out.fence_keys != nullptr) oracle_build_fences(out.entries, m, out.fence_stride, static_cast<uint8_t*>(out.fence_keys));
        *out.n_out = m;
    });
    return done();
}
int lsm_build_fences(const lsm_run_t* run, uint32_t stride, uint8_t* keys, void*) {
    if (refused()) return LSM_ERR_HIP;
    oracle_build_fences(run->entries, run->n, stride, keys);
    return done();
}
uint64_t lsm_bloom_blocks(uint64_t n, uint32_t bits_per_key) { return oracle_bloom_blocks(n, bits_per_key); }
int lsm_build_bloom(const lsm_run_t* run, void* filter, uint64_t n_blocks, void*) {
    if (refused()) return LSM_ERR_HIP;
    oracle_build_bloom(run->entries, run->n, static_cast<uint8_t*>(filter), n_blocks);
    return done();
}
size_t lsm_bloom_workspace_bytes(uint64_t, uint64_t) { return 0; }  // lsm_build_bloom is used instead
int lsm_build_bloom_hashed(const uint64_t*, uint64_t, void*, uint64_t, void*, size_t, void*) { return LSM_ERR_INTERNAL; }
int lsm_hash_keys(const lsm_run_t* run, uint64_t* hashes, void*) {
    if (refused()) return LSM_ERR_HIP;
    std::memset(hashes, 0, run->n * 8);
    return done();
}
uint64_t lsm_hash_index_buckets(uint64_t n) { return n ? (n + 3) / 4 : 1; }
size_t lsm_hash_index_workspace_bytes(uint64_t n) { return 16 * n + 256; }
int lsm_build_hash_index(const uint64_t*, uint64_t n, void* buckets, void*, size_t, void*) {  // a mark: built
    if (refused()) return LSM_ERR_HIP;
    std::memset(buckets, 0x11, lsm_hash_index_buckets(n) * 64);
    return done();
}
// A lookup believes the filters, as the kernel does: a run whose filter excludes the key is not searched.
int lsm_probe(const lsm_queries_t* q, const lsm_tree_t* tree, const lsm_hits_t* out, void*) {
    if (refused()) return LSM_ERR_HIP;
    for (uint32_t r = 0; r < q->n_req; r++) {
        lsm_hit_t* row = out->hits + (uint64_t)r * q->max_blocks;
        std::memset(row, 0, sizeof(lsm_hit_t) * q->max_blocks);
        uint32_t j = 0;
        for (; j < q->n_blocks[r]; j++) {
            const uint8_t* key = q->keys + ((uint64_t)r * q->max_blocks + j) * LSM_KEY_BYTES;
            const lsm_entry_t* found = nullptr;
            for (uint32_t i = 0; i < tree->n_runs && found == nullptr; i++) {
                const lsm_tree_run_t& t = tree->runs[i];
                if (t.bloom.n_blocks != 0 && !oracle_bloom_may_contain(static_cast<const uint8_t*>(t.bloom.blocks), t.bloom.n_blocks, key)) continue;
                for (uint64_t e = 0; e < t.run.n; e++)
                    if (std::memcmp(t.run.entries[e].key, key, LSM_KEY_BYTES) == 0) found = t.run.entries + e;
                if (found != nullptr) row[j].run_idx = i;
            }
            if (found == nullptr || found->type != LSM_PUT) {
                row[j].run_idx = 0;
                break;
            }
            row[j].vptr = found->vptr, row[j].vlen = found->vlen;
        }
        out->hit_len[r] = j;
    }
    return done();
}
}  // extern "C"

namespace lsm {
// The launch that was to zero the status words has not been made; the call had counted on it.
static int not_launched(const ClearSpan& clear) {
    clear.status_zeroed = clear.status != nullptr && clear.epoch == 0;
    return LSM_ERR_HIP;
}
int compact_clearing(const lsm_run_t* runs, uint32_t n_runs, uint32_t flags, const lsm_out_t* out, void* workspace, size_t workspace_bytes, const ClearSpan& clear,
                     bool* cleared, hipStream_t) {
    *cleared = false;
    if (n_runs > LSM_MAX_RUNS) return LSM_ERR_BAD_ARG;
    if (refused()) return not_launched(clear);
    *cleared = clear.bytes != 0;
    lsm_compact_job_t job{};
    job.runs = runs, job.n_runs = n_runs, job.flags = flags, job.out = *out;
    merge_all(&job, 1, workspace, workspace_bytes, &clear);
    return done();
}
int compact_batch_clearing(const lsm_compact_job_t* jobs, uint32_t n_jobs, void* workspace, size_t workspace_bytes, const ClearSpan* clear, hipStream_t) {
    for (uint32_t j = 0; j < n_jobs; j++)
        if (jobs[j].n_runs > LSM_MAX_RUNS) return LSM_ERR_BAD_ARG;
    if (refused()) return clear != nullptr ? not_launched(clear[0]) : (int)LSM_ERR_HIP;
    merge_all(jobs, n_jobs, workspace, workspace_bytes, clear);
    return done();
}
int ingest_runs(const IngestJob* jobs, uint32_t count, uint32_t fence_stride, hipStream_t) {
    if (refused()) return LSM_ERR_HIP;
    for (uint32_t j = 0; j < count; j++) {
        std::memcpy(jobs[j].to, jobs[j].from, jobs[j].n * sizeof(lsm_entry_t));
        oracle_build_fences(jobs[j].to, jobs[j].n, fence_stride, static_cast<uint8_t*>(jobs[j].fences));
        if (jobs[j].clear_n != 0) std::memset(jobs[j].clear, 0, jobs[j].clear_n * 16);
    }
    return done();
}
int build_filters(const lsm_run_t* runs, void* const* filters, const uint64_t* n_blocks, uint32_t n_runs, bool cleared, hipStream_t) {
    if (refused()) return LSM_ERR_HIP;
    for (uint32_t j = 0; j < n_runs; j++) {
        const uint8_t* f = static_cast<const uint8_t*>(filters[j]);
        if (cleared && std::any_of(f, f + 16 * n_blocks[j], [](uint8_t b) { return b != 0; })) host_dirty_filters++;
        oracle_build_bloom(runs[j].entries, runs[j].n, static_cast<uint8_t*>(filters[j]), n_blocks[j]);
    }
    return done();
}
int probe_stats(const uint32_t* hit_len, uint32_t n_req, uint64_t* stats, uint64_t ticket, hipStream_t) {
    if (refused()) return LSM_ERR_HIP;
    uint64_t blocks = 0, hits = 0;
    for (uint32_t i = 0; i < n_req; i++) blocks += hit_len[i], hits += hit_len[i] > 0;
    enqueue(host_slow_stats, [=] { stats[0] = blocks, stats[1] = hits, stats[2] = ticket; });
    return done();
}
}  // namespace lsm
