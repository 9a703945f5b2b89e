// lsm_driver_*: the host driver of one tree.  Level bookkeeping of section 2.2 (a flushed run enters level 1; a level
// that holds more than K runs is merged; a merged run larger than M * T^level moves down), the controller of section
// 3.3 (operation counts over a sliding window, a new (T, K) search when the mix has moved by more than a threshold)
// and the lazy transition of appendix C (a level takes the current T and K when a run next arrives at it).  Nothing
// here touches entries: merging, fence indices, filters, hash indices, lookups and the cost model are the library's
// own entry points, and all of their work is enqueued on the caller's stream.
//
// A flush is a chain of small kernels whose lengths the host has to learn one by one (it decides by the number of entries a
// merge left), so what counts is the number of launches and how the host learns a count.  It watches the word in pinned
// memory that the merge writes: launch to count is 6 us where a stream synchronisation takes 11 (it enqueues a marker and
// waits for that).  A merge of two runs is one launch, on status words that the driver keeps.  A merge zeroes the memory of the filter on
// the way (a long filter's is built from the keys' hashes, which the merge writes), so that the filter is one launch; where
// the merged run is certain to stay at its level, whatever its length, that launch follows the merge at once and finds the
// length on the device, so that the GPU works on while the host sees the count and sets out on the next flush (96 flushes 3.06 -> 2.71 ms).
// A flushed run that comes to rest is copied, fenced and has its filter zeroed in one launch.  (With the filters on a second stream, every cascade waited for that stream before
// memory could go back to the pool, and the single workgroup that built a filter took 22 us beside a merge of 19:
// 59 us a flush.)
//
// Device memory of the runs the driver creates comes from a pool that keeps every block for reuse (hipMalloc and
// hipFree cost more than a small compaction, and hipFree waits for the device).  A block that is given back may still
// be read by work already enqueued on the caller's stream; that is safe because its next user's work is enqueued later
// on the same stream.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>
#include <cstring>
#include <deque>
#include <map>
#include <new>
#include <unordered_map>
#include <utility>
#include <vector>

#include "lsm_common.h"
#include "lsm_index.h"

namespace {

class DevicePool {
public:
    void* take(size_t bytes) {
        const size_t c = size_class(bytes);
        std::vector<void*>& idle = idle_[c];
        if (!idle.empty()) {
            void* p = idle.back();
            idle.pop_back();
            return p;
        }
        void* p = nullptr;
        if (hipMalloc(&p, c) != hipSuccess) return nullptr;
        size_of_[p] = c;
        return p;
    }
    void give(const void* p) {
        if (p == nullptr) return;
        auto it = size_of_.find(const_cast<void*>(p));
        if (it != size_of_.end()) idle_[it->second].push_back(it->first);
    }
    void free_all() {  // the caller has waited for the stream
        for (auto& kv : size_of_) (void)hipFree(kv.first);
        size_of_.clear();
        idle_.clear();
    }

private:
    // four classes per power of two from 256 bytes up: at most a quarter of a block is unused
    static size_t size_class(size_t bytes) {
        if (bytes > (size_t(1) << 60)) return bytes;  // no such allocation succeeds; keeps the loop below finite
        for (size_t s = 256;; s *= 2)
            for (size_t j = 0; j < 4; j++)
                if (s / 4 * (4 + j) >= bytes) return s / 4 * (4 + j);
    }
    std::map<size_t, std::vector<void*>> idle_;
    std::unordered_map<void*, size_t> size_of_;
};

struct Run {
    const lsm_entry_t* entries = nullptr;
    uint64_t n = 0;
    bool owned = false;      // entries came from the pool
    bool transient = false;  // entries belong to the caller of a flush: copied if the run comes to rest
    uint8_t* fences = nullptr;
    void* bloom = nullptr;
    uint64_t n_blocks = 0;     // 0: bloom is memory for a filter at most
    bool bloom_clear = false;  // bloom is memory that has been zeroed, not a filter yet
    void* index = nullptr;
    uint64_t n_buckets = 0;
    bool settled = false;  // has every lookup structure it is to get (see settle_all)
};

struct Level {
    std::vector<Run> runs;  // newest first
    uint32_t T, K;
};

struct Batch {
    uint64_t writes, hits, empties;
    double blocks;
};

uint64_t ceil_div(uint64_t a, uint64_t b) { return (a + b - 1) / b; }

constexpr uint64_t kCountUnset = UINT64_MAX - 1;  // a count word that no kernel has written yet (UINT64_MAX reports a failed merge)
// Runs of at least this many entries get their filter from the keys' hashes, sorted by block range.
constexpr uint64_t kHashedFilterEntries = 1ull << 20;

void cpu_pause() {
#if defined(__x86_64__)
    __builtin_ia32_pause();
#endif
}

}  // namespace

struct lsm_driver {
    lsm_driver_config_t cfg;
    hipStream_t stream = nullptr;  // the caller's
    double p = 1.0;
    uint32_t T = 0, K = 0;  // what the controller asks for now
    std::vector<Level> levels;
    std::vector<lsm_driver_event_t> log;
    std::deque<Batch> window;
    Batch sum{0, 0, 0, 0.0};
    bool searched = false;
    double last_mix[4] = {0, 0, 0, 0};
    DevicePool pool;
    // Memory of one compaction after the other: status words for merges in one launch (see lsm::ClearSpan), the compaction's workspace, scratch
    // memory for filters.
    struct Workspace {
        char* p = nullptr;
        size_t bytes = 0;
        uint32_t epoch = 0;  // of the next merge; 0: the status words are not zero yet
    };
    Workspace workspace, batch_workspace;  // of compactions on their own, and of batches (lsm_driver_flush_many)
    uint64_t* n_host = nullptr;  // pinned: the kernels write a compaction's count here
    uint64_t* stats_host = nullptr;  // pinned: what a probe batch found, and a ticket that says which batch
    uint64_t tickets = 0;
    uint64_t* counts_host = nullptr;  // pinned: the counts of a batch of compactions (lsm_driver_flush_many)
    size_t counts_host_count = 0;

    void record(uint32_t kind, uint32_t level, uint32_t a, uint32_t b, uint64_t n_in, uint64_t n_out) {
        lsm_driver_event_t e;
        std::memset(&e, 0, sizeof(e));
        e.kind = kind, e.level = level, e.a = a, e.b = b, e.n_in = n_in, e.n_out = n_out;
        log.push_back(e);
    }

    void drop(Run& r) {
        if (r.owned) pool.give(r.entries);
        pool.give(r.fences);
        pool.give(r.bloom);
        pool.give(r.index);
        r = Run();
    }

    void ensure_level(uint32_t level) {  // 0-based
        while (levels.size() <= level) levels.push_back(Level{{}, T, K});
    }

    uint64_t total_entries() const {
        uint64_t n = 0;
        for (const Level& lv : levels)
            for (const Run& r : lv.runs) n += r.n;
        return n;
    }

    // M * T^(level + 1), saturating
    uint64_t capacity(uint32_t level) const {
        unsigned __int128 c = cfg.buffer_entries;
        for (uint32_t i = 0; i <= level; i++) {
            c *= levels[level].T;
            if (c > UINT64_MAX) return UINT64_MAX;
        }
        return (uint64_t)c;
    }

    int wait() { return hipStreamSynchronize(stream) == hipSuccess ? LSM_OK : LSM_ERR_HIP; }

    // Waits until a kernel of the stream has made ready(*word) true.  The stream is asked now and then, so that an error
    // there ends the wait.
    template <typename Ready>
    int watch(const uint64_t* word, Ready ready) {
        const volatile uint64_t* w = word;
        for (uint32_t spins = 1; !ready(*w); spins++) {
            cpu_pause();
            if (spins % 16384 != 0) continue;
            const hipError_t e = hipStreamQuery(stream);
            if (e == hipErrorNotReady) {
                (void)hipGetLastError();  // not an error of the next launch
                continue;
            }
            if (e != hipSuccess || !ready(*w)) return LSM_ERR_HIP;
        }
        std::atomic_thread_fence(std::memory_order_acquire);
        return LSM_OK;
    }
    int watch_count(const uint64_t* word) {
        return watch(word, [](uint64_t v) { return v != kCountUnset; });
    }

    // What the driver needs of the GPU runtime is created by the first call that works on runs, so that the controller
    // (note_writes, note_reads, the log) can be used, and tested, on its own.  Words that the host watches are asked for as
    // coherent memory: where the default is another, a count would be seen only when its kernel has ended.
    int gpu_ready() {
        if (n_host != nullptr) return LSM_OK;
        if (stats_host == nullptr && hipHostMalloc(reinterpret_cast<void**>(&stats_host), 4 * sizeof(uint64_t), hipHostMallocCoherent) != hipSuccess)
            return LSM_ERR_HIP;
        stats_host[2] = 0;
        return hipHostMalloc(reinterpret_cast<void**>(&n_host), sizeof(uint64_t), hipHostMallocCoherent) == hipSuccess ? LSM_OK : LSM_ERR_HIP;
    }

    bool wants_index(uint64_t n) const { return cfg.hash_index_from != 0 && n >= cfg.hash_index_from && n <= (1ull << 27); }
    // filters that are built straight from the entries, on memory zeroed beforehand (of 32 GiB and more they are not: the memory is no span)
    bool plain_filter(uint64_t n) const {
        const uint64_t blocks = lsm_bloom_blocks(n, cfg.bloom_bits);
        return blocks != 0 && blocks < lsm::kMostClearWords && n < kHashedFilterEntries && !wants_index(n);
    }

    // Filter and hash index of a run that has come to rest, from the keys' hashes (computed once for both).  The
    // temporaries go back to the pool at once: their next user's work comes later on the stream.  The run gets both when
    // the launches that fill them have been made, or neither.
    int build_hashed(Run& r) {
        std::vector<void*> scratch;
        auto take = [&](size_t bytes) {
            void* p = pool.take(bytes);
            if (p != nullptr) scratch.push_back(p);
            return p;
        };
        const bool indexed = wants_index(r.n) && r.index == nullptr;
        const lsm_run_t run{r.entries, r.n};
        void *bloom = nullptr, *index = nullptr;
        uint64_t n_blocks = 0, n_buckets = 0;
        uint64_t* hashes = static_cast<uint64_t*>(take(r.n * 8));
        int rc = hashes == nullptr ? (int)LSM_ERR_HIP : lsm_hash_keys(&run, hashes, stream);
        if (rc == LSM_OK && cfg.bloom_bits != 0 && r.bloom == nullptr) n_blocks = lsm_bloom_blocks(r.n, cfg.bloom_bits);
        if (n_blocks != 0) {
            bloom = pool.take(n_blocks * 16);
            if (bloom == nullptr) rc = LSM_ERR_HIP;
            const size_t ws_bytes = lsm_bloom_workspace_bytes(r.n, n_blocks);
            void* ws = rc == LSM_OK && ws_bytes != 0 ? take(ws_bytes) : nullptr;
            if (rc == LSM_OK && ws_bytes != 0)
                rc = ws == nullptr ? (int)LSM_ERR_HIP : lsm_build_bloom_hashed(hashes, r.n, bloom, n_blocks, ws, ws_bytes, stream);
            else if (rc == LSM_OK)
                rc = lsm_build_bloom(&run, bloom, n_blocks, stream);
        }
        if (rc == LSM_OK && indexed) {
            n_buckets = lsm_hash_index_buckets(r.n);
            const size_t ws_bytes = lsm_hash_index_workspace_bytes(r.n);
            index = pool.take(n_buckets * 64);
            void* ws = take(ws_bytes);
            rc = (index == nullptr || ws == nullptr) ? (int)LSM_ERR_HIP : lsm_build_hash_index(hashes, r.n, index, ws, ws_bytes, stream);
        }
        for (void* p : scratch) pool.give(p);
        if (rc != LSM_OK) {
            pool.give(bloom);
            pool.give(index);
            return rc;
        }
        if (bloom != nullptr) r.bloom = bloom, r.n_blocks = n_blocks;
        if (index != nullptr) r.index = index, r.n_buckets = n_buckets;
        r.settled = true;
        return LSM_OK;
    }

    // Memory for the filter of a merged run of at most `n` entries, to be zeroed by a launch that is made anyway.  A run that is
    // certain to stay at `level` gets its filter in the same call: the launch does not wait for the host to see the count.
    // A long filter is built in *scratch_bytes of scratch memory, which the caller gives as clear->p.
    int take_filter(Run& r, uint64_t n, uint32_t level, lsm::ClearSpan* clear, size_t* scratch_bytes) {
        *scratch_bytes = 0;
        r.bloom = nullptr, r.bloom_clear = false;
        clear->p = nullptr, clear->bytes = 0;
        clear->filter_bits = 0, clear->filter_built = false, clear->filter = nullptr;
        if (n == 0 || !plain_filter(n)) return LSM_OK;
        const uint64_t blocks = lsm_bloom_blocks(n, cfg.bloom_bits);
        const bool small = lsm::small_filter(n, blocks);
        const lsm::FilterScratch scratch = lsm::filter_scratch(n, blocks);
        if (n <= capacity(level) && (small || scratch.n_ranges != 0)) clear->filter_bits = cfg.bloom_bits;
        r.bloom = pool.take(blocks * 16);
        if (r.bloom == nullptr) return LSM_ERR_HIP;
        if (clear->filter_bits != 0 && !small) {
            clear->filter = r.bloom;
            clear->bytes = scratch.zeroed;
            *scratch_bytes = scratch.total;
            return LSM_OK;
        }
        clear->p = r.bloom;
        clear->bytes = blocks * 16;
        return LSM_OK;
    }

    // The workspace for one call, with `need` bytes behind the status words.  It starts well below the 2 MB from which on the runtime asks the kernel
    // driver for every block on its own (30 to 300 us each, and what a tree allocates next takes longer as well), and when it is outgrown the
    // next has room for twice the need, so that a young tree does not grow it time and again.  First passes of new trees, geometric mean over 18
    // cases (one to 12 trees of 100,000 to 4M entries, 8 to 96 flushes) against blocks that start with 2 MB and hold twice the need: from 256 KB
    // on, in powers of two 0.96, with twice the need 0.86.
    // Eight trees of 1M entries, 24 flushes, us: 4,420 / 4,960 / 4,640; ten of 0.9M 4,000 / 3,240 / 2,990; one of 0.9M, 52 flushes 2,250 / 2,840 / 1,560.
    static constexpr size_t kStatusBytes = lsm::kShortTiles * sizeof(uint64_t), kLeastWorkspace = size_t(256) << 10;
    int reserve(Workspace& w, size_t need) {
        if (kStatusBytes + need <= w.bytes) return LSM_OK;
        pool.give(w.p);
        w = Workspace();
        if (need > (size_t(1) << 60)) return LSM_ERR_HIP;  // no such allocation succeeds
        const size_t twice = 2 * (kStatusBytes + need), bytes = twice > kLeastWorkspace ? twice : kLeastWorkspace;
        w.p = static_cast<char*>(pool.take(bytes));
        if (w.p == nullptr) return LSM_ERR_HIP;
        w.bytes = bytes;
        return LSM_OK;
    }
    // Its status words for the call, and what the call has made of them: from the first that has zeroed them on, every call has
    // an epoch of its own, until these are used up or a call has failed.
    static void lend_status(const Workspace& w, lsm::ClearSpan* clear) {
        clear->status = reinterpret_cast<uint64_t*>(w.p), clear->epoch = w.epoch, clear->status_zeroed = false;
    }
    static void status_used(Workspace& w, const lsm::ClearSpan& clear, int rc) {
        const bool known = rc == LSM_OK && (w.epoch != 0 || clear.status_zeroed);
        w.epoch = known && w.epoch + 1 < lsm::kStEpochs ? w.epoch + 1 : 0;
    }

    // A merged run whose filter has been built by the call that merged it has every structure it is to get (what holds for the
    // upper bound of its length, a plain filter and no index, holds for the length).
    void take_built_filter(Run& r, const lsm::ClearSpan& clear) {
        if (!clear.filter_built) return;
        r.n_blocks = lsm_bloom_blocks(r.n, cfg.bloom_bits);
        r.bloom_clear = false, r.settled = true;
    }

    // The runs that have come to rest in `count` drivers (of one stream) get whatever lookup structure they still lack: the
    // copies of flushed runs in one launch, and the filters of all short runs in one.  (Runs that are merged away at once -
    // a flushed run arriving at a full level, a run moved down onto another - never get any.)
    // A run is changed only when the launch that fills the memory it points to has been made, and what fails for one run
    // (memory, mostly) leaves out that run and no other; the first error is returned.  A run that was left out has no
    // structure rather than an unfinished one, and the next call completes it.
    static int settle_all(lsm_driver* const* drivers, uint32_t count) {
        struct Resting {
            lsm_driver* d;
            Run* r;
            lsm_entry_t* copy;  // of a flushed run
            uint8_t* fences;
            void* bloom;
        };
        int first_error = LSM_OK;
        auto fails = [&](int rc) {
            if (rc != LSM_OK && first_error == LSM_OK) first_error = rc;
            return rc != LSM_OK;
        };
        std::vector<Resting> resting;
        for (uint32_t i = 0; i < count; i++)
            for (Level& lv : drivers[i]->levels)
                for (Run& r : lv.runs)
                    if (!r.settled && r.n != 0) resting.push_back(Resting{drivers[i], &r, nullptr, nullptr, nullptr});
        if (resting.empty()) return LSM_OK;
        const hipStream_t stream = drivers[0]->stream;
        std::vector<lsm::IngestJob> ingest;
        std::vector<size_t> ingested;
        ingest.reserve(resting.size()), ingested.reserve(resting.size());
        uint32_t stride = 1;
        auto launch_ingest = [&] {
            const bool failed = !ingest.empty() && fails(lsm::ingest_runs(ingest.data(), (uint32_t)ingest.size(), stride, stream));
            for (size_t i : ingested) {
                const Resting& x = resting[i];
                if (failed) {
                    x.d->pool.give(x.copy);
                    x.d->pool.give(x.fences);
                    x.d->pool.give(x.bloom);
                    continue;
                }
                x.r->entries = x.copy, x.r->owned = true, x.r->transient = false;
                x.r->fences = x.fences;
                x.r->bloom = x.bloom, x.r->bloom_clear = x.bloom != nullptr;
            }
            ingest.clear(), ingested.clear();
        };
        for (size_t i = 0; i < resting.size(); i++) {
            Resting& x = resting[i];
            lsm_driver* const d = x.d;
            Run& r = *x.r;
            if (!r.transient && r.fences != nullptr) continue;
            x.fences = static_cast<uint8_t*>(d->pool.take(ceil_div(r.n, d->cfg.fence_stride) * LSM_KEY_BYTES));
            if (!r.transient) {
                const lsm_run_t run{r.entries, r.n};
                if (fails(x.fences == nullptr ? (int)LSM_ERR_HIP : lsm_build_fences(&run, d->cfg.fence_stride, x.fences, stream))) d->pool.give(x.fences);
                else r.fences = x.fences;
                continue;
            }
            x.copy = static_cast<lsm_entry_t*>(d->pool.take(r.n * sizeof(lsm_entry_t)));
            lsm::ClearSpan clear;
            if (d->plain_filter(r.n)) {
                clear.bytes = lsm_bloom_blocks(r.n, d->cfg.bloom_bits) * 16;
                clear.p = x.bloom = d->pool.take(clear.bytes);
            }
            if (x.copy == nullptr || x.fences == nullptr || (clear.bytes != 0 && x.bloom == nullptr)) {
                (void)fails(LSM_ERR_HIP);
                d->pool.give(x.copy);
                d->pool.give(x.fences);
                d->pool.give(x.bloom);
                continue;
            }
            if (stride != d->cfg.fence_stride) launch_ingest();  // one stride per launch
            stride = d->cfg.fence_stride;
            ingest.push_back(lsm::IngestJob{r.entries, x.copy, r.n, x.fences, static_cast<uint4*>(clear.p), clear.bytes / 16});
            ingested.push_back(i);
        }
        launch_ingest();
        // filters: [1] on memory that is zeroed by then
        std::vector<lsm_run_t> runs[2];
        std::vector<void*> filters[2];
        std::vector<uint64_t> blocks[2];
        std::vector<size_t> filtered[2];
        for (size_t i = 0; i < resting.size(); i++) {
            Resting& x = resting[i];
            lsm_driver* const d = x.d;
            Run& r = *x.r;
            if (r.transient || r.fences == nullptr) continue;  // left out above
            if (d->plain_filter(r.n)) {
                const int zeroed = r.bloom != nullptr && r.bloom_clear ? 1 : 0;
                x.bloom = r.bloom != nullptr ? r.bloom : d->pool.take(lsm_bloom_blocks(r.n, d->cfg.bloom_bits) * 16);
                if (x.bloom == nullptr) {
                    (void)fails(LSM_ERR_HIP);
                    continue;
                }
                r.bloom = x.bloom;  // n_blocks stays 0: not a filter yet
                runs[zeroed].push_back(lsm_run_t{r.entries, r.n});
                filters[zeroed].push_back(x.bloom);
                blocks[zeroed].push_back(lsm_bloom_blocks(r.n, d->cfg.bloom_bits));
                filtered[zeroed].push_back(i);
            } else if (d->cfg.bloom_bits != 0 || d->wants_index(r.n)) {
                (void)fails(d->build_hashed(r));
            } else {
                r.settled = true;
            }
        }
        for (int zeroed = 0; zeroed < 2; zeroed++) {
            if (runs[zeroed].empty()) continue;
            const bool failed = fails(lsm::build_filters(runs[zeroed].data(), filters[zeroed].data(), blocks[zeroed].data(), (uint32_t)runs[zeroed].size(),
                                                         zeroed == 1, stream));
            for (size_t q = 0; q < filtered[zeroed].size(); q++) {
                Run& r = *resting[filtered[zeroed][q]].r;
                r.bloom_clear = false;  // a launch that failed may have set bits all the same
                if (!failed) r.n_blocks = blocks[zeroed][q], r.settled = true;
            }
        }
        return first_error;
    }
    int settle() {
        lsm_driver* self = this;
        return settle_all(&self, 1);
    }

    // All runs of a level into one; the fence index of the output is written in the same pass.  Waits for the count (the
    // kernels store it to pinned host memory); what else the merge does is ordered before whatever is enqueued next.
    int compact(const std::vector<Run>& in, uint32_t flags, uint32_t level, Run* merged) {
        if (in.size() > LSM_MAX_RUNS) return LSM_ERR_BAD_ARG;
        lsm_run_t runs[LSM_MAX_RUNS];
        uint64_t lens[LSM_MAX_RUNS];
        uint64_t total = 0;
        for (size_t j = 0; j < in.size(); j++) {
            runs[j] = lsm_run_t{in[j].entries, in[j].n};
            lens[j] = in[j].n;
            total += in[j].n;
        }
        const uint32_t k = (uint32_t)in.size();
        const uint64_t room = total > 0 ? total : 1;
        lsm_entry_t* entries = static_cast<lsm_entry_t*>(pool.take(room * sizeof(lsm_entry_t)));
        uint8_t* fences = static_cast<uint8_t*>(pool.take(ceil_div(room, cfg.fence_stride) * LSM_KEY_BYTES));
        *merged = Run();
        lsm::ClearSpan clear;
        size_t scratch_bytes = 0;
        auto fails = [&](int rc) {
            pool.give(entries);
            pool.give(fences);
            pool.give(merged->bloom);
            *merged = Run();
            return rc;
        };
        if (entries == nullptr || fences == nullptr || take_filter(*merged, total, level, &clear, &scratch_bytes) != LSM_OK) return fails(LSM_ERR_HIP);
        const size_t own = lsm_compact_workspace_bytes(lens, k);  // a multiple of 256 bytes
        if (reserve(workspace, own + scratch_bytes) != LSM_OK) return fails(LSM_ERR_HIP);
        char* const room_at = workspace.p + kStatusBytes;
        if (scratch_bytes != 0) clear.p = room_at + own;
        lend_status(workspace, &clear);
        const lsm_out_t out{entries, room, n_host, fences, cfg.fence_stride, nullptr};
        *static_cast<volatile uint64_t*>(n_host) = kCountUnset;
        int rc = lsm::compact_clearing(runs, k, flags, &out, room_at, own, clear, &merged->bloom_clear, stream);
        if (clear.filter != nullptr) merged->bloom_clear = false;
        status_used(workspace, clear, rc);
        // an error may be that of the filter's launch, or of an earlier call, with the merge under way: its count must not meet the next one's
        if (rc != LSM_OK) (void)wait();
        if (rc == LSM_OK) rc = watch_count(n_host);
        if (rc == LSM_OK && *n_host > room) rc = LSM_ERR_INTERNAL;  // the device-side failure mark, or nonsense
        if (rc == LSM_OK && cfg.observer != nullptr) rc = wait();   // the observer sees a complete output
        if (rc != LSM_OK) return fails(rc);
        merged->n = *n_host;
        if (cfg.observer != nullptr) cfg.observer(cfg.observer_ctx, level + 1, entries, merged->n);
        merged->entries = entries, merged->owned = true, merged->fences = fences;
        take_built_filter(*merged, clear);
        if (merged->n == 0) drop(*merged);
        return LSM_OK;
    }

    // A run arrives at a level (0-based).  The cascade this starts is cut into steps, so that a caller who drives several
    // trees can run the compactions of their current steps as one batch: arrive_begin places the run and leaves a
    // compaction to be done in `due` if the level is too full; arrive_merged takes that compaction's output and either
    // places it, or moves it down (arrive_begin at the next level, which may leave the next compaction in `due`).
    // settle_all completes the runs that stay where they were placed.
    struct Due {
        bool active = false;
        uint32_t level = 0, flags = 0;
        uint64_t n_in = 0;
    } due;

    int arrive_begin(uint32_t level, const Run& moving) {
        ensure_level(level);
        Level& lv = levels[level];
        if (lv.T != T || lv.K != K) record(LSM_EV_ADOPT, level + 1, T, K, 0, 0);
        lv.T = T, lv.K = K;  // lazy transition: the level takes the current parameters when data flows into it
        lv.runs.insert(lv.runs.begin(), moving);
        if (lv.runs.size() <= lv.K) return LSM_OK;
        bool deeper_empty = true;
        for (size_t i = level + 1; i < levels.size(); i++) deeper_empty = deeper_empty && levels[i].runs.empty();
        due.active = true, due.level = level, due.flags = deeper_empty ? (uint32_t)LSM_BOTTOMMOST : 0u, due.n_in = 0;
        for (const Run& r : lv.runs) due.n_in += r.n;
        return LSM_OK;
    }

    int arrive_merged(const Run& merged) {
        const uint32_t level = due.level;
        Level& lv = levels[level];
        due.active = false;
        record(LSM_EV_COMPACT, level + 1, (uint32_t)lv.runs.size(), due.flags, due.n_in, merged.n);
        for (Run& r : lv.runs) drop(r);
        lv.runs.clear();
        if (merged.n > capacity(level)) {
            record(LSM_EV_MOVE, level + 1, level + 2, 0, 0, merged.n);
            return arrive_begin(level + 1, merged);
        }
        if (merged.n > 0) lv.runs.push_back(merged);
        return LSM_OK;
    }

    // The compaction that is due, on its own (one lsm_compact).
    int compact_due() {
        Run merged;
        const int rc = compact(levels[due.level].runs, due.flags, due.level, &merged);
        return rc != LSM_OK ? rc : arrive_merged(merged);
    }

    // The whole cascade of one arrival, one compaction after the other.
    int arrive(uint32_t level, const Run& moving) {
        int rc = arrive_begin(level, moving);
        while (rc == LSM_OK && due.active) rc = compact_due();
        return rc == LSM_OK ? settle() : rc;
    }

    // One batch of operation counts enters the window; the (T, K) search is re-run when the mix has moved.
    int count(uint64_t writes, uint64_t hits, uint64_t empties, double blocks) {
        window.push_back(Batch{writes, hits, empties, blocks});
        sum.writes += writes, sum.hits += hits, sum.empties += empties, sum.blocks += blocks;
        // slide: drop the oldest batches while the rest still covers window_ops operations
        while (window.size() > 1) {
            const Batch& f = window.front();
            if (sum.writes + sum.hits + sum.empties - (f.writes + f.hits + f.empties) < cfg.window_ops) break;
            sum.writes -= f.writes, sum.hits -= f.hits, sum.empties -= f.empties, sum.blocks -= f.blocks;
            window.pop_front();
        }
        const uint64_t total = sum.writes + sum.hits + sum.empties;
        if (total < cfg.window_ops) return LSM_OK;  // the window is not full yet
        const double mix[4] = {(double)sum.writes / (double)total, (double)sum.hits / (double)total / 2, (double)sum.hits / (double)total / 2,
                               (double)sum.empties / (double)total};  // w, s, r, z
        const double d = sum.hits ? sum.blocks / (double)sum.hits : 0.0;
        if (searched) {
            double moved = 0.0;
            for (int i = 0; i < 4; i++) moved += mix[i] > last_mix[i] ? mix[i] - last_mix[i] : last_mix[i] - mix[i];
            if (moved <= cfg.shift_threshold) return LSM_OK;
        }
        std::memcpy(last_mix, mix, sizeof(mix));
        searched = true;
        const uint64_t n = total_entries();
        const lsm_policy_input_t in{mix[0], mix[1], mix[2], mix[3], n > 0 ? n : 1, cfg.buffer_entries, cfg.page_entries, p, d};
        uint32_t best_T = 0, best_K = 0;
        const int rc = lsm_policy_choose(&in, cfg.t_min, cfg.t_max, &best_T, &best_K);
        if (rc != LSM_OK) return rc;
        lsm_driver_event_t e;
        std::memset(&e, 0, sizeof(e));
        e.kind = LSM_EV_POLICY, e.a = best_T, e.b = best_K, e.d = d;
        std::memcpy(e.mix, mix, sizeof(mix));
        log.push_back(e);
        T = best_T, K = best_K;
        return LSM_OK;
    }

    uint32_t tree(lsm_tree_run_t* out, uint32_t capacity) const {
        uint32_t n = 0;
        for (size_t l = 0; l < levels.size(); l++)
            for (const Run& r : levels[l].runs) {
                if (n < capacity) {
                    lsm_tree_run_t t;
                    std::memset(&t, 0, sizeof(t));
                    t.run = lsm_run_t{r.entries, r.n};
                    t.fence = lsm_fence_t{r.fences, r.fences ? ceil_div(r.n, cfg.fence_stride) : 0, cfg.fence_stride};
                    t.bloom = lsm_bloom_t{r.n_blocks ? r.bloom : nullptr, r.n_blocks};  // n_blocks is set when the filter is built
                    t.level = (uint32_t)l + 1;
                    t.index = lsm_hash_index_t{r.index, r.index ? r.n_buckets : 0};
                    out[n] = t;
                }
                n++;
            }
        return n;
    }
};

extern "C" int lsm_driver_create(const lsm_driver_config_t* config, void* stream, lsm_driver_t** driver_out) {
    if (config == nullptr || driver_out == nullptr) return LSM_ERR_NULL;
    *driver_out = nullptr;
    if (config->buffer_entries == 0 || config->size_ratio < 2 || config->runs_per_level == 0 || config->window_ops == 0 ||
        config->t_min < 2 || config->t_max < config->t_min || !(config->page_entries > 0) || config->fence_stride == 0)
        return LSM_ERR_BAD_ARG;
    lsm_driver* d = new (std::nothrow) lsm_driver();
    if (d == nullptr) return LSM_ERR_HIP;
    d->cfg = *config;
    d->stream = static_cast<hipStream_t>(stream);
    d->p = config->filter_fpr < 0 ? lsm_policy_filter_fpr(config->bloom_bits) : config->filter_fpr;
    d->T = config->size_ratio, d->K = config->runs_per_level;
    *driver_out = d;
    return LSM_OK;
}

extern "C" void lsm_driver_destroy(lsm_driver_t* d) {
    if (d == nullptr) return;
    if (d->n_host != nullptr) (void)hipStreamSynchronize(d->stream);  // else no GPU call was ever made
    d->pool.free_all();
    if (d->n_host != nullptr) (void)hipHostFree(d->n_host);
    if (d->stats_host != nullptr) (void)hipHostFree(d->stats_host);
    if (d->counts_host != nullptr) (void)hipHostFree(d->counts_host);
    delete d;
}

extern "C" int lsm_driver_load_run(lsm_driver_t* d, uint32_t level, const lsm_entry_t* entries, uint64_t n) try {
    if (d == nullptr || (n > 0 && entries == nullptr)) return LSM_ERR_NULL;
    if (level == 0 || level > 64 || (reinterpret_cast<uintptr_t>(entries) & 63) != 0) return LSM_ERR_BAD_ARG;
    const int ready = d->gpu_ready();
    if (ready != LSM_OK) return ready;
    d->ensure_level(level - 1);
    Run r;
    r.entries = entries, r.n = n;
    std::vector<Run>& runs = d->levels[level - 1].runs;
    runs.push_back(r);
    return d->settle();
} catch (...) {  // host memory ran out: nothing may be thrown through the C ABI
    return LSM_ERR_INTERNAL;
}

extern "C" int lsm_driver_note_writes(lsm_driver_t* d, uint64_t n_ops) try {
    if (d == nullptr) return LSM_ERR_NULL;
    return d->count(n_ops, 0, 0, 0.0);
} catch (...) {  // host memory ran out: nothing may be thrown through the C ABI
    return LSM_ERR_INTERNAL;
}

extern "C" int lsm_driver_note_reads(lsm_driver_t* d, uint64_t successful, uint64_t empty, uint64_t blocks) try {
    if (d == nullptr) return LSM_ERR_NULL;
    if (successful + empty > UINT32_MAX) return LSM_ERR_BAD_ARG;
    d->record(LSM_EV_PROBE, 0, (uint32_t)(successful + empty), (uint32_t)successful, 0, blocks);
    return d->count(0, successful, empty, (double)blocks);
} catch (...) {  // host memory ran out: nothing may be thrown through the C ABI
    return LSM_ERR_INTERNAL;
}

extern "C" int lsm_driver_flush(lsm_driver_t* d, const lsm_entry_t* run, uint64_t n) try {
    if (d == nullptr || (n > 0 && run == nullptr)) return LSM_ERR_NULL;
    if ((reinterpret_cast<uintptr_t>(run) & 63) != 0) return LSM_ERR_BAD_ARG;
    const int ready = d->gpu_ready();
    if (ready != LSM_OK) return ready;
    Run r;
    if (n > 0) r.entries = run, r.n = n, r.transient = true;
    return d->arrive(0, r);
} catch (...) {  // host memory ran out: nothing may be thrown through the C ABI
    return LSM_ERR_INTERNAL;
}

extern "C" int lsm_driver_flush_unsorted(lsm_driver_t* d, const lsm_entry_t* buffer, uint64_t n) try {
    if (d == nullptr || (n > 0 && buffer == nullptr)) return LSM_ERR_NULL;
    if (n > LSM_MAX_BUFFER) return LSM_ERR_BAD_ARG;
    const int ready = d->gpu_ready();
    if (ready != LSM_OK) return ready;
    const uint64_t room = n > 0 ? n : 1;
    const size_t ws_bytes = lsm_flush_workspace_bytes(n);
    Run r;
    r.owned = true;
    lsm_entry_t* sorted = static_cast<lsm_entry_t*>(d->pool.take(room * sizeof(lsm_entry_t)));
    r.entries = sorted;
    r.fences = static_cast<uint8_t*>(d->pool.take(ceil_div(room, d->cfg.fence_stride) * LSM_KEY_BYTES));
    void* ws = d->pool.take(ws_bytes > 0 ? ws_bytes : 4);
    int rc = (sorted == nullptr || r.fences == nullptr || ws == nullptr) ? (int)LSM_ERR_HIP : (int)LSM_OK;
    if (rc == LSM_OK) {
        const lsm_out_t out{sorted, room, d->n_host, r.fences, d->cfg.fence_stride, nullptr};
        *static_cast<volatile uint64_t*>(d->n_host) = kCountUnset;
        rc = lsm_flush_buffer(buffer, n, &out, ws, ws_bytes > 0 ? ws_bytes : 4, d->stream);
        if (rc != LSM_OK) (void)d->wait();  // some of its launches may have been made: see compact
    }
    if (rc == LSM_OK) rc = d->watch_count(d->n_host);
    d->pool.give(ws);
    if (rc == LSM_OK && *d->n_host > room) rc = LSM_ERR_INTERNAL;
    if (rc != LSM_OK) {
        d->drop(r);
        return rc;
    }
    r.n = *d->n_host;
    if (r.n == 0) d->drop(r);
    return d->arrive(0, r);
} catch (...) {  // host memory ran out: nothing may be thrown through the C ABI
    return LSM_ERR_INTERNAL;
}

// Jobs of at least this many input entries are merged on their own: lsm_compact_batch takes jobs below 2,048 tiles.
static constexpr uint64_t kBatchJobEntries = 1ull << 21;

extern "C" int lsm_driver_flush_many(lsm_driver_t* const* drivers, const lsm_entry_t* const* runs, const uint64_t* n, uint32_t count) try {
    if (count == 0) return LSM_OK;
    if (drivers == nullptr || runs == nullptr || n == nullptr) return LSM_ERR_NULL;
    for (uint32_t i = 0; i < count; i++) {
        if (drivers[i] == nullptr || (n[i] > 0 && runs[i] == nullptr)) return LSM_ERR_NULL;
        if (drivers[i]->stream != drivers[0]->stream || (reinterpret_cast<uintptr_t>(runs[i]) & 63) != 0) return LSM_ERR_BAD_ARG;
        for (uint32_t j = 0; j < i; j++)
            if (drivers[j] == drivers[i]) return LSM_ERR_BAD_ARG;
    }
    lsm_driver_t* const first = drivers[0];
    for (uint32_t i = 0; i < count; i++) {
        const int ready = drivers[i]->gpu_ready();
        if (ready != LSM_OK) return ready;
    }
    if (count > first->counts_host_count) {
        if (first->counts_host != nullptr) (void)hipHostFree(first->counts_host);
        first->counts_host = nullptr, first->counts_host_count = 0;
        if (hipHostMalloc(reinterpret_cast<void**>(&first->counts_host), (size_t)count * sizeof(uint64_t), hipHostMallocCoherent) != hipSuccess)
            return LSM_ERR_HIP;
        first->counts_host_count = count;
    }
    std::vector<int> status(count, LSM_OK);  // a tree that has failed takes no further step; the others end as they would alone
    for (uint32_t i = 0; i < count; i++) {
        if (runs[i] == nullptr) continue;  // nothing to flush for this tree
        Run r;
        if (n[i] > 0) r.entries = runs[i], r.n = n[i], r.transient = true;
        status[i] = drivers[i]->arrive_begin(0, r);
    }
    struct Step {  // one compaction of a batch
        uint32_t tree;
        Run merged;
    };
    std::vector<Step> steps;
    std::vector<std::vector<lsm_run_t>> inputs;
    std::vector<lsm_compact_job_t> jobs;
    std::vector<lsm::ClearSpan> clear;
    std::vector<size_t> scratch;  // bytes of the filters' scratch memory
    for (;;) {
        // the compactions that are due now: the long ones on their own, the others as one batch
        steps.clear(), inputs.clear(), jobs.clear(), clear.clear(), scratch.clear();
        for (uint32_t i = 0; i < count; i++) {
            lsm_driver_t* d = drivers[i];
            while (status[i] == LSM_OK && d->due.active && d->due.n_in >= kBatchJobEntries) status[i] = d->compact_due();
            if (status[i] != LSM_OK || !d->due.active) continue;
            const std::vector<Run>& in = d->levels[d->due.level].runs;
            if (in.size() > LSM_MAX_RUNS) {
                status[i] = LSM_ERR_BAD_ARG;
                continue;
            }
            const uint64_t room = d->due.n_in > 0 ? d->due.n_in : 1;
            Run merged;
            lsm::ClearSpan zeroed;
            size_t scratch_bytes = 0;
            lsm_entry_t* entries = static_cast<lsm_entry_t*>(d->pool.take(room * sizeof(lsm_entry_t)));
            merged.entries = entries, merged.owned = true;  // given back through drop() on failure
            merged.fences = static_cast<uint8_t*>(d->pool.take(ceil_div(room, d->cfg.fence_stride) * LSM_KEY_BYTES));
            status[i] = d->take_filter(merged, d->due.n_in, d->due.level, &zeroed, &scratch_bytes);
            if (entries == nullptr || merged.fences == nullptr) status[i] = LSM_ERR_HIP;
            if (status[i] != LSM_OK) {
                d->drop(merged);
                continue;
            }
            merged.bloom_clear = merged.bloom != nullptr && zeroed.filter == nullptr;
            inputs.emplace_back();
            for (const Run& r : in) inputs.back().push_back(lsm_run_t{r.entries, r.n});
            lsm_compact_job_t job{};
            job.runs = inputs.back().data(), job.n_runs = (uint32_t)inputs.back().size(), job.flags = d->due.flags;
            job.out = lsm_out_t{entries, room, first->counts_host + jobs.size(), merged.fences, d->cfg.fence_stride, nullptr};
            static_cast<volatile uint64_t*>(first->counts_host)[jobs.size()] = kCountUnset;
            jobs.push_back(job);
            clear.push_back(zeroed);
            scratch.push_back((scratch_bytes + 255) & ~size_t(255));
            steps.push_back(Step{i, merged});
        }
        const uint32_t n_jobs = (uint32_t)jobs.size();
        if (n_jobs == 0) break;
        int rc = LSM_OK;
        const size_t own = lsm_compact_batch_workspace_bytes(jobs.data(), n_jobs);
        if (own == 0) rc = LSM_ERR_BAD_ARG;
        size_t need = own;
        for (size_t bytes : scratch) need += bytes;
        lsm_driver::Workspace& shared = first->batch_workspace;
        if (rc == LSM_OK) rc = first->reserve(shared, need);
        if (rc == LSM_OK) {
            char* const room_at = shared.p + lsm_driver::kStatusBytes;
            char* at = room_at + own;
            for (uint32_t j = 0; j < n_jobs; j++) {
                if (clear[j].filter == nullptr) continue;
                clear[j].p = at;
                at += scratch[j];
            }
            lsm_driver::lend_status(shared, &clear[0]);
            rc = lsm::compact_batch_clearing(jobs.data(), n_jobs, room_at, own, clear.data(), first->stream);
            lsm_driver::status_used(shared, clear[0], rc);
            // an error may be that of an earlier call, with this launch under way: its counts must not meet the next batch's
            if (rc != LSM_OK) (void)first->wait();
        }
        if (rc != LSM_OK) {  // what the trees shared failed: every tree's compaction on its own
            for (Step& step : steps) {
                drivers[step.tree]->drop(step.merged);
                status[step.tree] = drivers[step.tree]->compact_due();
            }
            continue;
        }
        bool observed = false;
        for (uint32_t j = 0; j < n_jobs; j++) {
            int& st = status[steps[j].tree];
            st = first->watch_count(first->counts_host + j);
            if (st == LSM_OK && first->counts_host[j] > jobs[j].out.capacity) st = LSM_ERR_INTERNAL;  // the device-side failure mark, or nonsense
            observed = observed || drivers[steps[j].tree]->cfg.observer != nullptr;
        }
        const int seen = observed ? first->wait() : (int)LSM_OK;  // observers see complete outputs
        for (uint32_t j = 0; j < n_jobs; j++) {
            lsm_driver_t* d = drivers[steps[j].tree];
            Run& merged = steps[j].merged;
            int& st = status[steps[j].tree];
            if (st == LSM_OK) st = seen;
            if (st != LSM_OK) {
                d->drop(merged);
                continue;
            }
            merged.n = first->counts_host[j];
            d->take_built_filter(merged, clear[j]);
            if (d->cfg.observer != nullptr) d->cfg.observer(d->cfg.observer_ctx, d->due.level + 1, merged.entries, merged.n);
            if (merged.n == 0) d->drop(merged);
            st = d->arrive_merged(merged);
        }
    }
    const int settled = lsm_driver::settle_all(drivers, count);
    for (int st : status)
        if (st != LSM_OK) return st;
    return settled;
} catch (...) {  // host memory ran out: nothing may be thrown through the C ABI
    return LSM_ERR_INTERNAL;
}

extern "C" int lsm_driver_probe(lsm_driver_t* d, const lsm_queries_t* queries, const lsm_hits_t* out_hits) try {
    if (d == nullptr || queries == nullptr || out_hits == nullptr) return LSM_ERR_NULL;
    lsm_tree_run_t runs[LSM_MAX_RUNS];
    const uint32_t n_runs = d->tree(runs, LSM_MAX_RUNS);
    if (n_runs > LSM_MAX_RUNS) return LSM_ERR_BAD_ARG;
    for (uint32_t i = 0; i < n_runs; i++) runs[i].level = i;
    const lsm_tree_t tree{runs, n_runs};
    int rc = d->gpu_ready();
    if (rc == LSM_OK) rc = lsm_probe(queries, &tree, out_hits, d->stream);
    if (rc != LSM_OK) return rc;
    const uint32_t n_req = queries->n_req;
    uint64_t hits = 0, blocks = 0;
    if (n_req > 0) {
        const uint64_t ticket = ++d->tickets;  // this batch's: after a call that failed the word may hold any earlier one
        rc = lsm::probe_stats(out_hits->hit_len, n_req, d->stats_host, ticket, d->stream);
        if (rc == LSM_OK) rc = d->watch(d->stats_host + 2, [ticket](uint64_t v) { return v == ticket; });
        if (rc != LSM_OK) return rc;
        blocks = d->stats_host[0], hits = d->stats_host[1];
    }
    d->record(LSM_EV_PROBE, 0, n_req, (uint32_t)hits, 0, blocks);
    return d->count(0, hits, n_req - hits, (double)blocks);
} catch (...) {  // host memory ran out: nothing may be thrown through the C ABI
    return LSM_ERR_INTERNAL;
}

extern "C" uint32_t lsm_driver_levels(const lsm_driver_t* d) { return d ? (uint32_t)d->levels.size() : 0; }

extern "C" int lsm_driver_level(const lsm_driver_t* d, uint32_t level, uint32_t* T, uint32_t* K, uint32_t* n_runs) {
    if (d == nullptr) return LSM_ERR_NULL;
    if (level == 0 || level > d->levels.size()) return LSM_ERR_BAD_ARG;
    const Level& lv = d->levels[level - 1];
    if (T) *T = lv.T;
    if (K) *K = lv.K;
    if (n_runs) *n_runs = (uint32_t)lv.runs.size();
    return LSM_OK;
}

extern "C" int lsm_driver_tree(lsm_driver_t* d, lsm_tree_run_t* runs_out, uint32_t capacity, uint32_t* n_runs) try {
    if (d == nullptr || n_runs == nullptr || (capacity > 0 && runs_out == nullptr)) return LSM_ERR_NULL;
    *n_runs = d->tree(runs_out, capacity);
    return d->n_host != nullptr ? d->wait() : (int)LSM_OK;
} catch (...) {  // host memory ran out: nothing may be thrown through the C ABI
    return LSM_ERR_INTERNAL;
}

extern "C" int lsm_driver_target(const lsm_driver_t* d, uint32_t* T, uint32_t* K) {
    if (d == nullptr) return LSM_ERR_NULL;
    if (T) *T = d->T;
    if (K) *K = d->K;
    return LSM_OK;
}

extern "C" uint64_t lsm_driver_log(const lsm_driver_t* d, uint64_t first, lsm_driver_event_t* out, uint64_t capacity) {
    if (d == nullptr) return 0;
    const uint64_t n = d->log.size();
    for (uint64_t i = first; out != nullptr && i < n && i - first < capacity; i++) out[i - first] = d->log[i];
    return n;
}

extern "C" int lsm_driver_read(lsm_driver_t* d, const void* device_src, void* dst, size_t bytes) try {
    if (d == nullptr || (bytes > 0 && (device_src == nullptr || dst == nullptr))) return LSM_ERR_NULL;
    int rc = d->gpu_ready();
    if (rc != LSM_OK) return rc;
    if (bytes > 0 && hipMemcpyAsync(dst, device_src, bytes, hipMemcpyDefault, d->stream) != hipSuccess) return LSM_ERR_HIP;
    return d->wait();
} catch (...) {  // host memory ran out: nothing may be thrown through the C ABI
    return LSM_ERR_INTERNAL;
}
