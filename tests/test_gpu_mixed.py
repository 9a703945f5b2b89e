"""Configuration 5 (mixed, shifting workload): the two host drivers of the GPU library (the Python one of tree.py and
the library's own, lsm_driver_*), each against the plain driver of oracle/lsm_driver_oracle.py on the CPU checker.
They share no code with it.  Every probe batch (all hit bytes), the
sequence of compactions (level, run count, sizes in and out, last-level flag), the moves between levels, the policy
decisions, the levels' transitions of (T, K) and the final tree must be identical."""
import numpy as np
import pytest
import torch

from gpu_util import dev

pytestmark = pytest.mark.gpu


def replay_both(oracle, tr, bloom_bits, t_grid, window_batches, shuffle=None, progress=None, hash_index_from=0, native=False):
    """Run the trace through both drivers in step: every compaction output and every probe batch is compared as it is
    produced (so that no more than one of each is alive at a time), the logs after every event.  native: the library's own
    driver (lsm_driver_*) is stepped along as a third participant and compared with the plain driver in the same way."""
    from gpu_util import oracle_probe_threads
    from oracle import lsm_driver_oracle as drv
    from paper_2511_16138_amd.tree import AdaptiveLsmTree, GpuBackend
    window = window_batches * tr.batch_requests
    gpu_out, cpu_out = [], []

    class Recording(GpuBackend):
        def compact(self, runs, flags):
            merged = super().compact(runs, flags)
            gpu_out.append(merged)
            return merged

    gpu = AdaptiveLsmTree(Recording(bloom_bits=bloom_bits, hash_index_from=hash_index_from), tr.buffer_entries, size_ratio=tr.size_ratio, window_ops=window,
                          t_grid=t_grid)
    cpu = drv.DriverOracle(tr.buffer_entries, T=tr.size_ratio, K=1, window_ops=window, threshold=0.2, t_grid=t_grid,
                           page_entries=64.0, fpr=drv.bloom_fpr(bloom_bits), on_compact=cpu_out.append,
                           probe_fn=lambda q, nb, runs: oracle_probe_threads(oracle, q, nb, runs))
    nat, nat_out = None, []
    if native:
        from paper_2511_16138_amd import LsmDriver
        nat = LsmDriver(tr.buffer_entries, size_ratio=tr.size_ratio, window_ops=window, t_grid=t_grid, bloom_bits=bloom_bits,
                        hash_index_from=hash_index_from, on_compaction=lambda level, out: nat_out.append(out))
    for level, r in enumerate(tr.workload.runs):
        gpu.load_level(level, [r])
        cpu.install(level + 1, [r.cpu()])
        if nat:
            nat.load_run(level + 1, r)
    n_probe = 0
    for (kind, i, _phase), n_writes in zip(tr.events, tr.write_ops_between):
        if n_writes:
            gpu.note_writes(n_writes)
            cpu.writes(n_writes)
            if nat:
                nat.note_writes(n_writes)
        if kind == "flush":
            run = tr.flush_runs[i]
            if shuffle is not None:   # the GPU side gets the write buffer in the order it was "written" and sorts it itself
                gpu.flush_unsorted(run[shuffle(i, int(run.shape[0]))])
            else:
                gpu.flush(run)
            if nat:
                nat.flush_unsorted(run[shuffle(i, int(run.shape[0]))].contiguous()) if shuffle is not None else nat.flush(run)
            cpu.flush(run.cpu())
            assert len(gpu_out) == len(cpu_out) and (nat is None or len(nat_out) == len(cpu_out))
            for got, want in zip(gpu_out, cpu_out):   # every compaction of this flush, byte for byte
                assert np.array_equal(oracle.as_run(got), want), f"flush {i}: a compaction output differs"
            for got, want in zip(nat_out, cpu_out):
                assert np.array_equal(oracle.as_run(got), want), f"flush {i}: a compaction output of the library's driver differs"
            gpu_out.clear()
            cpu_out.clear()
            nat_out.clear()
        else:
            q, nb = tr.probe_batch(i)
            ghl, ghits = gpu.probe(q, nb)
            chl, chits = cpu.probe(q.cpu(), nb.cpu())
            assert np.array_equal(ghl.cpu().numpy().astype(np.uint32), chl), f"probe batch {i}: hit_len"
            assert np.array_equal(ghits.cpu().numpy().view(oracle.HIT_DTYPE).reshape(chits.shape), chits), f"probe batch {i}"
            if nat:
                nhl, nhits = nat.probe(q, nb)
                assert np.array_equal(nhl.cpu().numpy().astype(np.uint32), chl), f"probe batch {i}: hit_len (library's driver)"
                assert np.array_equal(nhits.cpu().numpy().view(oracle.HIT_DTYPE).reshape(chits.shape), chits), f"probe batch {i} (library's driver)"
            n_probe += 1
            if progress:
                progress(f"probe batch {i} ok, {len(gpu.trace)} log records")
        assert len(gpu.trace) == len(cpu.log) and gpu.trace[-1:] == cpu.log[-1:], (kind, i, gpu.trace[-3:], cpu.log[-3:])
        if nat:
            log = nat.trace
            assert len(log) == len(cpu.log) and log[-1:] == cpu.log[-1:], (kind, i, log[-3:], cpu.log[-3:])
    assert gpu.trace == cpu.log
    if nat:
        assert nat.trace == cpu.log
        check_native_tree(oracle, nat, cpu, bloom_bits, hash_index_from, progress,
                          borrowed={int(r.data_ptr()) for r in tr.workload.runs})
        nat.close()
    assert [len(lv) for lv in gpu.levels] == [len(lv.runs) for lv in cpu.levels]
    for glv, clv in zip(gpu.levels, cpu.levels):
        for gr, cr in zip(glv, clv.runs):
            if progress:
                progress(f"final tree: run of {cr.shape[0]} entries")
            assert np.array_equal(oracle.as_run(gr.run), cr)
            assert np.array_equal(gr.fences.cpu().numpy().view(np.uint8).reshape(-1, 32), oracle.build_fences(cr, 64))
            if bloom_bits:
                assert np.array_equal(gr.bloom.cpu().numpy().view(np.uint8).reshape(-1, 16), oracle.build_bloom(cr, int(gr.bloom.shape[0])))
            if hash_index_from and cr.shape[0] >= hash_index_from:
                assert oracle.hash_index_check(cr, gr.index.cpu().numpy()) == 0
            else:
                assert gr.index is None
    assert [(t, k) for t, k in zip(gpu.level_t, gpu.level_k)] == [(lv.T, lv.K) for lv in cpu.levels]
    return gpu, n_probe


@pytest.mark.parametrize("tree_total,buffer_entries,ops,bloom_bits,t_grid,shuffled,hash_index_from", [
    (400_000, 360, 4096, 16, (2, 16), False, 0),    # filters on: p = 0.0022, the full (T, K) grid
    (2_000_000, 900, 8192, 16, (10, 10), False, 0),  # T fixed at 10: only K moves
    (400_000, 360, 4096, 0, (2, 16), False, 0),     # no filters: p = 1
    (400_000, 360, 4096, 16, (2, 16), True, 0),     # write buffers handed over unsorted (lsm_flush_buffer)
    (400_000, 360, 4096, 16, (2, 16), False, 2000),  # runs of 2,000 entries and more also get a hash index
])
def test_mixed_trace_gpu_equals_plain_driver(oracle, tree_total, buffer_entries, ops, bloom_bits, t_grid, shuffled, hash_index_from):
    from workloads import lsm
    print("mixed trace", tree_total, buffer_entries, ops, bloom_bits, t_grid, shuffled, hash_index_from, flush=True)
    tr = lsm.config5(device=dev(), tree_total=tree_total, buffer_entries=buffer_entries, ops_per_phase=ops, batch_requests=128)
    assert len([e for e in tr.events if e[0] == "flush"]) > 50 and len([e for e in tr.events if e[0] == "probe"]) >= 6
    shuffle = (lambda i, n: torch.from_numpy(np.random.RandomState(i).permutation(n)).to(dev())) if shuffled else None
    gpu, n_probe = replay_both(oracle, tr, bloom_bits, t_grid, 16, shuffle, hash_index_from=hash_index_from, native=True)
    kinds = {e[0] for e in gpu.trace}
    assert {"compact", "probe", "policy", "move"} <= kinds and n_probe >= 6
    pol = [(e[1], e[2]) for e in gpu.trace if e[0] == "policy"]
    assert pol[0][1] == 1, pol                     # leveling while reads dominate (phase 90:10)
    if bloom_bits:
        # with filters the lookups are cheap enough that the write-heavy phase (10:90) leaves leveling
        assert max(k for _, k in pol) > 1, pol
        assert "adopt" in kinds
        assert any(e[0] == "compact" and e[2] > 2 for e in gpu.trace)   # several runs of a level merged at once
    if t_grid[0] != t_grid[1]:
        assert len({t for t, _ in pol}) > 1 or pol[0][0] != tr.size_ratio, pol   # the size ratio moves as well


def check_native_tree(oracle, gpu, cpu, bloom_bits, hash_index_from, progress=None, borrowed=()):
    """The tree of the library's driver against the plain driver's: levels, parameters, every run with its fence index,
    filter and hash index.  borrowed: addresses of the runs the test itself handed to load_run - the driver must still
    point at them (their content is the generator's and is not read back)."""
    assert gpu.levels() == [(lv.T, lv.K, len(lv.runs)) for lv in cpu.levels]
    assert gpu.target() == (cpu.target_T, cpu.target_K)
    want_runs = [(li + 1, r) for li, lv in enumerate(cpu.levels) for r in lv.runs]
    tree = gpu.tree()
    assert len(tree) == len(want_runs)
    for t, (level, cr) in zip(tree, want_runs):
        n = int(cr.shape[0])
        assert (t.level, t.run.n) == (level, n)
        if n == 0:                       # an empty write buffer that came to rest: a run without structures
            assert not t.bloom.blocks and not t.index.buckets and t.fence.n == 0
            continue
        if progress:
            progress(f"final tree of the library's driver: run of {n} entries")
        if t.run.entries in borrowed:   # the right one of them: its two ends
            m = min(n, 1000)
            assert np.array_equal(oracle.as_run(gpu.read(t.run.entries, m, 8)), cr[:m])
            assert np.array_equal(oracle.as_run(gpu.read(t.run.entries + 64 * (n - m), m, 8)), cr[n - m:])
        else:
            assert np.array_equal(oracle.as_run(gpu.read(t.run.entries, n, 8)), cr)
        assert (t.fence.n, t.fence.stride) == ((n + 63) // 64, 64)
        assert np.array_equal(gpu.read(t.fence.keys, t.fence.n, 4).cpu().numpy().view(np.uint8).reshape(-1, 32), oracle.build_fences(cr, 64))
        if bloom_bits:
            assert t.bloom.n_blocks == (n * bloom_bits + 127) // 128
            assert np.array_equal(gpu.read(t.bloom.blocks, t.bloom.n_blocks, 4, torch.int32).cpu().numpy().view(np.uint8).reshape(-1, 16),
                                  oracle.build_bloom(cr, int(t.bloom.n_blocks)))
        else:
            assert not t.bloom.blocks
        if hash_index_from and n >= hash_index_from:
            assert t.index.n_buckets == oracle.hash_index_buckets(n)
            assert oracle.hash_index_check(cr, gpu.read(t.index.buckets, t.index.n_buckets, 8).cpu().numpy()) == 0
        else:
            assert not t.index.buckets


def test_sharded_trees_with_batched_compactions(oracle):
    """Four independent trees stepped together: the compactions of every round go to the library as one batch
    (lsm_compact_batch).  Every tree's log, probe results and final runs equal the plain driver's for that tree alone."""
    from oracle import lsm_driver_oracle as drv
    from paper_2511_16138_amd.tree import AdaptiveLsmTree, GpuBackend, ShardedLsmTrees
    from workloads import lsm, rng
    print("sharded trees", flush=True)
    n_shards, window = 4, 16 * 128
    traces = [lsm.config5(device=dev(), seed=rng.SEED + 1000 * i, tree_total=200_000 + 50_000 * i, buffer_entries=360,
                          ops_per_phase=2048, batch_requests=128) for i in range(n_shards)]
    backend = GpuBackend(bloom_bits=16, hash_index_from=5000)   # runs of 5,000 entries and more also get a hash index
    batches = []
    real = backend.compact_batch
    backend.compact_batch = lambda jobs: (batches.append(len(jobs)), real(jobs))[1]
    trees = [AdaptiveLsmTree(backend, tr.buffer_entries, size_ratio=tr.size_ratio, window_ops=window, t_grid=(2, 16)) for tr in traces]
    cpus = [drv.DriverOracle(tr.buffer_entries, T=tr.size_ratio, K=1, window_ops=window, threshold=0.2, t_grid=(2, 16),
                             page_entries=64.0, fpr=drv.bloom_fpr(16)) for tr in traces]
    for tr, tree, cpu in zip(traces, trees, cpus):
        for level, r in enumerate(tr.workload.runs):
            tree.load_level(level, [r])
            cpu.install(level + 1, [r.cpu()])
    sharded = ShardedLsmTrees(trees, backend)
    at = [0] * n_shards
    while any(at[i] < len(traces[i].events) for i in range(n_shards)):
        runs = [None] * n_shards
        for i, (tr, tree, cpu) in enumerate(zip(traces, trees, cpus)):
            if at[i] >= len(tr.events):
                continue
            (kind, idx, _phase), n_writes = tr.events[at[i]], tr.write_ops_between[at[i]]
            at[i] += 1
            if n_writes:
                tree.note_writes(n_writes)
                cpu.writes(n_writes)
            if kind == "flush":
                runs[i] = tr.flush_runs[idx]
                cpu.flush(runs[i].cpu())
            else:
                q, nb = tr.probe_batch(idx)
                ghl, ghits = tree.probe(q, nb)
                chl, chits = cpu.probe(q.cpu(), nb.cpu())
                assert np.array_equal(ghl.cpu().numpy().astype(np.uint32), chl)
                assert np.array_equal(ghits.cpu().numpy().view(oracle.HIT_DTYPE).reshape(chits.shape), chits)
        sharded.flush_all(runs)
        for i, (tree, cpu) in enumerate(zip(trees, cpus)):
            assert tree.trace[-2:] == cpu.log[-2:] and len(tree.trace) == len(cpu.log), (i, tree.trace[-3:], cpu.log[-3:])
    assert max(batches) == n_shards and sum(batches) == sum(1 for t in trees for e in t.trace if e[0] == "compact")
    for tree, cpu in zip(trees, cpus):
        assert tree.trace == cpu.log
        assert [len(lv) for lv in tree.levels] == [len(lv.runs) for lv in cpu.levels]
        for glv, clv in zip(tree.levels, cpu.levels):
            for gr, cr in zip(glv, clv.runs):
                assert np.array_equal(oracle.as_run(gr.run), cr)
                assert np.array_equal(gr.fences.cpu().numpy().view(np.uint8).reshape(-1, 32), oracle.build_fences(cr, 64))
                assert np.array_equal(gr.bloom.cpu().numpy().view(np.uint8).reshape(-1, 16), oracle.build_bloom(cr, int(gr.bloom.shape[0])))
                if cr.shape[0] >= 5000:
                    assert oracle.hash_index_check(cr, gr.index.cpu().numpy()) == 0
                else:
                    assert gr.index is None


def test_sharded_trees_in_the_library_driver(oracle):
    """The same four trees driven by the library (lsm_driver_flush_many): every compaction output, probe batch, log and
    final tree equal the plain driver's for that tree alone.  One tree also gets hash indices, one has no filters."""
    from oracle import lsm_driver_oracle as drv
    from paper_2511_16138_amd import LsmDriver, lsm_driver_flush_many
    from workloads import lsm, rng
    print("sharded trees, library driver", flush=True)
    n_shards, window = 4, 16 * 128
    traces = [lsm.config5(device=dev(), seed=rng.SEED + 1000 * i, tree_total=200_000 + 50_000 * i, buffer_entries=360,
                          ops_per_phase=2048, batch_requests=128) for i in range(n_shards)]
    bits = [16, 16, 0, 16]
    index_from = [0, 5000, 0, 0]
    outs = [[] for _ in range(n_shards)]
    want_outs = [[] for _ in range(n_shards)]
    trees = [LsmDriver(tr.buffer_entries, size_ratio=tr.size_ratio, window_ops=window, t_grid=(2, 16), bloom_bits=bits[i],
                       hash_index_from=index_from[i], on_compaction=(lambda level, out, i=i: outs[i].append(out)))
             for i, tr in enumerate(traces)]
    cpus = [drv.DriverOracle(tr.buffer_entries, T=tr.size_ratio, K=1, window_ops=window, threshold=0.2, t_grid=(2, 16),
                             page_entries=64.0, fpr=drv.bloom_fpr(bits[i]), on_compact=want_outs[i].append) for i, tr in enumerate(traces)]
    for tr, tree, cpu in zip(traces, trees, cpus):
        for level, r in enumerate(tr.workload.runs):
            tree.load_run(level + 1, r)
            cpu.install(level + 1, [r.cpu()])
    at = [0] * n_shards
    rounds = together = 0
    while any(at[i] < len(traces[i].events) for i in range(n_shards)):
        runs = [None] * n_shards
        for i, (tr, tree, cpu) in enumerate(zip(traces, trees, cpus)):
            if at[i] >= len(tr.events):
                continue
            (kind, idx, _phase), n_writes = tr.events[at[i]], tr.write_ops_between[at[i]]
            at[i] += 1
            if n_writes:
                tree.note_writes(n_writes)
                cpu.writes(n_writes)
            if kind == "flush":
                runs[i] = tr.flush_runs[idx]
                cpu.flush(runs[i].cpu())
            else:
                q, nb = tr.probe_batch(idx)
                ghl, ghits = tree.probe(q, nb)
                chl, chits = cpu.probe(q.cpu(), nb.cpu())
                assert np.array_equal(ghl.cpu().numpy().astype(np.uint32), chl)
                assert np.array_equal(ghits.cpu().numpy().view(oracle.HIT_DTYPE).reshape(chits.shape), chits)
        lsm_driver_flush_many(trees, runs)
        rounds += 1
        together += sum(1 for r in runs if r is not None) > 1
        for i, (tree, cpu) in enumerate(zip(trees, cpus)):
            assert len(outs[i]) == len(want_outs[i])
            for got, want in zip(outs[i], want_outs[i]):
                assert np.array_equal(oracle.as_run(got), want), f"tree {i}: a compaction output differs"
            outs[i].clear()
            want_outs[i].clear()
            log = tree.trace
            assert log[-2:] == cpu.log[-2:] and len(log) == len(cpu.log), (i, log[-3:], cpu.log[-3:])
    assert together > rounds // 2          # most rounds flushed several trees at once
    for i, (tree, cpu) in enumerate(zip(trees, cpus)):
        assert tree.trace == cpu.log and any(e[0] == "move" for e in cpu.log)
        check_native_tree(oracle, tree, cpu, bits[i], index_from[i])
        tree.close()


@pytest.mark.parametrize("seed,start_k,t_grid", [(11, 1, (2, 5)), (12, 3, (2, 5)), (13, 2, (4, 4))])
def test_drivers_on_degenerate_trees(oracle, seed, start_k, t_grid):
    """Both drivers against the plain one where the trees are tiny and awkward: a key space of 300 keys with half of
    all writes tombstones (compactions whose output is empty, levels that empty out again), empty write buffers,
    several runs per level from the start, a window so short that (T, K) is searched again every few operations."""
    import brute
    from gpu_util import to_dev
    from oracle import lsm_driver_oracle as drv
    from paper_2511_16138_amd import LsmDriver
    from paper_2511_16138_amd.tree import AdaptiveLsmTree, GpuBackend
    print("degenerate trees", seed, start_k, t_grid, flush=True)
    rs = np.random.RandomState(seed)
    key_of = lambda k: int(k).to_bytes(32, "big")
    M, window = 40, 64
    py = AdaptiveLsmTree(GpuBackend(bloom_bits=16, hash_index_from=50), M, size_ratio=4, runs_per_level=start_k, window_ops=window,
                         t_grid=t_grid)
    nat = LsmDriver(M, size_ratio=4, runs_per_level=start_k, window_ops=window, t_grid=t_grid, bloom_bits=16, hash_index_from=50)
    cpu = drv.DriverOracle(M, T=4, K=start_k, window_ops=window, threshold=0.2, t_grid=t_grid, page_entries=64.0, fpr=drv.bloom_fpr(16))
    seq = 0
    empties = empty_outputs = 0
    for step in range(260):
        if step < 4 or rs.rand() < 0.7:
            n = 0 if rs.rand() < 0.1 else int(rs.randint(1, M + 1))
            keys = sorted(rs.choice(300, size=n, replace=False).tolist())
            raw = []
            for k in keys:
                seq += 1
                tomb = step < 4 or rs.rand() < 0.5     # the first buffers hold deletions only: they merge to nothing
                raw.append(brute.pack_entry(key_of(k), seq, brute.TOMBSTONE if tomb else brute.PUT, vptr=seq, vlen=k))
            run = brute.run_from_raw(raw)
            empties += n == 0
            for d in (py, nat):
                d.note_writes(max(n, 1))
            cpu.writes(max(n, 1))
            g_run = to_dev(run)
            py.flush(g_run)
            nat.flush(g_run)
            cpu.flush(run)
        else:
            n_req, max_blocks = 24, 6
            q = np.zeros((n_req, max_blocks, 32), np.uint8)
            nb = rs.randint(0, max_blocks + 1, size=n_req).astype(np.int32)
            for r in range(n_req):
                for j in range(max_blocks):
                    q[r, j] = np.frombuffer(key_of(rs.randint(0, 300)), np.uint8)
            gq = torch.from_numpy(q.view(np.int64).reshape(n_req, max_blocks, 4).copy()).to(dev())
            gnb = torch.from_numpy(nb).to(dev())
            want_len, want_hits = cpu.probe(q, nb.astype(np.uint32))
            for d in (py, nat):
                hl, hits = d.probe(gq, gnb)
                assert np.array_equal(hl.cpu().numpy().astype(np.uint32), want_len), step
                assert np.array_equal(hits.cpu().numpy().view(oracle.HIT_DTYPE).reshape(want_hits.shape), want_hits), step
        assert py.trace == cpu.log and nat.trace == cpu.log, (step, py.trace[-3:], nat.trace[-3:], cpu.log[-3:])
        empty_outputs = sum(1 for e in cpu.log if e[0] == "compact" and e[4] == 0)
    assert empties >= 5 and (empty_outputs >= 1 or start_k == 3)   # with three runs per level the deletions are not merged alone
    kinds = {e[0] for e in cpu.log}
    assert {"compact", "move", "policy", "adopt", "probe"} <= kinds
    assert len({e[1:3] for e in cpu.log if e[0] == "policy"}) > 1
    assert [len(lv) for lv in py.levels] == [len(lv.runs) for lv in cpu.levels]
    for glv, clv in zip(py.levels, cpu.levels):
        for gr, cr in zip(glv, clv.runs):
            assert np.array_equal(oracle.as_run(gr.run), cr)
    check_native_tree(oracle, nat, cpu, 16, 50)
    nat.close()


@pytest.mark.parametrize("seed", [1, 2, 3, 4])
def test_flush_many_on_degenerate_trees(oracle, seed):
    """lsm_driver_flush_many where it is awkward: one to four tiny trees with different settings, trees that sit a round
    out, empty write buffers (still a flush), deletion-only buffers that merge to nothing."""
    import brute
    from gpu_util import to_dev
    from oracle import lsm_driver_oracle as drv
    from paper_2511_16138_amd import LsmDriver, lsm_driver_flush_many
    print("flush_many on degenerate trees", seed, flush=True)
    rs = np.random.RandomState(1000 + seed)
    key_of = lambda k: int(k).to_bytes(32, "big")
    n_trees, M, window = int(rs.randint(2, 5)), 40, 64
    cfgs = [(int(rs.randint(1, 4)), (2, int(rs.randint(2, 6))), int(rs.choice([0, 16])), int(rs.choice([0, 30]))) for _ in range(n_trees)]
    nats = [LsmDriver(M, size_ratio=4, runs_per_level=k, window_ops=window, t_grid=tg, bloom_bits=b, hash_index_from=ix) for k, tg, b, ix in cfgs]
    cpus = [drv.DriverOracle(M, T=4, K=k, window_ops=window, threshold=0.2, t_grid=tg, page_entries=64.0, fpr=drv.bloom_fpr(b))
            for k, tg, b, ix in cfgs]
    seq = skipped = empty = 0
    for step in range(150):
        runs = []
        for i in range(n_trees):
            if rs.rand() < 0.25:
                runs.append(None)               # this tree has nothing to flush in this round
                skipped += 1
                continue
            n = 0 if rs.rand() < 0.1 else int(rs.randint(1, M + 1))
            empty += n == 0
            raw = []
            for k in sorted(rs.choice(300, size=n, replace=False).tolist()):
                seq += 1
                tomb = step < 3 or rs.rand() < 0.5
                raw.append(brute.pack_entry(key_of(k), seq, brute.TOMBSTONE if tomb else brute.PUT, vptr=seq, vlen=k))
            run = brute.run_from_raw(raw)
            nats[i].note_writes(max(n, 1))
            cpus[i].writes(max(n, 1))
            cpus[i].flush(run)
            runs.append(to_dev(run))
        lsm_driver_flush_many(nats, runs)
        if step % 5 == 4:
            n_req, max_blocks = 16, 5
            q = np.zeros((n_req, max_blocks, 32), np.uint8)
            nb = rs.randint(0, max_blocks + 1, size=n_req).astype(np.int32)
            for r in range(n_req):
                for j in range(max_blocks):
                    q[r, j] = np.frombuffer(key_of(rs.randint(0, 300)), np.uint8)
            gq = torch.from_numpy(q.view(np.int64).reshape(n_req, max_blocks, 4).copy()).to(dev())
            gnb = torch.from_numpy(nb).to(dev())
            for nat, cpu in zip(nats, cpus):
                want_len, want_hits = cpu.probe(q, nb.astype(np.uint32))
                hl, hits = nat.probe(gq, gnb)
                assert np.array_equal(hl.cpu().numpy().astype(np.uint32), want_len), step
                assert np.array_equal(hits.cpu().numpy().view(oracle.HIT_DTYPE).reshape(want_hits.shape), want_hits), step
        for i, (nat, cpu) in enumerate(zip(nats, cpus)):
            assert nat.trace == cpu.log, (step, i, nat.trace[-3:], cpu.log[-3:])
    assert skipped > 20 and empty > 5
    for (k, tg, b, ix), nat, cpu in zip(cfgs, nats, cpus):
        check_native_tree(oracle, nat, cpu, b, ix)
        nat.close()


def test_flush_many_when_one_tree_fails(oracle):
    """A tree whose compaction is refused (65 runs in a level) ends lsm_driver_flush_many with an error; the run that has
    come to rest in the other tree is complete all the same: a copy of the caller's buffer, with fences and a filter."""
    import brute
    from gpu_util import to_dev
    from paper_2511_16138_amd import LsmDriver, LsmError, lsm_driver_flush_many
    key_of = lambda k: int(k).to_bytes(32, "big")
    run_of = lambda keys: brute.run_from_raw([brute.pack_entry(key_of(k), 1, brute.PUT, vptr=k, vlen=k) for k in keys])
    good, bad = LsmDriver(200, size_ratio=4, bloom_bits=16), LsmDriver(200, size_ratio=4, bloom_bits=16)
    for i in range(64):
        bad.load_run(1, to_dev(run_of([i])))
    want = run_of(range(150))
    buffer = to_dev(want)
    with pytest.raises(LsmError):
        lsm_driver_flush_many([good, bad], [buffer, to_dev(run_of([70]))])
    buffer.zero_()
    q = np.stack([np.stack([np.frombuffer(key_of(k), np.uint8) for k in range(r, r + 8)]) for r in range(0, 200, 8)])
    gq = torch.from_numpy(q.view(np.int64).reshape(len(q), 8, 4).copy()).to(dev())
    nb = np.full(len(q), 8, np.int32)
    hit_len, hits = good.probe(gq, torch.from_numpy(nb).to(dev()))
    want_len, want_hits = oracle.probe(gq.cpu(), torch.from_numpy(nb), [to_dev(want).cpu()])
    assert np.array_equal(hit_len.cpu().numpy(), np.asarray(want_len).reshape(-1))
    for r, n in enumerate(np.asarray(want_len).reshape(-1)):
        assert hits[r, :n].cpu().numpy().tobytes() == np.asarray(want_hits)[r, :n].tobytes()
    good.flush(to_dev(run_of(range(150, 180))))  # the tree goes on
    assert good.levels()[0][2] == 1


@pytest.mark.parametrize("buffer_entries,trees", [(300, 1), (1500, 1), (3600, 1), (9000, 1), (40, 2), (1500, 18), (9000, 3), (30_000, 1), (70_000, 2)])
@pytest.mark.parametrize("bits", [3, 16, 64])
def test_filters_of_driver_runs_byte_for_byte(oracle, buffer_entries, trees, bits):
    """Every run of a live tree has the filter of its entries whenever a flush has returned: filters built right behind the
    merge (in LDS, one share and several, two sizes, from the keys' hashes, and with atomics), those of runs that may move down, and those of flushed runs;
    a third of all writes repeat keys or delete, so that lengths fall short of their upper bounds."""
    from paper_2511_16138_amd import LsmDriver, lsm_driver_flush_many
    print("driver filters", buffer_entries, trees, bits, flush=True)
    rs = np.random.RandomState(buffer_entries + bits)
    drivers = [LsmDriver(buffer_entries, size_ratio=4, window_ops=1 << 30, bloom_bits=bits) for _ in range(trees)]
    seq = 0
    for step in range(7):
        runs = []
        for _ in drivers:
            lead = np.unique(rs.randint(0, buffer_entries * 12, size=buffer_entries))
            a = np.zeros((len(lead), 64), dtype=np.uint8)
            a[:, :8] = lead.astype(">u8").view(np.uint8).reshape(-1, 8)
            rec = a.view(oracle.ENTRY_DTYPE).reshape(-1)
            rec["seqno"] = seq + np.arange(len(lead))
            rec["type"] = rs.rand(len(lead)) < 0.2
            seq += len(lead)
            runs.append(torch.from_numpy(a.view(np.int64).reshape(-1, 8)).to(dev()))
        if trees == 1:
            drivers[0].flush(runs[0])
        else:
            lsm_driver_flush_many(drivers, runs)
        for d in drivers[:: max(1, trees // 3)]:
            for t in d.tree():
                n, blocks = int(t.run.n), int(t.bloom.n_blocks)
                assert n > 0 and blocks == oracle.bloom_blocks(n, bits)
                entries = d.read(t.run.entries, n, 8).cpu()
                got = d.read(t.bloom.blocks, blocks, 2).cpu().numpy().view(np.uint8).reshape(-1, 16)
                assert np.array_equal(got, oracle.build_bloom(entries, blocks)), (step, n, blocks)


def test_filter_of_keys_whose_hashes_are_close_together(oracle):
    """A merged run all of whose hashes fall into a twentieth of the filter: ranges of blocks with far more hashes than there is room
    for are built all the same, and the others stay empty."""
    from paper_2511_16138_amd import LsmDriver
    rs = np.random.RandomState(5)
    a = np.zeros((1_700_000, 64), dtype=np.uint8)
    a[:, :16] = rs.randint(0, 256, size=(a.shape[0], 16), dtype=np.uint8)
    a = a[oracle.key_hashes(a) < (1 << 64) // 20][:80_000]
    assert a.shape[0] == 80_000
    driver = LsmDriver(40_000, size_ratio=4, window_ops=1 << 30, bloom_bits=16)
    for part in (a[:40_000], a[40_000:]):
        words = part[:, :16].copy().view(">u8")
        part = np.ascontiguousarray(part[np.lexsort((words[:, 1], words[:, 0]))])
        driver.flush(torch.from_numpy(part.view(np.int64).reshape(-1, 8)).to(dev()))
    t, = driver.tree()
    n, blocks = int(t.run.n), int(t.bloom.n_blocks)
    assert n == 80_000 and blocks == oracle.bloom_blocks(n, 16)
    got = driver.read(t.bloom.blocks, blocks, 2).cpu().numpy().view(np.uint8).reshape(-1, 16)
    assert np.array_equal(got, oracle.build_bloom(driver.read(t.run.entries, n, 8).cpu(), blocks))
