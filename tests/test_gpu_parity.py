"""GPU parity: the HIP library, called through its C ABI, against the CPU checker, bit for bit.

Sizes here are ones the checker finishes in seconds; they still span many tiles (a tile is
about a thousand entries) and ragged tails.  Full-size cases are in test_gpu_fullsize.py.
"""
import ctypes

import numpy as np
import pytest
import torch

import brute
from brute import PUT, TOMBSTONE
from gpu_util import as_bytes, assert_probe_equal, build_tree, compact_gpu, dev, probe_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    import paper_2511_16138_amd as lsmgpu
    lsmgpu.binding._load()  # raises if the HIP library has not been built
    assert torch.cuda.is_available()
    return lsmgpu


@pytest.fixture(scope="module")
def cfg1():
    from workloads import lsm
    return lsm.config1(device=dev())


def _check_compact(g, oracle, runs, flags):
    got = compact_gpu(g, runs, flags)
    want = oracle.compact([r.cpu() for r in runs], flags & 1)
    assert got.shape[0] == want.shape[0]
    assert np.array_equal(as_bytes(got).reshape(-1, 64), want)
    return got


# ------------------------------------------------------------------ compaction
SHORT, FILL = 512, 256  # shortest tile spacing, tiles an input is spread over before its tiles grow


@pytest.mark.parametrize("flags", [0, 1])
def test_config1_compaction(g, oracle, cfg1, flags):
    print("config1 compaction flags", flags, flush=True)
    _check_compact(g, oracle, cfg1.runs, flags)


def test_generator_is_identical_on_cpu_and_gpu(cfg1):
    from workloads import lsm
    w = lsm.config1(device="cpu")
    assert all(torch.equal(a.cpu(), b) for a, b in zip(cfg1.runs, w.runs))


@pytest.mark.parametrize("scale,flags", [(256, 1), (256, 0), (64, 1), (12, 1), (6, 1)])  # 5.6M and 11.2M entries: boundaries searched between rows
def test_scaled_config3_tiered_16way(g, oracle, scale, flags):
    from workloads import lsm
    print("config3 scale", scale, "flags", flags, flush=True)
    w = lsm.config3(device=dev(), scale=scale)
    _check_compact(g, oracle, w.runs, flags)


@pytest.mark.parametrize("flags", [0, 1])
def test_scaled_config2_leveled_two_way(g, oracle, flags):
    from workloads import lsm
    print("config2 scale 50 flags", flags, flush=True)
    w = lsm.config2(device=dev(), scale=50)  # 40,000 + 400,000 entries
    _check_compact(g, oracle, w.runs, flags)


@pytest.mark.parametrize("k", [1, 2, 3, 5, 7, 16, 17, 33, 64])
def test_run_counts_and_ragged_lengths(g, oracle, k):
    """Any run count up to the maximum, uneven and empty runs, lengths that are not tile multiples."""
    from workloads import lsm
    print("ragged k", k, flush=True)
    w = lsm.config3(device=dev(), scale=1024)  # 16 runs x 4096
    rs = np.random.RandomState(k)
    runs = []
    for j in range(k):
        src = w.runs[j % 16]
        n = int(rs.choice([0, 1, 7, 959, 960, 961, 1024, 2500, 4096]))
        start = int(rs.randint(0, 4096 - n + 1))
        r = src[start:start + n].clone()
        r[:, 4] = r[:, 4] ^ (j * 0x9E3779B1)  # different versions in different runs
        runs.append(r)
    for flags in (0, 1):
        _check_compact(g, oracle, runs, flags)


def test_runs_from_any_iterable(g, oracle):
    """lsm_compact takes its runs as any iterable: a list, a generator, one tensor of runs of the same length."""
    rs = np.random.RandomState(3)
    stacked = torch.stack(_runs_of(oracle, rs, [500, 500, 500], 4000))
    want = oracle.compact([r.cpu() for r in stacked], 0)
    for runs in (list(stacked), (r for r in stacked), stacked):
        out, n_out = g.lsm_compact(runs, 0)
        assert int(n_out.item()) == want.shape[0]
        assert np.array_equal(as_bytes(out[: want.shape[0]]).reshape(-1, 64), want)


@pytest.mark.parametrize("k", [3, 4, 5, 16, 32, 33, 64])
@pytest.mark.parametrize("shape", ["nested", "stairs", "copies", "one long"])
def test_tile_boundaries_of_uneven_runs(g, oracle, k, shape):
    """Boundary searches where evenly spaced records say little: every run inside one gap of the run before, runs one
    behind the other, the same keys in every run, one long run beside runs of a few entries."""
    print("boundaries", k, shape, flush=True)
    rs = np.random.RandomState(k)
    total = 30000
    runs = []
    for j in range(k):
        n = total // k if shape != "one long" else (total if j == k // 2 else 3)
        if shape == "nested":
            half = 1 << (62 - (58 * j) // k)
            lead = (1 << 62) + rs.randint(-(half >> 1), half >> 1, size=n)
        elif shape == "stairs":
            lead = ((k - j) << 56) + rs.randint(0, 1 << 56, size=n)
        elif shape == "copies":
            lead = np.arange(n, dtype=np.int64) * 12345
        else:
            lead = rs.randint(0, 1 << 40, size=n)
        a = np.zeros((n, 64), dtype=np.uint8)
        a[:, :8] = lead.astype(">u8").view(np.uint8).reshape(n, 8)
        a = a[np.unique(lead, return_index=True)[1]]
        rec = a.view(oracle.ENTRY_DTYPE).reshape(-1)
        rec["seqno"] = rs.randint(0, 1 << 40, size=rec.shape[0])
        rec["type"] = (rs.rand(rec.shape[0]) < 0.1).astype(np.uint8)
        runs.append(to_dev(a))
    for flags in (0, 1):
        _check_compact(g, oracle, runs, flags)


@pytest.mark.parametrize("case", ["same_keys", "interleaved", "one_inside_the_other", "short_and_long", "batch"])
def test_two_runs_many_tiles(g, oracle, case):
    """Two runs (boundaries by bisection on the merge path): every key in both runs (each boundary falls between the
    two versions of some key), keys that alternate between the runs, one run's key range inside the other's, a short
    run against a long one, and the same pairs as jobs of a batch - dozens of tiles each, both flags."""
    from workloads import lsm
    print("two runs", case, flush=True)
    w = lsm.config3(device=dev(), scale=64)           # runs of 65,536 entries
    base = torch.from_numpy(oracle.compact([w.runs[0].cpu(), w.runs[1].cpu()], 0).view(np.int64).reshape(-1, 8).copy()).to(dev())
    older = base.clone()
    older[:, 4] = older[:, 4] - 1                     # the same keys with smaller seqnos
    if case == "same_keys":
        pairs = [(base[:60_000], older[:60_000])]
    elif case == "interleaved":
        pairs = [(base[0:100_000:2].contiguous(), older[1:100_000:2].contiguous())]
    elif case == "one_inside_the_other":
        pairs = [(base[30_000:50_000].contiguous(), older[:90_000].contiguous()), (older[:90_000].contiguous(), base[30_000:50_000].contiguous())]
    elif case == "short_and_long":
        pairs = [(base[77:78].contiguous(), older[:70_000].contiguous()), (base[:70_000].contiguous(), older[5_000:5_003].contiguous())]
    else:
        pairs = [(base[:9_000].contiguous(), older[:9_000].contiguous()), (base[0:30_000:2].contiguous(), older[1:30_000:2].contiguous()),
                 (base[100:101].contiguous(), older[:5_000].contiguous())]
    for flags in (0, 1):
        if case == "batch":
            outs, n_out = g.lsm_compact_batch([(list(p), flags) for p in pairs])
            torch.cuda.synchronize()
            for p, out, n in zip(pairs, outs, n_out.cpu().tolist()):
                want = oracle.compact([r.cpu() for r in p], flags & 1)
                assert n == want.shape[0] and np.array_equal(as_bytes(out[:n]).reshape(-1, 64), want)
        else:
            for p in pairs:
                _check_compact(g, oracle, list(p), flags)


def test_degenerate_inputs(g, oracle):
    from workloads import lsm
    print("degenerate inputs", flush=True)
    w = lsm.config3(device=dev(), scale=1024)
    a = w.runs[0]
    empty = a[:0]
    assert compact_gpu(g, [empty], 1).shape[0] == 0
    assert compact_gpu(g, [empty, empty, empty], 0).shape[0] == 0
    _check_compact(g, oracle, [empty, a[:5], empty], 0)
    _check_compact(g, oracle, [a], 1)  # single run: tombstone filter
    _check_compact(g, oracle, [a], 0)  # single run: copy
    # k identical key sets: the run with the largest seqnos survives whole
    runs = []
    for j, base in enumerate([300, 900, 100, 500]):
        r = a.clone()
        r[:, 4] = base * 100000 + torch.arange(a.shape[0], device=a.device)
        r[:, 6] = j
        runs.append(r)
    got = _check_compact(g, oracle, runs, 0)
    assert bool((got[:, 6] == 1).all())
    # all tombstones into the last level: nothing survives
    t = a.clone()
    t[:, 5] = 1
    assert compact_gpu(g, [t, t[:100].clone()], 1).shape[0] == 0
    # equal seqnos: lowest run index wins
    r0, r1 = a.clone(), a.clone()
    r0[:, 6], r1[:, 6] = 111, 222
    got = _check_compact(g, oracle, [r0, r1], 0)
    assert bool((got[:, 6] == 111).all())
    # disjoint key ranges given in the "wrong" order: concatenation
    _check_compact(g, oracle, [a[3000:], a[:1000], a[1000:3000]], 0)


def test_adversarial_keys_long_common_prefixes(g, oracle):
    """Keys that differ only in their last bytes, and heavy duplication across runs."""
    print("adversarial keys", flush=True)
    rs = np.random.RandomState(77)
    runs = []
    for j in range(6):
        codes = np.unique(rs.randint(0, 6000, size=4000))
        raws = []
        for c in codes:
            key = b"\xAB" * 29 + bytes([(c >> 16) & 0xFF, (c >> 8) & 0xFF, c & 0xFF])
            raws.append(brute.pack_entry(key, int(rs.randint(0, 1 << 62)), TOMBSTONE if rs.rand() < 0.2 else PUT,
                                         vptr=int(rs.randint(1 << 60)), vlen=j, pad0=bytes([j] * 7), pad1=j))
        runs.append(to_dev(brute.run_from_raw(raws)))
    for flags in (0, 1):
        _check_compact(g, oracle, runs, flags)


@pytest.mark.parametrize("n_runs,n_heads,long_groups", [(5, 3000, 0), (16, 1500, 0), (4, 2500, 6)])
def test_keys_that_tie_in_their_first_14_bytes(g, oracle, n_runs, n_heads, long_groups):
    """Small groups of keys equal in the bytes the merge orders by and different after them; with
    long_groups some groups are longer than the in-place repair handles."""
    print("prefix-tie groups", n_runs, n_heads, long_groups, flush=True)
    rs = np.random.RandomState(1000 + n_runs)
    runs = [to_dev(brute.run_from_raw(r)) for r in brute.tie_group_runs(rs, n_runs, n_heads, long_groups)]
    for flags in (0, 1):
        _check_compact(g, oracle, runs, flags)


def _tied_runs(oracle, rs, k, group, total, seqnos):
    """k runs of about `total` entries in all; keys come in groups of `group` that share 14 bytes and differ behind, and are in one to three runs."""
    runs = []
    for j in range(k):
        code = np.unique(rs.randint(0, max(4, int(total * 0.8)), size=total // k))
        head, tail = code // group, code % group
        a = np.zeros((code.size, 64), dtype=np.uint8)
        a[:, :8] = (head.astype(np.uint64) * np.uint64(0x9E3779B97F4A7C15) >> np.uint64(1)).astype(">u8").view(np.uint8).reshape(-1, 8)
        spot = np.array([14, 20, 30])[head % 3]
        a[np.arange(code.size), spot] = tail >> 8
        a[np.arange(code.size), spot + 1] = tail & 255
        words = a[:, :32].copy().view(">u8")
        a = a[np.lexsort((words[:, 3], words[:, 2], words[:, 1], words[:, 0]))]
        rec = a.view(oracle.ENTRY_DTYPE).reshape(-1)
        rec["seqno"] = rs.randint(0, seqnos, size=code.size)
        rec["type"] = (rs.rand(code.size) < 0.1).astype(np.uint8)
        rec["vptr"] = np.arange(code.size) + (j << 40)
        runs.append(a)
    return runs


@pytest.mark.parametrize("k", [2, 5, 17])
@pytest.mark.parametrize("group", [2, 33, 34, 600])  # members of a prefix-tie group in all runs together, about: settled by neighbours, or not
def test_prefix_ties_on_both_sides_of_the_short_form(g, oracle, k, group):
    """One tile, tiles of up to and of more than 1,024 entries, 256 tiles and more: keys that share 14 bytes with others and differ behind."""
    rs = np.random.RandomState(100 * k + group)
    for total in (1000, 1100, 1900, 60_000, 300_000, 256 * (2048 - k) - 1, 256 * (2048 - k) + 3000):
        print("prefix ties, short form", k, group, total, flush=True)
        runs = [to_dev(r) for r in _tied_runs(oracle, rs, k, group, total, 1 << 40 if total & 1 else 3)]
        _check_compact(g, oracle, runs, int(group & 1))


@pytest.mark.parametrize("k", [1, 3, 17])
@pytest.mark.parametrize("group", [1, 40, 600])
def test_ranges_of_about_as_many_entries_as_threads(g, oracle, k, group):
    """Key ranges that hold 1, 505 .. 520, 1,000 and 1,500 entries of the runs: one entry per thread up to 512; keys that share 14 bytes."""
    print("ranges around 512 entries", k, group, flush=True)
    rs = np.random.RandomState(k + group)
    runs = _tied_runs(oracle, rs, k, group, 4000, 4)
    keys = sorted(bytes(e[:32]) for r in runs for e in r)  # of all runs, in order: range i holds the first n[i] of them, and other versions of the last
    n = [1, *range(505, 521), 1000, 1500]
    hi = np.frombuffer(b"".join(keys[i] for i in n), dtype=np.uint8).reshape(-1, 32)
    lo = np.zeros_like(hi)
    tree = build_tree(g, [to_dev(r) for r in runs])
    as_key = lambda x: torch.from_numpy(x.copy().view(np.int64).reshape(-1, 4)).to(dev())  # noqa: E731
    for slot in (1500, 400):
        entries, counts = g.lsm_range_scan(tree, as_key(lo), as_key(hi), slot)
        torch.cuda.synchronize()
        for i, end in enumerate(hi):
            cut = [np.ascontiguousarray(r[[bytes(e[:32]) < bytes(end) for e in r]]) for r in runs]
            want = oracle.compact(cut, 1)
            count = int(counts[i].item()) & 0xFFFFFFFF
            if want.shape[0] > slot:
                assert count == 0xFFFFFFFF
                continue
            assert count == want.shape[0]
            assert np.array_equal(as_bytes(entries[i, :count]).reshape(-1, 64), want)


@pytest.mark.parametrize("separate", [False, True])
def test_first_key_words_that_differ_in_one_bit(g, oracle, separate):
    """Two first key words that differ in their last bit next to one far away (any scaled or
    shortened form of the first word confuses the close pair), mixed inside every run or
    kept in separate runs; the rest of the key is random."""
    print("close first words, separate =", separate, flush=True)
    rs = np.random.RandomState(31 + separate)
    runs = [to_dev(brute.run_from_raw(r)) for r in brute.close_first_words_runs(rs, 6, 1500, separate)]
    for flags in (0, 1):
        _check_compact(g, oracle, runs, flags)


def test_results_do_not_depend_on_repetition(g, cfg1):
    print("determinism", flush=True)
    first = compact_gpu(g, cfg1.runs, 1).clone()
    for _ in range(5):
        assert torch.equal(compact_gpu(g, cfg1.runs, 1), first)


def test_compaction_is_associative_on_gpu(g, oracle, cfg1):
    print("associativity", flush=True)
    newest_first = cfg1.runs
    inner = compact_gpu(g, newest_first[2:], 0).contiguous()        # the two oldest runs
    nested = compact_gpu(g, [newest_first[0], newest_first[1], inner], 1)
    flat = compact_gpu(g, newest_first, 1)
    assert torch.equal(nested, flat)


def test_validate_flag(g, cfg1):
    print("validate", flush=True)
    a = cfg1.runs[0].clone()
    out, n_out = g.lsm_compact([a, cfg1.runs[1]], g.LSM_VALIDATE)
    assert int(n_out.item()) > 0
    bad = a.clone()
    bad[[10, 11]] = bad[[11, 10]]
    with pytest.raises(g.LsmError) as e:
        g.lsm_compact([bad, cfg1.runs[1]], g.LSM_VALIDATE)
    assert e.value.code == -5
    bad = a.clone()
    bad[5, 5] = 7
    with pytest.raises(g.LsmError) as e:
        g.lsm_compact([cfg1.runs[1], bad], g.LSM_VALIDATE)
    assert e.value.code == -6
    small = torch.empty((10, 8), dtype=torch.int64, device=a.device)
    with pytest.raises(g.LsmError) as e:
        g.lsm_compact([a], 0, out=small)
    assert e.value.code == -3


# ------------------------------------------------------------------ fences
@pytest.mark.parametrize("stride", [1, 3, 64, 100, 16383, 16384, 100000])
def test_fences(g, oracle, cfg1, stride):
    print("fences stride", stride, flush=True)
    run = cfg1.runs[0]
    f = g.lsm_build_fences(run, stride)
    torch.cuda.synchronize()
    assert np.array_equal(as_bytes(f).reshape(-1, 32), oracle.build_fences(run.cpu(), stride))


# ------------------------------------------------------------------ probe
def test_config1_probe_before_and_after_compaction(g, oracle, cfg1):
    from workloads import lsm
    print("config1 probe", flush=True)
    q, nb = lsm.queries_config1(cfg1, 4096)
    runs_cpu = [r.cpu() for r in cfg1.runs]
    want = oracle.probe(q, nb, runs_cpu)
    got = probe_gpu(g, q, nb, build_tree(g, cfg1.runs))
    assert_probe_equal(oracle, got, want)
    assert 0.05 < float((want[0] == 0).mean()) < 0.6 and want[0].max() > 32
    for flags in (0, 1):
        merged = compact_gpu(g, cfg1.runs, flags).contiguous()
        got2 = probe_gpu(g, q, nb, build_tree(g, [merged]))
        assert_probe_equal(oracle, got2, oracle.probe(q, nb, [merged.cpu()]))
        assert np.array_equal(got2[0], got[0])                      # same prefix lengths
        assert np.array_equal(got2[1][..., 0], got[1][..., 0])      # same pointers
        assert np.array_equal(got2[1][..., 1] & 0xFFFFFFFF, got[1][..., 1] & 0xFFFFFFFF)  # same lengths


@pytest.mark.parametrize("stride", [1, 7, 64, 1000])
def test_probe_fence_strides_and_row_pitches(g, oracle, cfg1, stride):
    from workloads import lsm
    print("probe stride", stride, flush=True)
    q, nb = lsm.make_queries(cfg1.universe, 300, 1, 100, 0.6, 0.3, None, stream=5, row_blocks=100)
    want = oracle.probe(q, nb, [r.cpu() for r in cfg1.runs])
    assert_probe_equal(oracle, probe_gpu(g, q, nb, build_tree(g, cfg1.runs, stride)), want)


def test_probe_holes_absent_keys_and_edges(g, oracle):
    """A hole ends the prefix even if later blocks are present; keys between, below and above
    the stored keys miss; tombstoned keys are not live; repeated keys are fine."""
    print("probe holes", flush=True)
    rs = np.random.RandomState(21)
    runs_raw = brute.random_runs(rs, 5, 400, 3000, (30, 31), tomb_p=0.25)
    runs = [to_dev(brute.run_from_raw(r)) for r in runs_raw]
    present = sorted({r[:32] for run in runs_raw for r in run})
    requests = []
    for _ in range(600):
        n = int(rs.randint(0, 41))
        req = []
        for _ in range(n):
            u = rs.rand()
            if u < 0.8:
                req.append(present[int(rs.randint(len(present)))])
            elif u < 0.9:
                k = bytearray(present[int(rs.randint(len(present)))]); k[29] = 1; req.append(bytes(k))
            else:
                req.append(bytes(rs.randint(0, 256, size=32).astype(np.uint8)))
        requests.append(req)
    requests += [[b"\x00" * 32], [b"\xff" * 32], []]
    q = np.zeros((len(requests), 40, 32), dtype=np.uint8)
    nb = np.zeros(len(requests), dtype=np.int32)
    for i, req in enumerate(requests):
        nb[i] = len(req)
        for j, k in enumerate(req):
            q[i, j] = np.frombuffer(k, dtype=np.uint8)
    qd = torch.from_numpy(q.view(np.int64).reshape(len(requests), 40, 4).copy()).to(dev())
    nbd = torch.from_numpy(nb).to(dev())
    # random_runs draws seqnos at random; the tree precondition wants newer runs to hold larger ones
    ordered = []
    for j, r in enumerate(runs):
        r = r.clone(); r[:, 4] = (len(runs) - j) * (1 << 40) + (r[:, 4] & 0xFFFFF); ordered.append(r)
    want = oracle.probe(q, nb.astype(np.uint32), [r.cpu() for r in ordered])
    assert_probe_equal(oracle, probe_gpu(g, qd, nbd, build_tree(g, ordered)), want)
    assert (want[0] > 3).any() and (want[0] == 0).any()


def test_probe_empty_tree_and_empty_runs(g, oracle, cfg1):
    from workloads import lsm
    print("probe empty", flush=True)
    q, nb = lsm.queries_config1(cfg1, 64)
    hl, hits = probe_gpu(g, q, nb, [])
    assert (hl == 0).all() and (hits == 0).all()
    empty = cfg1.runs[0][:0]
    tree = build_tree(g, [empty, cfg1.runs[3], empty])
    want = oracle.probe(q, nb, [empty.cpu(), cfg1.runs[3].cpu(), empty.cpu()])
    assert_probe_equal(oracle, probe_gpu(g, q, nb, tree), want)


def _runs_of(oracle, rs, lens, keys):
    """Sorted runs of these lengths, keys spread evenly over about range(keys)."""
    runs = []
    for n in lens:
        lead = np.cumsum(rs.randint(1, max(2, 2 * keys // max(n, 1)), size=n))
        a = np.zeros((n, 64), dtype=np.uint8)
        a[:, :8] = lead.astype(">u8").view(np.uint8).reshape(n, 8)
        rec = a.view(oracle.ENTRY_DTYPE).reshape(-1)
        rec["seqno"] = rs.randint(0, 1 << 40, size=n)
        rec["type"] = (rs.rand(n) < 0.1).astype(np.uint8)
        runs.append(to_dev(a))
    return runs


def _best_us(call, passes=5, reps=5):
    """Shortest mean time of `reps` calls, in us."""
    call()
    best = float("inf")
    for _ in range(passes):
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0.record()
        for _ in range(reps):
            call()
        t1.record()
        t1.synchronize()
        best = min(best, t0.elapsed_time(t1) / reps * 1e3)
    return best


@pytest.mark.parametrize("k,total", [(64, 1024 * 1984), (64, 1024 * 1984 + 1), (33, 200_001)])  # 65,536 pieces of tiles in runs, more
@pytest.mark.parametrize("shape", ["mixed", "stairs", "one long"])
def test_many_runs(g, oracle, k, total, shape):
    """More than 32 runs on both sides of the line where the boundaries' search changes; runs one after the other or one
    long run must not take the boundaries apart."""
    print("many runs", k, total, shape, flush=True)
    rs = np.random.RandomState(k)
    lens = np.full(k, total // k)
    if shape == "one long":
        lens[:] = rs.randint(0, 40, size=k)
    lens[k // 2] += total - lens.sum()
    runs = _runs_of(oracle, rs, lens, 2 * total)
    if shape == "stairs":
        for j, r in enumerate(runs):  # the keys' first byte, as stored
            r[:, 0] |= (j * 7) % k + 1
    _check_compact(g, oracle, runs, 1)
    if total < 1 << 20:  # a batch of it and a small job
        few = _runs_of(oracle, rs, [700, 900, 30], 4000)
        outs, n_out = g.lsm_compact_batch([(runs, 1), (few, 0)])
        for rr, flags, out, n in zip((runs, few), (1, 0), outs, n_out.tolist()):
            want = oracle.compact([r.cpu() for r in rr], flags)
            assert n == want.shape[0]
            assert np.array_equal(as_bytes(out[:n]).reshape(-1, 64), want)


def test_many_runs_one_after_the_other_are_not_slow(g, oracle):
    """64 runs that cover different keys take at most three times as long as 64 mixed ones.  (Trying the records of one run
    after the other for every boundary took five times as long.)"""
    rs = np.random.RandomState(8)
    runs = _runs_of(oracle, rs, [1024] * 64, 1 << 18)
    apart = [r.clone() for r in runs]
    for j, r in enumerate(apart):
        r[:, 0] |= j + 1
    out, n_out = torch.empty((1 << 16, 8), dtype=torch.int64, device=dev()), torch.zeros(1, dtype=torch.int64, device=dev())
    base, took = [_best_us(lambda: g.lsm_compact(rr, 0, out, n_out)) for rr in (runs, apart)]
    print(f"64 runs of 1,024 entries: mixed {base:.0f} us, one after the other {took:.0f} us", flush=True)
    assert took < 3 * base


def _launches(call):
    """Kernels (and other work) that a call puts on the stream: the nodes of a graph that records it."""
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    n = ctypes.c_size_t(0)
    assert ctypes.CDLL(path).hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


# For 3 to 16 runs both totals are searched between rows: see test_lines_between_the_ways_of_finding_boundaries.
@pytest.mark.parametrize("k,tiles,shape", [(k, tiles, "uneven") for k, tiles in [(1, 10240), (3, 10240), (5, 8192), (16, 5120), (17, 2048), (40, 2048)]]
                         + [(17, 2048, "copies"), (40, 2048, "copies")])
def test_searched_directly_or_on_samples(g, oracle, k, tiles, shape):
    """The longest input whose boundaries are searched in the runs themselves and the shortest that is sampled; runs of very
    different lengths, an empty one among them, and ones that cover a part of the keys only; or the same keys in every run, so
    that the samples tie."""
    rs = np.random.RandomState(k)
    for total in ((tiles - 1) * (2048 - k), (tiles - 1) * (2048 - k) + 1):
        print("direct or sampled", k, total, shape, flush=True)
        if shape == "copies":
            lens = np.full(k, total // k)
            lens[0] += total - lens.sum()
            one = _runs_of(oracle, rs, [int(lens[0])], 2 * total)[0]
            runs = [one[:n].clone() for n in lens]
            for r in runs:
                r[:, 4] = torch.randint(0, 1 << 40, (r.shape[0],), device=dev())
        else:
            lens = np.maximum(1, (total * rs.dirichlet(np.full(k, 0.7)) * 0.999).astype(np.int64))
            lens[0] = 0
            lens[-1] += total - lens.sum()
            runs = _runs_of(oracle, rs, lens, 2 * total)
            runs[min(1, k - 1)][:, 0] |= 1  # the keys' first byte, as stored: a run behind all others
        _check_compact(g, oracle, runs, int(total & 1))
        del runs
        torch.cuda.empty_cache()


# The longest input whose boundaries are found one way and the shortest of another way, and the launches of either with the merge's: a wave per
# boundary over the whole runs 2, between rows 3, on copied samples 6.  The last four: totals that nothing changes at.
@pytest.mark.parametrize("k,tiles,below,above", [(3, 2048, 2, 3), (4, 2048, 2, 3), (17, 2048, 3, 6), (32, 2048, 3, 6), (33, 2048, 2, 6), (40, 2048, 2, 6),
                                                 (64, 2048, 2, 6), (1, 10240, 2, 2), (3, 10240, 3, 3), (5, 8192, 3, 3), (16, 5120, 3, 3)])
def test_lines_between_the_ways_of_finding_boundaries(g, oracle, k, tiles, below, above):
    """Both sides of every line, by the launches that a call makes, and the results there."""
    for total, launches in (((tiles - 1) * (2048 - k), below), ((tiles - 1) * (2048 - k) + 1, above)):
        print("line", k, total, flush=True)
        out, n_out = torch.empty((total, 8), dtype=torch.int64, device=dev()), torch.zeros(1, dtype=torch.int64, device=dev())
        runs = list(torch.empty((total, 8), dtype=torch.int64, device=dev()).split(-(-total // k)))
        workspace = torch.empty(g.lsm_compact_workspace_bytes([r.shape[0] for r in runs]), dtype=torch.uint8, device=dev())
        assert len(runs) == k and _launches(lambda: g.lsm_compact(runs, 0, out, n_out, workspace)) == launches  # noqa: B023
        del out, n_out, runs, workspace
    torch.cuda.empty_cache()
    test_searched_directly_or_on_samples(g, oracle, k, tiles, "uneven")


@pytest.mark.parametrize("k,total", [(16, 1 << 26), (8, 1 << 27), (12, 89_478_486)])
def test_long_inputs_of_up_to_16_runs_are_cut_one_way(g, k, total):
    """No line between two ways at 2^30 entries times runs, where measurements show none: the launches are recorded, not run."""
    print("one way", k, total, flush=True)
    out, n_out = torch.empty((total + 1, 8), dtype=torch.int64, device=dev()), torch.zeros(1, dtype=torch.int64, device=dev())
    for n in (total - 1, total, total + 1):
        runs = list(torch.empty((n, 8), dtype=torch.int64, device=dev()).split(-(-n // k)))
        workspace = torch.empty(g.lsm_compact_workspace_bytes([r.shape[0] for r in runs]), dtype=torch.uint8, device=dev())
        assert _launches(lambda: g.lsm_compact(runs, 0, out, n_out, workspace)) == 3  # noqa: B023
        del runs, workspace
        torch.cuda.empty_cache()


@pytest.mark.parametrize("tiles", [2, 256, 257, 2047, 2048, 10240, 10241])
def test_one_run_is_cut_without_a_search(g, oracle, tiles):
    """One run of any length: the boundaries are multiples of the tile, one launch before the merge's."""
    print("one run", tiles, flush=True)
    rs = np.random.RandomState(tiles)
    full = 2047
    for n in ((tiles - 1) * full + 1, tiles * full):
        run = _runs_of(oracle, rs, [n], 2 * n)[0]
        _check_compact(g, oracle, [run], tiles & 1)
        out, n_out = torch.empty_like(run), torch.zeros(1, dtype=torch.int64, device=dev())
        workspace = torch.empty(g.lsm_compact_workspace_bytes([n]), dtype=torch.uint8, device=dev())
        assert _launches(lambda: g.lsm_compact([run], 1, out, n_out, workspace)) == 2


@pytest.mark.parametrize("k", [1, 2, 3, 16, 64])
def test_tile_spacing_edges(g, oracle, k):
    """Inputs around the totals where the tile spacing changes: one tile or several, the shortest spacing, one that grows
    with the input, the longest."""
    rs = np.random.RandomState(k)
    full = 2048 - k
    for total in (full, full + 1, SHORT, SHORT * FILL, SHORT * FILL + 1, 777 * FILL + 5, full * FILL - 1, full * FILL + 1):
        print("tile spacing", k, total, flush=True)
        cuts = np.sort(rs.randint(0, total + 1, size=k - 1)) if k > 1 else np.zeros(0, np.int64)
        lens = np.diff(np.concatenate([[0], cuts, [total]])).astype(int)
        _check_compact(g, oracle, _runs_of(oracle, rs, lens, 2 * total + 100), int(total & 1))


@pytest.mark.parametrize("jobs", [1, 3, 30])  # 30: the job table is copied
def test_batch_tile_spacing_edges(g, oracle, jobs):
    """The same for a batch: its spacing follows from the entries of all jobs, a job's own run count caps it."""
    rs = np.random.RandomState(jobs)
    for total in (SHORT * FILL - 3, SHORT * FILL + 3, 2000 * FILL, 2047 * FILL):
        print("batch tile spacing", jobs, total, flush=True)
        todo = []
        for j in range(jobs):
            k, n = (1, 2, 3, 17)[(j + jobs) % 4], total // jobs
            todo.append((_runs_of(oracle, rs, [n // k] * (k - 1) + [n - (k - 1) * (n // k)], 2 * n + 100), j & 1))
        outs, n_out = g.lsm_compact_batch(todo)
        for (runs, flags), out, n in zip(todo, outs, n_out.tolist()):
            want = oracle.compact([r.cpu() for r in runs], flags)
            assert n == want.shape[0]
            assert np.array_equal(as_bytes(out[:n]).reshape(-1, 64), want)


@pytest.mark.parametrize("k", [3, 4, 9, 17, 40, 64])  # 16, 16, 4, 2, 1 and 1 lanes per search
@pytest.mark.parametrize("shape", ["mixed", "copies", "ragged"])
def test_boundaries_at_ranked_samples(g, oracle, k, shape):
    """Three runs or more of up to 512 tiles: totals at the shortest mean tile, where it grows, and on both sides of the
    longest (samples get denser up to there; with many runs the limit on samples is met first).  Copies: every sample key is
    in every run.  Ragged: empty runs and runs shorter than the distance between two samples."""
    rs = np.random.RandomState(k)
    totals = [2048 - k + 1, 4099, 512 * 512, 512 * 512 + 1, 512 * 700 + 3]
    if shape == "mixed":
        totals += [512 * 1200, 512 * 2030 + 1, 512 * 2047 - 1, 512 * 2047 + 1]
    for total in totals:
        print("ranked samples", k, shape, total, flush=True)
        lens = np.full(k, total // k)
        if shape == "ragged":
            lens = np.where(rs.rand(k) < 0.4, rs.randint(0, 12, size=k), lens)
        lens[rs.randint(k)] += max(0, total - lens.sum())
        if shape == "copies":
            one = _runs_of(oracle, rs, [int(lens.max())], 3 * int(lens.max()))[0]
            runs = [one[:n].clone() for n in lens]
            for r in runs:
                r[:, 4] = torch.randint(0, 1 << 40, (r.shape[0],), device=dev())
        else:
            runs = _runs_of(oracle, rs, lens, 2 * total)
        _check_compact(g, oracle, runs, int(total & 1))
    few = _runs_of(oracle, rs, [700, 900], 4000)  # a batch: a job with samples, one without
    outs, n_out = g.lsm_compact_batch([(few, 1), (runs, 0), (few, 0)])
    for rr, flags, out, n in zip((few, runs, few), (1, 0, 0), outs, n_out.tolist()):
        want = oracle.compact([r.cpu() for r in rr], flags)
        assert n == want.shape[0]
        assert np.array_equal(as_bytes(out[:n]).reshape(-1, 64), want)


@pytest.mark.parametrize("k,total", [(3, 2048 * 2045 + 1), (4, 2048 * 2044 - 1), (5, 1_100_000), (16, 1_300_003), (17, 2_000_000), (32, 1_500_000)])
@pytest.mark.parametrize("shape", ["ragged", "copies", "apart"])
def test_boundaries_between_rows(g, oracle, k, total, shape):
    """Boundaries that are searched between ranked rows (every 4,096th entry of a run), and with four runs just below.  Ragged: empty runs, runs
    of one entry, around 4,096 and far longer.  Copies: rows of the same key in every run.  Apart: between two rows lies one run only."""
    print("between rows", k, total, shape, flush=True)
    rs = np.random.RandomState(k)
    lens = np.full(k, total // k)
    if shape == "ragged":
        few = np.array([0, 1, 4095, 4096, 4097, 8193])
        lens = np.where(rs.rand(k) < 0.6, few[rs.randint(0, 6, size=k)], (total * rs.dirichlet(np.full(k, 0.7))).astype(np.int64))
    lens[rs.randint(k)] += max(0, total - lens.sum())
    if shape == "copies":
        one = _runs_of(oracle, rs, [int(lens.max())], 3 * int(lens.max()))[0]
        runs = [one[:n].clone() for n in lens]
        for r in runs:
            r[:, 4] = torch.randint(0, 1 << 40, (r.shape[0],), device=dev())
    else:
        runs = _runs_of(oracle, rs, lens, 2 * total)
        for j in range(k if shape == "apart" else 0):
            runs[j][:, 0] |= (j * 7) % 64 + 1  # the keys' first byte, as stored
    _check_compact(g, oracle, runs, int(total & 1))

@pytest.mark.parametrize("k,total", [(4, 2047 * 2044), (4, 2047 * 2044 + 1), (5, 1_499_999), (5, 1_500_000), (12, 2_499_999), (12, 2_500_000), (16, 7_999_999), (16, 8_000_000)])
@pytest.mark.parametrize("shape", ["ragged", "copies", "apart", "turns"])
def test_distances_between_rows(g, oracle, k, total, shape):
    """Both sides of the totals where the distance between ranked rows changes (1,024 entries of a run to 16,384), and of four runs' first rows.
    Turns: runs that advance together, 100 entries each."""
    if shape != "turns":
        test_boundaries_between_rows(g, oracle, k, total, shape)
        return
    print("between rows", k, total, shape, flush=True)
    one = _runs_of(oracle, np.random.RandomState(k), [total], 3 * total)[0]
    turn = torch.arange(total, device=dev()) // 100 % k
    _check_compact(g, oracle, [one[turn == j].contiguous() for j in range(k)], int(total & 1))


@pytest.mark.parametrize("k,total", [(3, 2048 * 2045 + 1), (5, 1_100_000), (16, 1_300_003), (17, 2_000_000), (32, 1_500_000)])
def test_rows_of_runs_in_turns(g, oracle, k, total):
    test_distances_between_rows(g, oracle, k, total, "turns")


@pytest.mark.parametrize("n_req", [1, 2, 3, 511, 512, 513, 2047, 2048, 2049])  # four, two and one wave per request
@pytest.mark.parametrize("row", [256, 192, 64, 17])                            # key rows that need four, three or one of them
def test_probe_batches_of_all_sizes(g, oracle, cfg1, n_req, row):
    from workloads import lsm
    print("probe batch", n_req, row, flush=True)
    q, nb = lsm.queries_config1(cfg1, n_req, stream=n_req)
    q, nb = q[:, :row].contiguous(), nb.clamp(max=row)
    want = oracle.probe(q, nb, [r.cpu() for r in cfg1.runs])
    assert_probe_equal(oracle, probe_gpu(g, q, nb, build_tree(g, cfg1.runs)), want)


@pytest.mark.parametrize("n_req", [1024, 1025])  # one wave per request: workgroups of 256 threads up to 1,024 requests, of 512 beyond
@pytest.mark.parametrize("indexed", [False, True])
def test_probe_workgroup_sizes(g, oracle, cfg1, n_req, indexed):
    """lsm_probe with rows of at most 64 keys and lsm_probe_length on both sides of the line, with and without the fence
    table in LDS."""
    from workloads import lsm
    print("probe workgroups", n_req, indexed, flush=True)
    q, nb = lsm.queries_config1(cfg1, n_req)
    q, nb = q[:, :64].contiguous(), nb.clamp(max=64)
    tree = build_tree(g, cfg1.runs)
    if indexed:
        tree = [g.TreeRun(t.run, t.fences, t.stride, t.level, None, g.lsm_build_hash_index(g.lsm_hash_keys(t.run))) for t in tree]
    want = oracle.probe(q, nb, [r.cpu() for r in cfg1.runs])
    assert_probe_equal(oracle, probe_gpu(g, q, nb, tree), want)
    assert np.array_equal(g.lsm_probe_length(q, nb, tree).cpu().numpy().astype(np.uint32), want[0])


@pytest.mark.parametrize("n_req", [2049, 4096, 4097, 9001])  # pooled lookups: the smallest batch, the largest; beyond, a wave per request
@pytest.mark.parametrize("row", [256, 65, 64])  # 64: one chunk of keys, a wave per request as before
@pytest.mark.parametrize("ruled_out_by", ["filters", "indices", "both", "either", "tiny filters"])
def test_probe_pooled_lookups(g, oracle, cfg1, n_req, row, ruled_out_by):
    """Batches of more than 2,048 requests on trees whose runs all have a filter or an index, an empty run without either
    among them; tiny filters admit every key, so that every key of every request is looked up."""
    from workloads import lsm
    print("pooled lookups", n_req, row, ruled_out_by, flush=True)
    q, nb = lsm.queries_config1(cfg1, n_req, stream=row)
    q, nb = q[:, :row].contiguous(), nb.clamp(max=row)
    nb[::7] = 0
    tree = build_tree(g, list(cfg1.runs) + [cfg1.runs[0][:0]])
    for i, t in enumerate(tree[:-1]):
        if ruled_out_by in ("filters", "both") or (ruled_out_by == "either" and i % 2 == 0):
            t.bloom = g.lsm_build_bloom(t.run, 16)
        if ruled_out_by == "tiny filters":
            t.bloom = g.lsm_build_bloom(t.run, 16, out=torch.empty((1, 4), dtype=torch.int32, device=dev()))
        if ruled_out_by in ("indices", "both") or (ruled_out_by == "either" and i % 2 == 1):
            t.index = g.lsm_build_hash_index(g.lsm_hash_keys(t.run))
    want = oracle.probe(q, nb, [r.cpu() for r in cfg1.runs])
    assert_probe_equal(oracle, probe_gpu(g, q, nb, tree), want)


def _stored_keys(g, n, tombstones):
    """Keys of a two-run tree with filters: n live ones and, behind them, some whose newest version is a tombstone."""
    rs = np.random.RandomState(5)
    old = np.zeros((n + tombstones, 64), dtype=np.uint8)
    old[:, :8] = np.cumsum(rs.randint(1, 1 << 40, size=n + tombstones)).astype(">u8").view(np.uint8).reshape(-1, 8)
    new = old[n:].copy()
    new[:, 32], new[:, 40] = 9, TOMBSTONE
    runs = [to_dev(new), to_dev(old)]
    tree = build_tree(g, runs)
    for t in tree:
        t.bloom = g.lsm_build_bloom(t.run, 16)
    return runs, tree, runs[1][:, :4].clone()


@pytest.mark.parametrize("n_req", [2049, 2305, 4096])  # 9, 10 and 16 requests in a workgroup
def test_probe_pooled_and_alone(g, oracle, n_req):
    """Requests whose prefix ends at an edge of a chunk of keys, by a key that is not in the tree or by a tombstone, in
    workgroups of every kind: keys shared out, just as many as threads and more, so that the waves go on with the rest, first
    chunks just full enough to go on without, and one key fewer."""
    print("pooled or alone", n_req, flush=True)
    n, dead = 40_000, 1_000
    runs, tree, stored = _stored_keys(g, n, dead)
    rs = np.random.RandomState(n_req)
    per = -(-n_req // 256)
    edges = [0, 1, 63, 64, 65, 127, 128, 129, 255, 256]
    groups = [lambda i: int(rs.choice(edges)), lambda i: 256, lambda i: 256 if i < 4 else 0, lambda i: 256 if i < 4 else (1 if i == 4 else 0),
              lambda i: 60, lambda i: 59 if i == 0 else 60,  # 60 keys on average go on alone
              lambda i: 0, lambda i: int(rs.choice([0, 200])), lambda i: int(rs.choice([0, 17, 64, 80]))]
    cut = np.array([groups[r // per % len(groups)](r % per) for r in range(n_req)])
    nb = np.where(rs.rand(n_req) < 0.3, np.maximum(cut, 1), 256)
    at = rs.randint(0, n - 256, size=n_req)[:, None] + np.arange(256)
    ends = rs.rand(n_req) < 0.2  # by a tombstone somewhere before the cut
    where = (rs.rand(n_req) * cut).astype(np.int64)
    at[np.arange(n_req)[ends], where[ends]] = n + rs.randint(0, dead, size=int(ends.sum()))
    q = stored[torch.from_numpy(at).to(dev())]
    q[:, :, 3] = torch.from_numpy(np.arange(256)[None, :] >= cut[:, None]).to(dev()).to(torch.int64)  # a key of no run from the cut on
    nb = torch.from_numpy(nb.astype(np.int32)).to(dev())
    want = oracle.probe(q, nb, [r.cpu() for r in runs])
    assert_probe_equal(oracle, probe_gpu(g, q, nb, tree), want)


def _times(calls, rounds=12, each=10):
    """Shortest time per call, in microseconds, of each of `calls`, measured in turn."""
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = [float("inf")] * len(calls)
    for call in calls:
        call()
    for _ in range(rounds):
        for i, call in enumerate(calls):
            torch.cuda.synchronize()
            a.record()
            for _ in range(each):
                call()
            b.record()
            b.synchronize()
            best[i] = min(best[i], a.elapsed_time(b) * 1e3 / each)
    return best


@pytest.mark.parametrize("n_req", [2048, 4096])
def test_an_empty_run_does_not_slow_lookups_down(g, oracle, cfg1, n_req):
    """A run without entries holds no key, filter or not: keys that every other run rules out are not looked up.  Requests
    that share nothing with the tree took 2.3 to 3.1 times as long beside such a run where it counted as a run to be
    searched, 4,096 of them."""
    tree = build_tree(g, cfg1.runs)
    for t in tree:
        t.bloom = g.lsm_build_bloom(t.run, 16)
    rs = np.random.RandomState(n_req)
    q = torch.from_numpy(rs.randint(-1 << 62, 1 << 62, size=(n_req, 256, 4))).to(dev())
    nb = torch.full((n_req,), 256, dtype=torch.int32, device=dev())
    hit_len, hits = torch.empty(n_req, dtype=torch.int32, device=dev()), torch.empty((n_req, 256, 2), dtype=torch.int64, device=dev())
    empty = build_tree(g, [cfg1.runs[0][:0]])
    calls = [lambda tr=tr: g.lsm_probe(q, nb, tr, hit_len, hits) for tr in (tree, tree[:2] + empty + tree[2:])]
    without, beside = _times(calls)
    print(f"{n_req} requests: {without:.1f} us, beside an empty run {beside:.1f}", flush=True)
    assert beside < 1.6 * without
    assert int(hit_len.max()) == 0 and not hits.any()


@pytest.mark.parametrize("n_req", [2049, 4096, 4097])
def test_keys_behind_a_tombstone_do_not_slow_lookups_down(g, n_req):
    """Requests of 256 stored keys, the first a tombstone, against their first 64 keys alone: looking all of them up took
    three times as long."""
    _, tree, stored = _stored_keys(g, 200_000, 5_000)
    rs = np.random.RandomState(n_req)
    at = rs.randint(0, 199_000, size=(n_req, 256))
    at[:, 0] = 200_000 + rs.randint(0, 5_000, size=n_req)
    q = stored[torch.from_numpy(at).to(dev())]
    hit_len, hits = torch.empty(n_req, dtype=torch.int32, device=dev()), torch.empty((n_req, 256, 2), dtype=torch.int64, device=dev())
    nb = [torch.full((n_req,), n, dtype=torch.int32, device=dev()) for n in (64, 256)]
    first, all_keys = _times([lambda b=b: g.lsm_probe(q, b, tree, hit_len, hits) for b in nb])
    print(f"{n_req} requests: 64 keys {first:.1f} us, 256 keys {all_keys:.1f}", flush=True)
    assert all_keys < 1.6 * first
    assert int(hit_len.max()) == 0 and not hits.any()


# ------------------------------------------------------------------ Bloom filters
@pytest.mark.parametrize("bits_per_key", [8, 16])
def test_bloom_filter_bytes_equal_the_checker(g, oracle, cfg1, bits_per_key):
    print("bloom filter", bits_per_key, flush=True)
    for run in list(cfg1.runs) + [cfg1.runs[0][:0], cfg1.runs[1][:1], cfg1.runs[2][:1000]]:
        n_blocks = g.lsm_bloom_blocks(int(run.shape[0]), bits_per_key)
        assert n_blocks == oracle.bloom_blocks(int(run.shape[0]), bits_per_key)
        got = g.lsm_build_bloom(run.contiguous(), bits_per_key)
        torch.cuda.synchronize()
        assert np.array_equal(as_bytes(got).reshape(-1, 16), oracle.build_bloom(run.cpu(), n_blocks))
        # building again into the same buffer clears it first
        again = g.lsm_build_bloom(run.contiguous(), bits_per_key, out=got.fill_(-1))
        torch.cuda.synchronize()
        assert np.array_equal(as_bytes(again).reshape(-1, 16), oracle.build_bloom(run.cpu(), n_blocks))


def test_probe_with_bloom_filters_gives_the_same_answers(g, oracle, cfg1):
    """Filters only let the probe skip runs that cannot hold a key: results equal the checker's (which
    has no filters) with filters on every run, on some runs, and with a deliberately tiny filter."""
    from workloads import lsm
    print("probe with bloom filters", flush=True)
    q, nb = lsm.queries_config1(cfg1, 2048)
    want = oracle.probe(q, nb, [r.cpu() for r in cfg1.runs])
    plain = build_tree(g, cfg1.runs)
    for choice in ("all", "some", "tiny"):
        tree = []
        for i, t in enumerate(plain):
            bloom = None
            if choice == "all" or (choice == "some" and i % 2 == 0):
                bloom = g.lsm_build_bloom(t.run, 16)
            elif choice == "tiny":
                bloom = g.lsm_build_bloom(t.run, 16, out=torch.empty((3, 4), dtype=torch.int32, device=dev()))  # nearly all ones
            tree.append(g.TreeRun(t.run, t.fences, t.stride, t.level, bloom))
        assert_probe_equal(oracle, probe_gpu(g, q, nb, tree), want)


# ------------------------------------------------------------------ hash index (section 2.2: in-memory indices of a run)
@pytest.mark.parametrize("n", [0, 1, 3, 9, 4096, 16384, 300_000, 65_536 * 5 + 123])
def test_hash_index_is_a_valid_index_of_the_run(g, oracle, n):
    """lsm_build_hash_index: the table passes the checker's validity check (every key in its bucket with its tag and
    position, or its bucket marked crowded and holding seven; nothing else in the table), whatever the buffers held
    before; the key hashes equal the checker's.  The table itself is not unique, so its bytes are not compared."""
    from workloads import lsm
    print("hash index", n, flush=True)
    w = lsm.config3(device=dev(), scale=64)      # 16 runs x 65,536 entries
    run = w.runs[0][:n].contiguous() if n <= 65_536 else torch.cat(list(w.runs))[:n].contiguous()
    if n > 65_536:   # several runs put together are not sorted and hold a key more than once: one sorted run
        cpu = oracle.compact([r.cpu() for r in w.runs], 0)[:n]
        run = torch.from_numpy(cpu.view(np.int64).reshape(-1, 8).copy()).to(dev())
    n = int(run.shape[0])
    hashes = g.lsm_hash_keys(run)
    torch.cuda.synchronize()
    assert np.array_equal(hashes.cpu().numpy().view(np.uint64), oracle.key_hashes(run.cpu()))
    n_buckets = g.lsm_hash_index_buckets(n)
    assert n_buckets == oracle.hash_index_buckets(n)
    table = g.lsm_build_hash_index(hashes, out=torch.full((n_buckets, 8), 0x5A5A5A5A, dtype=torch.int64, device=dev()))
    torch.cuda.synchronize()
    assert oracle.hash_index_check(run.cpu(), table.cpu().numpy()) == 0
    if n >= 4096:
        marks = int(((table[:, 0] >> 15) & 1).sum().item())   # bit 15 of the first tag field
        assert 0 < marks < n_buckets // 10          # some buckets are crowded, most are not


def test_probe_with_hash_indices_gives_the_same_answers(g, oracle, cfg1):
    """A hash index only tells the probe where to look: results equal the checker's (which has none) with an index on
    every run (no fence table in the kernel) or on some, with and without filters, and for the search over the prefix
    length.  Requests made of a run's own keys reach every key of every crowded bucket (the fence path behind the
    mark)."""
    from workloads import lsm
    print("probe with hash indices", flush=True)
    q, nb = lsm.queries_config1(cfg1, 2048)
    runs_cpu = [r.cpu() for r in cfg1.runs]
    want = oracle.probe(q, nb, runs_cpu)
    plain = build_tree(g, cfg1.runs)
    indices = [g.lsm_build_hash_index(g.lsm_hash_keys(t.run)) for t in plain]
    for choice in ("all", "some", "all+filters", "some+filters"):
        tree = []
        for i, t in enumerate(plain):
            index = indices[i] if (not choice.startswith("some") or i % 2 == 0) else None
            bloom = g.lsm_build_bloom(t.run, 16) if choice.endswith("filters") else None
            tree.append(g.TreeRun(t.run, t.fences, t.stride, t.level, bloom, index))
        assert_probe_equal(oracle, probe_gpu(g, q, nb, tree), want)
        got_len = g.lsm_probe_length(q, nb, tree)
        torch.cuda.synchronize()
        assert np.array_equal(got_len.cpu().numpy().astype(np.uint32), want[0])
    # every key of the oldest run as a request of its own row of keys
    run = cfg1.runs[-1]
    n = int(run.shape[0]) // 256 * 256
    own_q = run[:n, :4].reshape(-1, 256, 4).contiguous()
    own_nb = torch.full((own_q.shape[0],), 256, dtype=torch.int32, device=dev())
    want_own = oracle.probe(own_q, own_nb, runs_cpu)
    for tree in ([g.TreeRun(t.run, t.fences, t.stride, t.level, None, ix) for t, ix in zip(plain, indices)],
                 [g.TreeRun(t.run, t.fences, t.stride, t.level, None, ix if i != 1 else None) for i, (t, ix) in enumerate(zip(plain, indices))]):
        assert_probe_equal(oracle, probe_gpu(g, own_q, own_nb, tree), want_own)
    # a table that does not belong to the run (positions far beyond it) must not send a read outside the run
    wrong = torch.full_like(indices[0], (2_000_000_000 << 32) | 2_000_000_000)   # every tag field set, positions beyond the run
    tree = [g.TreeRun(t.run, t.fences, t.stride, t.level, None, wrong if t.run.shape[0] == plain[0].run.shape[0] else None) for t in plain]
    hl, _ = probe_gpu(g, q, nb, tree)
    assert hl.shape == want[0].shape   # the answers are meaningless, the call must simply stay inside the runs


# ------------------------------------------------------------------ pointer rewrite during compaction (section 3.4)
def test_compaction_with_pointer_rewrite(g, oracle, cfg1):
    """lsm_compact_remap = compaction followed by the checker's pointer rewrite: several tensor files folded into
    fewer, files outside the table and tombstones untouched; an empty table is plain compaction."""
    print("pointer rewrite", flush=True)
    runs = cfg1.runs
    files = torch.cat([(r[:, 6] >> 32) & 0xFFFFFFFF for r in runs])
    n_files = int(files.max().item()) + 1
    assert n_files > 4
    table_len = n_files - 2  # the two highest file ids stay as they are
    rs = np.random.RandomState(9)
    # old files f -> new file f // 4, placed one after the other inside it
    starts = rs.randint(0, 1 << 20, size=table_len).cumsum()
    base = torch.tensor([((f // 4) << 32) + int(starts[f]) for f in range(table_len)], dtype=torch.int64, device=dev())
    for flags in (0, 1):
        out, n_out = g.lsm_compact(runs, flags, remap=base)
        torch.cuda.synchronize()
        got = out[: int(n_out.item())]
        plain = oracle.compact([r.cpu() for r in runs], flags & 1)
        want = oracle.remap_pointers(plain, base.cpu().numpy().astype(np.uint64))
        assert np.array_equal(as_bytes(got).reshape(-1, 64), want)
        assert not np.array_equal(want, plain)
        out2, n2 = g.lsm_compact(runs, flags, remap=base[:0])
        torch.cuda.synchronize()
        assert np.array_equal(as_bytes(out2[: int(n2.item())]).reshape(-1, 64), plain)


@pytest.mark.parametrize("stride", [1, 64, 100])
def test_fence_index_written_by_the_compaction(g, oracle, cfg1, stride):
    """The fence keys lsm_compact writes along with the run equal those lsm_build_fences and the checker give."""
    print("fused fences", stride, flush=True)
    total = sum(int(r.shape[0]) for r in cfg1.runs)
    for flags in (0, 1):
        fences = torch.full(((total + stride - 1) // stride, 4), -1, dtype=torch.int64, device=dev())
        out, n_out = g.lsm_compact(cfg1.runs, flags, fences=fences, fence_stride=stride)
        torch.cuda.synchronize()
        n = int(n_out.item())
        want = oracle.build_fences(oracle.compact([r.cpu() for r in cfg1.runs], flags & 1), stride)
        n_f = (n + stride - 1) // stride
        assert np.array_equal(as_bytes(fences[:n_f]).reshape(-1, 32), want)
        assert bool((fences[n_f:] == -1).all())  # nothing written past the end


@pytest.mark.parametrize("case", ["cfg1", "one_tile", "empty", "sampled"])
def test_filter_hashes_written_by_the_compaction(g, oracle, cfg1, case):
    """The key hashes lsm_compact writes along with the run are those lsm_hash_keys gives for the merged run, and the
    filter lsm_build_bloom_hashed builds from them is byte for byte the checker's filter of the merged run (so also
    lsm_build_bloom's); fences asked for in the same call are written as well."""
    from workloads import lsm
    print("key hashes from the compaction", case, flush=True)
    if case == "cfg1":
        runs = list(cfg1.runs)
    elif case == "one_tile":
        runs = [cfg1.runs[0][:700].contiguous(), cfg1.runs[1][:300].contiguous()]
    elif case == "empty":
        runs = [cfg1.runs[0][:0].contiguous()]
    else:
        runs = lsm.config3(device=dev(), scale=12).runs
        runs = runs[:-1] + [runs[-1][::2].contiguous(), runs[-1][1::2].contiguous()]  # 17 runs, 5.6M entries: the sampled partition, thousands of tiles
    total = sum(int(r.shape[0]) for r in runs)
    for flags, bits in ((1, 16), (0, 7)):
        hashes = torch.full((max(total, 1),), -1, dtype=torch.int64, device=dev())
        fences = torch.full(((max(total, 1) + 63) // 64, 4), -1, dtype=torch.int64, device=dev()) if flags else None
        out, n_out = g.lsm_compact(runs, flags, key_hashes=hashes, fences=fences, fence_stride=64)
        torch.cuda.synchronize()
        n = int(n_out.item())
        want = oracle.compact([r.cpu() for r in runs], flags & 1)
        assert n == want.shape[0] and np.array_equal(as_bytes(out[:n]).reshape(-1, 64), want)
        assert torch.equal(hashes[:n], g.lsm_hash_keys(out[:n]))
        assert bool((hashes[n:] == -1).all())   # nothing written past the end
        n_blocks = g.lsm_bloom_blocks(n, bits)
        assert n_blocks == oracle.bloom_blocks(n, bits)
        bloom = g.lsm_build_bloom_hashed(hashes[:n], n_blocks, out=torch.full((n_blocks, 4), -1, dtype=torch.int32, device=dev()))
        torch.cuda.synchronize()
        assert np.array_equal(as_bytes(bloom).reshape(-1, 16), oracle.build_bloom(want, n_blocks))
        assert torch.equal(bloom, g.lsm_build_bloom(out[:n], bits))
        if fences is not None:
            assert np.array_equal(as_bytes(fences[:(n + 63) // 64]).reshape(-1, 32), oracle.build_fences(want, 64))
    if case == "cfg1":   # the entry point that allocates nothing takes the same request
        out = torch.empty((total, 8), dtype=torch.int64, device=dev())
        n_out = torch.zeros(1, dtype=torch.int64, device=dev())
        hashes = torch.full((total,), -1, dtype=torch.int64, device=dev())
        g.lsm_compact_static(runs, 1, out, n_out, key_hashes=hashes)
        torch.cuda.synchronize()
        n = int(n_out.item())
        assert torch.equal(hashes[:n], g.lsm_hash_keys(out[:n]))


@pytest.mark.parametrize("n,bits", [(0, 16), (1, 16), (5000, 16), (40_000, 16), (300_000, 16), (300_000, 3), (65_536 * 3 + 17, 10)])
def test_filter_built_from_hashes_equals_the_checker(g, oracle, n, bits):
    """lsm_hash_keys + lsm_build_bloom_hashed on runs from one bucket's worth to several chunks and dozens of buckets:
    the same bytes as the checker's filter, whatever the buffers held before; a filter with more blocks than the key
    count asks for (as a caller who sizes it from an upper bound would pass) as well."""
    from workloads import lsm
    print("hashed bloom", n, bits, flush=True)
    w = lsm.config3(device=dev(), scale=64)      # 16 runs x 65,536 entries
    run = torch.cat([r for r in w.runs])[:n].contiguous()   # not sorted across runs: a filter does not care
    for n_blocks in (g.lsm_bloom_blocks(n, bits), g.lsm_bloom_blocks(n, bits) * 3 + 5):
        hashes = g.lsm_hash_keys(run)
        ws = torch.full((max(g.lsm_bloom_workspace_bytes(n, n_blocks), 256),), 0xA5, dtype=torch.uint8, device=dev())
        got = g.lsm_build_bloom_hashed(hashes, n_blocks, out=torch.full((n_blocks, 4), -1, dtype=torch.int32, device=dev()), workspace=ws)
        torch.cuda.synchronize()
        assert np.array_equal(as_bytes(got).reshape(-1, 16), oracle.build_bloom(run.cpu(), n_blocks))
    if n == 300_000 and bits == 16:   # a long run with a filter of three blocks: lsm_build_bloom's path for long runs
        tiny = g.lsm_build_bloom(run, 16, out=torch.full((3, 4), -1, dtype=torch.int32, device=dev()))
        torch.cuda.synchronize()
        assert np.array_equal(as_bytes(tiny).reshape(-1, 16), oracle.build_bloom(run.cpu(), 3))


@pytest.mark.parametrize("n", [4096, 4097, 32_768, 32_769,     # filters in LDS: one share, two, the largest, atomics
                               65_535, 65_536, 65_537, 262_145])  # from hashes: unsorted up to 65,536, sorted by range beyond
def test_filter_and_index_at_the_edges_of_their_builds(g, oracle, n):
    """lsm_build_bloom, lsm_build_bloom_batch, lsm_build_bloom_hashed and lsm_build_hash_index where the build changes."""
    from workloads import lsm
    print("filter and index edges", n, flush=True)
    w = lsm.config3(device=dev(), scale=64)
    run = torch.from_numpy(oracle.compact([r.cpu() for r in w.runs[:8]], 0)[:n].view(np.int64).reshape(-1, 8).copy()).to(dev())
    assert int(run.shape[0]) == n
    want = oracle.build_bloom(run.cpu(), g.lsm_bloom_blocks(n, 16))
    hashes = g.lsm_hash_keys(run)
    short = run[:77].contiguous()
    batch = g.lsm_build_bloom_batch([short, run], 16)
    for got in (g.lsm_build_bloom(run, 16), batch[1], g.lsm_build_bloom_hashed(hashes, g.lsm_bloom_blocks(n, 16))):
        torch.cuda.synchronize()
        assert np.array_equal(as_bytes(got).reshape(-1, 16), want)
    assert np.array_equal(as_bytes(batch[0]).reshape(-1, 16), oracle.build_bloom(short.cpu(), int(batch[0].shape[0])))
    table = g.lsm_build_hash_index(hashes)
    torch.cuda.synchronize()
    assert oracle.hash_index_check(run.cpu(), table.cpu().numpy()) == 0


@pytest.mark.parametrize("n", [2048, 2049, 4095, 4097, 8192, 8193])  # keys per thread: two, four, shares; in a batch eight up to 8,192
@pytest.mark.parametrize("bits", [3, 16, 64])                        # 64: filters of more than 64 KiB from 8,192 keys on
def test_short_filters_in_one_launch(g, oracle, n, bits):
    from workloads import lsm
    print("short filters", n, bits, flush=True)
    run = torch.cat([r for r in lsm.config3(device=dev(), scale=1024).runs])[:n].contiguous()
    assert int(run.shape[0]) == n
    blocks = g.lsm_bloom_blocks(n, bits)
    want = oracle.build_bloom(run.cpu(), blocks)
    got = g.lsm_build_bloom(run, bits, out=torch.full((blocks, 4), -1, dtype=torch.int32, device=dev()))
    rows = torch.full((3 * blocks, 4), -1, dtype=torch.int32, device=dev())  # what the allocations below start with
    del rows
    batch = g.lsm_build_bloom_batch([run, run[:1], run], bits)
    torch.cuda.synchronize()
    for f in (got, batch[0], batch[2], g.lsm_build_bloom_batch([run], bits)[0]):
        assert np.array_equal(as_bytes(f).reshape(-1, 16), want)


# ------------------------------------------------------------------ prefix length by search (appendix B)
def test_probe_length_equals_probe_on_prefix_closed_data(g, oracle, cfg1):
    """The generator evicts leaf first, so its trees are prefix-closed: the search over the prefix length gives the
    checker's first-miss length, with and without Bloom filters, on several runs and on the compacted run."""
    from workloads import lsm
    print("probe length", flush=True)
    q, nb = lsm.queries_config1(cfg1, 4096)
    want = oracle.probe(q, nb, [r.cpu() for r in cfg1.runs])[0]
    tree = build_tree(g, cfg1.runs)
    got = g.lsm_probe_length(q, nb, tree)
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy().astype(np.uint32), want)
    filtered = [g.TreeRun(t.run, t.fences, t.stride, t.level, g.lsm_build_bloom(t.run, 16)) for t in tree]
    assert np.array_equal(g.lsm_probe_length(q, nb, filtered).cpu().numpy().astype(np.uint32), want)
    merged = compact_gpu(g, cfg1.runs, 1).contiguous()
    assert np.array_equal(g.lsm_probe_length(q, nb, build_tree(g, [merged])).cpu().numpy().astype(np.uint32), want)
    # long and short rows, rows of length 0
    nb2 = nb.clone()
    nb2[::7] = 0
    nb2[1::7] = 1
    want2 = oracle.probe(q, nb2, [r.cpu() for r in cfg1.runs])[0]
    assert np.array_equal(g.lsm_probe_length(q, nb2, tree).cpu().numpy().astype(np.uint32), want2)


def test_probe_length_on_data_with_holes(g, oracle):
    """Without prefix closure the result is still a boundary: block j-1 live (or j = 0), block j not (or j = n)."""
    print("probe length with holes", flush=True)
    rs = np.random.RandomState(12)
    keys = sorted({bytes(rs.randint(0, 256, size=32).astype(np.uint8)) for _ in range(300)})
    present = [k for i, k in enumerate(keys) if rs.rand() < 0.7]
    run = brute.run_from_raw([brute.pack_entry(k, i + 1, TOMBSTONE if rs.rand() < 0.1 else PUT, 1000 + i, 5) for i, k in enumerate(present)])
    live = {brute.unpack(r)[0] for r in brute.raws_of(run) if brute.unpack(r)[2] == PUT}
    n_req, max_blocks = 64, 200
    q = np.zeros((n_req, max_blocks, 32), dtype=np.uint8)
    rows = []
    for r in range(n_req):
        row = [keys[i] for i in rs.choice(len(keys), size=max_blocks, replace=False)]
        rows.append(row)
        q[r] = np.frombuffer(b"".join(row), dtype=np.uint8).reshape(max_blocks, 32)
    nb = rs.randint(0, max_blocks + 1, size=n_req).astype(np.int32)
    qd = torch.from_numpy(q.view(np.int64).reshape(n_req, max_blocks, 4)).to(dev())
    got = g.lsm_probe_length(qd, torch.from_numpy(nb).to(dev()), build_tree(g, [to_dev(run)])).cpu().numpy()
    for r in range(n_req):
        j = int(got[r])
        assert 0 <= j <= nb[r]
        assert j == 0 or rows[r][j - 1] in live
        assert j == nb[r] or rows[r][j] not in live


# ------------------------------------------------------------------ write-buffer flush (section 2.2)
@pytest.mark.parametrize("n,n_keys", [(0, 10), (1, 10), (255, 40), (256, 4000), (3600, 3000), (3600, 50), (8192, 6000),
                                      # beyond 8,192 entries: sorted segments of 4,096, merged by the compaction kernels
                                      (8193, 5000), (10000, 100000), (50000, 40), (100000, 30000), (20000, 10 ** 7),
                                      (262144, 200000)])
def test_flush_of_the_write_buffer(g, oracle, n, n_keys):
    """Unsorted entries with repeated keys and repeated seqnos -> the checker's sorted run, with its fence index."""
    print("flush", n, n_keys, flush=True)
    rs = np.random.RandomState(n + n_keys)
    alphabet = rs.randint(0, 256, size=(n_keys, 32)).astype(np.uint8)
    a = np.zeros((n, 64), dtype=np.uint8)
    if n:
        a[:, :32] = alphabet[rs.randint(0, n_keys, size=n)]
        rec = a.view(oracle.ENTRY_DTYPE).reshape(-1)
        rec["seqno"] = rs.randint(0, 6, size=n) if n_keys <= 50 else rs.randint(0, 1 << 40, size=n)
        rec["type"] = (rs.rand(n) < 0.2).astype(np.uint8)
        rec["vptr"] = np.arange(n)
        rec["vlen"] = 655360
    buf = to_dev(a)
    fences = torch.full(((n + 63) // 64 + 1, 4), -1, dtype=torch.int64, device=dev())
    out, n_out = g.lsm_flush_buffer(buf, fences=fences, fence_stride=64)
    torch.cuda.synchronize()
    want = oracle.flush_buffer(a)
    m = int(n_out.item())
    assert m == want.shape[0]
    assert np.array_equal(as_bytes(out[:m]).reshape(-1, 64), want)
    assert np.array_equal(as_bytes(fences[: (m + 63) // 64]).reshape(-1, 32), oracle.build_fences(want, 64))
    if m:  # a flushed buffer is a run like any other: it compacts and probes
        assert np.array_equal(as_bytes(compact_gpu(g, [out[:m].contiguous()], 0)).reshape(-1, 64), want)


@pytest.mark.parametrize("n", [2, 16, 17, 63, 65, 2048, 2049, 4097, 8192,          # ranks by comparing all pairs: tiles, slices
                               8193, 12288, 12289, 16385 + 4095])                  # segments sorted in LDS: full, one entry, ragged
@pytest.mark.parametrize("shared", [8, 14, 29])
def test_flush_of_keys_with_common_prefixes(g, oracle, n, shared):
    """Keys that agree in their first `shared` bytes, so that the order is decided behind the 14 (or 16) bytes that are
    compared first; a few thousand distinct keys and seqnos that repeat.  Exact: bytes are copied, not computed."""
    print("flush, common prefix", n, shared, flush=True)
    rs = np.random.RandomState(n * 31 + shared)
    a = np.zeros((n, 64), dtype=np.uint8)
    a[:, :32] = 0x5A
    a[:, shared:32] = rs.randint(0, 14 if shared == 29 else 256, size=(n, 32 - shared))
    if shared < 29:  # tails from a small set: groups of equal and of nearly equal keys
        a[:, shared:32] = a[rs.randint(0, max(1, n // 3), size=n), shared:32]
        a[:, 31] = rs.randint(0, 3, size=n)
    rec = a.view(oracle.ENTRY_DTYPE).reshape(-1)
    rec["seqno"] = rs.randint(0, 5, size=n)
    rec["type"] = (rs.rand(n) < 0.2).astype(np.uint8)
    rec["vptr"] = np.arange(n)
    out, n_out = g.lsm_flush_buffer(to_dev(a))
    torch.cuda.synchronize()
    want = oracle.flush_buffer(a)
    assert int(n_out.item()) == want.shape[0]
    assert np.array_equal(as_bytes(out[: want.shape[0]]).reshape(-1, 64), want)


@pytest.mark.parametrize("n", [3, 127, 128, 129, 255, 8193, 131_072, 131_073])  # one launch up to 128; segments of 2,048 and, beyond 64 of them, 4,096
@pytest.mark.parametrize("lead", [0, 14, 16])
def test_flush_around_its_kernels(g, oracle, n, lead):
    """Keys that share their first `lead` bytes, every third of them all ones there (what unused records hold), each written
    about three times, seqnos that repeat."""
    print("flush kernels", n, lead, flush=True)
    rs = np.random.RandomState(n + lead)
    keys = rs.randint(0, 256, size=(n // 3 + 1, 32)).astype(np.uint8)
    keys[:, :lead] = 7
    keys[::3, :16] = 255
    a = np.zeros((n, 64), dtype=np.uint8)
    a[:, :32] = keys[rs.randint(0, len(keys), size=n)]
    rec = a.view(oracle.ENTRY_DTYPE).reshape(-1)
    rec["seqno"] = rs.randint(0, max(2, n // 2), size=n)
    rec["type"] = (rs.rand(n) < 0.2).astype(np.uint8)
    rec["vptr"] = np.arange(n)
    fences = torch.full(((n + 6) // 7, 4), -1, dtype=torch.int64, device=dev())
    out, n_out = g.lsm_flush_buffer(to_dev(a), fences=fences, fence_stride=7)
    want = oracle.flush_buffer(a)
    m = int(n_out.item())
    assert m == want.shape[0]
    assert np.array_equal(as_bytes(out[:m]).reshape(-1, 64), want)
    assert np.array_equal(as_bytes(fences[: (m + 6) // 7]).reshape(-1, 32), oracle.build_fences(want, 7))


WALK = 16  # members up to which a segment's groups of equal 14-byte prefixes are settled one position at a time


@pytest.mark.parametrize("sizes", [[WALK - 1, WALK, 1, 2], [WALK + 1, 1, 2, 3], [WALK, 200, 1, 5], [4096], [8192 + WALK], [8192 + WALK + 1], [700, 1300, 90]])
@pytest.mark.parametrize("kind", ["versions", "tails", "both"])
def test_flush_of_groups_of_equal_prefixes(g, oracle, sizes, kind):
    """Groups of entries that share the 14 bytes a segment is sorted by first, around the size at which they are sorted
    instead of compared one by one: versions of one key, keys that differ further on, both; sequence numbers in no order."""
    print("flush, groups", sizes, kind, flush=True)
    rs = np.random.RandomState(sum(sizes))
    n = max(8193 + 77, sum(sizes))
    heads = np.repeat(np.arange(len(sizes)), sizes)
    heads = np.concatenate([heads, len(sizes) + np.arange(n - heads.size)])[rs.permutation(n)]
    a = np.zeros((n, 64), dtype=np.uint8)
    a[:, :8] = heads.astype(">u8").view(np.uint8).reshape(n, 8)
    if kind != "versions":
        a[:, 14 + rs.randint(0, 18, size=n)[0]] = rs.randint(0, 5, size=n)
        a[:, 20] = rs.randint(0, 256 if kind == "tails" else 2, size=n)
    rec = a.view(oracle.ENTRY_DTYPE).reshape(-1)
    rec["seqno"] = rs.randint(0, 1 << 40, size=n) if kind == "versions" else rs.randint(0, 3, size=n)
    rec["vptr"] = np.arange(n)
    out, n_out = g.lsm_flush_buffer(to_dev(a))
    torch.cuda.synchronize()
    want = oracle.flush_buffer(a)
    assert int(n_out.item()) == want.shape[0]
    assert np.array_equal(as_bytes(out[: want.shape[0]]).reshape(-1, 64), want)


@pytest.mark.parametrize("kind", ["one key", "prefixes"])
def test_flush_of_hot_keys_is_not_quadratic(g, oracle, kind):
    """A buffer of versions of one key, or of keys with a common prefix, takes at most five times as long as one of
    scattered keys: two sorts of every segment instead of one, of longer records.  (Comparing every entry of a segment
    with every other takes more than a hundred times as long.)"""
    rs = np.random.RandomState(5)
    spread = torch.from_numpy(rs.randint(0, 1 << 62, size=(20_000, 8))).to(dev())
    spread[:, 5] = 0
    hot = spread.clone()
    hot[:, :4 if kind == "one key" else 2] = 0
    out, n_out = torch.empty_like(hot), torch.zeros(1, dtype=torch.int64, device=dev())
    base, took = [_best_us(lambda: g.lsm_flush_buffer(buf, out, n_out)) for buf in (spread, hot)]
    print(f"flush of 20,000 entries: {base:.0f} us, {kind} {took:.0f} us", flush=True)
    assert took < 5 * base


# ------------------------------------------------------------------ range lookups (section 2.2, appendix B get_batch)
def test_range_scan_equals_filtered_compaction(g, oracle, cfg1):
    """Entries of a key range, newest version of each, live only = the checker's last-level compaction of all runs
    cut to the range; one family's range, a range between two stored keys, an empty one and everything."""
    from paper_2511_16138_amd.tree import range_scan
    print("range scan", flush=True)
    tree = build_tree(g, cfg1.runs)
    full = oracle.compact([r.cpu() for r in cfg1.runs], 1)
    keys = [bytes(k) for k in full[:, :32]]
    fam = keys[len(keys) // 3][:8]
    ranges = [(fam + bytes(24), fam + b"\xff" * 24), (keys[100], keys[5000]), (keys[7], keys[7]),
              (bytes(32), b"\xff" * 32), (keys[-1], b"\xff" * 32)]
    for lo, hi in ranges:
        want = full[[i for i, k in enumerate(keys) if lo <= k < hi]] if lo < hi else full[:0]
        bounds = g.lsm_range_bounds(tree, lo, hi).cpu().numpy()
        for (a, b), r in zip(bounds, cfg1.runs):  # every bound is the lower bound of its key in its run
            rk = as_bytes(r).reshape(-1, 64)[:, :32]
            for at, key in ((int(a), lo), (int(b), hi)):
                assert (at == 0 or bytes(rk[at - 1]) < key) and (at == r.shape[0] or bytes(rk[at]) >= key)
        got = range_scan(tree, lo, hi)
        torch.cuda.synchronize()
        assert np.array_equal(as_bytes(got).reshape(-1, 64), want)


def _keys_tensor(keys):
    a = np.frombuffer(b"".join(keys), dtype=np.uint8).reshape(-1, 32).copy()
    return torch.from_numpy(a.view(np.int64).reshape(-1, 4)).to(dev())


@pytest.mark.parametrize("which", ["config1", "tiered16"])
def test_batched_range_scans(g, oracle, cfg1, which):
    """Many key ranges in one call (appendix B, get_batch): every range's entries equal the checker's last-level
    compaction of all runs cut to the range - families, ranges between stored keys, single keys, empty and inverted
    ranges, keys outside the tree; ranges too large for their slot or for a tile are reported as overflow."""
    from workloads import lsm
    print("batched range scans", which, flush=True)
    w = cfg1 if which == "config1" else lsm.config3(device=dev(), scale=256)
    tree = build_tree(g, w.runs)
    full = oracle.compact([r.cpu() for r in w.runs], 1)
    keys = [bytes(k) for k in full[:, :32]]
    run_keys = [[bytes(k) for k in as_bytes(r).reshape(-1, 64)[:, :32]] for r in w.runs]
    all_in = sorted({k for rk in run_keys for k in rk})  # every version's key, dead ones too
    rs = np.random.RandomState(11)
    ranges = []
    for i in rs.randint(0, len(keys), size=300):          # the family of a stored key: all keys with the same first 8 bytes
        fam = keys[i][:8]
        ranges.append((fam + bytes(24), fam + b"\xff" * 24))
    for i in rs.randint(0, len(keys) - 300, size=200):    # between two stored keys, a few to a few hundred entries apart
        ranges.append((keys[i], keys[i + int(rs.randint(0, 300))]))
    for i in rs.randint(0, len(all_in), size=100):        # exactly one key, live or not
        k = all_in[i]
        ranges.append((k, (int.from_bytes(k, "big") + 1).to_bytes(32, "big")))
    ranges += [(keys[7], keys[7]), (keys[50], keys[10]), (bytes(32), keys[0]), (keys[-1], b"\xff" * 32),
               (b"\xff" * 32, b"\xff" * 32), (bytes(32), bytes(32))]
    ranges += [(bytes(32), b"\xff" * 32), (keys[0], keys[len(keys) // 2])]   # far more than a tile: overflow
    import bisect
    max_entries = 512
    ent, cnt = g.lsm_range_scan(tree, _keys_tensor([lo for lo, _ in ranges]), _keys_tensor([hi for _, hi in ranges]), max_entries)
    torch.cuda.synchronize()
    cnt = cnt.cpu().numpy()
    got = as_bytes(ent).reshape(len(ranges), max_entries, 64)
    n_over = 0
    for i, (lo, hi) in enumerate(ranges):
        a, b = (bisect.bisect_left(keys, lo), bisect.bisect_left(keys, hi)) if lo < hi else (0, 0)
        in_pieces = sum(bisect.bisect_left(rk, hi) - bisect.bisect_left(rk, lo) for rk in run_keys) if lo < hi else 0
        if b - a > max_entries or in_pieces > 2048:   # more results than the slot, or more entries (all versions) than a tile
            assert cnt[i] == g.binding.LSM_RANGE_OVERFLOW, (i, cnt[i], b - a, in_pieces)
            n_over += 1
        else:
            assert cnt[i] == b - a, (i, cnt[i], b - a)
            assert np.array_equal(got[i, : b - a], full[a:b]), i
    assert 2 <= n_over < len(ranges) // 2   # the two huge ranges and the large families
    # a small slot: ranges with more results than the slot are reported, the others are unchanged
    ent2, cnt2 = g.lsm_range_scan(tree, _keys_tensor([lo for lo, _ in ranges]), _keys_tensor([hi for _, hi in ranges]), 8)
    cnt2 = cnt2.cpu().numpy()
    got2 = as_bytes(ent2).reshape(len(ranges), 8, 64)
    for i, (lo, hi) in enumerate(ranges):
        a, b = (bisect.bisect_left(keys, lo), bisect.bisect_left(keys, hi)) if lo < hi else (0, 0)
        if b - a > 8:
            assert cnt2[i] == g.binding.LSM_RANGE_OVERFLOW
        elif cnt[i] != g.binding.LSM_RANGE_OVERFLOW:
            assert cnt2[i] == b - a and np.array_equal(got2[i, : b - a], full[a:b])
    # the driver's helper: ranges that overflow their slot are redone one by one, so every range has its content
    from paper_2511_16138_amd.tree import range_scan_batch
    pick = [0, 150, 310, 420, 560, len(ranges) - 1]
    parts = range_scan_batch(tree, _keys_tensor([ranges[i][0] for i in pick]), _keys_tensor([ranges[i][1] for i in pick]), 8)
    for i, part in zip(pick, parts):
        lo, hi = ranges[i]
        a, b = (bisect.bisect_left(keys, lo), bisect.bisect_left(keys, hi)) if lo < hi else (0, 0)
        assert np.array_equal(as_bytes(part).reshape(-1, 64), full[a:b]), i
    # an empty tree and an empty batch
    e0, c0 = g.lsm_range_scan([], _keys_tensor([bytes(32)]), _keys_tensor([b"\xff" * 32]), 4)
    assert c0.cpu().tolist() == [0]
    e1, c1 = g.lsm_range_scan(tree, _keys_tensor([bytes(32)])[:0], _keys_tensor([bytes(32)])[:0], 4)
    assert c1.numel() == 0


def _numbered_runs(oracle, rs, lengths, spread):
    """Runs of the given lengths as [n, 64] uint8 arrays, sorted.  Keys carry a random number below 2^spread behind a common
    prefix: in the last eight bytes (dense, many keys in several runs, all first halves equal) for spreads up to 18, else
    in bytes 8..15."""
    runs = []
    for n in lengths:
        some = np.arange(1 << spread) if spread <= 18 else np.unique(rs.randint(0, 1 << spread, size=2 * n + 8))
        lead = np.sort(rs.permutation(some)[:n]).astype(np.int64)
        a = np.zeros((n, 64), dtype=np.uint8)
        a[:, :32] = 0x33
        at = 24 if spread <= 18 else 8
        a[:, at:at + 8] = lead.astype(">u8").view(np.uint8).reshape(n, 8)
        rec = a.view(oracle.ENTRY_DTYPE).reshape(-1)
        rec["seqno"] = ((len(lengths) - len(runs)) << 32) + rs.permutation(n)  # newest run first
        rec["type"] = (rs.rand(n) < 0.1).astype(np.uint8)
        rec["vptr"] = np.arange(n)
        runs.append(a)
    return runs


@pytest.mark.parametrize("k", [1, 2, 8, 9, 16, 17, 32, 33, 64])   # 32, 16, 8 or 4 lanes per search
@pytest.mark.parametrize("spread", [13, 40])                      # keys that differ behind byte 24, or in the first 16
def test_range_scan_by_runs(g, oracle, k, spread):
    """Range ends found by shared searches: runs from empty to a few thousand entries, bounds below, between, at and
    above the stored keys."""
    print("range scan by runs", k, spread, flush=True)
    rs = np.random.RandomState(100 * k + spread)
    runs = _numbered_runs(oracle, rs, [(0, 1, 31, 33, 700, 4099)[(j + 5) % 6] if j else 4099 for j in range(k)], spread)
    tree = build_tree(g, [to_dev(a) for a in runs])
    full = oracle.compact(runs, 1)
    every = np.unique(np.concatenate([a[:, :32] for a in runs]), axis=0)
    cut = np.sort(rs.randint(0, len(every), size=(200, 2)), axis=1)
    cut[:, 1] = np.minimum(cut[:, 1], cut[:, 0] + rs.randint(0, 40, size=200))
    ranges = [(bytes(every[i]), bytes(every[j])) for i, j in cut]
    ranges += [(bytes(32), bytes(every[3])), (bytes(every[-5]), b"\xff" * 32), (bytes(every[5]), bytes(every[2])), (b"\xff" * 32, b"\xff" * 32)]
    ranges += [(lo[:31] + b"\x01", hi[:31] + b"\x02") for lo, hi in ranges[:40]]
    ent, cnt = g.lsm_range_scan(tree, _keys_tensor([lo for lo, _ in ranges]), _keys_tensor([hi for _, hi in ranges]), 2048)
    cnt, got = cnt.cpu().numpy(), as_bytes(ent).reshape(len(ranges), 2048, 64)
    keys = [bytes(x) for x in full[:, :32]]
    for i, (lo, hi) in enumerate(ranges):
        want = full[[j for j, x in enumerate(keys) if lo <= x < hi]]
        assert cnt[i] == want.shape[0], (i, cnt[i], want.shape[0])
        assert np.array_equal(got[i, : want.shape[0]], want), i


def test_batch_of_small_compactions(g, oracle, cfg1):
    """Many independent compactions in one call: every job's output and count equal the checker's for that job -
    1 to 9 runs per job, empty runs and empty jobs, both flag values, jobs of one tile and of dozens of tiles."""
    from workloads import lsm
    print("batch of small compactions", flush=True)
    rs = np.random.RandomState(3)
    src = [r for r in cfg1.runs] + [r for r in lsm.config3(device=dev(), scale=128).runs]
    jobs = []
    for j in range(160):
        k = int(rs.randint(1, 10))
        runs = []
        for r in rs.choice(len(src), size=k, replace=False):   # distinct source runs: one version per key per run
            n = int(src[r].shape[0])
            lo = int(rs.randint(0, n))
            ln = int(rs.choice([0, 1, 7, 100, 1000, 3000, 9000]))
            runs.append(src[r][lo:min(n, lo + ln)].contiguous())
        jobs.append((runs, int(rs.randint(0, 2))))
    jobs.append(([src[0][:0].contiguous()], 1))                       # nothing at all
    jobs.append(([src[0][:0].contiguous(), src[1][:5].contiguous()], 0))
    jobs.append(([r.contiguous() for r in cfg1.runs], 0))              # configuration 1 as one job of the batch
    outs, n_out = g.lsm_compact_batch(jobs)
    torch.cuda.synchronize()
    n_out = n_out.cpu().numpy()
    for j, ((runs, flags), out) in enumerate(zip(jobs, outs)):
        want = oracle.compact([r.cpu() for r in runs], flags)
        assert int(n_out[j]) == want.shape[0], (j, int(n_out[j]), want.shape[0])
        assert np.array_equal(as_bytes(out[: want.shape[0]]).reshape(-1, 64), want), j
    # the same batch again into fresh buffers (the workspace of the first call is gone), with fence indices: same
    # result, and every job's fences are the strided keys of its output
    outs2, n_out2, fences = g.lsm_compact_batch(jobs, fence_stride=64)
    torch.cuda.synchronize()
    assert np.array_equal(n_out2.cpu().numpy(), n_out)
    for a, b, m, f in zip(outs, outs2, n_out, fences):
        assert torch.equal(a[: int(m)], b[: int(m)])
        want_f = as_bytes(a[: int(m)]).reshape(-1, 64)[::64, :32]
        assert np.array_equal(as_bytes(f[: (int(m) + 63) // 64]).reshape(-1, 32), want_f)
    assert g.lsm_compact_batch([])[1].numel() == 0


def test_get_batch_under_a_shared_prefix_with_ladder_keys(g, oracle):
    """get_batch (appendix B) on keys in the segment-ladder layout: the cached blocks below a shared prefix of 512 g
    tokens are one tight key range, fetched for many prefixes in one lsm_range_scan - newest versions, no tombstoned
    blocks - and nothing that is not below the prefix."""
    from test_workloads import _prefix_tree_tokens
    from workloads import keys as K
    print("get_batch with ladder keys", flush=True)
    toks = _prefix_tree_tokens(n_seq=120, length=100, seed=21)
    n, length = toks.shape[0], toks.shape[1]
    words = K.chain_keys(toks, "ladder")                                  # [n, L, 4]
    mem = K.key_bytes_words(words.reshape(-1, 4)).numpy().view(np.uint8).reshape(-1, 32)
    uniq, first_at = np.unique(mem.view("V32").reshape(-1), return_index=True)
    keys_all = mem[np.sort(first_at)]                                     # distinct keys, one per cached block
    rs = np.random.RandomState(5)
    runs, seq = [], 1000
    for r in range(3):                                                    # three runs: random subsets, some tombstones, newer = earlier run
        pick = np.sort(rs.choice(keys_all.shape[0], size=keys_all.shape[0] * 2 // 3, replace=False))
        a = np.zeros((pick.shape[0], 64), dtype=np.uint8)
        a[:, :32] = keys_all[pick]
        rec = a.view(oracle.ENTRY_DTYPE).reshape(-1)
        rec["seqno"] = (3 - r) * 1_000_000 + np.arange(pick.shape[0])
        rec["type"] = (rs.rand(pick.shape[0]) < 0.1).astype(np.uint8)
        rec["vptr"] = rec["seqno"] * 16
        rec["vlen"] = 655360
        order = np.argsort(a[:, :32].view("V32").reshape(-1), kind="stable")
        runs.append(a[order])
    full = oracle.compact(runs, 1)
    full_keys = [bytes(k) for k in full[:, :32]]
    tree = build_tree(g, [to_dev(r) for r in runs])
    kb = [bytes(k) for k in mem]
    t = toks.numpy()
    ranges, below = [], []
    for i in range(0, n, 2):
        for grp in (1, 2, 3):
            deep = kb[i * length + 32 * grp]
            ranges.append((deep[:3 * grp] + bytes(32 - 3 * grp), deep[:3 * grp] + b"\xff" * (32 - 3 * grp)))
            below.append({kb[j * length + k] for j in range(n) if (t[j, :32 * grp] == t[i, :32 * grp]).all() for k in range(32 * grp, length)})
    ent, cnt = g.lsm_range_scan(tree, _keys_tensor([lo for lo, _ in ranges]), _keys_tensor([hi for _, hi in ranges]), 1024)
    torch.cuda.synchronize()
    cnt = cnt.cpu().numpy()
    got = as_bytes(ent).reshape(len(ranges), 1024, 64)
    for i, ((lo, hi), sub) in enumerate(zip(ranges, below)):
        want = full[[j for j, k in enumerate(full_keys) if k in sub]]     # live newest versions of the blocks below the prefix
        assert cnt[i] == want.shape[0], (i, cnt[i], want.shape[0])
        assert np.array_equal(got[i, : cnt[i]], want), i
    assert max(cnt) > 100 and min(cnt) > 0


def test_bloom_filters_of_many_runs_in_one_call(g, oracle, cfg1):
    """lsm_build_bloom_batch: every filter is byte for byte the checker's filter of that run (and so lsm_build_bloom's)."""
    print("bloom batch", flush=True)
    rs = np.random.RandomState(8)
    src = [r for r in cfg1.runs]
    runs = []
    for j in range(70):                      # more than one launch's worth of runs, sizes 0 .. 16,384
        r = src[j % len(src)]
        lo = int(rs.randint(0, r.shape[0]))
        runs.append(r[lo:lo + int(rs.choice([0, 1, 9, 300, 5000, 16384]))].contiguous())
    for bits in (16, 5):
        filters = g.lsm_build_bloom_batch(runs, bits)
        torch.cuda.synchronize()
        for r, f in zip(runs, filters):
            assert int(f.shape[0]) == oracle.bloom_blocks(int(r.shape[0]), bits)
            assert np.array_equal(as_bytes(f).reshape(-1, 16), oracle.build_bloom(r.cpu(), int(f.shape[0])))
    one = g.lsm_build_bloom(runs[5], 16)
    assert torch.equal(one, g.lsm_build_bloom_batch(runs, 16)[5])
    assert g.lsm_build_bloom_batch([], 16) == []
