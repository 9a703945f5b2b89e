"""The library's driver on the CPU (tests/driver_host.cpp answers its calls): what becomes of the trees when device memory
runs out or a launch is refused, at every place where that can happen.  A run that lookups can reach is complete or has no
filter: never an unwritten copy, never a filter that rules out keys of its run."""
import ctypes as C
import os
import subprocess

import brute
import numpy as np
import pytest

from oracle.lsm_driver_oracle import DriverOracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_16138_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
BAD_ARG, HIP = -2, -7


@pytest.fixture(scope="module")
def host(tmp_path_factory, oracle):
    import paper_2511_16138_amd.binding as B
    d = tmp_path_factory.mktemp("driver_host")
    inc = ["-I" + os.path.join(ROOT, "include"), "-I" + CSRC]
    objects = []
    for src in (os.path.join(CSRC, "lsm_driver.cpp"), os.path.join(ROOT, "tests", "driver_host.cpp")):
        objects.append(str(d / (os.path.basename(src) + ".o")))
        subprocess.check_call([HIPCC, "-O1", "-std=c++17", "-fPIC", "--offload-host-only", "-x", "hip", "-DLSM_STATUS_EPOCH_BITS=3", *inc, "-c", src, "-o", objects[-1]])
    objects.append(str(d / "oracle.o"))
    subprocess.check_call(["gcc", "-O1", "-fPIC", "-c", os.path.join(ROOT, "oracle", "lsm_oracle.c"), "-o", objects[-1]])
    lib = str(d / "libdriver_host.so")
    # calls stay inside the library, whatever else the process has loaded
    subprocess.check_call(["g++", "-shared", "-fPIC", "-Wl,-Bsymbolic", "-Wl,--no-undefined", "-o", lib, *objects, *inc,
                           os.path.join(CSRC, "lsm_policy.cpp"), "-lpthread"])
    L = C.CDLL(lib)
    L.lsm_driver_create.argtypes = [C.POINTER(B._DriverConfig), C.c_void_p, C.POINTER(C.c_void_p)]
    L.lsm_driver_destroy.argtypes = [C.c_void_p]
    L.lsm_driver_destroy.restype = None
    L.lsm_driver_load_run.argtypes = [C.c_void_p, C.c_uint32, C.c_void_p, C.c_uint64]
    L.lsm_driver_flush.argtypes = L.lsm_driver_flush_unsorted.argtypes = [C.c_void_p, C.c_void_p, C.c_uint64]
    L.lsm_driver_flush_many.argtypes = [C.POINTER(C.c_void_p), C.POINTER(C.c_void_p), C.POINTER(C.c_uint64), C.c_uint32]
    L.lsm_driver_probe.argtypes = [C.c_void_p, C.POINTER(B._Queries), C.POINTER(B._Hits)]
    L.lsm_driver_tree.argtypes = [C.c_void_p, C.POINTER(B._TreeRun), C.c_uint32, C.POINTER(C.c_uint32)]
    L.lsm_driver_log.argtypes = [C.c_void_p, C.c_uint64, C.POINTER(B._DriverEvent), C.c_uint64]
    L.lsm_driver_log.restype = C.c_uint64
    return L


@pytest.fixture
def knobs(host):
    host.host_reset()

    class Knobs:
        def __setattr__(self, name, value):
            C.c_int64.in_dll(host, "host_" + name).value = value

        def read(self, name, kind=C.c_uint64):
            return kind.in_dll(host, "host_" + name).value
    return Knobs()


def run_of(keys, seq):
    """Sorted run of these key numbers, 64-byte aligned."""
    raw = np.zeros(len(keys) * 64 + 64, np.uint8)
    at = -raw.ctypes.data % 64
    run = raw[at:at + len(keys) * 64].reshape(-1, 64)
    for i, k in enumerate(sorted(keys)):
        run[i] = np.frombuffer(brute.pack_entry(int(k).to_bytes(32, "big"), seq, brute.PUT, vptr=1000 * seq + k, vlen=k + 1), np.uint8)
    return run


class Tree:
    """A driver beside the plain replay of the same tree."""

    def __init__(self, host, buffer=100, T=4, K=1, bits=16, stride=64, index=0, loaded=()):
        import paper_2511_16138_amd.binding as B
        self.B, self.host, self.bits, self.stride, self.index = B, host, bits, stride, index
        cfg = B._DriverConfig(buffer, T, K, 1 << 40, 0.2, 2, 16, 64.0, 0.01, stride, bits, index, B._DriverObserver(), None)
        self.h = C.c_void_p()
        assert host.lsm_driver_create(C.byref(cfg), None, C.byref(self.h)) == 0
        self.plain = DriverOracle(buffer, T, K, window_ops=1 << 40)
        self.loaded = [(level, run) for level, run in loaded]
        for level, run in self.loaded:
            assert host.lsm_driver_load_run(self.h, level, run.ctypes.data, len(run)) == 0
        for level in {level for level, _ in self.loaded}:
            self.plain.install(level, [run for at, run in self.loaded if at == level])

    def close(self):
        self.host.lsm_driver_destroy(self.h)

    def runs(self):
        n = C.c_uint32(0)
        assert self.host.lsm_driver_tree(self.h, None, 0, C.byref(n)) == 0
        out = (self.B._TreeRun * max(1, n.value))()
        assert self.host.lsm_driver_tree(self.h, out, n.value, C.byref(n)) == 0
        return [out[i] for i in range(n.value)]

    def unfinished(self, oracle):
        """What the tree lacks against the plain replay ("" = it is complete).  Anything wrong, as opposed to missing, fails."""
        lacks = []
        got = self.runs()
        want = [r for r in self.plain.runs_newest_first()]
        same_runs = len(got) == len(want)
        for i, t in enumerate(got):
            n = t.run.n
            if n == 0:
                continue
            entries = np.ctypeslib.as_array(C.cast(t.run.entries, C.POINTER(C.c_uint8)), (n, 64))
            if same_runs and not np.array_equal(entries, want[i]):
                same_runs = False
            keys = [bytes(e[:32]) for e in entries]
            assert keys == sorted(keys) and not any(k.startswith(b"\xab" * 8) for k in keys), "a run of unwritten memory"
            if t.fence.n == 0:
                lacks.append(f"fences of run {i}")  # a lookup is refused
            else:
                fences = np.ctypeslib.as_array(C.cast(t.fence.keys, C.POINTER(C.c_uint8)), (t.fence.n, 32))
                assert np.array_equal(fences, oracle.build_fences(entries, self.stride)), "wrong fences"
            if t.bloom.n_blocks != 0:
                words = np.ctypeslib.as_array(C.cast(t.bloom.blocks, C.POINTER(C.c_uint8)), (t.bloom.n_blocks, 16))
                assert np.array_equal(words, oracle.build_bloom(entries, t.bloom.n_blocks)), "a filter that is not the run's"
            elif self.bits:
                lacks.append(f"filter of run {i}")
            if t.index.n_buckets != 0:
                table = np.ctypeslib.as_array(C.cast(t.index.buckets, C.POINTER(C.c_uint8)), (t.index.n_buckets * 64,))
                assert (table == 0x11).all(), "an index that was not built"
            elif self.index and n >= self.index:
                lacks.append(f"index of run {i}")
        if not same_runs:
            lacks.append("runs")
        return ", ".join(lacks)

    def log(self):
        total = self.host.lsm_driver_log(self.h, 0, None, 0)
        out = (self.B._DriverEvent * max(1, total))()
        self.host.lsm_driver_log(self.h, 0, out, total)
        names = {1: lambda e: ("adopt", e.level, e.a, e.b), 2: lambda e: ("compact", e.level, e.a, e.n_in, e.n_out, e.b),
                 3: lambda e: ("move", e.level, e.a, e.n_out), 4: lambda e: ("probe", e.a, e.b, e.n_out)}
        return [names[out[i].kind](out[i]) for i in range(total)]


def flush_many(host, trees, runs):
    hd = (C.c_void_p * len(trees))(*[t.h for t in trees])
    ptr = (C.c_void_p * len(trees))(*[None if r is None else r.ctypes.data for r in runs])
    n = (C.c_uint64 * len(trees))(*[0 if r is None else len(r) for r in runs])
    for t, r in zip(trees, runs):
        if r is not None:
            t.plain.flush(r.copy())
    return host.lsm_driver_flush_many(hd, ptr, n, len(trees))


def resting_trees(host):
    """Trees whose flushed run comes to rest at once: copies with two fence strides, a filter from hashes and an index, no
    filter at all."""
    old = lambda: [(1, run_of(range(0, 300, 3), 1))]  # noqa: E731
    return [Tree(host, K=3, loaded=old()), Tree(host, K=3), Tree(host, K=3, stride=16, loaded=old()), Tree(host, K=3, index=1, loaded=old()),
            Tree(host, K=3, bits=0), Tree(host, K=3, stride=16)]


FAULTS = ["malloc_in", "kernel_in", "late_in"]


def sweep(host, knobs, oracle, fault, trees_of, flushes):
    """Every place at which `fault` can strike one flush_many: yields (place, status, trees, what each lacks)."""
    for place in range(1, 1000):
        trees = trees_of(host)
        runs = flushes()
        setattr(knobs, fault, place)
        rc = flush_many(host, trees, runs)
        struck = knobs.read(fault, C.c_int64) == 0
        setattr(knobs, fault, 0)
        lacks = [t.unfinished(oracle) for t in trees]
        for t, r, missing in zip(trees, runs, lacks):
            if r is not None and not missing:
                r[:] = 0xEE  # the caller's memory again: a complete tree does not refer to it
                assert t.unfinished(oracle) == ""
        yield place, rc, trees, lacks
        assert knobs.read("dirty_filters") == 0
        for t in trees:
            t.close()
        if not struck:
            assert rc == 0
            return
    raise AssertionError("the sweep did not end")


@pytest.mark.parametrize("fault", FAULTS)
def test_a_failure_while_runs_are_completed_leaves_out_no_other_tree(host, knobs, oracle, fault):
    flushes = lambda: [run_of(range(j, 90 + j), 2) for j in range(6)]  # noqa: E731
    for place, rc, trees, lacks in sweep(host, knobs, oracle, fault, resting_trees, flushes):
        missing = [x for x in lacks if x]
        assert rc == (HIP if missing else 0), (place, rc, lacks)
        if fault == "malloc_in":
            assert len(missing) <= 1, (place, lacks)
        # the next call that gets through makes up for what was left out
        assert flush_many(host, trees, [run_of(range(200 + j, 260 + j), 3) for j in range(6)]) == 0
        assert not any(t.unfinished(oracle) for t in trees), place


def merging_trees(host):
    """Trees with compactions due: one that stays, one whose output moves down onto a run, one that only rests, one with an
    index, a chain of three levels."""
    return [Tree(host, loaded=[(1, run_of(range(0, 300, 3), 1))]),
            Tree(host, loaded=[(1, run_of(range(0, 790, 2), 2)), (2, run_of(range(1, 1800, 2), 1))]),
            Tree(host, K=2, stride=16, loaded=[(1, run_of(range(40, 90), 1))]),
            Tree(host, index=150, loaded=[(1, run_of(range(0, 300, 3), 1)), (2, run_of(range(600, 700), 0))]),
            Tree(host, buffer=50, T=2, loaded=[(1, run_of(range(0, 99), 3)), (2, run_of(range(150, 349), 2)), (3, run_of(range(500, 600), 1))])]


@pytest.mark.parametrize("fault", FAULTS)
def test_a_failure_in_one_tree_s_compaction_leaves_the_others_as_after_their_own_flush(host, knobs, oracle, fault):
    flushes = lambda: [run_of(range(j, 90 + j), 4) for j in range(5)]  # noqa: E731
    places = 0
    for place, rc, trees, lacks in sweep(host, knobs, oracle, fault, merging_trees, flushes):
        places += 1
        missing = [x for x in lacks if x]
        if fault == "malloc_in":  # memory is the tree's own, and what the trees share can be done without
            assert len(missing) <= 1, (place, lacks)
        assert rc == (HIP if missing else 0), (place, rc, lacks)
        for t, x in zip(trees, lacks):
            assert x or t.log() == t.plain.log, place
    assert places > (20 if fault == "malloc_in" else 5)


def test_a_tree_with_too_many_runs_does_not_stop_the_others(host, knobs, oracle):
    """65 runs in a level are refused; the compactions that were due beside that one are done, in the first step of the call
    and in later ones."""
    trees = merging_trees(host) + [Tree(host, loaded=[(1, run_of([j], 1)) for j in range(64)])]
    runs = [run_of(range(j, 90 + j), 4) for j in range(6)]
    assert flush_many(host, trees, runs) == BAD_ARG
    for r in runs[:5]:
        r[:] = 0xEE
    for t in trees[:5]:
        assert t.unfinished(oracle) == ""
        assert t.log() == t.plain.log
    assert flush_many(host, trees[:5], [run_of(range(100 + j, 190 + j), 5) for j in range(5)]) == 0  # the trees go on
    for t in trees[:5]:
        assert t.unfinished(oracle) == ""
        assert t.log() == t.plain.log
    for t in trees:
        t.close()


def probe(host, tree, keys, blocks=4):
    """One request per key: the numbers from it upwards.  Returns the call's status and hit_len."""
    B = tree.B
    q = np.zeros((len(keys), blocks, 32), np.uint8)
    for r, k in enumerate(keys):
        for j in range(blocks):
            q[r, j] = np.frombuffer(int(k + j).to_bytes(32, "big"), np.uint8)
    nb, hit_len = np.full(len(keys), blocks, np.uint32), np.zeros(len(keys), np.uint32)
    hits = np.zeros((len(keys), blocks, 16), np.uint8)
    qd, hd = B._Queries(q.ctypes.data, nb.ctypes.data, len(keys), blocks), B._Hits(hit_len.ctypes.data, hits.ctypes.data)
    return host.lsm_driver_probe(tree.h, C.byref(qd), C.byref(hd)), hit_len


@pytest.mark.parametrize("fault", ["kernel_in", "late_in"])
@pytest.mark.parametrize("place", [1, 2])  # the lookup, the launch that adds up what it found
def test_what_a_batch_found_is_its_own_after_a_batch_that_failed(host, knobs, oracle, fault, place):
    """The statistics that reach the log are those of the batch of this call, however long they take to arrive."""
    tree = Tree(host, loaded=[(1, run_of(range(100), 1))])
    knobs.slow_stats = 1
    assert probe(host, tree, [0, 50, 98, 200])[0] == 0           # 4 + 4 + 2 blocks
    setattr(knobs, fault, place)
    assert probe(host, tree, [300])[0] == HIP
    assert probe(host, tree, [10])[0] == 0
    assert probe(host, tree, [97, 98, 99])[0] == 0               # 3 + 2 + 1
    assert tree.log() == [("probe", 4, 3, 10), ("probe", 1, 1, 4), ("probe", 3, 3, 6)]
    tree.close()


@pytest.mark.parametrize("call", ["flush", "flush_unsorted"])
def test_a_count_is_that_of_its_own_merge_after_a_call_that_failed(host, knobs, oracle, call):
    """A call that reports an error may leave a merge (or a sort) under way, which stores its count when it ends: the next
    call's runs have their own lengths all the same, however long that takes."""
    old, failed, last = run_of(range(0, 300, 3), 1), run_of(range(90), 2), run_of(range(1000, 1040), 3)
    tree = Tree(host, loaded=[(1, old)])
    flush = getattr(host, "lsm_driver_" + call)
    knobs.slow_merges = 1
    knobs.late_in = 1
    assert flush(tree.h, failed.ctypes.data, len(failed)) == HIP
    assert flush(tree.h, last.ctypes.data, len(last)) == 0
    # the sorted run had entered the tree when its merge failed; a write buffer that was not sorted had not
    want = oracle.compact([last, failed, old] if call == "flush" else [last, old], 1)
    runs = tree.runs()
    assert len(runs) == 1 and runs[0].run.n == len(want)
    assert np.array_equal(np.ctypeslib.as_array(C.cast(runs[0].run.entries, C.POINTER(C.c_uint8)), (len(want), 64)), want)
    tree.close()


def test_words_the_host_watches_are_in_coherent_memory(host, knobs):
    """The host reads counts and statistics while kernels run: whatever the runtime's default for pinned memory is, these
    words are asked for as coherent."""
    tree = Tree(host, loaded=[(1, run_of(range(100), 1))])
    assert flush_many(host, [tree], [run_of(range(50), 2)]) == 0
    assert probe(host, tree, [0])[0] == 0
    assert knobs.read("pinned_flags", C.c_uint32) & 0x40000000  # hipHostMallocCoherent, in every allocation
    tree.close()


@pytest.mark.parametrize("trees", [1, 2])
def test_a_small_tree_takes_little_memory(host, knobs, trees):
    """The first flushes of new trees with a buffer of 100 entries: alone and in a batch, no block is as large as those that the runtime asks
    the kernel driver for one by one (2 MB), and all of them together are less than that."""
    new = [Tree(host, T=10) for _ in range(trees)]
    for step in range(8):
        runs = [run_of(range(7 * step + j, 7 * step + j + 90), step) for j in range(trees)]
        assert flush_many(host, new, runs) == 0
        assert all(host.lsm_driver_flush(t.h, r.ctypes.data, len(r)) == 0 for t, r in zip(new, runs))
    assert 0 < knobs.read("largest") <= 512 << 10
    assert knobs.read("bytes") < 2 << 20
    for t in new:
        t.close()


def flush(host, trees, runs):
    """One tree by its own call, several by the shared one."""
    if len(trees) > 1:
        return flush_many(host, trees, runs)
    trees[0].plain.flush(runs[0].copy())
    return host.lsm_driver_flush(trees[0].h, runs[0].ctypes.data, len(runs[0]))


def memory_was_used_as_promised(knobs):
    return knobs.read("stale_words") == 0 and knobs.read("outside") == 0 and knobs.read("dirty_filters") == 0


def check(oracle, trees):
    for t in trees:
        assert t.unfinished(oracle) == ""
        assert t.log() == t.plain.log


@pytest.mark.parametrize("count", [1, 3])
def test_no_status_word_of_an_earlier_call_is_taken_for_this_one_s(host, knobs, oracle, count):
    """Merges in one launch find their status words zero or of a smaller epoch, far beyond the eight epochs of this build, in a workspace that grows
    (several times) and holds the scratch memory of long filters (4,096 bits a key) beside the compaction's."""
    sizes = [600] if count == 1 else [100, 200, 300]
    trees = [Tree(host, buffer=n, T=6, bits=4096) for n in sizes]
    for step in range(60):
        runs = [run_of(range(n // 10 * step, n // 10 * step + n), step) for n in sizes]
        assert flush(host, trees, runs) == 0
        check(oracle, trees)
    assert memory_was_used_as_promised(knobs)
    assert knobs.read("largest") > 256 << 10  # the workspace has grown
    assert knobs.read("whole_merges") > 30 and knobs.read("zeroings") > 5 and knobs.read("hashed_filters") > 10
    for t in trees:
        t.close()


def newest_versions(oracle, runs):
    return oracle.compact([np.array(r) for r in runs if len(r)], 1)


@pytest.mark.parametrize("fault", FAULTS)
@pytest.mark.parametrize("count", [1, 3])
def test_status_words_are_zeroed_after_a_call_that_failed(host, knobs, oracle, fault, count):
    """A call that is refused, one that reports an error although its work is done (and its status words are written), memory that runs out where the
    workspace grows: whatever comes next meets no word of that call, and the trees hold what was flushed."""
    struck_at = 0
    for place in range(1, 14):
        trees = [Tree(host, T=6, bits=4096, loaded=[(1, run_of(range(0, 300, 3), 1))]) for _ in range(count)]
        kept, results = [], []
        for step in range(24):
            if step == 4:
                zeroed = knobs.read("zeroings")
                setattr(knobs, fault, place)
            kept.append([run_of(range(5 * step + j, 5 * step + j + 60), 2 + step) for j in range(count)])  # a call that failed may still refer to them
            results.append(flush(host, trees, kept[-1]))
        struck = knobs.read(fault, C.c_int64) == 0
        setattr(knobs, fault, 0)
        struck_at += struck
        assert set(results) <= {0, HIP} and results[-1] == 0 and (HIP in results) <= struck
        assert memory_was_used_as_promised(knobs), place
        assert knobs.read("zeroings") > zeroed and knobs.read("whole_merges") > 0
        for t in trees:
            got = [np.ctypeslib.as_array(C.cast(r.run.entries, C.POINTER(C.c_uint8)), (r.run.n, 64)) for r in t.runs() if r.run.n]
            assert np.array_equal(newest_versions(oracle, got), newest_versions(oracle, t.plain.runs_newest_first())), place
            t.close()
    assert struck_at > 5


def test_filters_that_are_no_span_do_not_go_through_the_merge(host, knobs):
    """A span of memory that a merge zeroes has fewer than 2^31 words of 16 bytes.  A filter of more (here 80 keys of 2^32 - 1 bits each, 43 GB)
    is left to the builds behind the merge: with no memory for it the merge is made all the same."""
    tree = Tree(host, T=4, bits=(1 << 32) - 1)
    runs = [run_of(range(40 * step, 40 * step + 40), step) for step in range(2)]
    for r in runs:
        tree.plain.flush(r.copy())
        assert host.lsm_driver_flush(tree.h, r.ctypes.data, len(r)) == HIP  # no memory for the filter
    assert tree.log() == tree.plain.log  # the merge among them
    assert [t.run.n for t in tree.runs()] == [80]
    tree.close()
