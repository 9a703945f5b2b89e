"""Performance cases of the LSM key index: what a serving system has the library do, through its public calls.

A case is a plain dict; its "kind" says which path it takes:

  flush     a write buffer as it was filled -> sorted run with fence index               (write side, smallest calls)
  compact   merge of sorted runs, the core of the index: flush-level, leveled and tiered shapes
  rebuild   a compaction that leaves a searchable run: merge + fences + key hashes, filter, hash index, first lookups
  batch     many independent small compactions (one per shard) in one call, with fence indices and filters
  probe     batched longest-prefix lookups in a leveled tree (read side)
  range     batched key-range scans of a leveled tree (the read list of get_batch)
  driver    a live tree under its own driver: write buffers flushed, lookups in between
  shards    several live trees stepped together, then looked up

Inputs follow the repository's synthetic workloads: sequences of 16..128 blocks, 60 % behind a Zipf-chosen shared
prefix of 32..96 blocks, 32-byte keys (8-byte family digest, block number, digest), 8 % overwrites and 3..5 %
tombstones in newer runs; tiered inputs hold 20 % of their keys in two to four runs with random sequence numbers.
Keys are digests of (owner, block) computed in closed form, so that 100 million entries are made in about a second.
"""
import math

import numpy as np
import torch

import paper_2511_16138_amd as lsm

DEVICE = "cuda"
STRIDE = 64            # entries per fence: one 4 KiB page
BLOOM_BITS = 16        # filter bits per key
MAX_BLOCKS = 256       # block keys per request
MAX_POOL_BLOCKS = 96
RANGE_SLOT = 128       # result entries per key range
BUFFER = 3600          # write buffer of the mixed workload, in entries
VLEN = 16 * 40 * 1024  # bytes of a block's tensors
OVERWRITES, TOMBSTONES = 0.08, 0.03


# ---------------------------------------------------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------------------------------------------------
def listed():
    return [
        # one full write buffer of the mixed workload: the smallest call of the write path, launch latency counts
        {"name": "flush 3600", "kind": "flush", "entries": 3600},
        # a large write buffer of a bulk load, an odd size
        {"name": "flush 100001", "kind": "flush", "entries": 100_001},
        # four flushed runs into level 1: the ordinary small compaction
        {"name": "compact 4 x 16k", "kind": "compact", "shape": "leveled", "runs": 4, "ratio": 1, "entries": 65_536, "last": False, "fences": True},
        # leveled compaction, size ratio 10: a 2M-entry level into the 20M-entry level below
        {"name": "compact 2M + 20M", "kind": "compact", "shape": "leveled", "runs": 2, "ratio": 10, "entries": 22_000_000, "last": False, "fences": True},
        # tiered compaction into the last level: 16 overlapping runs of about 4M entries
        {"name": "compact 16 x 4M", "kind": "compact", "shape": "tiered", "runs": 16, "ratio": 1, "entries": 67_108_864, "last": True, "fences": False},
        # a mid-size tiered compaction with everything lookups need of the new run, and the first batch of lookups
        {"name": "rebuild 8 x 500k", "kind": "rebuild", "runs": 8, "entries": 4_000_000, "requests": 1024},
        # one round of small compactions of 16 shards
        {"name": "batch of 16", "kind": "batch", "jobs": 16, "entries": 30_000, "runs": 2},
        # lookup-heavy serving: full request batches against a 5-level tree of 100M entries with filters
        {"name": "probe 100M, 4096", "kind": "probe", "entries": 100_000_000, "requests": 4096, "filters": True, "index": False},
        # the lookups of one scheduler tick against a mid-size tree with hash indices: few requests, latency counts
        {"name": "probe 20M indexed, 64", "kind": "probe", "entries": 20_000_000, "requests": 64, "filters": True, "index": True},
        # read lists for one tick's prefixes
        {"name": "range 500", "kind": "range", "entries": 4_000_000, "ranges": 500},
        # mixed serving on one live tree: a flush every buffer, lookups after every 16th
        {"name": "driver mixed", "kind": "driver", "entries": 4_000_000, "buffer": BUFFER, "flushes": 96, "probe_every": 16, "requests": 1024, "sorted": True},
        # eight live trees (key-range shards) flushed in step
        {"name": "shards 8", "kind": "shards", "trees": 8, "entries": 1_000_000, "buffer": BUFFER, "flushes": 24, "requests": 512},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["flush", "compact", "compact", "compact", "rebuild", "batch", "probe", "probe", "range", "driver", "shards"])
    if kind == "flush":
        return {"kind": kind, "entries": _log_int(rng, 1, 262_144)}
    if kind == "compact":
        shape = rng.choice(["leveled", "tiered"])
        runs = rng.choice([2, 2, 3, 4]) if shape == "leveled" else rng.randint(2, 24)
        most = 22_000_000 if shape == "leveled" else 50_000_000
        return {"kind": kind, "shape": shape, "runs": runs, "ratio": rng.choice([1, 2, 4, 10]) if shape == "leveled" else 1,
                "entries": _log_int(rng, 2_000, most), "last": rng.random() < 0.5, "fences": rng.random() < 0.5}
    if kind == "rebuild":
        return {"kind": kind, "runs": rng.randint(2, 16), "entries": _log_int(rng, 20_000, 16_000_000), "requests": _log_int(rng, 16, 4096)}
    if kind == "batch":
        return {"kind": kind, "jobs": rng.randint(2, 20), "entries": _log_int(rng, 2_000, 200_000), "runs": rng.choice([2, 2, 3, 5])}
    if kind == "probe":
        return {"kind": kind, "entries": _log_int(rng, 50_000, 60_000_000), "requests": _log_int(rng, 1, 4096), "filters": rng.random() < 0.8,
                "index": rng.random() < 0.5}
    if kind == "range":
        return {"kind": kind, "entries": _log_int(rng, 50_000, 20_000_000), "ranges": _log_int(rng, 1, 2000)}
    if kind == "driver":
        return {"kind": kind, "entries": _log_int(rng, 200_000, 8_000_000), "buffer": _log_int(rng, 500, 8000), "flushes": rng.randint(16, 96),
                "probe_every": rng.choice([4, 8, 16]), "requests": _log_int(rng, 16, 2048), "sorted": rng.random() < 0.5}
    return {"kind": kind, "trees": rng.randint(2, 12), "entries": _log_int(rng, 100_000, 1_000_000), "buffer": _log_int(rng, 500, 8000),
            "flushes": rng.randint(8, 24), "requests": _log_int(rng, 16, 512)}


def tolerance(case):
    return "exact"  # integers and bytes


# ---------------------------------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------------------------------
def _i64(x):
    x &= (1 << 64) - 1
    return x - (1 << 64) if x >= 1 << 63 else x


_ODD = [_i64(v) for v in (0x9E3779B97F4A7C15, 0xBF58476D1CE4E5B9, 0x94D049BB133111EB)]


def _lsr(x, s):
    return (x >> s) & ((1 << (64 - s)) - 1)


def _mix(x, salt):
    """64-bit digest (the splitmix64 output function) of x under a salt."""
    x = (x ^ salt) + _ODD[0]
    x = (x ^ _lsr(x, 30)) * _ODD[1]
    x = (x ^ _lsr(x, 27)) * _ODD[2]
    return x ^ _lsr(x, 31)


def _bswap(x):
    x = ((x & 0x00FF00FF00FF00FF) << 8) | (_lsr(x, 8) & 0x00FF00FF00FF00FF)
    x = ((x & 0x0000FFFF0000FFFF) << 16) | (_lsr(x, 16) & 0x0000FFFF0000FFFF)
    return (x << 32) | _lsr(x, 32)


class Keys:
    """The keys of a stream of sequences in arrival order: the shared prefixes first, then every sequence's own blocks."""

    def __init__(self, n, seed):
        self.n = n
        self.gen = g = torch.Generator(device=DEVICE)
        g.manual_seed(seed)
        self.salt = [_i64((seed + 1) * 0x9E3779B97F4A7C15 + i * 0xD6E8FEB86659FD93) for i in range(4)]
        self.n_pool = max(16, min(4096, n // 16_384))
        self.plen = torch.randint(32, MAX_POOL_BLOCKS + 1, (self.n_pool,), generator=g, device=DEVICE)
        n_seq = n // 30 + 1024  # a sequence brings about 45 blocks of its own
        length = torch.randint(16, 129, (n_seq,), generator=g, device=DEVICE)
        pid = torch.searchsorted(self._zipf(0.9), torch.rand(n_seq, generator=g, device=DEVICE, dtype=torch.float64)).clamp_(max=self.n_pool - 1)
        pid = torch.where(torch.rand(n_seq, generator=g, device=DEVICE) < 0.6, pid, torch.full_like(pid, -1))
        shared = torch.where(pid >= 0, torch.minimum(self.plen[pid.clamp(min=0)], length), torch.zeros_like(length))
        owner_len = torch.cat([self.plen, length - shared])  # owners: the pool prefixes, then the sequences
        ends = torch.cumsum(owner_len, 0)
        n_owners = int(torch.searchsorted(ends, torch.tensor([n], device=DEVICE)).item()) + 1
        owner_len = owner_len[:n_owners].clone()
        owner_len[-1] -= ends[n_owners - 1] - n
        self.n_seq = max(0, n_owners - self.n_pool)
        self.pid, self.shared, self.own_len = pid[: self.n_seq], shared[: self.n_seq], owner_len[self.n_pool:]
        first_block = torch.cat([torch.zeros_like(self.plen), self.shared])[:n_owners]
        family = torch.cat([torch.arange(self.n_pool, device=DEVICE),
                            torch.where(self.pid >= 0, self.pid, self.n_pool + torch.arange(self.n_seq, device=DEVICE))])[:n_owners]
        self.owner = torch.repeat_interleave(torch.arange(n_owners, device=DEVICE), owner_len, output_size=n)
        self.block = torch.arange(n, device=DEVICE) - (torch.cumsum(owner_len, 0) - owner_len - first_block)[self.owner]
        self.family = family[self.owner]
        # ascending key order: (family digest, block number, digest)
        fam_rank = torch.empty(self.n_pool + self.n_seq, dtype=torch.int64, device=DEVICE)
        all_fam = self.family_word(torch.arange(self.n_pool + self.n_seq, device=DEVICE))
        fam_rank[torch.argsort(all_fam ^ _i64(1 << 63))] = torch.arange(all_fam.numel(), device=DEVICE)
        order = torch.argsort(_mix(self.owner * 4096 + self.block, self.salt[1]) ^ _i64(1 << 63))
        order = order[torch.sort(fam_rank[self.family[order]] * 4096 + self.block[order], stable=True)[1]]
        self.rank = torch.empty(n, dtype=torch.int64, device=DEVICE)
        self.rank[order] = torch.arange(n, device=DEVICE)

    def _zipf(self, a):
        w = torch.arange(1, self.n_pool + 1, dtype=torch.float64, device=DEVICE) ** -a
        return torch.cumsum(w, 0) / w.sum()

    def family_word(self, family):
        return _mix(family, self.salt[0])

    def words(self, family, block, owner):
        """Big-endian key words of block `block` of `owner` in `family`, as stored (byte-swapped): [..., 4]."""
        c0 = _mix(owner * 4096 + block, self.salt[1])
        c1 = _mix(c0, self.salt[2])
        c2 = _mix(c1, self.salt[3])
        w = [self.family_word(family), (block << 48) | _lsr(c0, 16), (c0 << 48) | _lsr(c1, 16), (c1 << 48) | _lsr(c2, 16)]
        return _bswap(torch.stack(w, dim=-1))

    def entries(self, idx, seqno, dead, ordered=True):
        """[n, 8] entries of the keys idx, ascending by key if `ordered`."""
        if ordered:
            order = torch.argsort(self.rank[idx])
            idx, seqno, dead = idx[order], seqno[order], dead[order]
        e = torch.empty((idx.numel(), 8), dtype=torch.int64, device=DEVICE)
        step = 1 << 24
        for a in range(0, idx.numel(), step):  # in pieces: the temporaries of a long run are several times its size
            i = idx[a:a + step]
            e[a:a + step, 0:4] = self.words(self.family[i], self.block[i], self.owner[i])
        e[:, 4] = seqno
        e[:, 5] = dead
        e[:, 6] = torch.where(dead, 0, (_lsr(seqno, 12) << 32) | (seqno & 0xFFF))
        e[:, 7] = torch.where(dead, 0, VLEN)
        return e

    def epochs(self, sizes, ordered=lambda epoch: True, repeats=0.0):
        """One operation stream cut into runs of `sizes` entries (oldest first); newer ones also overwrite and delete
        older keys.  `repeats`: share of an unordered epoch's entries that write a key of the same epoch again."""
        runs, fresh, seq = [], 0, 0
        for e, n in enumerate(sizes):
            m = min(int(round(n * (OVERWRITES + TOMBSTONES))), fresh) if e else 0
            edge = torch.arange(m + 1, device=DEVICE) * fresh // max(m, 1)
            pick = edge[:-1] + torch.randint(0, 1 << 40, (m,), generator=self.gen, device=DEVICE) % (edge[1:] - edge[:-1]).clamp(min=1)
            dead = torch.rand(m, generator=self.gen, device=DEVICE) < TOMBSTONES / (OVERWRITES + TOMBSTONES)
            idx = torch.cat([fresh + torch.arange(n - m, device=DEVICE), pick])
            dead = torch.cat([torch.zeros(n - m, dtype=torch.bool, device=DEVICE), dead])
            fresh += n - m
            if not ordered(e):
                shuffle = torch.randperm(n, generator=self.gen, device=DEVICE)
                idx, dead = idx[shuffle], dead[shuffle]
                again = torch.rand(n, generator=self.gen, device=DEVICE) < repeats
                earlier = (torch.rand(n, generator=self.gen, device=DEVICE, dtype=torch.float64) * torch.arange(n, device=DEVICE)).to(torch.int64)
                idx = torch.where(again, idx[earlier], idx)
            runs.append(self.entries(idx, seq + torch.arange(n, device=DEVICE), dead, ordered(e)))
            seq += n
        return runs

    def overlapping(self, n_runs, run_len):
        """Runs of run_len entries for a tiered merge: every key in one run, 20 % of them in two to four; random sequence
        numbers."""
        copies = torch.where(torch.rand(self.n, generator=self.gen, device=DEVICE) < 0.2,
                             torch.randint(2, min(4, n_runs) + 1, (self.n,), generator=self.gen, device=DEVICE), 1)
        first = torch.randint(0, n_runs, (self.n,), generator=self.gen, device=DEVICE)
        runs = []
        for r in range(n_runs):
            idx = torch.nonzero((r - first) % n_runs < copies).squeeze(1)
            idx = idx[torch.randperm(idx.numel(), generator=self.gen, device=DEVICE)[:run_len]]
            assert idx.numel() == run_len
            seqno = torch.randint(0, 1 << 62, (idx.numel(),), generator=self.gen, device=DEVICE)
            runs.append(self.entries(idx, seqno, torch.rand(idx.numel(), generator=self.gen, device=DEVICE) < 0.05))
        return runs

    def requests(self, n):
        """Longest-prefix requests of 16..256 blocks: 70 % follow a stored sequence behind a Zipf(0.99)-chosen shared
        prefix for a random part of its own blocks, the others share nothing with the tree."""
        g = self.gen
        nb = torch.randint(16, MAX_BLOCKS + 1, (n,), generator=g, device=DEVICE)
        hit = torch.rand(n, generator=g, device=DEVICE) < 0.7
        pid = torch.searchsorted(self._zipf(0.99), torch.rand(n, generator=g, device=DEVICE, dtype=torch.float64)).clamp_(max=self.n_pool - 1)
        shared, follow, owner = self.plen[pid], torch.zeros_like(pid), torch.zeros_like(pid)
        if self.n_seq:
            by_pid = torch.argsort(self.pid, stable=True)
            count = torch.bincount(self.pid + 1, minlength=self.n_pool + 1)
            start = torch.cumsum(count, 0) - count
            c = count[pid + 1]
            nth = torch.randint(0, 1 << 40, (n,), generator=g, device=DEVICE) % c.clamp(min=1)
            seq = by_pid[(start[pid + 1] + nth).clamp(max=self.n_seq - 1)]
            follows = c > 0
            shared = torch.where(follows, self.shared[seq], shared)
            part = torch.rand(n, generator=g, device=DEVICE)
            follow = torch.where(follows, (self.own_len[seq] * part).to(torch.int64), follow)
            owner = self.n_pool + seq
        shared, follow = torch.where(hit, shared, 0), torch.where(hit, follow, 0)
        t = torch.arange(MAX_BLOCKS, device=DEVICE).unsqueeze(0)
        stranger = (1 << 40) + torch.arange(n, device=DEVICE)
        col = lambda x: x.unsqueeze(1)  # noqa: E731
        own = torch.where(t < col(shared), col(pid), torch.where(t < col(shared + follow), col(owner), col(stranger)))
        fam = col(torch.where(hit, pid, stranger)).expand(-1, MAX_BLOCKS)
        keys = self.words(fam, t.expand(n, -1), own)
        keys[(t >= col(nb))] = 0
        return keys.contiguous(), nb.to(torch.int32)

    def ranges(self, n):
        """Key ranges of one prefix each: a shared prefix, or a slice of a sequence that has none."""
        g = self.gen
        fam = torch.randint(0, self.n_pool, (n,), generator=g, device=DEVICE)
        last = self.plen[fam]
        alone = torch.nonzero(self.pid < 0).squeeze(1)
        if alone.numel():
            seq = alone[torch.randint(0, alone.numel(), (n,), generator=g, device=DEVICE)]
            own = torch.rand(n, generator=g, device=DEVICE) < 0.6
            fam, last = torch.where(own, self.n_pool + seq, fam), torch.where(own, self.own_len[seq], last)
        first = (torch.rand(n, generator=g, device=DEVICE) * last * 0.5).to(torch.int64)
        zero = torch.zeros_like(fam)
        bound = lambda k: _bswap(torch.stack([self.family_word(fam), k << 48, zero, zero], dim=-1)).contiguous()  # noqa: E731
        return bound(first), bound(last)


def _level_sizes(total, buffer):
    """Runs of a leveled tree with size ratio 10, newest (smallest) first."""
    levels = 1
    while buffer * 10 ** levels < total:
        levels += 1
    share = sum(10 ** i for i in range(levels))
    sizes = [max(1, total * 10 ** i // share) for i in range(levels)]
    sizes[-1] = max(1, total - sum(sizes[:-1]))
    return sizes


def _indexed_tree(case, seed, filters, index):
    sizes = _level_sizes(case["entries"], BUFFER)
    keys = Keys(sum(sizes), seed)
    tree = []
    for level, run in enumerate(reversed(keys.epochs(sizes[::-1]))):
        hashes = lsm.lsm_hash_keys(run) if filters or index else None
        bloom = lsm.lsm_build_bloom_hashed(hashes, lsm.lsm_bloom_blocks(run.shape[0], BLOOM_BITS)) if filters else None
        tree.append(lsm.TreeRun(run, lsm.lsm_build_fences(run, STRIDE), STRIDE, level + 1, bloom,
                                lsm.lsm_build_hash_index(hashes) if index else None))
    return keys, tree


def _ceil(a, b):
    return -(-a // b)


def _compact_runs(case, seed):
    n, k = case["entries"], case["runs"]
    if case.get("shape", "tiered") == "tiered":
        run_len = max(1, n // k)
        mean = 1.4 if k >= 4 else 1 + 0.2 * (0.5 * (2 + min(4, k)) - 1)
        keys = Keys(int(k * (run_len + 6 * math.sqrt(run_len) + 16) / mean) + 1, seed)  # enough candidates for every run
        return keys, keys.overlapping(k, run_len)
    share = [case["ratio"] ** i for i in range(k)]  # newest first
    sizes = [max(1, n * s // sum(share)) for s in share]
    keys = Keys(sum(sizes), seed)
    return keys, keys.epochs(sizes[::-1])[::-1]


def _hit_buffers(n):
    return (torch.zeros(n, dtype=torch.int32, device=DEVICE), torch.zeros((n, MAX_BLOCKS, 2), dtype=torch.int64, device=DEVICE))


def _driver(case, seed):
    """A driver with its starting tree, the write buffers of one pass, and the keys for requests."""
    sizes = _level_sizes(case["entries"], case["buffer"])
    flushes = case["flushes"]
    keys = Keys(sum(sizes) + flushes * case["buffer"], seed)
    ordered = case.get("sorted", True)
    runs = keys.epochs(sizes[::-1] + [case["buffer"]] * flushes, lambda e: ordered or e < len(sizes), 0.03)
    d = lsm.LsmDriver(case["buffer"], window_ops=16_384, t_grid=(2, 16), bloom_bits=BLOOM_BITS)
    for level, run in enumerate(reversed(runs[: len(sizes)])):
        d.load_run(level + 1, run)
    return keys, d, runs[len(sizes):]


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "flush":
        n = case["entries"]
        keys = Keys(2 * n + 64, seed)
        s["buffer"] = keys.epochs([n, n], lambda e: False, 0.05)[1]
        s["out"] = torch.zeros((n, 8), dtype=torch.int64, device=DEVICE)
        s["n_out"] = torch.zeros(1, dtype=torch.int64, device=DEVICE)
        s["fences"] = torch.zeros((_ceil(n, STRIDE), 4), dtype=torch.int64, device=DEVICE)
    elif kind in ("compact", "rebuild"):
        keys, s["runs"] = _compact_runs(case, seed)
        total = sum(r.shape[0] for r in s["runs"])
        s["out"] = torch.zeros((total, 8), dtype=torch.int64, device=DEVICE)
        s["fences"] = torch.zeros((_ceil(total, STRIDE), 4), dtype=torch.int64, device=DEVICE)
        s["workspace"] = torch.empty(lsm.lsm_compact_workspace_bytes([r.shape[0] for r in s["runs"]]), dtype=torch.uint8, device=DEVICE)
        if kind == "compact":
            s["n_out"] = torch.zeros(1, dtype=torch.int64, device=DEVICE)
        else:
            s["n_out"] = torch.zeros(1, dtype=torch.int64, pin_memory=True)
            s["hashes"] = torch.zeros(total, dtype=torch.int64, device=DEVICE)
            s["bloom"] = torch.zeros((lsm.lsm_bloom_blocks(total, BLOOM_BITS), 4), dtype=torch.int32, device=DEVICE)
            s["queries"] = keys.requests(case["requests"])
            s["hits"] = _hit_buffers(case["requests"])
    elif kind == "batch":
        s["jobs"] = []
        for j in range(case["jobs"]):
            n = max(64, int(case["entries"] * (0.5 + ((j * 5) % 8) / 8)))  # shards fill unevenly
            newer = [max(1, n // 11)] * (case["runs"] - 1)
            sizes = [max(1, n - sum(newer))] + newer
            s["jobs"].append((Keys(sum(sizes), seed * 1000 + j).epochs(sizes)[::-1], 0))
    elif kind == "probe":
        keys, s["tree"] = _indexed_tree(case, seed, case["filters"], case["index"])
        s["queries"] = keys.requests(case["requests"])
        s["hits"] = _hit_buffers(case["requests"])
    elif kind == "range":
        keys, s["tree"] = _indexed_tree(case, seed, False, False)
        s["lo"], s["hi"] = keys.ranges(case["ranges"])
        s["entries"] = torch.zeros((case["ranges"], RANGE_SLOT, 8), dtype=torch.int64, device=DEVICE)
        s["counts"] = torch.zeros(case["ranges"], dtype=torch.int32, device=DEVICE)
    elif kind == "driver":
        keys, s["driver"], s["buffers"] = _driver(case, seed)
        probes = _ceil(case["flushes"], case["probe_every"])
        s["queries"] = [keys.requests(case["requests"]) for _ in range(probes)]
        s["hits"] = [_hit_buffers(case["requests"]) for _ in range(probes)]
    else:
        s["trees"] = [_driver(case, seed * 100 + i) for i in range(case["trees"])]
        s["queries"] = [t[0].requests(case["requests"]) for t in s["trees"]]
        s["hits"] = [_hit_buffers(case["requests"]) for _ in s["trees"]]
        s["trees"] = [t[1:] for t in s["trees"]]
    return s


# ---------------------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------------------
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "flush":
        out, n_out = lsm.lsm_flush_buffer(s["buffer"], s["out"], s["n_out"], fences=s["fences"], fence_stride=STRIDE)
        return out, n_out, s["fences"]
    if kind == "compact":
        flags = lsm.LSM_BOTTOMMOST if case["last"] else 0
        if not case["fences"]:
            return lsm.lsm_compact(s["runs"], flags, s["out"], s["n_out"], s["workspace"])
        out, n_out = lsm.lsm_compact(s["runs"], flags, s["out"], s["n_out"], s["workspace"], fences=s["fences"], fence_stride=STRIDE)
        return out, n_out, s["fences"]
    if kind == "rebuild":
        out, n_out = lsm.lsm_compact(s["runs"], lsm.LSM_BOTTOMMOST, s["out"], s["n_out"], s["workspace"], fences=s["fences"],
                                     fence_stride=STRIDE, key_hashes=s["hashes"])
        torch.cuda.current_stream().synchronize()  # the new run's length, in pinned memory
        n = int(n_out)
        run_, fences, hashes = out[:n], s["fences"][: _ceil(n, STRIDE)], s["hashes"][:n]
        blocks = lsm.lsm_bloom_blocks(n, BLOOM_BITS)
        bloom = lsm.lsm_build_bloom_hashed(hashes, blocks, s["bloom"][:blocks])
        index = lsm.lsm_build_hash_index(hashes)  # where a key's slot lies is free: checked through the lookups
        hit_len, hits = lsm.lsm_probe(*s["queries"], [lsm.TreeRun(run_, fences, STRIDE, 1, bloom, index)], *s["hits"])
        return out, n, s["fences"], s["hashes"], s["bloom"], hit_len, hits
    if kind == "batch":
        outs, n_out, fences = lsm.lsm_compact_batch(s["jobs"], fence_stride=STRIDE)
        counts = n_out.tolist()
        runs = [o[:n] for o, n in zip(outs, counts)]
        return runs, [f[: _ceil(n, STRIDE)] for f, n in zip(fences, counts)], lsm.lsm_build_bloom_batch(runs, BLOOM_BITS)
    if kind == "probe":
        return lsm.lsm_probe(*s["queries"], s["tree"], *s["hits"])
    if kind == "range":
        return lsm.lsm_range_scan(s["tree"], s["lo"], s["hi"], RANGE_SLOT, s["entries"], s["counts"])
    if kind == "driver":
        d, out = s["driver"], []
        for i, buffer in enumerate(s["buffers"]):
            d.note_writes(case["buffer"] // 16)
            d.flush(buffer) if case["sorted"] else d.flush_unsorted(buffer)
            if (i + 1) % case["probe_every"] == 0 or i + 1 == len(s["buffers"]):
                p = len(out)
                out.append(d.probe(*s["queries"][p], *s["hits"][p]))
        return out, np.array(d.levels())
    drivers = [d for d, _ in s["trees"]]
    for i in range(case["flushes"]):
        for d in drivers:
            d.note_writes(case["buffer"] // 16)
        lsm.lsm_driver_flush_many(drivers, [buffers[i] for _, buffers in s["trees"]])
    return [d.probe(*q, *h) for d, q, h in zip(drivers, s["queries"], s["hits"])], [len(d.levels()) for d in drivers]


# ---------------------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------------------------------
def _probe_bytes(requests):
    """Every request: its keys up to the first miss (about 38 are found), an entry for each, the whole row of hits."""
    return requests * (39 * 32 + 38 * 64 + 8 + MAX_BLOCKS * 16)


def _merge_bytes(n_in, survive, fences=False, hashes=False):
    n_out = n_in * survive
    return 64 * (n_in + n_out) + (n_out / STRIDE * 32 if fences else 0) + (8 * n_out if hashes else 0)


def work(case):
    kind = case["kind"]
    if kind == "flush":
        b = _merge_bytes(case["entries"], 0.95, True)
    elif kind == "compact":
        tiered = case["shape"] == "tiered"
        survive = (1 / 1.4 if tiered else 0.97) * (0.95 if case["last"] and tiered else 1)
        b = _merge_bytes(case["entries"], survive, case["fences"])
    elif kind == "rebuild":
        n = case["entries"] * 0.95 / 1.4
        b = _merge_bytes(case["entries"], 0.95 / 1.4, True, True) + 8 * n + 2 * n + 16 * n + _probe_bytes(case["requests"])
    elif kind == "batch":
        n = case["jobs"] * case["entries"] * 0.94
        b = _merge_bytes(n, 0.98, True) + 2 * n
    elif kind == "probe":
        b = _probe_bytes(case["requests"])
    elif kind == "range":
        b = case["ranges"] * (64 + 2 * 64 * 40 + 4)
    else:
        trees, flushes, m = case.get("trees", 1), case["flushes"], case["buffer"]
        levels = len(_level_sizes(case["entries"], m))
        # leveling with size ratio 10: a flushed entry is rewritten about T / 2 times in the first level and, while the
        # pass lasts, some three times in the second, each time read and written; the tree's lookups come on top
        b = trees * flushes * m * 64 * 2 * (5 + 3 * (levels > 1)) + _probe_bytes(case["requests"]) * (
            trees if kind == "shards" else _ceil(flushes, case["probe_every"]))
    return {"bytes": float(b), "flops": 0.0}
