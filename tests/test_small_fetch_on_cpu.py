"""fetch_kv_small, compiled for the CPU and run lane by lane (tests/emulate/small_fetch.cpp), while the directory changes under it.
Every workgroup reads the directory for itself, each at times of its own: whatever mixture of older and younger entries they meet, every
byte of the destination has to be there - of the blocks that are edited and of those that are not."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"
pytestmark = pytest.mark.skipif(shutil.which(CLANG) is None, reason="needs clang's vector extensions")
HOST, CACHE, LOCAL = 0, 1, 2
NEVER = 1 << 30
u32, u64, vp = ctypes.c_uint32, ctypes.c_uint64, ctypes.c_void_p


class Fetch(ctypes.Structure):
    _fields_ = [(n, u32) for n in ("n_planes", "nthr", "head_major", "n_layers", "n_objects", "n_seq", "max_blocks", "n_host", "lg_groups", "seen",
                                   "n_versions", "n_heads", "block_tokens", "n_slots", "unrolled", "pad")]
    _fields_ += [("chunk_bytes", u64), ("dst_cap", u64), ("dst_step", u64), ("pool", u64 * 2 * 3), ("dst", u64 * 2)]
    _fields_ += [(n, vp) for n in ("table", "n_blocks", "seq_dst", "seq_cap", "versions", "when", "cnt", "miss")]


@pytest.fixture(scope="module")
def emulated(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("emulate") / "libsmall_fetch.so")
    here = os.path.join(ROOT, "tests", "emulate")
    subprocess.check_call([CLANG, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", here, "-I", os.path.join(ROOT, "paper_2602_00328_amd", "csrc"),
                           "-o", so, os.path.join(here, "small_fetch.cpp")])
    return ctypes.CDLL(so)


def aligned(shape, dtype=np.uint8):
    n = int(np.prod(shape)) * np.dtype(dtype).itemsize
    raw = np.zeros(n + 64, dtype=np.uint8)
    at = -raw.ctypes.data % 64
    return raw[at:at + n].view(dtype).reshape(shape)


def entry(tier, slot, edit):
    return np.uint64(int(tier) | int(slot) << 2 | (int(edit) & 0xFFFFFFFF) << 32)


class Case:
    """Objects have one slot number in every tier, which all hold the same bytes; `tiers[v]` are their tiers in version v."""

    def __init__(self, lib, rng, lens, width, chunk, n_planes=2, nthr=256, head_major=False, n_layers=1, n_host=32, lg=0, heads=(2, 1)):
        self.lib, self.rng, self.n_layers, self.n_planes = lib, rng, n_layers, n_planes
        self.n_objects = n = len(lens) * width
        f = self.f = Fetch(n_planes=n_planes, nthr=nthr, head_major=head_major, n_layers=n_layers, n_objects=n, n_seq=len(lens), max_blocks=width,
                           n_host=n_host, lg_groups=lg, seen=7, n_heads=heads[0], block_tokens=heads[1], n_slots=n, chunk_bytes=chunk)
        self.cap = sum(lens)
        f.dst_cap, f.dst_step = self.cap, self.cap * chunk
        self.payload = aligned((n_planes, n_layers, n, chunk))
        self.payload[:] = rng.integers(0, 256, self.payload.shape, dtype=np.uint8)
        self.pools = [[aligned(self.payload.shape[1:]) for _ in range(n_planes)] for _ in range(3)]
        for t in range(3):
            for p in range(n_planes):
                self.pools[t][p][:] = self.payload[p]
                f.pool[t][p] = self.pools[t][p].ctypes.data
        self.table = np.arange(n, dtype=np.int32)
        rng.shuffle(self.table)
        self.n_blocks = np.array(lens, dtype=np.int32)
        self.first = np.cumsum([0] + list(lens[:-1])).astype(np.uint64)
        self.caps = np.array(lens, dtype=np.uint32)
        self.cells = np.concatenate([np.arange(k) + s * width for s, k in enumerate(lens)])
        f.table, f.n_blocks, f.seq_dst, f.seq_cap = (x.ctypes.data for x in (self.table, self.n_blocks, self.first, self.caps))
        self.heads = heads

    def run(self, tiers, when=None):
        f, n = self.f, self.n_objects
        versions = np.empty((len(tiers), n), dtype=np.uint64)
        for v, tier in enumerate(tiers):
            for i in range(n):
                versions[v, i] = entry(tier[i], i, 3) if v == 0 else (versions[v - 1, i] if tier[i] == tiers[v - 1][i] else entry(tier[i], i, 7 + v))
        tiles = -(-f.chunk_bytes // (f.nthr * 16)) * n * f.n_planes * f.n_layers
        n_wgs = f.n_host + 1 + int(tiles)
        if when is None:                      # every workgroup at its own time, most of them within the walk
            when = self.rng.choice([0, 1, 2, 3, 4, 5, 7, 9, NEVER], (n_wgs, len(tiers) - 1))
        when = np.ascontiguousarray(np.sort(np.broadcast_to(when, (n_wgs, len(tiers) - 1)), axis=1), dtype=np.uint32)
        dst = [aligned((self.n_layers, self.cap, f.chunk_bytes)) for _ in range(f.n_planes)]
        cnt, miss = np.zeros(16, dtype=np.uint32), np.zeros(n, dtype=np.uint32)
        f.n_versions, f.versions, f.when, f.cnt, f.miss = len(tiers), versions.ctypes.data, when.ctypes.data, cnt.ctypes.data, miss.ctypes.data
        for p in range(f.n_planes):
            f.dst[p] = dst[p].ctypes.data
        self.lib.run_fetch(ctypes.byref(f))
        for p in range(f.n_planes):
            want = self.payload[p][:, self.table[self.cells]]
            got = dst[p]
            if f.head_major:
                h, t = self.heads
                want = want[0].reshape(self.cap, t, h, -1)
                want = np.concatenate([want[a:a + k].reshape(k * t, h, -1).transpose(1, 0, 2).reshape(-1) for a, k in zip(self.first.astype(int), self.caps)])
                got = got.reshape(-1)
                assert np.array_equal(got, want), f"plane {p}: {np.count_nonzero(got != want)} bytes missing"
                continue
            wrong = (got != want).any(axis=2)
            assert not wrong.any(), f"plane {p}: {wrong.sum()} of {wrong.size} chunks are not whole"
        return cnt, miss


SHAPES = [         # threads, planes, layers, chunk, lengths, width, workgroups at the host, shares (log2)
    (256, 2, 1, 8192, [300, 280], 300, 32, 1),
    (256, 2, 1, 32768, [60, 70], 140, 32, 0),
    (256, 2, 1, 4096 + 16, [513], 513, 7, 0),
    (256, 1, 1, 4096, [512, 90], 512, 25, 2),
    (256, 1, 3, 16384, [140], 140, 32, 0),
    (256, 2, 2, 12288, [130, 1], 200, 25, 2),
    (64, 2, 1, 1024, [128], 128, 128, 0),
    (64, 1, 5, 2048 + 16, [17, 30], 40, 7, 0),
    (64, 2, 3, 3072, [20], 20, 1, 0),
]


@pytest.mark.parametrize("edit", ["revoked", "placed", "placed and revoked"])
@pytest.mark.parametrize("nthr,n_planes,n_layers,chunk,lens,width,n_host,lg", SHAPES)
def test_every_block_is_whole_when_entries_change_under_the_fetch(emulated, edit, nthr, n_planes, n_layers, chunk, lens, width, n_host, lg):
    rng = np.random.default_rng(n_host * 100 + lg * 10 + len(edit))
    c = Case(emulated, rng, lens, width, chunk, n_planes, nthr, n_layers=n_layers, n_host=n_host, lg=lg)
    tier = rng.choice([HOST, CACHE, LOCAL], c.n_objects, p=[0.4, 0.5, 0.1])
    for how_many in (1, 20):
        tiers = [tier]
        if edit == "revoked":
            tiers.append(tier.copy())
            tiers[1][rng.permutation(np.flatnonzero(tier == CACHE))[:how_many]] = HOST
        else:
            moved = rng.permutation(np.flatnonzero(tier == HOST))[:how_many]
            tiers.append(tier.copy())
            tiers[1][moved] = CACHE
            if edit != "placed":
                tiers.append(tiers[1].copy())
                tiers[2][moved[::2]] = HOST
        c.run(tiers)


@pytest.mark.parametrize("n_planes,nthr,heads,lens,width", [(2, 256, (8, 16), [300, 250], 300), (1, 256, (3, 5), [400], 400), (2, 64, (2, 4), [60, 61], 64)])
@pytest.mark.parametrize("edit", ["revoked", "placed"])
def test_every_head_major_block_is_whole_when_entries_change_under_the_fetch(emulated, edit, n_planes, nthr, heads, lens, width):
    rng = np.random.default_rng(3)
    c = Case(emulated, rng, lens, width, heads[0] * heads[1] * 48, n_planes, nthr, head_major=True, n_host=9, lg=1 if nthr == 256 else 0, heads=heads)
    tier = rng.choice([HOST, CACHE, LOCAL], c.n_objects, p=[0.4, 0.5, 0.1])
    after = tier.copy()
    after[rng.permutation(np.flatnonzero(tier == (CACHE if edit == "revoked" else HOST)))[:9]] = HOST if edit == "revoked" else CACHE
    c.run([tier, after])


def test_counters_and_misses_of_a_directory_that_holds_still(emulated):
    rng = np.random.default_rng(5)
    for nthr, lens, width, lg in ((256, [513, 300], 600, 1), (64, [40, 50], 64, 0)):
        c = Case(emulated, rng, lens, width, 1040, 2, nthr, n_layers=2, n_host=24, lg=lg)
        tier = rng.choice([HOST, CACHE, LOCAL], c.n_objects, p=[0.4, 0.5, 0.1])
        cnt, miss = c.run([tier])
        asked = tier[c.table[c.cells]]
        assert cnt[:6].tolist() == [len(asked), (asked == LOCAL).sum(), (asked == CACHE).sum(), (asked == HOST).sum(), 0, 0]
        assert miss[:(asked == HOST).sum()].tolist() == c.cells[asked == HOST].tolist()


@pytest.mark.parametrize("n_planes", [1, 2])
@pytest.mark.parametrize("nthr", [64, 256])
def test_head_major_cells_beyond_a_sequences_room_are_invalid(emulated, n_planes, nthr):
    """The last sequence's destination has room for two blocks less than it has."""
    rng = np.random.default_rng(6)
    c = Case(emulated, rng, [65, 62], 65, 16, n_planes, nthr, head_major=True, n_host=8, heads=(1, 1))
    c.n_blocks[1] = 64
    tier = rng.choice([HOST, CACHE, LOCAL], c.n_objects, p=[0.4, 0.5, 0.1])
    cnt, miss = c.run([tier])
    asked = tier[c.table[c.cells]]
    assert cnt[:6].tolist() == [129, (asked == LOCAL).sum(), (asked == CACHE).sum(), (asked == HOST).sum(), 0, 2]
    assert miss[:(asked == HOST).sum()].tolist() == c.cells[asked == HOST].tolist()


@pytest.mark.parametrize("edit", ["revoked", "placed"])
@pytest.mark.parametrize("n_planes,n_layers,chunk,lens,width,heads", [(2, 1, 16384, [140, 60], 150, None), (1, 1, 8192 + 16, [200], 200, None), (2, 3, 4096 + 16, [70, 71], 71, None),
                                                                      (2, 1, 16, [129], 129, None), (2, 1, 8 * 16 * 64, [90, 50], 90, (8, 16)), (1, 1, 5 * 3 * 592, [140], 140, (5, 3))])
def test_blocks_are_whole_with_two_loads_a_thread(emulated, edit, n_planes, n_layers, chunk, lens, width, heads):
    """Tiles of 8 KiB: chunks of some of them, of one and a bit, of less than half of one."""
    rng = np.random.default_rng(chunk)
    c = Case(emulated, rng, lens, width, chunk, n_planes, 256, head_major=heads is not None, n_layers=n_layers, n_host=9, heads=heads or (2, 1))
    c.f.unrolled = 1
    tier = rng.choice([HOST, CACHE, LOCAL], c.n_objects, p=[0.2, 0.7, 0.1])
    after = tier.copy()
    after[rng.permutation(np.flatnonzero(tier == (CACHE if edit == "revoked" else HOST)))[:9]] = HOST if edit == "revoked" else CACHE
    c.run([tier, after])


class Experts(ctypes.Structure):
    _fields_ = [(n, u32) for n in ("n_experts", "n_known", "n_ids", "n_staging", "n_host", "hbm_wgs", "seen", "n_versions", "n_slots", "pad")]
    _fields_ += [("chunk_bytes", u64), ("pool", u64 * 2), ("staging", u64)] + [(n, vp) for n in ("topk", "versions", "when", "expert_ptr", "cnt", "miss")]


@pytest.mark.parametrize("edit", [None, "revoked", "placed", "placed and revoked"])
@pytest.mark.parametrize("n_experts,n_known,n_ids,n_staging,n_host,short,chunk", [(60, 60, 16, 60, 5, 1, 24576 + 16), (64, 64, 50, 64, 3, 0.4, 8192), (128, 128, 64, 128, 7, 0.7, 4096),
                                                                                  (65, 50, 30, 65, 1, 1, 16), (100, 100, 40, 9, 24, 1, 8192 + 4112), (1, 1, 1, 1, 2, 1, 40960), (33, 33, 5, 33, 0, 1, 8208), (16, 16, 256, 16, 3, 1, 8192),
                                                                                  (128, 128, 129, 128, 5, 1, 2048)])
def test_routed_experts_are_whole_when_entries_change_under_the_fetch(emulated, edit, n_experts, n_known, n_ids, n_staging, n_host, short, chunk):
    """A grid of a tile each and shorter ones, ids that are out of range, experts that nobody has registered, less staging than experts; entries
    change between two experts of a reader's walk and between two tiles of a workgroup too."""
    rng = np.random.default_rng(n_experts + n_ids)
    ids = rng.integers(0, n_experts, n_ids).astype(np.int32)
    if n_ids > 4:
        ids[1], ids[3] = -1, n_experts
    weights = aligned((n_experts, chunk))
    weights[:] = rng.integers(0, 256, weights.shape, dtype=np.uint8)
    pools = [aligned(weights.shape) for _ in range(2)]
    for x in pools:
        x[:] = weights
    inside = sorted({int(i) for i in ids if 0 <= i < n_experts})
    routed = [i for i in inside if i < n_known]
    staged = routed[:n_staging]
    tier = rng.choice([HOST, CACHE], n_experts, p=[0.3, 0.7]) if n_host else np.full(n_experts, CACHE)
    tiers = [tier]
    if edit and n_host:
        moved = rng.permutation(np.flatnonzero(tier == (CACHE if edit == "revoked" else HOST)))[:7]
        tiers.append(tier.copy())
        tiers[1][moved] = HOST if edit == "revoked" else CACHE
        if edit == "placed and revoked":
            tiers.append(tiers[1].copy())
            tiers[2][moved[::2]] = HOST
    versions = np.empty((len(tiers), n_experts), dtype=np.uint64)
    for v, t in enumerate(tiers):
        for i in range(n_experts):
            versions[v, i] = entry(t[i], i, 3) if v == 0 else (versions[v - 1, i] if t[i] == tiers[v - 1][i] else entry(t[i], i, 7 + v))
    versions[:, n_known:] = np.uint64(0xFFFFFFFFFFFFFFFF)
    tiles = -(-chunk // 8192)
    wgs = max(1, int(short * len(staged) * tiles))
    # before a workgroup's first look, never, or at one of its meetings: four wavefronts have 32 for every 32 experts, then each one an expert
    walk = 4 * 32 * (2 if n_experts <= 64 else 4) + np.arange(-4, 4 * len(staged) + 8)
    times = np.concatenate([np.repeat([0, NEVER], len(walk) // 2), np.repeat([1, 2, 3, 5, 8], len(walk) // 8 + 1), walk])
    when = np.sort(rng.choice(times, (n_host + 1 + wgs, len(tiers) - 1)), axis=1).astype(np.uint32)
    staging, ptr = aligned((n_staging, chunk)), np.full(n_experts, 7, dtype=np.uint64)
    staging[:] = 0xEE
    cnt, miss = np.zeros(16, dtype=np.uint32), np.zeros(n_experts, dtype=np.uint32)
    f = Experts(n_experts=n_experts, n_known=n_known, n_ids=n_ids, n_staging=n_staging, n_host=n_host, hbm_wgs=wgs, seen=7, n_versions=len(tiers),
                n_slots=n_experts, chunk_bytes=chunk, staging=staging.ctypes.data, topk=ids.ctypes.data, versions=versions.ctypes.data,
                when=when.ctypes.data, expert_ptr=ptr.ctypes.data, cnt=cnt.ctypes.data, miss=miss.ctypes.data)
    f.pool[0], f.pool[1] = pools[0].ctypes.data, pools[1].ctypes.data
    hbm = emulated.run_experts(ctypes.byref(f))
    assert np.array_equal(staging[:len(staged)], weights[staged]) and (staging[len(staged):] == 0xEE).all()
    want = np.zeros(n_experts, dtype=np.uint64)
    want[staged] = staging.ctypes.data + np.arange(len(staged), dtype=np.uint64) * chunk
    assert np.array_equal(ptr, want)
    assert cnt[0] == len(inside) and cnt[2] + cnt[3] == len(staged) and hbm == cnt[2]
    assert cnt[5] == len(inside) - len(staged) + (2 if n_ids > 4 else 0)
    if len(tiers) == 1:
        assert cnt[3] == sum(tier[i] == HOST for i in staged) and sorted(miss[:cnt[3]]) == [i for i in staged if tier[i] == HOST]


@pytest.mark.parametrize("n_seg,seg_cells,fill", [(1, 0, 7), (1, 256, 256), (2, 256, 3), (5, 256, 0.3), (64, 256, 0.02), (255, 1024, 0.01), (256, 1024, 0.1), (256, 256, "last")])
@pytest.mark.parametrize("step", [1, 3, 24, 96, 300, "back", "any"])
def test_the_hosts_list_over_its_segments(emulated, n_seg, seg_cells, fill, step):
    """Entries in the order in which a workgroup asks for them, and in others: segments of none, of one, of all their cells."""
    rng = np.random.default_rng(n_seg)
    if isinstance(fill, int):
        counts = np.full(n_seg, fill)
    elif fill == "last":
        counts = np.where(np.arange(n_seg) == n_seg - 1, 200, 0)
    else:
        counts = rng.binomial(seg_cells, fill, n_seg) * (rng.random(n_seg) < 0.8)
        counts[rng.integers(n_seg)] = seg_cells
    recs = rng.integers(0, 1 << 60, (n_seg, max(seg_cells, 7), 2), dtype=np.uint64)
    want = np.concatenate([recs[s, :k] for s, k in enumerate(counts)])
    total = len(want)
    order = np.arange(total)[::-1] if step == "back" else rng.integers(0, total, 100) if step == "any" else np.arange(step % 7, total, step)
    order = order[:300] if step != 1 else order[-300:]
    padded = np.zeros(256, dtype=np.uint32)
    padded[:n_seg] = counts
    idx, out = np.ascontiguousarray(order, dtype=np.uint32), np.zeros((len(order), 2), dtype=np.uint64)
    got = emulated.host_list(padded.ctypes.data_as(vp), u32(n_seg), u32(seg_cells), recs.ctypes.data_as(vp), idx.ctypes.data_as(vp), u32(len(idx)), out.ctypes.data_as(vp))
    assert got == total and np.array_equal(out, want[order])
