"""The kernels of the fetch at the edges of their tiles, pages and grids, against numpy indexing of the payload.

A fetch moves bytes, so the comparison is exact.  Sizes are in 16-byte units around what one workgroup takes at a time:
1 KiB tiles, 4 KiB host pages (64 threads x 4 loads), read two loads at a time.
"""
import numpy as np
import pytest
import torch

from paper_2602_00328_amd import binding as B

pytestmark = pytest.mark.gpu


class Rig:
    """A KV class of n objects with tiers mixed by object number, and its payload [plane][layer][object][chunk] in numpy."""

    def __init__(self, chunk, n, n_layers=1, n_planes=2, host_every=3, local_every=7, seed=0, **kw):
        rng = np.random.default_rng(seed)
        self.chunk, self.n, self.n_layers, self.n_planes = chunk, n, n_layers, n_planes
        self.payload = rng.integers(0, 256, (n_planes, n_layers, n, chunk), dtype=np.uint8)
        local = np.array([i for i in range(n) if local_every and i % local_every == 3], dtype=np.int64)
        rest = np.setdiff1d(np.arange(n), local)
        self.order = np.concatenate([rest, local])                # object number -> payload row
        host_slots = rng.permutation(n).astype(np.int64)
        self.h = B.Harvest(kv=B.ClassSpec(n_layers=n_layers, n_planes=n_planes, chunk_bytes=chunk, max_objects=n, n_host_slots=n,
                                          n_cache_slots=max(1, len(rest)), n_local_slots=len(local)), **kw)
        for p in range(n_planes):
            self.h.host_plane(B.KV, p)[:, host_slots] = self.payload[p][:, self.order]
        self.h.register(B.KV, len(rest), host_slots[:len(rest)])
        if len(local):
            self.h.register(B.KV, len(local), host_slots[len(rest):], tier=B.LOCAL)
            for p in range(n_planes):
                self.h.dev_plane(B.KV, B.LOCAL, p).copy_(torch.from_numpy(self.payload[p][:, local]))
        self.on_host = np.array([bool(host_every) and i % host_every == 1 for i in range(len(rest))])
        cached = rng.permutation(np.flatnonzero(~self.on_host))
        if len(cached):
            self.h.place(B.KV, cached)
        torch.cuda.synchronize()

    def tables(self, lens, width, seed=1):
        rng = np.random.default_rng(seed)
        t = np.full((len(lens), width), -1, dtype=np.int32)
        for s, k in enumerate(lens):
            t[s, :k] = rng.integers(0, self.n, k)
        first = np.cumsum([0] + list(lens[:-1])).astype(np.int64)
        dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
        return t, dev(t), dev(np.array(lens, dtype=np.int32)), dev(first), int(sum(lens))

    def expected(self, t, lens, plane, layer):
        ids = np.concatenate([t[s, :k] for s, k in enumerate(lens)])
        return self.payload[plane][layer][self.order[ids]].reshape(-1)

    def misses(self, t, lens):
        return [s * t.shape[1] + j for s, k in enumerate(lens) for j in range(k)
                if t[s, j] < len(self.on_host) and self.on_host[t[s, j]]]

    def buffers(self, cap):
        return [torch.full((self.n_layers * cap * self.chunk + 64,), 0xEE, dtype=torch.uint8, device="cuda") for _ in range(2)]


@pytest.mark.parametrize("n_planes,layout", [(1, 0), (2, 0), (2, B.FLAG_CACHE_PLANES_ADJACENT)])
@pytest.mark.parametrize("chunk", [16, 1008, 1024, 2064, 4080, 4096, 4112, 8208, 16384 + 48])
@pytest.mark.parametrize("threads,host_wgs", [(64, 0), (64, 1), (128, 3), (256, 0)])
def test_both_tiers_in_one_launch(n_planes, layout, chunk, threads, host_wgs):
    """Plane after plane, and both planes of a request in one pass where the cache tier keeps them side by side."""
    rig = Rig(chunk, 41, n_layers=3, n_planes=n_planes, flags=B.FLAG_GENERAL_FETCH | layout, gather_threads=threads, host_wgs=host_wgs)
    lens = [13, 1, 0, 22]
    t, dt, dn, df, cap = rig.tables(lens, 23)
    for _ in range(2):                                # the second call's grid is sized by the first one's report
        k, v = rig.buffers(cap)
        rig.h.fetch_kv_layers(0, 3, dt, dn, k, v if n_planes == 2 else None, cap * chunk, df, cap)
        counts, miss, n_miss = rig.h.fetch_info(miss_cap=t.size)
        assert miss.tolist() == rig.misses(t, lens) and counts["n_host"] == n_miss
        for p, buf in enumerate([k, v][:n_planes]):
            got = buf.cpu().numpy()
            for layer in range(3):
                assert np.array_equal(got[layer * cap * chunk:(layer + 1) * cap * chunk], rig.expected(t, lens, p, layer)), (p, layer)
            assert (got[3 * cap * chunk:] == 0xEE).all()
    rig.h.close()


@pytest.mark.parametrize("n_planes,layout", [(1, 0), (2, 0), (2, B.FLAG_CACHE_PLANES_ADJACENT)])
@pytest.mark.parametrize("chunk", [16, 1008, 2064, 4096, 4112, 16384 + 48])
@pytest.mark.parametrize("threads", [64, 256])
def test_a_few_blocks_from_the_host(n_planes, layout, chunk, threads):
    """The second fetch knows from the first that HBM is what it waits for and reads the host with fewer wavefronts."""
    rig = Rig(chunk, 300, n_layers=2, n_planes=n_planes, host_every=100, flags=B.FLAG_GENERAL_FETCH | layout, gather_threads=threads)
    lens = [200, 0, 113]
    t, dt, dn, df, cap = rig.tables(lens, 201)
    t[np.isin(t, np.flatnonzero(rig.on_host))] = 0       # a block of the cache tier
    t[0, :3] = np.flatnonzero(rig.on_host)[:3]
    dt.copy_(torch.from_numpy(t))
    for _ in range(3):
        k, v = rig.buffers(cap)
        rig.h.fetch_kv_layers(0, 2, dt, dn, k, v if n_planes == 2 else None, cap * chunk, df, cap)
        counts, miss, _ = rig.h.fetch_info(miss_cap=t.size)
        assert miss.tolist() == rig.misses(t, lens) and 0 < counts["n_host"] * 55 <= counts["n_cache"] + counts["n_local"]
        for p, buf in enumerate([k, v][:n_planes]):
            got = buf.cpu().numpy()
            for layer in range(2):
                assert np.array_equal(got[layer * cap * chunk:(layer + 1) * cap * chunk], rig.expected(t, lens, p, layer)), (p, layer)
            assert (got[2 * cap * chunk:] == 0xEE).all()
    rig.h.close()


@pytest.mark.parametrize("flags", [0, B.FLAG_GENERAL_FETCH])
@pytest.mark.parametrize("host_wgs", [0, 1, 5])
@pytest.mark.parametrize("n_planes,chunk,n_host", [(1, 1040, 1), (2, 1040, 3), (1, 4112, 2), (2, 32768, 1), (2, 16384, 5)])
def test_layers_with_fewer_host_pages_than_workgroups(n_planes, chunk, n_host, host_wgs, flags):
    """The host's pages of all layers are dealt out as one sequence; the small tables walk their cells in 64 and in 256 threads."""
    for width in (40, 150):
        rig = Rig(chunk, 40, n_layers=7, n_planes=n_planes, host_every=4, flags=flags, host_wgs=host_wgs)
        lens = [width, 3]
        t, dt, dn, df, cap = rig.tables(lens, width)
        t[np.isin(t, np.flatnonzero(rig.on_host))] = 0       # a block of the cache tier
        t[0, 7:7 + n_host] = np.flatnonzero(rig.on_host)[:n_host]
        dt.copy_(torch.from_numpy(t))
        for _ in range(2):
            k, v = rig.buffers(cap)
            rig.h.fetch_kv_layers(0, 7, dt, dn, k, v if n_planes == 2 else None, cap * chunk, df, cap)
            assert rig.h.fetch_info(miss_cap=t.size)[0]["n_host"] == n_host
            for p, buf in enumerate([k, v][:n_planes]):
                got = buf.cpu().numpy()
                for layer in range(7):
                    assert np.array_equal(got[layer * cap * chunk:(layer + 1) * cap * chunk], rig.expected(t, lens, p, layer)), (p, layer)
        rig.h.close()


@pytest.mark.parametrize("host_every,local_every", [(0, 0), (1, 0), (2, 5)])
def test_again_counts_its_requests(host_every, local_every):
    """All in the cache tier, all but one request in three on the host, and a mix: a repeated fetch adds to the totals."""
    rig = Rig(2048, 30, n_layers=2, host_every=host_every, local_every=local_every, flags=B.FLAG_GENERAL_FETCH)
    lens = [9, 17]
    t, dt, dn, df, cap = rig.tables(lens, 20)
    k, v = rig.buffers(cap)
    rig.h.fetch_kv(0, dt, dn, k, v, df, cap)
    once = rig.h.stats().fetch[B.KV].as_dict()
    rig.h.fetch_kv_again(1, k, v)
    for p, buf in enumerate([k, v]):
        assert np.array_equal(buf.cpu().numpy()[:cap * 2048], rig.expected(t, lens, p, 1))
    assert rig.h.stats().fetch[B.KV].as_dict() == {name: 2 * x for name, x in once.items()}
    assert once["n_requests"] == 26 and once["n_host"] == len(rig.misses(t, lens))
    rig.h.close()


@pytest.mark.parametrize("n_planes", [1, 2])
@pytest.mark.parametrize("lens,width", [([1], 1), ([64], 64), ([65], 65), ([60, 62], 64), ([64, 0], 64), ([50, 79], 129), ([255], 255), ([256, 0], 256), ([200, 55, 257], 257), ([3, 510], 513), ([0, 0], 600),
                                        ([1, 2, 0, 5], 1024)])
def test_one_kernel_fetch_at_the_edges_of_its_rounds(n_planes, lens, width):
    """Tables of one cell up to several rounds of 512, twice: the second call of a mostly empty table takes the general path."""
    rig = Rig(4112, 37, n_layers=2, n_planes=n_planes)
    t, dt, dn, df, cap = rig.tables(lens, width)
    if lens[0] > 100:
        t[0, 5], t[0, 70] = -4, rig.n                 # blocks that do not exist: invalid requests
        dt.copy_(torch.from_numpy(t))
    ids = np.concatenate([t[s, :k] for s, k in enumerate(lens)])
    bad = (ids < 0) | (ids >= rig.n)
    for _ in range(2):
        k, v = rig.buffers(max(cap, 1))
        rig.h.fetch_kv_layers(0, 2, dt, dn, k, v if n_planes == 2 else None, max(cap, 1) * 4112, df, max(cap, 1))
        counts, miss, _ = rig.h.fetch_info(miss_cap=t.size)
        assert miss.tolist() == rig.misses(np.where(t >= 0, t, rig.n), lens)
        assert counts["n_requests"] == cap and counts["n_invalid"] == bad.sum()
        for p, buf in enumerate([k, v][:n_planes]):
            for layer in range(2):
                got = buf.cpu().numpy()[layer * max(cap, 1) * 4112:][:cap * 4112].reshape(cap, 4112)
                want = rig.payload[p][layer][rig.order[np.where(bad, 0, ids)]]
                want[bad] = 0xEE
                assert np.array_equal(got, want), (p, layer)
    rig.h.close()


@pytest.mark.parametrize("where", ["every cell", "every other cell", "every other row", "one"])
@pytest.mark.parametrize("host_wgs", [0, 11, 49, 100])        # two, one, four and eight shares of a table that has the rounds
@pytest.mark.parametrize("lens,width", [([512], 512), ([513], 513), ([512, 500], 512), ([1, 1024], 1025), ([300] * 7, 300), ([4096], 4096)])
def test_one_kernel_fetch_shares_out_the_walk_for_the_hosts_cells(lens, width, host_wgs, where):
    """Every cell is in one share, whatever the number of shares and wherever the host's cells are."""
    rig = Rig(1040, 64, n_layers=2, host_every=2, local_every=0, host_wgs=host_wgs)
    t, dt, dn, df, cap = rig.tables(lens, width)
    on_host, cached = np.flatnonzero(rig.on_host), np.flatnonzero(~rig.on_host)
    cell = np.arange(t.size).reshape(t.shape)
    hit = {"every cell": cell >= 0, "every other cell": cell % 2 == 1, "every other row": cell // width % 2 == 0, "one": cell == lens[0] - 1}[where]
    t[t >= 0] = np.where(hit, on_host[cell % len(on_host)], cached[cell % len(cached)])[t >= 0]
    dt.copy_(torch.from_numpy(t))
    k, v = rig.buffers(cap)
    rig.h.fetch_kv_layers(0, 2, dt, dn, k, v, cap * 1040, df, cap)
    counts, miss, _ = rig.h.fetch_info(miss_cap=t.size)
    assert miss.tolist() == rig.misses(t, lens) and counts["n_host"] == len(miss) > 0
    for p, buf in enumerate([k, v]):
        got = buf.cpu().numpy()
        for layer in range(2):
            assert np.array_equal(got[layer * cap * 1040:(layer + 1) * cap * 1040], rig.expected(t, lens, p, layer)), (p, layer)
        assert (got[2 * cap * 1040:] == 0xEE).all()
    rig.h.close()


@pytest.mark.parametrize("n_planes", [1, 2])
@pytest.mark.parametrize("heads,tokens,head_bytes", [(1, 1, 16), (3, 5, 48), (8, 16, 256), (2, 16, 512)])     # blocks of 16 B, 720 B, 32 KiB, 16 KiB
@pytest.mark.parametrize("lens,width", [([1], 1), ([128, 0], 64), ([65, 64], 65), ([256, 200, 1], 256), ([513], 513), ([30, 0, 7, 700], 701)])
def test_one_kernel_head_major_fetch_at_the_edges_of_its_rounds(n_planes, heads, tokens, head_bytes, lens, width):
    """Against the general path and numpy: blocks of all three tiers, blocks that do not exist, and a sequence whose destination
    has less room than its length."""
    chunk, outs = heads * tokens * head_bytes, []
    lens = [min(k, width) for k in lens]
    caps = np.array([k + i for i, k in enumerate(lens)], dtype=np.int32)
    caps[-1] = max(lens[-1] - 2, 1)
    first = np.cumsum([0] + caps[:-1].tolist())
    room = int(caps.sum())
    for flags in (0, B.FLAG_GENERAL_FETCH):
        rig = Rig(chunk, 37, n_planes=n_planes, flags=flags)
        t, dt, dn, _, _ = rig.tables(lens, width)
        if lens[0] > 100:
            t[0, 5], t[0, 70] = -4, rig.n
            dt.copy_(torch.from_numpy(t))
        k, v = rig.buffers(room)
        df, dc = torch.from_numpy(first.astype(np.int64)).cuda(), torch.from_numpy(caps).cuda()
        rig.h.fetch_kv_head_major(0, dt, dn, k, v if n_planes == 2 else None, df, dc, room, heads, tokens)
        counts, miss, _ = rig.h.fetch_info(miss_cap=t.size)
        outs.append((k.cpu().numpy(), v.cpu().numpy(), counts, miss.tolist()))
        if not flags:
            for p, buf in enumerate(outs[0][:n_planes]):
                for s, n in enumerate(lens):
                    got = buf[first[s] * chunk:(first[s] + caps[s]) * chunk].reshape(heads, caps[s] * tokens, head_bytes)
                    for j in range(min(n, caps[s])):
                        if 0 <= t[s, j] < rig.n:
                            want = rig.payload[p][0][rig.order[t[s, j]]].reshape(tokens, heads, head_bytes).transpose(1, 0, 2)
                            assert np.array_equal(got[:, j * tokens:(j + 1) * tokens], want), (p, s, j)
        rig.h.close()
    assert all(np.array_equal(a, b) for a, b in zip(*(o[:2] for o in outs))) and outs[0][2:] == outs[1][2:]


@pytest.mark.parametrize("recorded", [False, True])
@pytest.mark.parametrize("edit,head_major", [("revoke", False), ("place", False), ("revoke", True)])
def test_a_one_kernel_fetch_is_whole_when_the_directory_changes_under_it(edit, head_major, recorded):
    """Its workgroups read the directory for themselves, and an edit that does not wait for the fetch - a revocation publishes
    first and drains then, a placement runs on another stream - must not make a block fall between those that copy from HBM and
    those that copy from the host: each would leave it to the other."""
    n, chunk = (4096, 32768) if edit == "revoke" else (1024, 32768)
    rng = np.random.default_rng(3)
    payload = [rng.integers(0, 2 ** 31, (n, chunk // 4), dtype=np.int32) for _ in range(2)]
    h = B.Harvest(kv=B.ClassSpec(n_layers=1, n_planes=2, chunk_bytes=chunk, max_objects=n, n_host_slots=n, n_cache_slots=n, n_local_slots=0))
    for p in range(2):
        h.host_plane(B.KV, p).view(np.int32).reshape(n, -1)[:] = payload[p]
    ids = h.register(B.KV, n, np.arange(n))
    for i in ids:
        h.register_cb(B.KV, int(i), enabled=False)
    table = torch.arange(n, dtype=torch.int32, device="cuda").reshape(1, n)
    n_blocks, first = torch.tensor([n], dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int64, device="cuda")
    k, v = (torch.zeros(n * chunk, dtype=torch.uint8, device="cuda") for _ in range(2))
    want = source = [torch.from_numpy(x).cuda().reshape(-1) for x in payload]
    if head_major:
        want = [x.view(n * 16, 8, -1).transpose(0, 1).reshape(-1) for x in source]
    side, main = torch.cuda.Stream(), torch.cuda.Stream()

    def fetch():
        if head_major:
            h.fetch_kv_head_major(0, table, n_blocks, k, v, first, n_blocks, n, 8, 16)
        else:
            h.fetch_kv(0, table, n_blocks, k, v, first, n)

    with torch.cuda.stream(main):
        fetch()                                                   # makes the stream's scratch
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        if recorded:
            with torch.cuda.graph(graph, stream=main):
                fetch()
    batches = np.array_split(ids, 12)
    for _ in range(3):
        h.revoke(B.KV, ids)
        if edit == "revoke":
            h.place(B.KV, ids, stream=side)
        torch.cuda.synchronize()
        k.zero_(), v.zero_()
        torch.cuda.synchronize()
        def place(b):                                             # from device memory: not behind the fetch on the link
            h.place_from(B.KV, b, source[0].data_ptr(), source[1].data_ptr(), b.astype(np.uint64), n, stream=side)

        if edit == "place":                                       # one that is under way when the fetch is enqueued
            place(batches[0])
        with torch.cuda.stream(main):
            graph.replay() if recorded else fetch()
        if edit == "revoke":
            h.revoke(B.KV, ids)
        else:
            for b in batches[1:]:
                place(b)
        torch.cuda.synchronize()
        for got, x in zip((k, v), want):
            assert torch.equal(got.view(torch.int32), x), int((got.view(torch.int32) != x).reshape(n, -1).any(1).sum())
    h.close()


@pytest.mark.parametrize("head_major", [False, True])
@pytest.mark.parametrize("n_planes", [1, 2])
@pytest.mark.parametrize("lens,width", [([60, 40], 60), ([300, 250], 300), ([40, 700], 700)])
def test_cells_without_room_are_counted_and_write_nothing(lens, width, n_planes, head_major):
    """The last sequence's region ends seven blocks early: blocks of every tier that do not fit, in a destination that goes on behind."""
    chunk, room = 2048, sum(lens) - 7
    rig = Rig(chunk, 50, n_planes=n_planes, host_every=2)
    t, dt, dn, df, cap = rig.tables(lens, width)
    k, v = rig.buffers(cap)
    if head_major:
        caps = torch.tensor([lens[0], lens[1] - 7], dtype=torch.int32, device="cuda")
        rig.h.fetch_kv_head_major(0, dt, dn, k, v if n_planes == 2 else None, df, caps, room, 4, 4)
    else:
        rig.h.fetch_kv(0, dt, dn, k, v if n_planes == 2 else None, df, room)
    counts, miss, _ = rig.h.fetch_info(miss_cap=t.size)
    fit = [lens[0], lens[1] - 7]
    assert miss.tolist() == rig.misses(t, fit) and counts["n_invalid"] == 7 and counts["n_requests"] == cap
    for p, buf in enumerate([k, v][:n_planes]):
        got, at = buf.cpu().numpy(), 0
        assert (got[room * chunk:] == 0xEE).all()
        for s, n in enumerate(fit):
            want = rig.payload[p][0][rig.order[t[s, :n]]]
            if head_major:
                want = want.reshape(n * 4, 4, -1).transpose(1, 0, 2)
            assert np.array_equal(got[at:at + n * chunk], want.reshape(-1)), (p, s)
            at += n * chunk
    rig.h.close()


@pytest.mark.parametrize("n_planes,n_layers,n,layout,entry", [(2, 1, 4090, 0, "fetch"), (1, 1, 4090, 0, "fetch"), (2, 3, 1301, 0, "layers"), (2, 40, 100, 0, "layers"),
                                                              (2, 1, 3001, B.FLAG_CACHE_PLANES_ADJACENT, "fetch"), (2, 1, 3001, 0, "static"), (2, 1, 3001, 0, "head_major")])
def test_blocks_that_nobody_edits_are_whole_when_others_change_under_a_one_kernel_fetch(n_planes, n_layers, n, layout, entry):
    """Half of the blocks are on the host; a few of those are placed by another stream while the fetch runs, and a few of the cached
    ones are revoked.  Workgroups that list the host's blocks before and after such an edit have different lists."""
    rig = Rig(32768, n, n_layers=n_layers, n_planes=n_planes, host_every=2, local_every=0, flags=layout)
    for i in range(n):
        rig.h.register_cb(B.KV, i, enabled=False)
    t, dt, dn, df, cap = rig.tables([n], n)
    t[0] = np.random.default_rng(7).permutation(n)
    dt.copy_(torch.from_numpy(t))
    k, v = rig.buffers(cap)
    bufs, side, span = [k, v][:n_planes], torch.cuda.Stream(), n * 32768
    info, miss = (torch.zeros(m, dtype=torch.int32, device="cuda") for m in (8, n))

    def fetch():
        if entry == "layers":
            rig.h.fetch_kv_layers(0, n_layers, dt, dn, k, v, span, df, cap)
        elif entry == "static":
            rig.h.fetch_kv_static(0, dt, dn, k, v, df, cap, info, miss)
        elif entry == "head_major":
            rig.h.fetch_kv_head_major(0, dt, dn, k, v, df, dn, cap, 8, 16)
        else:
            rig.h.fetch_kv(0, dt, dn, k, v if n_planes == 2 else None, df, cap)

    want = [[torch.from_numpy(rig.expected(t, [n], p, layer)).cuda() for layer in range(n_layers)] for p in range(n_planes)]
    if entry == "head_major":
        want = [[x.view(n * 16, 8, -1).transpose(0, 1).reshape(-1) for x in w] for w in want]
    hosts, cached = np.flatnonzero(rig.on_host), np.flatnonzero(~rig.on_host)
    fetch()
    some = max(1, n // 300)
    rig.h.revoke(B.KV, cached[:some])                             # there is room for the placements
    for turn in range(1, 5):
        torch.cuda.synchronize()
        [b.zero_() for b in bufs]
        torch.cuda.synchronize()
        fetch()
        placed, revoked = hosts[turn * some:(turn + 1) * some], cached[turn * some:(turn + 1) * some]
        rig.h.place(B.KV, placed, stream=side)
        rig.h.revoke(B.KV, revoked)
        torch.cuda.synchronize()
        for p, b in enumerate(bufs):
            for layer in range(n_layers):
                got = b[layer * span:(layer + 1) * span]
                assert torch.equal(got, want[p][layer]), (turn, p, layer, int((got != want[p][layer]).reshape(n, -1).any(1).sum()))
    rig.h.close()


@pytest.mark.parametrize("lens,width", [([1], 1), ([65], 65), ([63, 64], 64), ([129], 129), ([300, 513], 600), ([5, 9], 4096), ([2, 1, 0], 4)])
def test_static_fetch_hands_out_counters_and_misses_in_order(lens, width):
    rig = Rig(2048, 50)
    t, dt, dn, df, cap = rig.tables(lens, width)
    for _ in range(2):
        k, v = rig.buffers(cap)
        info = torch.full((8,), 77, dtype=torch.int32, device="cuda")
        miss = torch.full((t.size,), -7, dtype=torch.int32, device="cuda")
        rig.h.fetch_kv_static(0, dt, dn, k, v, df, cap, info, miss)
        want = rig.misses(t, lens)
        ids = np.concatenate([t[s, :n] for s, n in enumerate(lens)])
        n_local = int((ids >= len(rig.on_host)).sum())
        assert info.tolist() == [cap, n_local, cap - n_local - len(want), len(want), 0, 0, len(want), 0]
        assert miss.tolist() == want + [-7] * (t.size - len(want))
        for p, buf in enumerate([k, v]):
            assert np.array_equal(buf.cpu().numpy()[:cap * 2048], rig.expected(t, lens, p, 0))
    empty = torch.zeros((0, 4), dtype=torch.int32, device="cuda")
    rig.h.fetch_kv_static(0, empty, dn, k, v, df, cap, info, miss)
    assert info.tolist() == [0] * 8
    rig.h.close()


@pytest.mark.parametrize("n_planes,cache", [(1, "slots"), (2, "slots"), (2, "adjacent"), (1, "segments"), (2, "segments")])
@pytest.mark.parametrize("chunk", [16, 1040, 16384, 32768 + 48])
@pytest.mark.parametrize("n", [1, 80, 81, 128, 129])
def test_moves_with_and_without_a_list_on_the_device(n_planes, cache, chunk, n):
    """place, place_from and evict of as many objects as travel with a launch, and one more; tiles of 1, 16 and 32 KiB; cache slots per
    plane, slots with the planes side by side, segments of a shared pool."""
    layers, rng, granule = 2, np.random.default_rng(n), 256
    segment = -(-layers * n_planes * chunk // granule) * granule
    h = B.Harvest(kv=B.ClassSpec(n_layers=layers, n_planes=n_planes, chunk_bytes=chunk, max_objects=n + 3, n_host_slots=n + 3,
                                 n_cache_slots=0 if cache == "segments" else n, n_local_slots=3),
                  flags=B.FLAG_CACHE_PLANES_ADJACENT if cache == "adjacent" else 0,
                  **(dict(shared_cache_bytes=n * segment, shared_granule=granule) if cache == "segments" else {}))
    dev = lambda a: torch.from_numpy(a).cuda()
    host_slots = rng.permutation(n + 3).astype(np.int64)
    h.register(B.KV, n, host_slots[:n])
    local = h.register(B.KV, 3, host_slots[n:], tier=B.LOCAL)
    bytes_of = lambda: rng.integers(0, 256, (n_planes, layers, n + 5, chunk), dtype=np.uint8)
    host = lambda: np.stack([h.host_plane(B.KV, p) for p in range(n_planes)])

    def pool(tier):
        if tier == B.CACHE and cache == "segments":        # taken from the low end on, each [layer][plane][chunk]
            segments = h.shared_cache.cpu().numpy().reshape(n, segment)[:, :layers * n_planes * chunk]
            return segments.reshape(n, layers, n_planes, chunk).transpose(2, 1, 0, 3).copy()
        return np.stack([h.dev_plane(B.KV, tier, p).cpu().numpy() for p in range(n_planes)])

    for p in range(n_planes):
        h.host_plane(B.KV, p)[:] = rng.integers(0, 256, (layers, n + 3, chunk), dtype=np.uint8)
    ids, block = rng.permutation(n), rng.permutation(n + 5)[:n]
    assert (h.place(B.KV, ids) == B.OK).all()                             # slots are handed out lowest first
    torch.cuda.synchronize()
    assert np.array_equal(pool(B.CACHE), host()[:, :, host_slots[ids]])
    h.revoke(B.KV, ids)
    src = bytes_of()
    d = [dev(x) for x in src] + [None]
    assert (h.place_from(B.KV, ids, d[0], d[1], block, n + 5) == B.OK).all()
    torch.cuda.synchronize()
    assert np.array_equal(pool(B.CACHE), src[:, :, block])
    # write-back of all layers, then of one, for cached objects and local ones (their slots are written through as well)
    every, where = np.concatenate([ids, local[:2]]), rng.permutation(n + 5)[:n + 2]
    want_host, want_cache, want_local = host(), pool(B.CACHE), pool(B.LOCAL)
    for layer in (-1, 1):
        src = bytes_of()
        d = [dev(x) for x in src] + [None]
        h.evict(B.KV, layer, every, d[0], d[1], where, n + 5)
        torch.cuda.synchronize()
        for at in range(layers) if layer < 0 else [layer]:
            new = src[:, at if layer < 0 else 0][:, where]
            want_host[:, at, host_slots[np.concatenate([ids, n + np.arange(2)])]] = new
            want_cache[:, at] = new[:, :n]
            want_local[:, at, :2] = new[:, n:]
        assert np.array_equal(host(), want_host)
        assert np.array_equal(pool(B.CACHE), want_cache) and np.array_equal(pool(B.LOCAL), want_local)
    h.close()


@pytest.mark.parametrize("chunk,n", [(16384, 64), (16384, 65), (32768, 32), (32768, 33), (32768 + 16, 32)])
def test_write_backs_around_the_size_from_which_stores_go_through(chunk, n):
    """2 MiB and the first size beyond, in tiles of 16 and 32 KiB and with a remainder: host copies and cache slots are the source's."""
    h = B.Harvest(kv=B.ClassSpec(n_layers=1, n_planes=2, chunk_bytes=chunk, max_objects=n, n_host_slots=n, n_cache_slots=n, n_local_slots=0))
    rng = np.random.default_rng(n)
    slots = rng.permutation(n).astype(np.int64)
    ids = h.register(B.KV, n, slots)
    h.place(B.KV, ids[:n // 2])
    src = [torch.from_numpy(rng.integers(0, 256, (n, chunk), dtype=np.uint8)).cuda() for _ in range(2)]
    at = rng.permutation(n).astype(np.uint64)
    h.evict(B.KV, -1, ids, src[0], src[1], at, n)
    torch.cuda.synchronize()
    for p in range(2):
        want = src[p].cpu().numpy()[at.astype(np.int64)]
        assert np.array_equal(h.host_plane(B.KV, p)[0][slots], want)
        assert np.array_equal(h.dev_plane(B.KV, B.CACHE, p)[0, :n // 2].cpu().numpy(), want[:n // 2])
    h.close()


def test_first_placement_on_a_stream_while_the_null_stream_is_busy():
    n, layers, chunk, rng = 40, 4, 16384, np.random.default_rng(3)
    h = B.Harvest(kv=B.ClassSpec(n_layers=layers, n_planes=1, chunk_bytes=chunk, max_objects=n, n_host_slots=n, n_cache_slots=n, n_local_slots=0))
    h.host_plane(B.KV, 0)[:] = rng.integers(0, 256, (layers, n, chunk), dtype=np.uint8)
    ids = h.register(B.KV, n, np.arange(n))
    torch.cuda.synchronize()
    for _ in range(6):          # a new stream's scratch each time (one that HIP maps to the null stream's hardware queue waits anyway)
        s = torch.cuda.Stream()
        torch.cuda._sleep(int(5e7))
        h.place(B.KV, ids, stream=s)
        s.synchronize()
        assert np.array_equal(h.dev_plane(B.KV, B.CACHE, 0).cpu().numpy(), h.host_plane(B.KV, 0))
        h.revoke(B.KV, ids)
        h.dev_plane(B.KV, B.CACHE, 0).zero_()
        torch.cuda.synchronize()
    h.close()


@pytest.mark.parametrize("flags", [B.FLAG_GENERAL_FETCH, 0])
def test_again_behind_a_replay_of_another_tables_fetch(flags):
    rig = Rig(2048, 30, n_layers=2, flags=flags)
    s, g, lens = torch.cuda.Stream(), torch.cuda.CUDAGraph(), [9, 17]
    t, dt, dn, df, cap = rig.tables(lens, 20)
    _, other_dt, other_dn, other_df, other_cap = rig.tables([30, 31], 33, seed=2)
    (k, v), (ok, ov) = rig.buffers(cap), rig.buffers(other_cap)
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        rig.h.fetch_kv(0, other_dt, other_dn, ok, ov, other_df, other_cap)       # the scratch is large enough for either
    with torch.cuda.graph(g, stream=s):
        rig.h.fetch_kv(1, other_dt, other_dn, ok, ov, other_df, other_cap)
    for layer in (1, 0, 1):
        with torch.cuda.stream(s):
            rig.h.fetch_kv(1 - layer, dt, dn, k, v, df, cap)
            g.replay()
            rig.h.fetch_kv_again(layer, k, v)
        torch.cuda.synchronize()
        for p, buf in enumerate([k, v]):
            got = buf.cpu().numpy()
            assert np.array_equal(got[:cap * 2048], rig.expected(t, lens, p, layer))
            assert (got[cap * 2048:] == 0xEE).all()
    rig.h.close()


@pytest.mark.parametrize("chunk", [16384, 32768])         # tiles of 16 and of 32 KiB
def test_a_write_back_beside_a_fetch_keeps_its_share_of_the_link(chunk):
    """Copies outside a fetch stand back while one needs the link, though never for longer than 60 us per 32 KiB and workgroup: the
    default 12 workgroups keep 6.5 GB/s.  Three quarters of that are asked for, with 0.1 ms for the host."""
    n, moved = 4000 * 32768 // chunk, 60 * 32768 // chunk
    h = B.Harvest(kv=B.ClassSpec(n_layers=1, n_planes=2, chunk_bytes=chunk, max_objects=n, n_host_slots=n, n_cache_slots=1, n_local_slots=0))
    h.register(B.KV, n, np.arange(n))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    dt, dn, df = dev(np.arange(n, dtype=np.int32)[None]), dev(np.array([n], dtype=np.int32)), dev(np.zeros(1, dtype=np.int64))
    k, v = (torch.empty(n * chunk, dtype=torch.uint8, device="cuda") for _ in range(2))
    src = [torch.zeros(moved * chunk, dtype=torch.uint8, device="cuda") for _ in range(2)]
    ids, at, us = np.arange(moved), np.arange(moved), []
    for _ in range(6):                                    # (two streams on one hardware queue run one after the other)
        a, b = torch.cuda.Stream(), torch.cuda.Stream()
        begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        h.evict(B.KV, -1, ids, src[0], src[1], at, moved, stream=b)
        torch.cuda.synchronize()
        h.fetch_kv(0, dt, dn, k, v, df, n, stream=a)      # 4.6 ms of the link
        begin.record(b)
        h.evict(B.KV, -1, ids, src[0], src[1], at, moved, stream=b)
        end.record(b)
        torch.cuda.synchronize()
        us.append(begin.elapsed_time(end) * 1e3)
    print("write-backs of 3.9 MB beside a fetch:", [round(x) for x in us], "us", flush=True)
    assert max(us) <= 2 * moved * chunk / 6.5e3 / 0.75 + 100
    h.close()


def test_a_fetch_beside_a_wide_placement_is_seen_by_the_next_tile():
    """32 workgroups that look for a fetch right before they load a tile: 200 blocks from the host take 4.0 times as long beside them
    as alone.  When they looked one tile earlier it was 5.4 to 6.4 times."""
    n, chunk, nx, xchunk = 200, 32768, 9, 96 << 20
    h = B.Harvest(kv=B.ClassSpec(n_layers=1, n_planes=2, chunk_bytes=chunk, max_objects=n, n_host_slots=n, n_cache_slots=1, n_local_slots=0),
                  expert=B.ClassSpec(n_layers=1, n_planes=1, chunk_bytes=xchunk, max_objects=nx, n_host_slots=nx, n_cache_slots=nx,
                                     n_local_slots=0, n_experts=nx), pcie_wgs=32, flags=B.FLAG_GENERAL_FETCH)
    h.register(B.KV, n, np.arange(n))
    ids = h.register(B.EXPERT, nx, np.arange(nx))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    dt, dn, df = dev(np.arange(n, dtype=np.int32)[None]), dev(np.array([n], dtype=np.int32)), dev(np.zeros(1, dtype=np.int64))
    k, v = (torch.empty(n * chunk, dtype=torch.uint8, device="cuda") for _ in range(2))
    fetches = torch.cuda.Stream()

    def fetch():
        begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        begin.record(fetches)
        h.fetch_kv(0, dt, dn, k, v, df, n, stream=fetches)
        end.record(fetches)
        fetches.synchronize()
        return begin.elapsed_time(end)

    alone = np.median([fetch() for _ in range(30)][10:])
    for _ in range(8):                                    # until HIP maps the two streams to different hardware queues
        places, beside = torch.cuda.Stream(), []
        h.place(B.EXPERT, ids, stream=places)
        while not places.query():
            beside.append(fetch())
        torch.cuda.synchronize()
        h.revoke(B.EXPERT, ids)
        if len(beside) > 5:
            break
    print(f"{len(beside)} fetches beside a placement: {np.median(beside):.3f} ms, alone {alone:.3f}", flush=True)
    assert np.median(beside) < 4.7 * alone
    h.close()


def test_a_fetch_from_the_host_keeps_its_rate_beside_a_kernel_that_fills_the_device():
    """The next layer's experts cross PCIe while this layer's are being read (the prefetch ring): loads from the host must go on
    arriving although every store queues behind the other kernel's.  Each wavefront waits for its own loads, so many with few
    loads keep the link busy: 96 of them with two loads each, 1.09 times the time alone; 48 with four, 1.38."""
    n, chunk = 6, 64 << 20
    h = B.Harvest(expert=B.ClassSpec(n_layers=1, n_planes=1, chunk_bytes=chunk, max_objects=n, n_host_slots=n, n_cache_slots=1,
                                     n_local_slots=0, n_experts=n))
    h.register(B.EXPERT, n, np.arange(n))
    topk = torch.arange(n, dtype=torch.int32, device="cuda")[None]
    staging, ptrs = torch.empty(n * chunk, dtype=torch.uint8, device="cuda"), torch.zeros(n, dtype=torch.int64, device="cuda")
    a, b = (torch.empty(1 << 30, dtype=torch.uint8, device="cuda") for _ in range(2))
    fetches = torch.cuda.Stream()

    def fetch():
        begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        begin.record(fetches)
        h.fetch_experts(0, topk, staging, n, ptrs, stream=fetches)
        end.record(fetches)
        fetches.synchronize()
        return begin.elapsed_time(end)

    alone, beside = np.median([fetch() for _ in range(6)][2:]), []
    for _ in range(6):                                    # (two streams on one hardware queue run one after the other)
        other = torch.cuda.Stream()
        torch.cuda.synchronize()
        for _ in range(40):                               # 13 ms and more beside 7
            B.plain_copy(b, a, a.numel(), stream=other)
        beside.append(fetch())
        torch.cuda.synchronize()
    print(f"402 MB from the host alone {alone:.2f} ms, beside a copy {[round(x, 2) for x in beside]}", flush=True)
    assert max(beside) < 1.18 * alone
    h.close()


@pytest.mark.parametrize("chunk", [16384, 32768])
def test_a_write_back_keeps_its_rate_beside_a_kernel_that_fills_the_device(chunk):
    """200 blocks beside a copy on another stream, against alone: 1.5 times as long with whole tiles of 16 KiB for chunks of 16 (2.7 with
    the remainder loop that a 32 KiB tile would make of each), 1.05 with tiles of 32 KiB for chunks of 32 (1.45 with 16)."""
    n = 200
    h = B.Harvest(kv=B.ClassSpec(n_layers=1, n_planes=2, chunk_bytes=chunk, max_objects=n, n_host_slots=n, n_cache_slots=n, n_local_slots=0))
    ids, at = h.register(B.KV, n, np.arange(n)), np.arange(n)
    h.place(B.KV, ids)
    src = [torch.zeros(n * chunk, dtype=torch.uint8, device="cuda") for _ in range(2)]
    a, b = (torch.empty(1 << 30, dtype=torch.uint8, device="cuda") for _ in range(2))
    writes = torch.cuda.Stream()

    def write():
        begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        begin.record(writes)
        h.evict(B.KV, -1, ids, src[0], src[1], at, n, stream=writes)
        end.record(writes)
        writes.synchronize()
        return begin.elapsed_time(end) * 1e3

    alone, beside = np.median([write() for _ in range(12)][4:]), []
    for _ in range(12):                                   # (two streams on one hardware queue run one after the other)
        other = torch.cuda.Stream()
        torch.cuda.synchronize()
        for _ in range(8):
            B.plain_copy(b, a, a.numel(), stream=other)
        beside.append(write())
        torch.cuda.synchronize()
    side_by_side = [x for x in beside if x > 1.02 * alone]
    print(f"write-back alone {alone:.0f} us, beside a copy {[round(x) for x in beside]}", flush=True)
    if side_by_side:
        assert np.median(side_by_side) < (2.1 if chunk < 32768 else 1.25) * alone
    h.close()


@pytest.mark.parametrize("revoked", [False, True])
@pytest.mark.parametrize("n_seq,width", [(1, 1), (1, 256), (1, 257), (3, 85), (7, 731), (300, 1), (256, 256), (4096, 16), (4097, 15), (5000, 3), (65537, 1), (9, 7300),
                                         (4200, 40), (2, 300000)])
def test_the_segments_of_a_resolve(n_seq, width, revoked):
    """One cell to several rounds of 1 024 a segment, one segment to 256 of them, more rows than one workgroup adds up: rows of no, of
    negative and of more than the table's length, blocks that do not exist and destinations that do not fit, of every tier."""
    chunk, n = 32, 500
    rig = Rig(chunk, n, n_layers=2, host_every=4, flags=B.FLAG_GENERAL_FETCH)
    rng = np.random.default_rng(n_seq + width)
    kinds = rng.integers(0, 6, n_seq)
    lens = np.where(kinds == 0, 0, np.where(kinds == 1, -3, np.where(kinds == 2, width + 5, rng.integers(0, width + 1, n_seq)))).astype(np.int32)
    lens[0] = min(width, 200000)
    live = np.clip(lens, 0, width).astype(np.int64)
    t = rng.integers(-1, n + 2, (n_seq, width), dtype=np.int32)
    asked = np.arange(width)[None, :] < live[:, None]
    first = np.cumsum(live) - live
    first[rng.random(n_seq) < 0.1] += 1 << 40                # some rows have no room at all
    first[0] = 0
    cap = int(live.sum())
    dst = first[:, None] + np.arange(width)[None, :]
    fits = dst < cap
    known = (t >= 0) & (t < n)
    good = asked & fits & known
    host = np.zeros(n + 2, dtype=bool)
    host[:len(rig.on_host)] = rig.on_host
    if revoked:
        gone = np.flatnonzero(~rig.on_host)[::5]
        rig.h.revoke(B.KV, gone)
        host[gone] = True
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    dt, dn, df = dev(t), dev(lens), dev(first.astype(np.int64))
    want_miss = np.flatnonzero((good & host[np.where(known, t, n)]).reshape(-1))
    n_local = int((good & (t >= len(rig.on_host))).sum())
    totals = []
    for turn in range(2):                                   # the second call's grid is sized by the first one's report
        k, v = rig.buffers(max(cap, 1))
        rig.h.fetch_kv(0, dt, dn, k, v, df, cap)
        counts, miss, n_miss = rig.h.fetch_info(miss_cap=t.size)
        assert n_miss == len(want_miss) and np.array_equal(miss, want_miss)
        assert counts == dict(n_requests=int(asked.sum()), n_local=n_local, n_cache=int(good.sum()) - n_local - n_miss, n_host=n_miss, n_lost=0,
                              n_invalid=int((asked & ~(fits & known)).sum()))
        rig.h.fetch_kv_again(1, k[rig.chunk * max(cap, 1):], v[rig.chunk * max(cap, 1):])
        for p, buf in enumerate([k, v]):
            got = buf.cpu().numpy()[:2 * max(cap, 1) * chunk].reshape(2, max(cap, 1), chunk)
            for layer in range(2):
                want = np.full((max(cap, 1), chunk), 0xEE, dtype=np.uint8)
                want[dst[good]] = rig.payload[p][layer][rig.order[t[good]]]
                assert np.array_equal(got[layer], want), (turn, p, layer)
        totals.append(rig.h.stats().fetch[B.KV].as_dict())
        assert totals[-1] == {name: 2 * (turn + 1) * x for name, x in counts.items()}
    if t.size <= 65536:
        info = torch.full((8,), 77, dtype=torch.int32, device="cuda")
        missed = torch.full((t.size,), -7, dtype=torch.int32, device="cuda")
        k, v = rig.buffers(max(cap, 1))
        rig.h.fetch_kv_static(0, dt, dn, k, v, df, cap, info, missed)
        c = counts
        assert info.tolist() == [c["n_requests"], c["n_local"], c["n_cache"], c["n_host"], 0, c["n_invalid"], n_miss, 0]
        assert np.array_equal(missed.cpu().numpy()[:n_miss], want_miss) and (missed.cpu().numpy()[n_miss:] == -7).all()
        want = np.full((max(cap, 1), chunk), 0xEE, dtype=np.uint8)
        want[dst[good]] = rig.payload[1][0][rig.order[t[good]]]
        assert np.array_equal(v.cpu().numpy()[:max(cap, 1) * chunk].reshape(-1, chunk), want)
    rig.h.close()


@pytest.mark.parametrize("n_host", [0, 1])
@pytest.mark.parametrize("n_planes,chunk,heads", [(2, 16, None), (2, 4112, None), (1, 8192, None), (2, 8208, None), (2, 32768 + 48, None), (1, 16384, (8, 16)), (2, 8880, (5, 3))])
@pytest.mark.parametrize("lens,width", [([129], 129), ([100, 64, 0, 40], 101), ([600, 3], 600)])
def test_one_kernel_fetch_with_two_loads_a_thread(n_planes, chunk, heads, lens, width, n_host):
    """From the second call on, which knows from a report that the link is not what the fetch waits for; tiles of 8 KiB."""
    rig = Rig(chunk, 400, n_planes=n_planes, host_every=100)
    t, dt, dn, df, cap = rig.tables(lens, width)
    hosts = np.flatnonzero(rig.on_host)
    t[np.isin(t, hosts)] = 0                                # a block of the cache tier
    t[0, 7:7 + n_host] = hosts[:n_host]
    t[0, 90] = -4
    dt.copy_(torch.from_numpy(t))
    for turn in range(3):
        k, v = rig.buffers(cap)
        if heads:
            rig.h.fetch_kv_head_major(0, dt, dn, k, v if n_planes == 2 else None, df, dn, cap, *heads)
        else:
            rig.h.fetch_kv(0, dt, dn, k, v if n_planes == 2 else None, df, cap)
        counts, miss, _ = rig.h.fetch_info(miss_cap=t.size)
        assert miss.tolist() == rig.misses(np.where(t >= 0, t, rig.n), lens) and len(miss) == n_host and counts["n_invalid"] == 1
        for p, buf in enumerate([k, v][:n_planes]):
            got = buf.cpu().numpy()
            assert (got[cap * chunk:] == 0xEE).all()
            at = 0
            for s, n in enumerate(lens):
                want = rig.payload[p][0][rig.order[t[s, :n]]]
                want[t[s, :n] < 0] = 0xEE
                if heads:
                    want = want.reshape(n * heads[1], heads[0], chunk // (heads[0] * heads[1])).transpose(1, 0, 2)
                assert np.array_equal(got[at:at + n * chunk], want.reshape(-1)), (turn, p, s)
                at += n * chunk
    rig.h.close()


@pytest.mark.parametrize("layout", [0, B.FLAG_CACHE_PLANES_ADJACENT])
@pytest.mark.parametrize("chunk", [32752, 32768, 32768 + 48, 65536 + 16])
@pytest.mark.parametrize("threads", [64, 256])
def test_chunks_around_the_size_from_which_planes_side_by_side_are_taken_in_one_pass(layout, chunk, threads):
    rig = Rig(chunk, 41, n_layers=2, host_every=5, flags=B.FLAG_GENERAL_FETCH | layout, gather_threads=threads)
    lens = [13, 0, 22]
    t, dt, dn, df, cap = rig.tables(lens, 23)
    for _ in range(2):
        k, v = rig.buffers(cap)
        rig.h.fetch_kv_layers(0, 2, dt, dn, k, v, cap * chunk, df, cap)
        assert rig.h.fetch_info(miss_cap=t.size)[1].tolist() == rig.misses(t, lens)
        for p, buf in enumerate([k, v]):
            got = buf.cpu().numpy()
            for layer in range(2):
                assert np.array_equal(got[layer * cap * chunk:(layer + 1) * cap * chunk], rig.expected(t, lens, p, layer)), (p, layer)
            assert (got[2 * cap * chunk:] == 0xEE).all()
    rig.h.close()


class ExpertRig:
    def __init__(self, e, chunk, known=None, on_host=(), **kw):
        rng = np.random.default_rng(e + chunk)
        self.e, self.chunk, self.known = e, chunk, e if known is None else known
        self.weights = rng.integers(0, 256, (e, chunk), dtype=np.uint8)
        slots = rng.permutation(e).astype(np.int64)
        self.h = B.Harvest(expert=B.ClassSpec(n_layers=1, n_planes=1, chunk_bytes=chunk, max_objects=e, n_host_slots=e, n_cache_slots=e, n_local_slots=0,
                                              n_experts=e), **kw)
        self.h.host_plane(B.EXPERT, 0)[0, slots] = self.weights
        self.h.register(B.EXPERT, self.known, slots[:self.known])
        self.on_host = np.zeros(e, dtype=bool)
        self.on_host[list(on_host)] = True
        cached = rng.permutation(np.flatnonzero(~self.on_host[:self.known]))
        if len(cached):
            self.h.place(B.EXPERT, cached)
        torch.cuda.synchronize()

    def fetch(self, ids, n_staging, stream=None):
        staging = torch.full((n_staging * self.chunk + 64,), 0xEE, dtype=torch.uint8, device="cuda")
        ptrs = torch.full((self.e,), 7, dtype=torch.int64, device="cuda")
        self.h.fetch_experts(0, torch.from_numpy(np.ascontiguousarray(ids[None])).cuda(), staging, n_staging, ptrs, stream=stream)
        counts, miss, _ = self.h.fetch_info(miss_cap=self.e)
        return staging.cpu().numpy(), ptrs.cpu().numpy() - staging.data_ptr(), counts, sorted(miss.tolist())


@pytest.mark.parametrize("e,known,chunk,n_ids,n_staging", [(1, 1, 16, 1, 1), (60, 60, 8192 * 3 + 48, 16, 60), (64, 64, 4096, 64, 64), (16, 16, 4096, 256, 16), (127, 127, 2048, 193, 127), (65, 65, 8208, 65, 65), (128, 128, 1 << 18, 64, 128),
                                                           (128, 100, 8192, 50, 128), (90, 90, 12288, 40, 5), (120, 120, 1040, 33, 120)])
@pytest.mark.parametrize("n_host", [0, 1])
def test_one_kernel_expert_fetch(e, known, chunk, n_ids, n_staging, n_host):
    """From the second fetch on, against numpy: repeated ids and ids that are out of range, experts that nobody has registered, less staging
    than experts; the grid is sized by the fetch before, which had fewer or more."""
    rig = ExpertRig(e, chunk, known, on_host=range(n_host))
    rng = np.random.default_rng(n_ids)
    totals = {}
    for turn in range(5):
        ids = rng.integers(-1 if n_ids > 4 else 0, e + (n_ids > 4), n_ids if turn % 2 else max(1, n_ids // 3)).astype(np.int32)
        if turn < 2:
            ids[ids < n_host] = n_host % e               # the first reports say that HBM is what the fetch waits for
        got, ptrs, counts, miss = rig.fetch(ids, n_staging)
        routed = [i for i in sorted(set(ids.tolist())) if 0 <= i < e]
        staged = [i for i in routed if i < known][:n_staging]
        assert np.array_equal(got[:len(staged) * chunk].reshape(-1, chunk), rig.weights[staged]) and (got[len(staged) * chunk:] == 0xEE).all(), turn
        at = np.zeros(e, dtype=np.int64)
        at[staged] = np.arange(len(staged)) * chunk
        there = np.isin(np.arange(e), staged)
        assert np.array_equal(ptrs[there], at[there]) and (ptrs[~there] < 0).all()
        assert miss == [i for i in staged if rig.on_host[i]] and counts["n_requests"] == len(routed)
        assert counts["n_invalid"] == int(((ids < 0) | (ids >= e)).sum()) + len(routed) - len(staged) and counts["n_cache"] == len(staged) - len(miss)
        for name, x in counts.items():
            totals[name] = totals.get(name, 0) + x
        assert rig.h.stats().fetch[B.EXPERT].as_dict() == totals
    rig.h.close()


@pytest.mark.parametrize("edit", ["revoked", "placed"])
def test_a_one_kernel_expert_fetch_is_whole_when_the_directory_changes_under_it(edit):
    e, chunk = 96, 1 << 20
    rig = ExpertRig(e, chunk, on_host=[0])
    for i in range(e):
        rig.h.register_cb(B.EXPERT, i, enabled=False)
    side = torch.cuda.Stream()
    every = np.arange(e, dtype=np.int32)
    staging, ptrs = torch.zeros(e * chunk, dtype=torch.uint8, device="cuda"), torch.zeros(e, dtype=torch.int64, device="cuda")
    d_ids = torch.from_numpy(every[None, :60].copy()).cuda()
    want = torch.from_numpy(rig.weights[:60].reshape(-1)).cuda()
    for turn in range(6):
        rig.fetch(every[30:62] if edit == "placed" else every[:60], e)          # reports about HBM
        if edit == "placed":
            rig.h.revoke(B.EXPERT, every[10:12])
        staging.zero_()
        torch.cuda.synchronize()
        rig.h.fetch_experts(0, d_ids, staging, e, ptrs)
        if edit == "revoked":
            rig.h.revoke(B.EXPERT, every[5 * turn + 1:5 * turn + 6])
        else:
            rig.h.place(B.EXPERT, every[10:12], stream=side)
        torch.cuda.synchronize()
        assert torch.equal(staging[:60 * chunk], want), (turn, int((staging[:60 * chunk] != want).reshape(60, -1).any(1).sum()))
        if edit == "revoked":
            rig.h.place(B.EXPERT, every[5 * turn + 1:5 * turn + 6])
    rig.h.close()


@pytest.mark.parametrize("pcie_wgs", [0, 1, 4])
@pytest.mark.parametrize("n", [1, 2, 3, 6, 7, 10, 11, 30])
def test_moves_of_fewer_and_of_more_tiles_than_workgroups(n, pcie_wgs):
    """Two tiles a block, against 12 workgroups from the host, 20 to it, or 1 and 4; three calls in a row on the same tile counter."""
    chunk = 32768
    h = B.Harvest(kv=B.ClassSpec(n_layers=1, n_planes=2, chunk_bytes=chunk, max_objects=n, n_host_slots=n, n_cache_slots=n, n_local_slots=0), pcie_wgs=pcie_wgs)
    rng = np.random.default_rng(n)
    slots = rng.permutation(n).astype(np.int64)
    ids = h.register(B.KV, n, slots)
    at = rng.permutation(n).astype(np.uint64)
    for turn in range(3):
        src = [torch.from_numpy(rng.integers(0, 256, (n, chunk), dtype=np.uint8)).cuda() for _ in range(2)]
        h.evict(B.KV, -1, ids, src[0], src[1], at, n)
        h.place(B.KV, ids)
        torch.cuda.synchronize()
        for p in range(2):
            want = src[p].cpu().numpy()[at.astype(np.int64)]
            assert np.array_equal(h.host_plane(B.KV, p)[0][slots], want), (turn, p)
            assert np.array_equal(h.dev_plane(B.KV, B.CACHE, p)[0].cpu().numpy(), want), (turn, p)
        h.revoke(B.KV, ids)
    h.close()


@pytest.mark.parametrize("flags", [0, B.FLAG_GENERAL_FETCH])
@pytest.mark.parametrize("e,n_ids", [(5, 255), (40, 256), (40, 257), (300, 511), (300, 2047), (33, 2048), (33, 2049), (2000, 4100), (64, 32768)])
def test_routing_ids_around_what_a_workgroup_loads_at_once(e, n_ids, flags):
    rig = ExpertRig(e, 64, on_host=range(0, e, 3), flags=flags)
    ids = np.random.default_rng(e).integers(0, e, n_ids).astype(np.int32)
    ids[[0, n_ids // 2, n_ids - 1]] = -5, e, 1 << 30
    for _ in range(2):
        got, ptrs, counts, miss = rig.fetch(ids, e)
        routed = [i for i in sorted(set(ids.tolist())) if 0 <= i < e]
        assert np.array_equal(got[:len(routed) * 64].reshape(-1, 64), rig.weights[routed]) and (got[len(routed) * 64:] == 0xEE).all()
        assert np.array_equal(ptrs[routed], np.arange(len(routed)) * 64) and (np.delete(ptrs, routed) < 0).all()
        assert counts["n_requests"] == len(routed) and counts["n_invalid"] == 3 and miss == [i for i in routed if i % 3 == 0]
    rig.h.close()


def with_a_lost_object(chunk, n, layout=0, **kw):
    """n objects in the cache tier, number n lost; every object's bytes are its number modulo 251."""
    h = B.Harvest(kv=B.ClassSpec(n_layers=1, n_planes=2, chunk_bytes=chunk, max_objects=n + 1, n_host_slots=n, n_cache_slots=n + 1, n_local_slots=1),
                  flags=B.FLAG_GENERAL_FETCH | layout, **kw)
    for p in range(2):
        h.host_plane(B.KV, p)[0] = (np.arange(n) % 251).astype(np.uint8)[:, None]
    h.register(B.KV, n, np.arange(n))
    h.place(B.KV, np.arange(n))
    h.register(B.KV, 1, None, tier=B.LOCAL)
    h.evict(B.KV, -1, [n], h.dev_plane(B.KV, B.LOCAL, 0), h.dev_plane(B.KV, B.LOCAL, 1), np.zeros(1, dtype=np.uint64), 1, B.EVICT_DEMOTE)
    torch.cuda.synchronize()
    h.revoke(B.KV, [n])
    return h


@pytest.mark.parametrize("n_seq,width,live,chunk,heads,most", [(256, 2048, 500224, 512, None, 0.55), (4, 4096, 12000, 32768, None, 0.16), (4, 4096, 12000, 32768, (8, 16), 0.16)])
def test_a_fetch_of_lost_blocks_takes_a_fraction_of_the_fetch_that_finds_them(n_seq, width, live, chunk, heads, most):
    """It moves no payload; the misses are long lists that no transfer hides (500 224 blocks: 245 us found, 17 lost; 198 with the misses put
    together by 16 wavefronts, a load at a time), and so is the list of what HBM might serve (12 000 blocks: 250 us found, 12.5 lost; 53 with
    one tile of it looked at after the other: 0.21 of the time, 0.19 head-major; the limit leaves a slow host 39 us for two launches)."""
    n = 4096
    h = with_a_lost_object(chunk, n)
    lens = np.full(n_seq, live // n_seq, dtype=np.int32)
    found = np.random.default_rng(0).integers(0, n, (n_seq, width), dtype=np.int32)
    dn, df = torch.from_numpy(lens).cuda(), torch.from_numpy((np.cumsum(lens) - lens).astype(np.int64)).cuda()
    k, v = (torch.zeros(live * chunk, dtype=torch.uint8, device="cuda") for _ in range(2))
    us = {}
    for what, table in (("found", found), ("lost", np.full_like(found, n))):
        dt = torch.from_numpy(table).cuda()
        if heads:
            fetch = lambda: h.fetch_kv_head_major(0, dt, dn, k, v, df, dn, live, *heads)
        else:
            fetch = lambda: h.fetch_kv(0, dt, dn, k, v, df, live)
        for _ in range(3):
            fetch()
        times = []
        for _ in range(7):
            begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            begin.record()
            for _ in range(10):
                fetch()
            end.record()
            end.synchronize()
            times.append(begin.elapsed_time(end) * 100)
        us[what] = np.median(times)
        counts, miss, n_miss = h.fetch_info(miss_cap=found.size)
        if what == "lost":
            cells = np.flatnonzero((np.arange(width)[None] < lens[:, None]).reshape(-1))
            assert counts["n_lost"] == n_miss == live and np.array_equal(miss, cells)
        else:
            assert counts["n_cache"] == live and n_miss == 0
    print({x: round(float(y), 1) for x, y in us.items()}, flush=True)
    assert us["lost"] < most * us["found"], us
    h.close()


@pytest.mark.parametrize("chunk,heads,threads,layout", [(1024, None, 0, 0), (2064, None, 128, 0), (32768, None, 0, B.FLAG_CACHE_PLANES_ADJACENT), (4096, (8, 16), 0, 0),
                                                        (8256, (3, 4), 0, 0)])
@pytest.mark.parametrize("where", [0.0, 0.001, 0.02, 0.3, 0.7, "runs", "first and last"])
def test_a_few_live_blocks_among_lost_ones(where, chunk, heads, threads, layout):
    """From the second call on the grid is sized by the live ones, far shorter than the list, and passes over the others."""
    n, n_seq = 1000, 3
    h = with_a_lost_object(chunk, n, layout, gather_threads=threads)
    live = 90000 if chunk < 2000 else 12000
    lens = np.array([live // 2, live // 3, live // 6], dtype=np.int32)
    cap, width = int(lens.sum()), int(lens.max())
    rng = np.random.default_rng(chunk)
    at = np.arange(cap)
    there = at // 1700 % 3 == 1 if where == "runs" else (at == 0) | (at == cap - 1) if where == "first and last" else rng.random(cap) < where
    asked = np.where(there, rng.integers(0, n, cap), n).astype(np.int32)
    first = np.cumsum(lens) - lens
    table = np.full((n_seq, width), -1, dtype=np.int32)
    for s in range(n_seq):
        table[s, :lens[s]] = asked[first[s]:first[s] + lens[s]]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    dt, dn, df = dev(table), dev(lens), dev(first.astype(np.int64))
    want = dev(np.where(there, asked % 251, 0xEE).astype(np.uint8))
    k, v = (torch.empty(cap * chunk, dtype=torch.uint8, device="cuda") for _ in range(2))
    for turn in range(3):
        k.fill_(0xEE), v.fill_(0xEE)
        if heads:
            h.fetch_kv_head_major(0, dt, dn, k, v, df, dn, cap, *heads)
        else:
            h.fetch_kv(0, dt, dn, k, v, df, cap)
        counts, miss, n_miss = h.fetch_info(miss_cap=table.size)
        cells = np.flatnonzero((np.arange(width)[None] < lens[:, None]).reshape(-1))
        assert counts["n_cache"] == there.sum() and counts["n_lost"] == n_miss == cap - there.sum() and np.array_equal(miss, cells[~there])
        for buf in (k, v):
            for s in range(n_seq):
                a, b = int(first[s]), int(first[s] + lens[s])
                got = buf[a * chunk:b * chunk]
                got = got.view(heads[0], b - a, -1) if heads else got.view(1, b - a, chunk)
                assert torch.equal(got, want[a:b][None, :, None].expand_as(got)), (turn, s)
    h.close()
