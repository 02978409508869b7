"""The HIP calls the library's host code makes, on a CPU: the host half of harvest.hip is linked with a runtime that writes the calls
down and fails the one a test names (tests/fakehip/fakehip.cpp).  Kernels do not run, so these tests are about order, choice of
path and error paths, never about payload bytes."""
import ctypes
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

from paper_2602_00328_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
POOL = 0x10000000                          # no kernel runs: pool and buffer addresses are only ever added up


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    d = tmp_path_factory.mktemp("fakehip")
    obj, run, so = str(d / "harvest.o"), str(d / "fakehip.o"), str(d / "libharvest_fake.so")
    flags = ["-O1", "-std=c++17", "-fPIC", "-Wno-unused-command-line-argument"]
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "--offload-host-only", *flags, "-c", "-o", obj,
                           os.path.join(ROOT, "paper_2602_00328_amd", "csrc", "harvest.hip")])
    fatbin = re.search(r"\b(__hip_fatbin\w*)$", subprocess.check_output(["nm", "-u", obj], text=True), re.M).group(1)
    subprocess.check_call(["hipcc", "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", *flags, f"-DHIP_FATBIN={fatbin}", "-c", "-o", run,
                           os.path.join(ROOT, "tests", "fakehip", "fakehip.cpp")])
    # -Bsymbolic: in a process where torch has loaded the real runtime, these calls still stay in this library
    subprocess.check_call(["g++", "-shared", "-Wl,-Bsymbolic", "-o", so, obj, run])
    lib = ctypes.CDLL(so)
    for name, (res, args) in B.SYMBOLS.items():
        fn = getattr(lib, name)
        fn.restype, fn.argtypes = res, args
    lib.fake_log.restype = ctypes.c_char_p
    lib.fake_fail.argtypes = [ctypes.c_char_p, ctypes.c_int]
    lib.fake_capture.argtypes = lib.fake_number.argtypes = [ctypes.c_void_p]
    lib.fake_stream.restype = lib.fake_pinned.restype = ctypes.c_void_p
    lib.fake_pinned.argtypes = [ctypes.c_size_t, ctypes.c_size_t]
    lib.fake_pinned_count.argtypes, lib.fake_pinned_count.restype = [ctypes.c_size_t], ctypes.c_size_t
    return lib


class Ctx:
    """A context with a KV class of n objects (32 KiB chunks unless said otherwise), all on the host."""

    def __init__(self, lib, n=200, n_local=0, n_layers=2, chunk=32768, flags=0, cb=None, **tuning):
        self.lib, cfg = lib, B.harvest_config()
        cfg.flags = flags
        for name, value in tuning.items():
            setattr(cfg, name, value)
        kv = cfg.cls[B.KV]
        kv.n_layers, kv.n_planes, kv.chunk_bytes, kv.max_objects = n_layers, 2, chunk, n + n_local
        kv.n_host_slots, kv.n_cache_slots, kv.n_local_slots = n + n_local, n, max(n_local, 1)
        for p in range(2):
            kv.host_pool[p], kv.d_cache_pool[p], kv.d_local_pool[p] = POOL * (p + 1), POOL * (p + 3), POOL * (p + 5)
        self.h, self.n, self.n_local = ctypes.c_void_p(), n, n_local
        assert lib.harvest_create(ctypes.byref(cfg), ctypes.byref(self.h)) == B.OK
        self.cb = B.REVOKE_CB(cb or (lambda *_: None))
        slots = np.arange(n + n_local, dtype=np.int64)
        for first, k, tier in ((0, n, B.HOST), (n, n_local, B.LOCAL)):
            if k:
                assert lib.harvest_register(self.h, B.KV, k, slots[first:].ctypes.data, tier, self.cb, None,
                                            np.empty(k, dtype=np.uint32).ctypes.data) == B.OK
        self.stream = lib.fake_stream()
        self.number = lib.fake_number(self.stream)

    def close(self):
        assert self.lib.harvest_destroy(self.h) == B.OK

    def tier(self, obj):
        t = ctypes.c_int()
        assert self.lib.harvest_lookup(self.h, B.KV, obj, ctypes.byref(t), None, None, None) == B.OK
        return t.value

    def stats(self):
        s = B.harvest_stats_t()
        assert self.lib.harvest_stats(self.h, ctypes.byref(s)) == B.OK
        return s

    def ids(self, ids):
        a = np.asarray(ids, dtype=np.uint32)
        return a, a.ctypes.data, a.size

    def place(self, ids):
        a, p, n = self.ids(ids)
        return self.lib.harvest_place(self.h, B.KV, p, n, self.stream, None)

    def place_from(self, ids):
        a, p, n = self.ids(ids)
        at = np.arange(n, dtype=np.uint64)
        return self.lib.harvest_place_from(self.h, B.KV, p, n, POOL * 8, POOL * 9, at.ctypes.data, n, self.stream, None)

    def evict(self, ids, flags=0):
        a, p, n = self.ids(ids)
        at = np.arange(n, dtype=np.uint64)
        return self.lib.harvest_evict(self.h, B.KV, -1, p, n, POOL * 8, POOL * 9, at.ctypes.data, n, flags, self.stream)

    def revoke(self, ids):
        a, p, n = self.ids(ids)
        return self.lib.harvest_revoke(self.h, B.KV, p, n)

    def log(self):
        return self.lib.fake_log().decode().splitlines()


def launches(log, name):
    """Where the log has a launch of the kernel that did not fail."""
    return [i for i, line in enumerate(log) if "LaunchKernel" in line and name in line and log[i + 1:i + 2] != ["  failed"]]


@pytest.mark.parametrize("n", [3, 81, 150])             # lists that travel with the launch; objects that do not; neither does
@pytest.mark.parametrize("what", ["place", "place_from", "evict", "demote"])
@pytest.mark.parametrize("failing", ["hipLaunchKernel", "hipEventRecord", "hipStreamWaitEvent", "hipHostGetDevicePointer", "hipMemcpyAsync"])
def test_a_call_that_fails_leaves_mirror_and_device_in_step(fake, what, n, failing):
    """Whichever HIP call fails: the mirror shows a new entry if and only if its dir_write was launched, and what was launched
    on the stream is either stood for by an event recorded behind it or has been waited for before the call returned."""
    reached = 0
    for nth in range(1, 9):
        c = Ctx(fake, n_local=150)
        assert c.place([199]) == B.OK                     # the stream's state and an earlier edit exist
        if what == "evict":
            assert c.place(range(n // 2)) == B.OK
        ids = np.arange(n) + (c.n if what == "demote" else 0)
        call = {"place": c.place, "place_from": c.place_from, "evict": c.evict, "demote": lambda i: c.evict(i, B.EVICT_DEMOTE)}[what]
        assert c.revoke([199]) == B.OK                    # the latest edit ran on another stream
        before, s0 = [c.tier(i) for i in ids], c.stats()
        c.log()
        fake.fake_fail(failing.encode(), nth)
        rc = call(ids)
        hit = not fake.fake_fail_pending()
        fake.fake_fail(b"", 0)
        log, after, s1 = c.log(), [c.tier(i) for i in ids], c.stats()
        if not hit:
            assert rc == B.OK
            c.close()
            break
        reached += 1
        assert rc == B.EHIP, log
        edited, moved = launches(log, "dir_write"), launches(log, "move_")
        changed = [a != b for a, b in zip(after, before)]
        if what != "evict":
            assert all(changed) == any(changed) == bool(edited), (nth, log)
        counted = s1.n_evicted[0] - s0.n_evicted[0] if what in ("evict", "demote") else s1.n_placed[0] - s0.n_placed[0]
        if what == "evict":
            assert counted == (n if moved else 0), (nth, log)
        else:
            assert counted == (n if edited else 0), (nth, log)
        for at in moved + edited:
            number = re.search(r"stream (\d+)", log[at]).group(1)
            rest = [line for i, line in enumerate(log) if i > at and log[i + 1:i + 2] != ["  failed"]]
            assert any(re.match(rf"(hipEventRecord|hipStreamSynchronize) stream {number}\b", line) for line in rest), (nth, log)
        # a slot that went back to the allocator is not being written: the copy had ended before the call gave it back
        if moved and not edited and what != "evict":
            tail = log[moved[0]:]
            assert any(line == f"hipStreamSynchronize stream {c.number}" for line in tail), (nth, log)
        # and the context goes on working
        assert call(ids) == B.OK
        c.close()
    assert reached or failing not in ("hipLaunchKernel", "hipEventRecord")


def test_a_fetch_whose_event_is_not_recorded_has_ended_when_the_call_returns(fake):
    """No event stands for it, so a revocation could not wait for it: the call does."""
    c = Ctx(fake)
    for how in (1, 2):                                    # the first fetch makes the stream's state
        c.log()
        if how == 2:
            fake.fake_fail(b"hipEventRecord", 1)
        rc = fake.harvest_fetch_kv(c.h, 0, POOL, POOL, 1, 8, POOL, POOL, POOL, 8, c.stream)
        assert rc == (B.OK if how == 1 else B.EHIP)
    assert c.log()[-1] == f"hipStreamSynchronize stream {c.number}"
    c.close()


@pytest.mark.parametrize("recorded", [False, True])
def test_a_revocation_hands_slots_back_behind_a_system_scope_release(fake, recorded):
    """Between the end of the drain's waits and the callbacks there is a fence at system scope that the host has waited for: the
    events of the drain carry none."""
    seen = []
    c = Ctx(fake, cb=lambda cls, obj, user: seen.append(c.log()))
    assert c.place([3, 4]) == B.OK
    assert fake.harvest_fetch_kv(c.h, 0, POOL, POOL, 1, 8, POOL, POOL, POOL, 8, c.stream) == B.OK
    if recorded:                                          # then the drain waits for the whole device
        fake.fake_capture(c.stream)
        assert fake.harvest_fetch_kv(c.h, 0, POOL, POOL, 1, 8, POOL, POOL, POOL, 8, c.stream) == B.OK
        fake.fake_capture(None)
    c.log()
    assert c.revoke([3, 4]) == B.OK
    log = seen[0]
    waits = [i for i, line in enumerate(log) if line.startswith("hipDeviceSynchronize" if recorded else "hipEventSynchronize")]
    fence = launches(log, "system_fence")
    assert len(seen) == 2 and waits and len(fence) == 1 and fence[0] > waits[-1], log
    number = re.search(r"stream (\d+)", log[fence[0]]).group(1)
    assert f"hipStreamSynchronize stream {number}" in log[fence[0]:], log
    if not recorded:                                      # nothing enqueued since: nothing to wait for and nothing to make visible
        assert c.place([5, 6]) == B.OK and c.revoke([5]) == B.OK
        c.log()
        assert c.revoke([6]) == B.OK
        assert not launches(seen[-1], "system_fence"), seen[-1]
    c.close()


def test_a_drain_whose_fence_fails_keeps_the_slots(fake):
    c = Ctx(fake, n=1)
    assert c.place([0]) == B.OK
    fake.fake_fail(b"hipStreamSynchronize", 1)
    assert c.revoke([0]) == B.EHIP
    fake.fake_fail(b"", 0)
    st = np.zeros(1, dtype=np.int32)
    a, p, n = c.ids([0])
    assert fake.harvest_place(c.h, B.KV, p, n, c.stream, st.ctypes.data) == B.OK and st[0] == B.ENOSPC
    c.close()


def test_scratch_is_cleared_on_the_stream_that_uses_it(fake):
    """hipMemset returns before the null stream has done it (21 us behind a null stream with 40 ms of work queued), and a stream
    made non-blocking does not wait for the null stream: a tile counter cleared that way may still hold anything at its first
    use, or be cleared in the middle of it."""
    c = Ctx(fake)
    for call in (lambda: c.place([1]), lambda: fake.harvest_fetch_kv(c.h, 0, POOL, POOL, 1, 8, POOL, POOL, POOL, 8, c.stream)):
        c.stream = fake.fake_stream()
        c.log()
        assert call() == B.OK
        log = c.log()
        assert "hipMemset" not in log, log
        cleared = [i for i, line in enumerate(log) if line == f"hipMemsetAsync stream {fake.fake_number(c.stream)}"]
        assert len(cleared) == 2 and cleared[-1] < launches(log, "")[0], log
    c.close()


def test_a_small_table_leaves_the_one_kernel_form_only_on_a_report_about_itself(fake):
    """The kernels report live requests (words 0 and 1: HBM and host tier) and which table they are about (words 2 and 3: rows and
    columns).  A table that is mostly padding goes through the general path; what another table reported says nothing about it,
    and neither does any report about the replays of a graph."""
    c = Ctx(fake)

    def path(n_seq, width, layers=1):
        c.log()
        assert fake.harvest_fetch_kv_layers(c.h, 0, layers, POOL, POOL, n_seq, width, POOL, POOL, 8 * 32768, POOL, 8, c.stream) == B.OK
        log = c.log()
        small = bool(launches(log, "fetch_kv_small"))
        assert small != bool(launches(log, "classify_kv")), log
        return "one kernel" if small else "general"

    assert path(1, 8) == "one kernel"
    words = (ctypes.c_uint32 * 16).from_address(fake.fake_pinned(64, fake.fake_pinned_count(64) - 1))

    def report(live_hbm, live_host, n_seq, width):
        words[:4] = [live_hbm, live_host, n_seq, width]

    report(8, 0, 1, 8)                                   # an 8-block fetch has run last: 2040 * 8 * 2 tiles fewer than the next table
    assert path(1, 2048) == "one kernel"
    assert path(1, 2048) == "one kernel"                 # still the report of the 8-block fetch: the others have not run yet
    assert path(2, 1024) == "one kernel"
    assert path(1, 48, layers=2) == "one kernel"
    report(8, 0, 1, 2048)
    assert path(1, 2048) == "general"
    assert path(2, 1024) == "one kernel"
    report(1000, 1048, 1, 2048)                          # full: both tiers together
    assert path(1, 2048) == "one kernel"
    report(8, 0, 1, 2048)
    fake.fake_capture(c.stream)
    assert path(1, 2048) == "one kernel"
    fake.fake_capture(None)
    c.close()


def test_a_static_state_that_goes_to_another_stream_takes_no_report_with_it(fake):
    c = Ctx(fake)
    words = [(ctypes.c_uint32 * 16).from_address(fake.fake_pinned(64, fake.fake_pinned_count(64) - 1 - i)) for i in range(4)]

    def path():
        c.log()
        assert fake.harvest_fetch_kv_static(c.h, 0, POOL, POOL, 1, 2048, POOL, POOL, POOL, 8, None, None, c.stream) == B.OK
        return "general" if launches(c.log(), "classify_kv") else "one kernel"

    assert path() == "one kernel"
    for w in words:
        w[:4] = [8, 0, 1, 2048]
    assert path() == "general"
    assert fake.harvest_release_stream(c.h, c.stream) == B.OK
    c.stream = fake.fake_stream()
    assert path() == "one kernel"
    assert path() == "one kernel"
    c.close()


def test_a_repeated_fetch_resolves_again_once_a_fetch_has_been_recorded_on_its_stream(fake):
    """A replay, which the library cannot see, writes the stream's counters and lists: they no longer belong to the eager fetch
    that the call repeats, and a count of one table with the list of another reaches beyond the destination."""
    c = Ctx(fake, flags=B.FLAG_GENERAL_FETCH)
    fetch = lambda width: fake.harvest_fetch_kv(c.h, 0, POOL, POOL, 1, width, POOL, POOL, POOL, 8, c.stream)
    again = lambda: fake.harvest_fetch_kv_again(c.h, 1, POOL, POOL, c.stream)
    assert fetch(32) == B.OK
    c.log()
    assert again() == B.OK and not launches(c.log(), "classify_kv")
    fake.fake_capture(c.stream)
    assert fetch(16) == B.OK
    fake.fake_capture(None)
    assert fetch(32) == B.OK
    for _ in range(2):                                    # a replay may come before either
        c.log()
        assert again() == B.OK and launches(c.log(), "classify_kv")
    c.close()


def test_the_host_tier_is_spread_wider_when_the_link_is_what_a_fetch_waits_for(fake):
    """Before anything is known, and when the last report says so: 96 single wavefronts at the head of the grid, otherwise 48."""
    c = Ctx(fake, flags=B.FLAG_GENERAL_FETCH)

    def head():
        c.log()
        assert fake.harvest_fetch_kv(c.h, 0, POOL, POOL, 1, 10000, POOL, POOL, POOL, 8, c.stream) == B.OK
        log = c.log()
        return int(re.search(r"grid (\d+),", log[launches(log, "gather")[0]]).group(1))

    tiles = 32                                           # of 1 KiB a block: the HBM tier's share of the grid is known
    assert head() == 96 + 10000 * tiles
    words = (ctypes.c_uint32 * 16).from_address(fake.fake_pinned(64, fake.fake_pinned_count(64) - 1))
    for hbm, host, wavefronts in ((9900, 100, 48), (9800, 200, 96), (10000, 0, 48), (5000, 5000, 96)):
        words[:4] = [hbm, host, 1, 10000]
        assert head() == wavefronts + hbm * tiles
    c.close()


@pytest.mark.parametrize("head_major", [False, True])
def test_the_gathers_grid_covers_the_list_where_that_is_not_much_longer_than_what_hbm_serves(fake, head_major):
    """Word 8 of the report: entries of the list, those of lost and invalid requests and of the host's among them.  Not beyond half as
    many again, and not where the link is what the fetch waits for."""
    c = Ctx(fake, flags=B.FLAG_GENERAL_FETCH)

    def hbm_tiles(at_host):
        c.log()
        if head_major:
            assert fake.harvest_fetch_kv_head_major(c.h, 0, POOL, POOL, 1, 10000, POOL, POOL, POOL, POOL, 8, 8, 16, c.stream) == B.OK
        else:
            assert fake.harvest_fetch_kv(c.h, 0, POOL, POOL, 1, 10000, POOL, POOL, POOL, 8, c.stream) == B.OK
        log = c.log()
        return int(re.search(r"grid (\d+),", log[launches(log, "gather")[0]]).group(1)) - (24 if head_major else at_host)

    tiles = 8 if head_major else 32
    assert hbm_tiles(96) == 10000 * tiles
    words = (ctypes.c_uint32 * 16).from_address(fake.fake_pinned(64, fake.fake_pinned_count(64) - 1))
    for hbm, host, listed, entries, at_host in ((7000, 0, 8000, 8000, 48), (7000, 100, 9000, 9000, 48), (6000, 0, 9000, 9000, 48), (6000, 0, 9001, 6000, 48), (6000, 3000, 9000, 6000, 96),
                                                (7000, 0, 0, 7000, 48), (9000, 0, 12000, 10000, 48)):
        words[:4], words[8] = [hbm, host, 1, 10000], listed
        assert hbm_tiles(at_host) == entries * tiles, (hbm, host, listed)
    c.close()


def test_a_head_major_gather_looks_ahead_in_its_list_where_its_grid_is_far_too_short(fake):
    c = Ctx(fake, flags=B.FLAG_GENERAL_FETCH)

    def looks_ahead():
        c.log()
        assert fake.harvest_fetch_kv_head_major(c.h, 0, POOL, POOL, 1, 10000, POOL, POOL, POOL, POOL, 8, 8, 16, c.stream) == B.OK
        log = c.log()
        return "gather_hmILi2ELb1E" in log[launches(log, "gather")[0]]

    assert not looks_ahead()
    words = (ctypes.c_uint32 * 16).from_address(fake.fake_pinned(64, fake.fake_pinned_count(64) - 1))
    for hbm, listed, expected in ((0, 2048, False), (0, 2049, True), (600, 2400, False), (600, 2401, True), (9000, 10000, False), (3000, 1 << 30, False)):
        words[:4], words[8] = [hbm, 0, 1, 10000], listed                # (never fewer than 16 workgroups of a tile on each of 256 compute units)
        assert looks_ahead() == expected, (hbm, listed)
    c.close()


def test_which_one_kernel_fetches_make_two_loads_a_thread(fake):
    """Their tiles are 8 KiB, not 4: more than 128 cells, up to 256 MiB (128 of several layers), once a report says that the link is not
    what the fetch waits for.  Both sides of each line, of that for tables that are mostly padding too."""
    c = Ctx(fake, n=16, n_layers=4, chunk=65536)

    def tiles(width, layers=1):
        """Of 64 KiB, by the grid: 16, or 8 with two loads a thread; 0: the general path."""
        c.log()
        assert fake.harvest_fetch_kv_layers(c.h, 0, layers, POOL, POOL, 1, width, POOL, POOL, 16 * 65536, POOL, 16, c.stream) == B.OK
        log = c.log()
        small = launches(log, "fetch_kv_small")
        if not small:
            return 0
        grid, block = (int(re.search(rf"{word} (\d+)", log[small[0]]).group(1)) for word in ("grid", "block"))
        hbm = grid if layers > 1 else grid - 1 - (32 if block == 256 else 64)
        assert hbm % width == 0, log
        return hbm // width * block // 256

    def report(hbm, host, width):
        words[:4] = [hbm, host, 1, width]

    assert tiles(600) == 16                               # nothing is known yet
    words = (ctypes.c_uint32 * 16).from_address(fake.fake_pinned(64, fake.fake_pinned_count(64) - 1))
    report(500, 0, 1)
    assert tiles(128) == 16 and tiles(129) == 8 and tiles(2048) == 8 and tiles(2049) == 16
    assert tiles(512, 2) == 8 and tiles(513, 2) == 16 and tiles(256, 4) == 8 and tiles(257, 4) == 16
    report(550, 10, 1)
    assert tiles(600) == 8
    report(549, 10, 1)                                    # the link
    assert tiles(600) == 16
    fake.fake_capture(c.stream)
    report(500, 0, 1)
    assert tiles(600) == 16
    fake.fake_capture(None)
    for loads, width, host in ((8, 2000, 0), (16, 2100, 0), (16, 2000, 50)):
        report(width - 625 - host, host, width)           # 625 cells that ask for nothing: 20 000 tiles of 4 KiB, 10 000 of 8
        assert tiles(width) == loads
        report(width - 626 - host, host, width)
        assert tiles(width) == 0
    c.close()


def test_the_one_kernel_fetch_knows_the_edits_it_comes_after(fake):
    """One that is being recorded learns them from a kernel in front of it.  With an object around that a revocation can leave
    nothing to copy from, every fetch resolves in one place."""
    c = Ctx(fake, n_local=4)
    fetch = lambda: fake.harvest_fetch_kv(c.h, 0, POOL, POOL, 1, 8, POOL, POOL, POOL, 8, c.stream)
    assert fetch() == B.OK
    for recorded in (False, True):
        fake.fake_capture(c.stream if recorded else None)
        c.log()
        assert fetch() == B.OK
        log = c.log()
        snap, small = launches(log, "snap_edit"), launches(log, "fetch_kv_small")
        assert len(small) == 1 and len(snap) == recorded and snap + small == sorted(snap + small), log
    fake.fake_capture(None)
    c.close()
    cfg = B.harvest_config()
    kv = cfg.cls[B.KV]
    kv.n_layers, kv.n_planes, kv.chunk_bytes, kv.max_objects, kv.n_host_slots, kv.n_cache_slots, kv.n_local_slots = 1, 1, 4096, 8, 4, 4, 4
    kv.host_pool[0], kv.d_cache_pool[0], kv.d_local_pool[0] = POOL, POOL * 2, POOL * 3
    h, stream, slots, out = ctypes.c_void_p(), fake.fake_stream(), np.arange(4, dtype=np.int64), np.empty(4, dtype=np.uint32)
    assert fake.harvest_create(ctypes.byref(cfg), ctypes.byref(h)) == B.OK
    for lossy in (False, True):
        assert fake.harvest_register(h, B.KV, 4, None if lossy else slots.ctypes.data, B.LOCAL if lossy else B.HOST, B.REVOKE_CB(), None, out.ctypes.data) == B.OK
        fake.fake_log()
        assert fake.harvest_fetch_kv(h, 0, POOL, POOL, 1, 8, POOL, None, POOL, 8, stream) == B.OK
        log = fake.fake_log().decode().splitlines()
        assert bool(launches(log, "classify_kv")) == lossy and bool(launches(log, "fetch_kv_small")) != lossy, log
    assert fake.harvest_destroy(h) == B.OK


def test_a_fetch_beside_another_streams_placement_and_recording(fake):
    """Whether the placement is through is asked so that it disturbs no recording on another stream; while it is not, the kernel in
    front of the one-kernel fetch asks the device which edits are complete."""
    c = Ctx(fake)
    other = fake.fake_stream()
    fetch = lambda s: fake.harvest_fetch_kv(c.h, 0, POOL, POOL, 1, 8, POOL, POOL, POOL, 8, s)
    assert fetch(other) == B.OK and fetch(c.stream) == B.OK and c.place([1, 2]) == B.OK
    fake.fake_capture(c.stream)
    for pending in (True, False):
        fake.fake_not_ready(pending)
        c.log()
        assert fetch(other) == B.OK
        log = c.log()
        assert len(launches(log, "snap_edit")) == pending and len(launches(log, "fetch_kv_small")) == 1, log
        assert [line.split()[-1] for line in log if line.startswith("hipEventQuery")] == ["relaxed"], log
    fake.fake_capture(None)
    fake.fake_not_ready(False)
    c.close()


@pytest.mark.parametrize("tuning,readers,writers", [({}, 32, 20), (dict(host_wgs=5, pcie_wgs=7), 5, 7)])
def test_a_callers_numbers_of_workgroups_are_taken_as_they_are(fake, tuning, readers, writers):
    """Of a one-kernel fetch (64 KiB blocks: 16 tiles a cell) those that read the host, and those of a write-back."""
    c = Ctx(fake, chunk=65536, **tuning)
    grid = lambda name: (lambda log: int(re.search(r"grid (\d+),", log[launches(log, name)[0]]).group(1)))(c.log())
    c.log()
    assert fake.harvest_fetch_kv(c.h, 0, POOL, POOL, 1, 300, POOL, POOL, POOL, 300, c.stream) == B.OK
    assert grid("fetch_kv_small") == 300 * 16 + readers + 1
    assert c.evict(np.arange(150)) == B.OK
    assert grid("move_pcie") == writers
    c.close()


def expert_context(lib, n=60, n_local=0, local=(), flags=0, chunk=1 << 20, **tuning):
    """n experts of 1 MiB, the last n_local of them registered as local; `local`: those without a host copy."""
    cfg = B.harvest_config()
    cfg.flags = flags
    for name, value in tuning.items():
        setattr(cfg, name, value)
    ex = cfg.cls[B.EXPERT]
    ex.n_layers, ex.n_planes, ex.chunk_bytes, ex.max_objects, ex.n_experts = 1, 1, chunk, n, n
    ex.n_host_slots, ex.n_cache_slots, ex.n_local_slots = n, n, 4
    ex.host_pool[0], ex.d_cache_pool[0], ex.d_local_pool[0] = POOL, POOL * 2, POOL * 3
    h, out = ctypes.c_void_p(), np.empty(n, dtype=np.uint32)
    assert lib.harvest_create(ctypes.byref(cfg), ctypes.byref(h)) == B.OK
    slots = np.arange(n, dtype=np.int64)
    assert lib.harvest_register(h, B.EXPERT, n - n_local, slots.ctypes.data, B.HOST, B.REVOKE_CB(), None, out.ctypes.data) == B.OK
    if n_local:
        assert lib.harvest_register(h, B.EXPERT, n_local, None if local == "lossy" else slots[n - n_local:].ctypes.data, B.LOCAL, B.REVOKE_CB(), None, out.ctypes.data) == B.OK
    return h


def test_a_few_routing_ids_are_fetched_by_one_kernel_when_ranks_and_edits_are_known(fake):
    """The rank of an expert has to follow from the ids alone, and the latest report to say that HBM is what the fetch waits for."""
    lib = fake

    def path(h, stream, n_ids=16, staging=60):
        lib.fake_log()
        assert lib.harvest_fetch_experts(h, 0, POOL * 4, n_ids, 1, POOL * 5, staging, POOL * 6, stream) == B.OK
        log = lib.fake_log().decode().splitlines()
        small = bool(launches(log, "fetch_experts_small"))
        assert small != bool(launches(log, "resolve_experts")), log
        return "one kernel" if small else "general"

    def report(hbm, host):
        words = (ctypes.c_uint32 * 16).from_address(lib.fake_pinned(64, lib.fake_pinned_count(64) - 1))
        words[4:8] = [hbm, host, 0, 0]

    h, s = expert_context(lib), lib.fake_stream()
    assert path(h, s) == "general"                        # nothing is known yet
    report(11, 0)
    assert path(h, s) == path(h, s, n_ids=256) == path(h, s, staging=1) == "one kernel"
    assert path(h, s, n_ids=257) == path(h, s, n_ids=0) == path(h, s, staging=0) == "general"
    report(11, 1)                                         # the link is what it waits for
    assert path(h, s) == "general"
    report(300, 0)                                        # 300 MiB
    assert path(h, s) == "general"
    report(11, 0)
    lib.fake_capture(s)
    assert path(h, s) == "general"
    lib.fake_capture(None)
    assert path(h, s) == "one kernel"
    other = lib.fake_stream()                             # another stream places: until its edit is seen
    assert path(h, other) == "general"
    report(11, 0)
    assert path(h, other) == "one kernel"
    ids = np.array([3], dtype=np.uint32)
    lib.fake_not_ready(True)
    assert lib.harvest_place(h, B.EXPERT, ids.ctypes.data, 1, s, None) == B.OK
    assert path(h, other) == "general"
    lib.fake_not_ready(False)
    assert path(h, other) == "one kernel"
    assert lib.harvest_destroy(h) == B.OK
    h, s = expert_context(lib, chunk=16 << 20), lib.fake_stream()
    assert path(h, s) == "general"
    report(11, 0)                                         # 176 MiB; 32 different ids would be 512 MiB, twice the limit
    assert path(h, s, n_ids=32) == "one kernel" and path(h, s, n_ids=33) == "general" and path(h, s, n_ids=33, staging=32) == "one kernel"
    assert lib.harvest_destroy(h) == B.OK
    for kw, expected in (({}, "one kernel"), (dict(n_local=2), "general"), (dict(n_local=2, local="lossy"), "general"), (dict(n=129), "general"),
                         (dict(flags=B.FLAG_GENERAL_FETCH), "general"), (dict(flags=B.FLAG_PROFILE), "general")):
        h, s = expert_context(lib, **kw), lib.fake_stream()
        assert path(h, s) == "general"
        report(11, 0)
        assert path(h, s) == expected, kw
        assert lib.harvest_destroy(h) == B.OK


@pytest.mark.parametrize("tuning,threads,cap", [(dict(gather_wg_per_cu=2), 64, 2), (dict(gather_threads=64), 64, None), (dict(gather_threads=256), 256, None),
                                                (dict(gather_wg_per_cu=1, gather_threads=128), 128, 1)])
def test_a_callers_gather_serves_every_expert_fetch(fake, tuning, threads, cap):
    """Workgroups per compute unit and threads of the HBM-tier gather hold for a few routing ids too, whatever is known from earlier fetches."""
    h, s = expert_context(fake, **tuning), fake.fake_stream()
    for turn in range(3):
        fake.fake_log()
        assert fake.harvest_fetch_experts(h, 0, POOL * 4, 16, 1, POOL * 5, 60, POOL * 6, s) == B.OK
        log = fake.fake_log().decode().splitlines()
        assert not launches(log, "fetch_experts_small"), log
        (at,) = launches(log, "gather")
        grid, block = (int(re.search(rf"{word} (\d+)", log[at]).group(1)) for word in ("grid", "block"))
        assert block == threads, log
        if cap:                                           # 256 compute units, and at most 192 KiB of reads of the host
            assert grid <= cap * 256 + 24 * 256 // threads, log
        words = (ctypes.c_uint32 * 16).from_address(fake.fake_pinned(64, fake.fake_pinned_count(64) - 1))
        words[4:8] = [11, 0, 0, 0]
    assert fake.harvest_destroy(h) == B.OK
