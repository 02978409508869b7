#!/usr/bin/env python3
"""Benchmark of the tiered cache fetch on one MI355X.

Workload (benchmark configs[1]): long-context KV decode fetch, Llama-3-8B-shaped - 32 layers, 8 KV heads x 128,
bf16, 16-token blocks (32 KiB K + 32 KiB V per block per layer), 4 sequences with seeded lengths in [32K, 128K] tokens,
70% of the closed blocks in the HBM cache tier, 30% host-only.  One step = one pass of the whole hot path: resolve every
block of every sequence through the device directory, gather one layer's K and V into the contiguous working layout
(HBM tier and, over PCIe, host tier at the same time), append one token per sequence, and,
when a tail block fills, write it back, demote it, place it in the cache tier and open a new tail.

Prints ONE JSON line on stdout; progress goes to stderr.
"""
import argparse
import gc
import json
import math
import os
import re
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0          # MI355X HBM3E, published


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--seed", type=int, default=0)
    ap.add_argument("--layers", type=int, default=32, help="layers materialised in the pools (footprint knob)")
    ap.add_argument("--iso-steps", type=int, default=20, help="fetches per isolation point (100%% cache / 100%% host)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-isolation", action="store_true")
    ap.add_argument("--host-wgs", type=int, default=0, help="tuning: workgroups of the host-tier gather (0 = default)")
    ap.add_argument("--workload", default="kv_decode",
                    choices=["kv_decode", "kv_tiny", "experts_phi", "experts_qwen", "latency_by_size", "link_contention",
                             "kv_and_experts"],
                    help="kv_decode = configs[1] (the benchmark line); kv_tiny = configs[0] (fetch latency, both forms of the "
                         "fetch); experts_* = configs[2] / configs[3], extra lines; latency_by_size = time of one fetch from "
                         "the cache tier against the same fetch from the host, by object size (the paper's Figures 3 and 7 "
                         "on this machine: context, not a benchmark line); link_contention = a PCIe-bound KV fetch repeated on one stream "
                         "while a placement of experts runs on another, by the number of workgroups the placement's copy runs "
                         "with (harvest_config.pcie_wgs): who gets the link; kv_and_experts = configs[4]: the KV decode fetch on one "
                         "stream and the Phi-shaped expert fetch on another at the same time, a quarter of each cache tier "
                         "revoked every 10 steps and placed again 5 steps later")
    ap.add_argument("--head-major", action="store_true", help="gather into the head-major working layout instead")
    ap.add_argument("--kv-elt-bytes", type=int, default=2, choices=[1, 2, 4],
                    help="bytes per KV element: 2 = the bf16 / fp16 of the named config, 1 = an fp8 KV cache (16 KiB blocks)")
    ap.add_argument("--placement", default="shuffled", choices=["shuffled", "in_sequence_order"],
                    help="kv_decode: order in which the resident blocks were placed (shuffled = scattered over the cache "
                         "tier, the default; in_sequence_order = a sequence's blocks are neighbours)")
    ap.add_argument("--no-profile", action="store_true",
                    help="kv_decode only: leave out the leg that times the tiers' kernels (per-kernel figures are then absent)")
    ap.add_argument("--fetch-layers", type=int, default=1,
                    help="variant: every step fetches this many consecutive layers with one harvest_fetch_kv_layers call "
                         "(must divide --layers); isolation and graph legs are skipped")
    ap.add_argument("--shared-cache", action="store_true",
                    help="variant: the cache tier is one pool of best-fit segments (an object's layers and planes are "
                         "contiguous) instead of equal-size slots per layer and plane")
    ap.add_argument("--place-from-host", action="store_true",
                    help="experts_qwen only: the LRU's placements read the host copies over PCIe (harvest_place) instead of "
                         "the staging buffer the fetch has just filled (harvest_place_from)")
    ap.add_argument("--fetch-again", action="store_true",
                    help="variant: after the first fetch every fetch is harvest_fetch_kv_again (same block table, another "
                         "layer): the request lists are made again only when the directory has been edited")
    ap.add_argument("--prefetch", action="store_true",
                    help="experts_phi only: also time the double-buffered prefetch ring against fetch-then-use")
    ap.add_argument("--graph-steps", type=int, default=64,
                    help="extra decode steps whose fetches replay recorded HIP graphs (one per layer); 0 = skip")
    ap.add_argument("--gather-threads", type=int, default=0, choices=[0, 64, 128, 256],
                    help="tuning: threads per workgroup of the HBM-tier gather (0 = the library's default, 64)")
    ap.add_argument("--cache-layout", default="adjacent", choices=["adjacent", "planes"],
                    help="kv_decode, equal-size slots: 'adjacent' = one cache pool [layer][slot][K|V][chunk] (a block's K and "
                         "V are neighbours, one 64 KiB source run per block); 'planes' = a K pool and a V pool")
    ap.add_argument("--no-other-legs", dest="other_legs", action="store_false",
                    help="kv_decode: skip the short extra legs (the next seed's draw, the two expert configurations with two "
                         "layers materialised) that the default run appends under 'other_legs'")
    ap.add_argument("--calibrate", type=int, default=3, help="plain-copy launches of 2 GiB (counter calibration)")
    args = ap.parse_args()
    if args.no_profile:
        args.no_isolation = True
    if args.fetch_layers > 1:
        if args.layers % args.fetch_layers or args.head_major:
            ap.error("--fetch-layers must divide --layers and excludes --head-major")
        args.no_isolation, args.graph_steps = True, 0
    return args


class DeviceDecode:
    """Keeps the decode state of workloads.scenarios.KVRun on the device so that a timed step moves no table or
    payload over PCIe except what the method itself moves."""

    def __init__(self, run, eng, wl, n_steps, head_major=False, fetch_layers=1, again=False):
        import numpy as np
        import torch
        import workloads as W
        self.run, self.eng, self.wl = run, eng, wl
        self.dev = eng.dev
        sh = wl.shape
        table, nb = run.table_arrays()
        self.d_table = torch.from_numpy(table).to(self.dev)
        self.d_nb = torch.from_numpy(nb).to(self.dev)
        self.d_sdb = torch.from_numpy(run.seq_dst_block.view(np.int64)).to(self.dev)
        self.fetch_layers = fetch_layers
        self.again, self.fetched_once = again, False
        self.layer_bytes = run.cap * sh.chunk_bytes
        self.dst_all = [torch.zeros(fetch_layers * self.layer_bytes, dtype=torch.uint8, device=self.dev) for _ in range(2)]
        self.dst = [t[:self.layer_bytes] for t in self.dst_all]            # the first fetched layer
        # the rows every step appends, generated up front: [step][plane][layer][seq][row_bytes]
        rows = np.empty((n_steps, 2, sh.n_layers, wl.n_seq, sh.row_bytes), dtype=np.uint8)
        for t in range(n_steps):
            for s in range(wl.n_seq):
                rows[t, :, :, s] = W.append_rows(wl, t, s)
        self.rows = torch.from_numpy(rows).to(self.dev)
        self.local = [eng.h.dev_plane(0, 2, p).view(sh.n_layers, -1, sh.row_bytes) for p in range(2)]
        self.t = 0
        self.graphs = None
        self.head_major = head_major
        idx = [eng.h.lookup(0, run.tables[s][-1])[1] * sh.block_tokens + run.lens[s] % sh.block_tokens
               for s in range(wl.n_seq)]
        self.d_idx = torch.tensor(idx, dtype=torch.int64, device=self.dev)
        self.roll = torch.zeros((sum(len(f) for f in wl.future_blocks) + 1, 2), dtype=torch.int64).pin_memory()
        self.n_roll = 0
        final = [len(t) + len(f) for t, f in zip(wl.tables, wl.future_blocks)]
        self.d_cap = torch.tensor(final, dtype=torch.int32, device=self.dev)

    def record_graphs(self):
        """One HIP graph per layer holding that layer's fetch: its launch parameters are fixed, tables and residency
        live in device memory and keep changing underneath."""
        import torch
        s = torch.cuda.Stream(self.dev)
        again, self.again = self.again, False          # a recorded fetch must resolve the table at every replay
        with torch.cuda.stream(s):
            self.fetch(0)                              # outside capture: this stream's scratch is allocated here
        s.synchronize()
        graphs = []
        for layer in range(self.wl.shape.n_layers):
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s):
                self.fetch(layer)
            graphs.append(g)
        self.graphs, self.again = graphs, again

    def first_layer(self, t):
        return (t * self.fetch_layers) % self.wl.shape.n_layers

    def fetch(self, layer):
        if self.fetch_layers > 1:
            self.eng.h.fetch_kv_layers(layer, self.fetch_layers, self.d_table, self.d_nb, self.dst_all[0], self.dst_all[1],
                                       self.layer_bytes, self.d_sdb, self.run.cap)
            return
        if self.graphs:
            self.graphs[layer].replay()
            return
        if self.again and self.fetched_once:
            # the same table as the fetch before (a roll-over edits the directory, which makes the library resolve again)
            self.eng.h.fetch_kv_again(layer, self.dst[0], self.dst[1])
            return
        self.fetched_once = True
        if self.head_major:
            sh = self.wl.shape
            self.eng.h.fetch_kv_head_major(layer, self.d_table, self.d_nb, self.dst[0], self.dst[1], self.d_sdb,
                                           self.d_cap, self.run.cap, sh.n_kv_heads, sh.block_tokens)
        else:
            self.eng.fetch_kv_device(layer, self.d_table, self.d_nb, self.d_sdb, self.run.cap, dst=self.dst)

    def step(self):
        import torch
        run, wl, sh = self.run, self.wl, self.wl.shape
        t = self.t
        self.fetch(self.first_layer(t))
        # append one token per sequence: rows go straight into the open tail blocks in local HBM.  The row index of every
        # tail lives on the device and is bumped there, so a step copies nothing from the host unless a tail rolls over.
        for p in range(2):
            self.local[p].index_copy_(1, self.d_idx, self.rows[t, p])
        self.d_idx += 1
        for s in range(wl.n_seq):
            run.lens[s] += 1
            if run.lens[s] % sh.block_tokens == 0:
                tail = run.tables[s][-1]
                self.eng.evict_from_local(0, [tail], 1)
                if wl.resident[tail] and self.eng.place(0, [tail])[0] == 0:
                    run.live.add(tail)
                new = int(wl.future_blocks[s][run.n_future[s]])
                run.n_future[s] += 1
                got = self.eng.register(0, 1, wl.host_slot[new:new + 1], 2)
                assert int(got[0]) == new
                run.tables[s].append(new)
                k = self.n_roll                       # one pinned row per roll-over: the copy below is asynchronous
                self.n_roll += 1
                self.roll[k, 0], self.roll[k, 1] = new, self.eng.h.lookup(0, new)[1] * sh.block_tokens
                r = self.roll[k].to(self.dev, non_blocking=True)
                self.d_table[s, len(run.tables[s]) - 1] = r[0].to(torch.int32)
                self.d_nb[s] += 1
                self.d_idx[s] = r[1]
        self.t += 1


COUNT_KEYS = ("n_requests", "n_local", "n_cache", "n_host", "n_lost", "n_invalid")


def kv_totals(stats):
    return {k: int(getattr(stats.fetch[0], k)) for k in COUNT_KEYS}


def bench_tiny(args, embed=False):
    """configs[0]: the tiny KV fetch (16 sequences x 16 blocks, 60 % in the cache tier), its write-back and the fetch
    again, checked against the oracle.  Its size says nothing about bandwidth; what it shows is the latency floor of a
    fetch, for the one-kernel form small tables take and for the general path."""
    import numpy as np
    import torch
    import workloads as W
    from workloads import scenarios as S
    from workloads.hip_engine import HipEngine
    wl = W.kv_tiny(args.seed)
    chunk = wl.shape.chunk_bytes
    want, cpu_baseline = None, None
    if not args.no_cpu_baseline:                         # the CPU-baseline leg: the oracle's result and its speed
        from oracle.engine import OracleEngine
        eo = OracleEngine(kv=S.kv_spec(wl))
        ro = S.KVRun(eo, wl)
        want = ro.fetch(0)
        a, n_rep = time.perf_counter(), 0
        while time.perf_counter() - a < 2.0:
            ro.fetch(0)
            n_rep += 1
        sec = (time.perf_counter() - a) / n_rep
        cpu_baseline = {"value": round(2 * 256 * 2 * chunk / sec / 1e9, 2), "unit": "GB/s", "cores": 1, "kind": "oracle",
                        "sample": f"the same fetch (256 blocks, 16 MiB), repeated for 2 s on one thread ({n_rep} times)"}
        eo.close()
    res, exact = {}, (True if want is not None else None)
    for name, general in (("one_kernel", False), ("general_path", True)):
        eng = HipEngine(kv=S.kv_spec(wl), general_fetch=general)
        run = S.KVRun(eng, wl)
        table, nb = run.table_arrays()
        dev = eng.dev
        d_table, d_nb = torch.from_numpy(table).to(dev), torch.from_numpy(nb).to(dev)
        d_sdb = torch.from_numpy(run.seq_dst_block.view(np.int64)).to(dev)
        dst = [torch.zeros(run.cap * chunk, dtype=torch.uint8, device=dev) for _ in range(2)]
        ids = np.concatenate(wl.tables).astype(np.uint32)
        blk = np.arange(ids.size)

        def fetch():
            eng.h.fetch_kv(0, d_table, d_nb, dst[0], dst[1], d_sdb, run.cap)

        for _ in range(args.warmup):
            fetch()
        torch.cuda.synchronize()
        lat = []
        for _ in range(args.steps):
            a = time.perf_counter()
            fetch()
            torch.cuda.synchronize()
            lat.append(time.perf_counter() - a)
        a = time.perf_counter()
        for _ in range(args.steps):
            fetch()
        torch.cuda.synchronize()
        b2b = (time.perf_counter() - a) / args.steps
        a = time.perf_counter()
        for _ in range(args.steps):                      # the round trip: gather, scatter the same bytes back, gather again
            fetch()
            eng.h.evict(0, 0, ids, dst[0], dst[1], blk, run.cap, 0)
        fetch()
        torch.cuda.synchronize()
        trip = (time.perf_counter() - a) / args.steps
        counts, _, _ = eng.h.fetch_info()
        if want is not None:
            exact &= bool(np.array_equal(dst[0].cpu().numpy(), want[0]) and np.array_equal(dst[1].cpu().numpy(), want[1])
                          and counts == want[3])
        res[name] = {"latency_us": round(float(np.median(lat)) * 1e6, 1), "back_to_back_us": round(b2b * 1e6, 1),
                     "fetch_plus_write_back_us": round(trip * 1e6, 1)}
        log(f"[bench] kv_tiny {name}: {res[name]}")
        served = counts
        eng.close()
    payload = ids.size * 2 * chunk
    best = res["one_kernel"]["back_to_back_us"] * 1e-6
    out = {
        "metric": "fetch GB/s (read+write) and % of HBM/PCIe peak; objects/s; bit-exact vs oracle",
        "value": round(2 * payload / best / 1e9, 2), "unit": "GB/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(best * 1e3, 5), "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "u8",
        "data": "synthetic",
        "config": {"workload": "configs[0]: tiny KV fetch, 16 sequences x 16 blocks of 2 x 32 KiB, 60% in the cache tier / 40% "
                               "on the host, one layer; a latency case - too small to say anything about bandwidth",
                   "seed": args.seed},
        "objects_per_s": round(ids.size / best), "bit_exact": exact, "served": served, "latency": res,
        "roofline": None, "cpu_baseline": cpu_baseline}
    if embed:
        return out
    print(json.dumps(out), flush=True)


def experts_vs_oracle(args, wl, run, eng, n_total, L):
    """The oracle walks the same steps (fetches, and for the LRU config the policy's revocations and placements), then
    both fetch every layer once more for the step after the timed ones: pointers, staged bytes, counts and miss list must
    agree.  Also times the oracle's fetch of one layer (single-threaded: a reported baseline, not a target)."""
    import numpy as np
    from workloads import scenarios as S
    from oracle.engine import OracleEngine
    t0 = time.time()
    eo = OracleEngine(expert=run._spec)
    xo = S.ExpertRun(eo, wl)
    for t in range(n_total):
        for l in range(L):
            if wl.lru_capacity:
                xo.fetch(t, l, digest=True)                 # the LRU's placements copy from the staging buffer of this fetch
                xo.lru_update(t, l, from_staging=not args.place_from_host)
    exact = True
    for l in range(L):
        a, b = xo.fetch(n_total, l), run.fetch(n_total, l)
        exact &= all((x is None) == (y is None) and (x is None or np.array_equal(x, y)) for x, y in zip(a[0], b[0]))
        exact &= bool(np.array_equal(np.where(a[1] >= 3, 0, a[1]), b[1]) and np.array_equal(a[3], b[3]) and a[4] == b[4])
    staged = sum(1 for x in a[0] if x is not None) - int((a[1] == 1).sum())
    n, t1 = 0, time.perf_counter()
    while n < 2 or time.perf_counter() - t1 < 3.0:
        xo.fetch(n_total, L - 1, digest=True)
        n += 1
    sec = (time.perf_counter() - t1) / n
    chunk = eng.spec[1].chunk_bytes
    base = {"value": round(2 * staged * chunk / sec / 1e9, 2), "unit": "GB/s", "cores": 1, "kind": "oracle",
            "sample": f"the fetch of one layer ({staged} experts of {chunk / 2**20:.1f} MiB copied into staging), repeated "
                      f"{n} times (>= 3 s), its checksum included; all tiers in host DRAM"}
    eo.close()
    log(f"[bench] experts vs oracle after {n_total} steps: bit_exact={bool(exact)}; oracle {base['value']} GB/s on one thread "
        f"({time.time() - t0:.1f}s)")
    return bool(exact), base


def bench_experts(args, embed=False):
    """configs[2] (Phi-3.5-MoE-shaped, static residency) and configs[3] (Qwen-MoE-shaped, LRU-driven cache tier): one step
    = the expert fetch of every materialised layer for one batch of routed tokens (plus, for the LRU config, the
    revocations and placements the policy asks for after each layer).  embed: return the result instead of printing it."""
    import numpy as np
    import torch
    import workloads as W
    from workloads import scenarios as S
    from workloads.hip_engine import HipEngine
    dev = torch.device("cuda", 0)
    phi = args.workload == "experts_phi"
    L = min(args.layers, 32 if phi else 24)

    def set_up(profile):
        if phi:
            wl = W.expert_offload(seed=args.seed, shape=W.ExpertShape(n_layers=L))
        else:
            wl = W.expert_lru(seed=args.seed, shape=W.ExpertShape(n_layers=L, n_experts=60, d_model=2048, d_ff=1408))
        t0 = time.time()
        spec = S.expert_spec(wl)
        if not args.no_isolation:
            spec.n_cache_slots = wl.n_objects          # room for the all-cache isolation point
        eng = HipEngine(expert=spec, profile=profile, host_wgs=args.host_wgs, gather_threads=args.gather_threads)
        run = S.ExpertRun(eng, wl)
        run._spec = spec
        torch.cuda.synchronize()
        sp = eng.spec[1]
        log(f"[bench] {args.workload}: {L} layers x {sp.n_experts} experts of {sp.chunk_bytes / 2**20:.1f} MiB, host pool "
            f"{sp.n_host_slots * sp.chunk_bytes / 2**30:.1f} GiB, set up in {time.time() - t0:.1f}s")
        return wl, eng, run

    # as in bench_kv: timed as callers run it, the tiers' kernels in a leg of their own
    wl, eng, run = set_up(False)
    sp = eng.spec[1]
    E = sp.n_experts
    staging = torch.empty(E * sp.chunk_bytes, dtype=torch.uint8, device=dev)
    ptrs = torch.zeros(E, dtype=torch.int64, device=dev)
    n_total = args.warmup + args.steps
    topk = {(t, l): torch.from_numpy(wl.routing(t, l)).to(dev) for t in range(n_total) for l in range(L)}

    def step(t):
        eng._last_staging = staging                    # what the LRU's placements copy from (harvest_place_from)
        for l in range(L):
            eng.h.fetch_experts(l, topk[(t, l)], staging, E, ptrs)
            if wl.lru_capacity:
                run.lru_update(t, l, from_staging=not args.place_from_host)

    for t in range(args.warmup):
        step(t)
    torch.cuda.synchronize()
    f0 = eng.h.stats()
    c0 = {k: int(getattr(f0.fetch[1], k)) for k in COUNT_KEYS}
    p0 = int(f0.n_placed[1])
    a = time.perf_counter()
    for t in range(args.warmup, n_total):
        step(t)
    torch.cuda.synchronize()
    sec = time.perf_counter() - a
    f1 = eng.h.stats()
    d = {k: int(getattr(f1.fetch[1], k)) - c0[k] for k in COUNT_KEYS}
    placed = int(f1.n_placed[1]) - p0
    chunk = sp.chunk_bytes
    payload = (d["n_cache"] + d["n_host"]) * chunk
    out = {
        "metric": "fetch GB/s (read+write) and % of HBM/PCIe peak; objects/s; bit-exact vs oracle",
        "value": round(2 * payload / sec / 1e9, 2), "unit": "GB/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(sec * 1e3 / args.steps, 4), "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "u8", "data": "synthetic",
        "config": {"workload": ("configs[2]: MoE expert fetch, Phi-3.5-MoE-shaped (16 experts/layer of 150 MiB, top-2 "
                                "Zipf(1.1), 64 tokens, 2 local, 50% of the rest cached)" if phi else
                                "configs[3]: MoE expert fetch, Qwen-MoE-shaped (60 experts/layer of 16.5 MiB, top-4 "
                                "Zipf(1.0), 256 tokens, LRU cache tier of 24 experts/layer)"),
                   "seed": args.seed, "layers_materialised": L,
                   **({"placements_read": "host copies" if args.place_from_host else "the staging buffer of the fetch"}
                      if wl.lru_capacity else {})},
        "objects_per_s": round(d["n_requests"] / sec), "bit_exact": None,
        "served_per_step": {k: round(v / args.steps, 2) for k, v in d.items()},
        "placed_per_step": round(placed / args.steps, 2),
        "cpu_baseline": None,
    }
    log(f"[bench] {args.steps} steps in {sec:.3f}s: {out['ms_per_step']} ms/step; per step {out['served_per_step']}, "
        f"placed {out['placed_per_step']}")
    if not args.no_cpu_baseline:
        out["bit_exact"], out["cpu_baseline"] = experts_vs_oracle(args, wl, run, eng, n_total, L)
    iso = {}

    def isolation():
        """The same routing with every non-local expert in the cache tier, then on the host."""
        everything = [i for i in range(wl.n_objects) if eng.lookup(1, i)[0] != 2]
        for name in ("all_cache", "all_host"):
            if name == "all_cache":
                st_all = eng.place(1, everything)
                assert (st_all == 0).all()
            else:
                eng.revoke(1, everything)
            torch.cuda.synchronize()
            eng.h.profile()
            s0 = eng.h.stats()
            a = time.perf_counter()
            for l in range(L):
                eng.h.fetch_experts(l, topk[(args.warmup, l)], staging, E, ptrs)
            torch.cuda.synchronize()
            dt = time.perf_counter() - a
            p, s1 = eng.h.profile(), eng.h.stats()
            n_c = int(s1.fetch[1].n_cache) - int(s0.fetch[1].n_cache)
            n_h = int(s1.fetch[1].n_host) - int(s0.fetch[1].n_host)
            if not p.hbm_launches:
                iso[name] = {"experts": n_c or n_h, "ms_per_layer": round(dt * 1e3 / L, 3)}
            elif name == "all_cache":
                g = 2 * n_c * chunk / (p.hbm_ms * 1e-3) / 1e9
                iso[name] |= {"kernel_ms_per_layer": round(p.hbm_ms / L, 3), "hbm_gbs_read_write": round(g, 1),
                              "frac_of_hbm_peak": round(g / HBM_PEAK_GBS, 4)}
            else:
                g = n_h * chunk / (p.host_ms * 1e-3) / 1e9
                iso[name] |= {"kernel_ms_per_layer": round(p.host_ms / L, 3), "pcie_gbs": round(g, 2)}
            log(f"[bench] isolation {name}: {iso[name]}")

    if not args.no_isolation:
        isolation()
        if not wl.lru_capacity:                          # back to the configured residency for the prefetch leg
            eng.place(1, [int(i) for i in wl.place_order])
    if args.prefetch and not wl.lru_capacity:
        out["prefetch"] = bench_prefetch(eng, wl, topk, staging, ptrs, L, E, sp.chunk_bytes, sec / (args.steps * L),
                                         range(args.warmup, n_total))
    eng.close()
    wl, eng, run = set_up(True)
    for t in range(args.warmup):
        step(t)
    torch.cuda.synchronize()
    eng.h.profile()
    f0 = eng.h.stats()
    for t in range(args.warmup, n_total):
        step(t)
    pr, f1 = eng.h.profile(), eng.h.stats()
    n_c, n_h = (int(getattr(f1.fetch[1], k)) - int(getattr(f0.fetch[1], k)) for k in ("n_cache", "n_host"))
    hbm_gbs = 2 * n_c * chunk / (pr.hbm_ms * 1e-3) / 1e9 if pr.hbm_ms > 0 and n_c else 0.0
    host_gbs = n_h * chunk / (pr.host_ms * 1e-3) / 1e9 if pr.host_ms > 0 and n_h else 0.0
    log(f"[bench] profiled: HBM tier {hbm_gbs:.0f} GB/s, host tier {host_gbs:.1f} GB/s")
    out["roofline"] = {"bound": "hbm", "kernel": "gather<64,1,false,false> (HBM-tier workgroups, whole experts)",
                       "achieved": round(hbm_gbs, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": round(hbm_gbs / HBM_PEAK_GBS, 4),
                       "traffic": None, "launches": int(pr.hbm_launches),
                       "note": "from a leg of the same steps in a profiled context, which launches the tiers apart"}
    out["host_tier"] = {"bound": "pcie", "kernel": "gather (host-tier workgroups)", "achieved": round(host_gbs, 2), "unit": "GB/s",
                        "launches": int(pr.host_launches)}
    if not args.no_isolation:
        isolation()
        out["isolation"] = iso
    eng.close()
    if embed:
        return out
    print(json.dumps(out), flush=True)


def bench_prefetch(eng, wl, topk, staging, ptrs, L, E, chunk, fetch_s_per_layer, steps):
    """Fetch-then-use on one stream against the prefetch ring (layer l+1 fetched while layer l is in use).  The stand-in
    for the FFN is a reader of the staging buffer (harvest_plain_copy into a sink), repeated so that one layer's use
    takes about 0.8 of one layer's fetch - the regime in which overlapping matters."""
    import torch
    from paper_2602_00328_amd import binding as B
    sink = torch.empty_like(staging)
    nbytes = staging.numel()

    def use(buf, passes):
        for _ in range(passes):
            B.plain_copy(sink, buf, nbytes)

    def timed(fn):
        torch.cuda.synchronize()
        a = time.perf_counter()
        fn()
        torch.cuda.synchronize()
        return time.perf_counter() - a

    one_pass = timed(lambda: use(staging, 8)) / 8
    passes = max(1, round(0.8 * fetch_s_per_layer / one_pass))
    work = [(t, l) for t in steps for l in range(L)]

    def use_only():
        for _ in work:
            use(staging, passes)

    def serial():
        for w in work:
            eng.h.fetch_experts(w[1], topk[w], staging, E, ptrs)
            use(staging, passes)

    pf = B.Prefetcher(eng.h, E)

    def pipelined():
        pf.issue(work[0][1], topk[work[0]])
        for i, w in enumerate(work):
            if i + 1 < len(work):
                pf.issue(work[i + 1][1], topk[work[i + 1]])
            buf, _ = pf.acquire()
            use(buf, passes)
            pf.release()

    pipelined()                                           # warm-up: scratch of the fetch stream
    n = len(work)
    t_use, t_serial, t_pipe = timed(use_only) / n, timed(serial) / n, timed(pipelined) / n
    pf.close()
    res = {"use": f"{passes} read passes over the staging buffer ({nbytes / 2**30:.2f} GiB each)",
           "fetch_only_ms_per_layer": round(fetch_s_per_layer * 1e3, 3), "use_only_ms_per_layer": round(t_use * 1e3, 3),
           "fetch_then_use_ms_per_layer": round(t_serial * 1e3, 3), "prefetch_ring_ms_per_layer": round(t_pipe * 1e3, 3),
           "ring_over_longer_leg": round(t_pipe / max(fetch_s_per_layer, t_use), 4)}
    log(f"[bench] prefetch: {res}")
    return res


def bench_latency(args):
    """The paper's two transfer-latency figures on this machine (Section 2.3 / Figure 3: copies the size of one expert,
    peer GPU against host; Section 5.4 / Figure 7: KV chunks of 100 ... 8 000 entries): the time of one fetch whose objects
    all sit in the cache tier against the same fetch after their revocation, when they come from the host.  Here the cache
    tier is HBM on the same GPU, so the ratio is HBM against PCIe, not NVLink against PCIe: context, not a target."""
    import numpy as np
    import torch
    from types import SimpleNamespace
    from paper_2602_00328_amd import binding as B
    dev = torch.device("cuda", 0)
    reps = max(5, args.steps // 10)

    def timed(fn):
        fn()
        torch.cuda.synchronize()
        ts = []
        for _ in range(reps):
            a = time.perf_counter()
            fn()
            torch.cuda.synchronize()
            ts.append(time.perf_counter() - a)
        return float(np.median(ts))

    out = {"experts": [], "kv": []}
    for name, mib in (("1 MiB", 1.0), ("4 MiB", 4.0), ("Qwen-MoE-shaped expert, 16.5 MiB", 16.5), ("64 MiB", 64.0),
                      ("Phi-3.5-MoE-shaped expert, 150 MiB", 150.0), ("Mixtral-8x7B-shaped expert (3 x 4096 x 14336 bf16), 336 MiB", 336.0)):
        chunk = int(mib * 2**20)
        E = 4
        h = B.Harvest(expert=B.ClassSpec(n_layers=1, n_planes=1, chunk_bytes=chunk, max_objects=E, n_host_slots=E,
                                         n_cache_slots=E, n_local_slots=0, n_experts=E))
        h.host_plane(B.EXPERT)[:] = np.random.default_rng(1).integers(0, 256, size=(1, E, 4096), dtype=np.uint8).repeat(chunk // 4096, axis=2)
        h.register(B.EXPERT, E, np.arange(E), B.HOST)
        assert (h.place(B.EXPERT, np.arange(E)) == 0).all()
        topk = torch.tensor([[2]], dtype=torch.int32, device=dev)
        staging = torch.zeros(chunk, dtype=torch.uint8, device=dev)
        ptrs = torch.zeros(E, dtype=torch.int64, device=dev)
        fetch = lambda: h.fetch_experts(0, topk, staging, 1, ptrs)
        t_cache = timed(fetch)
        from_cache = staging.clone()
        h.revoke(B.EXPERT, np.arange(E))
        t_host = timed(fetch)
        same = bool(torch.equal(from_cache, staging))
        out["experts"].append({"object": name, "bytes": chunk, "cache_tier_us": round(t_cache * 1e6, 1), "host_tier_us": round(t_host * 1e6, 1),
                               "speed_up": round(t_host / t_cache, 2), "same_bytes": same})
        log(f"[bench] one expert, {name}: cache tier {t_cache * 1e6:.1f} us, host {t_host * 1e6:.1f} us, x{t_host / t_cache:.1f}, same bytes {same}")
        h.close()
        del staging, from_cache
    chunk, n_max = 32768, 8000
    h = B.Harvest(kv=B.ClassSpec(n_layers=1, n_planes=2, chunk_bytes=chunk, max_objects=n_max, n_host_slots=n_max,
                                 n_cache_slots=n_max, n_local_slots=0), flags=B.FLAG_CACHE_PLANES_ADJACENT)
    rng = np.random.default_rng(2)
    for p in range(2):
        h.host_plane(B.KV, p)[:] = rng.integers(0, 256, size=(1, n_max, 64), dtype=np.uint8).repeat(chunk // 64, axis=2)
    h.register(B.KV, n_max, rng.permutation(n_max), B.HOST)
    dst = [torch.zeros(n_max * chunk, dtype=torch.uint8, device=dev) for _ in range(2)]
    order = rng.permutation(n_max).astype(np.int32)
    for n in (100, 500, 1000, 2000, 4000, 8000):
        assert (h.place(B.KV, np.arange(n_max)) == 0).all()
        d_table = torch.from_numpy(order[:n].reshape(1, n).copy()).to(dev)
        d_nb = torch.tensor([n], dtype=torch.int32, device=dev)
        d_sdb = torch.zeros(1, dtype=torch.int64, device=dev)
        fetch = lambda: h.fetch_kv(0, d_table, d_nb, dst[0], dst[1], d_sdb, n_max)
        t_cache = timed(fetch)
        from_cache = [t[:n * chunk].clone() for t in dst]
        h.revoke(B.KV, np.arange(n_max))
        t_host = timed(fetch)
        same = all(bool(torch.equal(a, t[:n * chunk])) for a, t in zip(from_cache, dst))
        out["kv"].append({"blocks": n, "bytes": 2 * n * chunk, "cache_tier_us": round(t_cache * 1e6, 1), "host_tier_us": round(t_host * 1e6, 1),
                          "speed_up": round(t_host / t_cache, 2), "same_bytes": same})
        log(f"[bench] {n} KV blocks of 2 x 32 KiB: cache tier {t_cache * 1e6:.1f} us, host {t_host * 1e6:.1f} us, x{t_host / t_cache:.1f}, same bytes {same}")
    h.close()
    print(json.dumps({"metric": "fetch latency of one request by object size, cache tier against host tier (call to completion, median of "
                                f"{reps})", "unit": "us", "n_gpus": 1, "data": "synthetic", "dtype": "u8",
                      "config": {"workload": "the paper's Figure 3 (expert-sized chunks) and Figure 7 (KV chunks of 100 ... 8000 entries) on one "
                                             "MI355X: cache tier = HBM on the same GPU, host tier = pinned DRAM over PCIe"},
                      "paper": "2 x H100, peer GPU over NVLink against host over PCIe 5: expert-sized chunks 7.5x ... 9.5x, KV chunks 3x ... 5.68x",
                      **out}), flush=True)


def bench_contention(args):
    """Who gets the PCIe link: a KV fetch that is bound by its host tier, repeated back to back on one stream, beside a
    placement of experts (host -> cache tier) on another, for several widths of the placement's copy kernel.  The paper
    puts the miss on the critical path, where its transfer contends with other traffic on the link (Section 2.2), and
    makes placement best effort (Section 3.1): the figures say what a fetch pays for a placement running beside it."""
    import numpy as np
    import torch
    import workloads as W
    from workloads import scenarios as S
    from workloads.hip_engine import HipEngine
    rows = []
    for wgs in (0, 4, 8, 16, 32, 64):
        wl = W.kv_decode(seed=30, n_layers=1, n_seq=2, min_len=20000, max_len=30000, n_steps=1)
        ex = W.expert_offload(seed=30, shape=W.ExpertShape(n_layers=1, n_experts=16, d_model=4096, d_ff=4096), n_local=0)
        eh = HipEngine(kv=S.kv_spec(wl, 0, 0), expert=S.expert_spec(ex), two_streams=True, pcie_wgs=wgs)
        try:
            rh, xh = S.KVRun(eh, wl), S.ExpertRun(eh, ex)
            eh.revoke(S.EXPERT, sorted(xh.live))                  # the whole expert cache tier is free
            ids = list(range(ex.n_objects))
            table, nb = rh.table_arrays()
            dev = eh.dev
            d_table, d_nb = torch.from_numpy(table).to(dev), torch.from_numpy(nb).to(dev)
            d_sdb = torch.from_numpy(rh.seq_dst_block.view(np.int64)).to(dev)
            dst = [torch.zeros(rh.cap * wl.shape.chunk_bytes, dtype=torch.uint8, device=dev) for _ in range(2)]
            ks, xs = eh.streams[S.KV], eh.streams[S.EXPERT]

            def fetch():
                a = time.perf_counter()
                with torch.cuda.stream(ks):
                    eh.h.fetch_kv(0, d_table, d_nb, dst[0], dst[1], d_sdb, rh.cap)
                ks.synchronize()
                return time.perf_counter() - a

            for _ in range(5):
                fetch()
            alone = float(np.median([fetch() for _ in range(20)]))
            want = [t.clone() for t in dst]
            counts, _, _ = eh.h.fetch_info(stream=ks, cls=S.KV)
            torch.cuda.synchronize()
            a = time.perf_counter()
            st = eh.place(S.EXPERT, ids)
            xs.synchronize()
            place_alone = time.perf_counter() - a
            n_placed = int((st == 0).sum())
            eh.revoke(S.EXPERT, ids)
            torch.cuda.synchronize()
            a = time.perf_counter()
            eh.place(S.EXPERT, ids)
            beside = []
            while not xs.query():
                beside.append(fetch())
            xs.synchronize()
            place_beside = time.perf_counter() - a
            same = all(bool(torch.equal(x, y)) for x, y in zip(want, dst))
            rows.append({"pcie_wgs": wgs or "default (12)", "fetch_alone_ms": round(alone * 1e3, 3),
                         "fetch_beside_placement_ms_median": round(float(np.median(beside)) * 1e3, 3),
                         "fetch_beside_placement_ms_max": round(float(np.max(beside)) * 1e3, 3), "fetches_beside": len(beside),
                         "placement_alone_ms": round(place_alone * 1e3, 2), "placement_beside_fetches_ms": round(place_beside * 1e3, 2),
                         "placement_bytes": n_placed * ex.shape.chunk_bytes, "fetch_host_tier_blocks": counts["n_host"],
                         "same_bytes": same})
            log(f"[bench] link contention, {rows[-1]}")
        finally:
            eh.close()
    print(json.dumps({"metric": "time of a PCIe-bound KV fetch alone and beside a placement on another stream, by the width of the "
                                "placement's copy kernel", "unit": "ms", "n_gpus": 1, "data": "synthetic", "dtype": "u8",
                      "config": {"workload": "2 sequences of 20K-30K tokens (Llama-3-8B-shaped blocks, 30 % of them on the host) fetched "
                                             "back to back on one stream; 16 experts of 96 MiB placed host -> cache tier on another"},
                      "rows": rows}), flush=True)


def bench_mixed(args, embed=False):
    """configs[4]: configs[1]'s KV decode on one stream and configs[2]'s expert fetch on another, both enqueued every step;
    at t = 10, 20, ... a seeded quarter of the live cache-tier allocations of each class is revoked with the step's fetches
    in flight (Section 3.2), at t = 5 mod 10 the revoked objects are placed again.  Timed: the two classes alone, then
    together; checked against the oracle at the end.  Both fetches are bound by the same PCIe link, so together they take
    about as long as one after the other - what the figure shows is that nothing else is lost."""
    import numpy as np
    import torch
    import workloads as W
    from workloads import scenarios as S
    from workloads.hip_engine import HipEngine
    steps = min(args.steps, 60)
    warm = min(args.warmup, 5)
    n_total = warm + 3 * steps
    layers_kv, layers_ex = min(args.layers, 8), 2
    t0 = time.time()
    wl = W.kv_decode(seed=args.seed, n_layers=layers_kv, n_steps=n_total, shape=W.KVShape(n_layers=layers_kv))
    ex = W.expert_offload(seed=args.seed, shape=W.ExpertShape(n_layers=layers_ex))
    sp = S.expert_spec(ex)
    eng = HipEngine(kv=S.kv_spec(wl), expert=sp, two_streams=True, poison=True, cache_planes_adjacent=True)
    run, xrun = S.KVRun(eng, wl), S.ExpertRun(eng, ex)
    dd = DeviceDecode(run, eng, wl, n_total)
    dev = eng.dev
    ks, xs = eng.streams[S.KV], eng.streams[S.EXPERT]
    E = ex.shape.n_experts
    staging = torch.empty(E * sp.chunk_bytes, dtype=torch.uint8, device=dev)
    ptrs = torch.zeros(E, dtype=torch.int64, device=dev)
    topk = {t: torch.from_numpy(ex.routing(t, t % layers_ex)).to(dev) for t in range(n_total)}
    torch.cuda.synchronize()
    log(f"[bench] kv_and_experts: KV {layers_kv} layers, experts {layers_ex} layers, set up in {time.time() - t0:.1f}s")

    def kv_step():
        with torch.cuda.stream(ks):
            dd.step()

    def ex_step(t):
        with torch.cuda.stream(xs):
            eng.h.fetch_experts(t % layers_ex, topk[t], staging, E, ptrs)

    def churn(t, kv, experts):
        if t % 10 == 0 and t > 0:
            if kv:
                run.revoke_quarter(t)
            if experts:
                xrun.revoke_quarter(t)
        if t % 10 == 5:
            if kv:
                run.replace_revoked()
            if experts:
                xrun.replace_revoked()

    def leg(t_first, n, kv, experts):
        torch.cuda.synchronize()
        s0 = eng.h.stats()
        a = time.perf_counter()
        for t in range(t_first, t_first + n):
            if kv:
                kv_step()
            if experts:
                ex_step(t)
            churn(t, kv, experts)
        torch.cuda.synchronize()
        sec = time.perf_counter() - a
        s1 = eng.h.stats()
        moved = 0
        for k, b in ((0, 2 * wl.shape.chunk_bytes), (1, sp.chunk_bytes)):
            served = sum(int(getattr(s1.fetch[k], f)) - int(getattr(s0.fetch[k], f)) for f in ("n_cache", "n_host"))
            moved += served * b
        return sec, moved, {"revoked": [int(s1.n_revoked[k] - s0.n_revoked[k]) for k in (0, 1)],
                            "placed": [int(s1.n_placed[k] - s0.n_placed[k]) for k in (0, 1)]}

    for t in range(warm):
        kv_step(); ex_step(t)
    t = warm
    # experts alone, KV alone (the decode state advances only in the legs that run the KV side), then both
    sec_x, moved_x, churn_x = leg(t, steps, False, True); t += steps
    sec_k, moved_k, churn_k = leg(t, steps, True, False); t += steps
    sec_b, moved_b, churn_b = leg(t, steps, True, True); t += steps
    log(f"[bench] {steps} steps: experts alone {sec_x / steps * 1e3:.2f} ms/step, KV alone {sec_k / steps * 1e3:.2f} ms/step, "
        f"together {sec_b / steps * 1e3:.2f} ms/step")

    bit_exact = None
    if not args.no_cpu_baseline:                              # the oracle goes through the same appends, revocations and placements
        from oracle.engine import OracleEngine
        layer = dd.first_layer(dd.t)
        wl1 = W.kv_decode(seed=args.seed, n_layers=layers_kv, n_steps=n_total, shape=W.KVShape(n_layers=layers_kv))
        eo = OracleEngine(kv=S.kv_spec(wl1), expert=sp, poison=True, kv_layers=[layer], threads=len(os.sched_getaffinity(0)))
        ro, xo = S.KVRun(eo, wl1), S.ExpertRun(eo, ex)
        kt = 0                                                # the KV side's own step count (DeviceDecode.t)
        for _ in range(warm):
            ro.append(kt); kt += 1
        tt = warm
        for kv, experts in ((False, True), (True, False), (True, True)):
            for _ in range(steps):
                if kv:
                    ro.append(kt); kt += 1
                if tt % 10 == 0 and tt > 0:
                    if kv:
                        ro.revoke_quarter(tt)
                    if experts:
                        xo.revoke_quarter(tt)
                if tt % 10 == 5:
                    if kv:
                        ro.replace_revoked()
                    if experts:
                        xo.replace_revoked()
                tt += 1
        assert kt == dd.t
        want = ro.fetch(layer)
        with torch.cuda.stream(ks):
            dd.fetch(layer)
        torch.cuda.synchronize()
        got_k, got_v = dd.dst[0].cpu().numpy(), dd.dst[1].cpu().numpy()
        counts, miss, _ = eng.h.fetch_info(stream=ks, miss_cap=dd.d_table.numel(), cls=S.KV)
        ok_kv = bool(np.array_equal(want[0], got_k) and np.array_equal(want[1], got_v) and counts == want[3]
                     and np.array_equal(np.sort(miss), want[2]))
        xw = xo.fetch(tt, tt % layers_ex)
        xg = xrun.fetch(tt, tt % layers_ex)
        ok_x = all((a is None and b is None) or (a is not None and b is not None and np.array_equal(a, b))
                   for a, b in zip(xw[0], xg[0])) and xw[4] == xg[4] and np.array_equal(xw[3], xg[3])
        bit_exact = bool(ok_kv and ok_x)
        log(f"[bench] after {n_total} steps vs oracle: KV {ok_kv}, experts {ok_x}")
        eo.close()
    out = {
        "metric": "fetch GB/s (read+write) and % of HBM/PCIe peak; objects/s; bit-exact vs oracle",
        "value": round(2 * moved_b / sec_b / 1e9, 2), "unit": "GB/s", "n_gpus": 1, "steps": steps, "warmup": warm,
        "ms_per_step": round(sec_b / steps * 1e3, 4), "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "u8", "data": "synthetic",
        "config": {"workload": "configs[4]: configs[1]'s KV decode fetch on one stream and configs[2]'s expert fetch (16 Phi-shaped "
                               "experts of 150 MiB per layer) on another, both every step; a quarter of each cache tier revoked every "
                               "10 steps with the fetches in flight, placed again 5 steps later; poisoning on",
                   "kv_layers_materialised": layers_kv, "expert_layers_materialised": layers_ex, "seed": args.seed},
        "bit_exact": bit_exact,
        "alone": {"kv_ms_per_step": round(sec_k / steps * 1e3, 4), "kv_gbs": round(2 * moved_k / sec_k / 1e9, 2),
                  "experts_ms_per_step": round(sec_x / steps * 1e3, 4), "experts_gbs": round(2 * moved_x / sec_x / 1e9, 2),
                  "churn": {"kv": churn_k, "experts": churn_x}},
        "together": {"ms_per_step": round(sec_b / steps * 1e3, 4), "churn": churn_b,
                     "over_sum_of_alone": round(sec_b / (sec_k + sec_x), 4),
                     "note": "both fetches and the placements are bound by the one PCIe link, so side by side cannot beat one "
                             "after the other; the three legs cover different steps, whose revocations and placements differ "
                             "somewhat (see churn): a ratio near 1 says that running side by side costs nothing on top"},
        "roofline": None, "cpu_baseline": None}
    eng.close()
    if embed:
        return out
    print(json.dumps(out), flush=True)


def no_nan(x):
    """JSON has no NaN: figures that were not measured (--no-profile) are reported as null."""
    if isinstance(x, dict):
        return {k: no_nan(v) for k, v in x.items()}
    if isinstance(x, list):
        return [no_nan(v) for v in x]
    return None if isinstance(x, float) and x != x else x


def main():
    args = parse()
    if args.gpus != 1:
        log(f"bench.py: this build runs on one GPU only (asked for --gpus {args.gpus}); the path has no collectives - "
            "objects are independent, so several GPUs would each run this same fetch over their own share.")
        sys.exit(2)
    import torch
    torch.cuda.set_device(0)
    if args.workload == "kv_tiny":
        return bench_tiny(args)
    if args.workload == "latency_by_size":
        return bench_latency(args)
    if args.workload == "link_contention":
        return bench_contention(args)
    if args.workload == "kv_and_experts":
        return bench_mixed(args)
    if args.workload != "kv_decode":
        return bench_experts(args)
    out = bench_kv(args, args.seed, full=True)
    if args.other_legs and not args.head_major and args.fetch_layers == 1:
        # Beside the benchmark line: the same configuration at another draw of the sequence lengths (seed 0 happens to draw
        # short ones), the two expert configurations with two layers materialised, the tiny configuration and the mixed
        # one - short runs, each checked against the oracle, so that one default run shows all five configurations and
        # every kernel at its real per-step shape.
        import copy
        extra = {}
        a2 = copy.copy(args)
        a2.steps, a2.warmup, a2.graph_steps, a2.no_isolation = min(args.steps, 40), 5, 0, True
        r = bench_kv(a2, args.seed + 1, full=False)
        extra["configs[1], seed %d" % (args.seed + 1)] = {
            k: r[k] for k in ("value", "unit", "ms_per_step", "objects_per_s", "bit_exact", "served")} | {
            "blocks_per_step": r["config"]["blocks_per_step"],
            "hbm_tier_gather_gbs": r["roofline"]["achieved"], "hbm_tier_gather_frac": r["roofline"]["frac"],
            "host_tier_gbs": r["host_tier"]["achieved"], "host_tier_frac": r["host_tier"]["frac"]}
        for wlname, key in (("experts_phi", "configs[2]"), ("experts_qwen", "configs[3]")):
            a3 = copy.copy(args)
            a3.workload, a3.layers, a3.steps, a3.warmup, a3.no_isolation, a3.prefetch = wlname, 2, 3, 1, True, False
            r = bench_experts(a3, embed=True)
            extra[key] = {k: r[k] for k in ("value", "unit", "ms_per_step", "objects_per_s", "bit_exact", "served_per_step",
                                            "placed_per_step", "cpu_baseline")} | {
                "layers_materialised": 2, "hbm_tier_gather_gbs": r["roofline"]["achieved"],
                "hbm_tier_gather_frac": r["roofline"]["frac"], "host_tier_gbs": r["host_tier"]["achieved"]}
        a4 = copy.copy(args)
        a4.steps, a4.warmup = 50, 10
        r = bench_tiny(a4, embed=True)
        extra["configs[0]"] = {k: r[k] for k in ("value", "unit", "ms_per_step", "objects_per_s", "bit_exact", "served", "latency")}
        a5 = copy.copy(args)
        a5.steps, a5.warmup = 30, 5
        r = bench_mixed(a5, embed=True)
        extra["configs[4]"] = {k: r[k] for k in ("value", "unit", "ms_per_step", "steps", "bit_exact", "alone", "together")}
        out["other_legs"] = extra
    print(json.dumps(no_nan(out)), flush=True)


def bench_kv(args, seed, full):
    """configs[1] at one seed.  full: every leg (calibration copies, graph replay, the oracle's speed, isolation points,
    write paths); otherwise the timed steps and the check against the oracle only.  Returns the result line as a dict."""
    import numpy as np
    import torch
    import workloads as W
    from workloads import scenarios as S
    from paper_2602_00328_amd import binding as B
    from workloads.hip_engine import HipEngine
    dev = torch.device("cuda", 0)
    n_total = args.warmup + args.steps + args.graph_steps
    kv_shape = W.KVShape(n_layers=args.layers, elt_bytes=args.kv_elt_bytes)
    wl = W.kv_decode(seed=seed, n_layers=args.layers, n_steps=n_total, shape=kv_shape, placement=args.placement)
    sh = wl.shape
    chunk = sh.chunk_bytes
    n_blocks0 = int(sum(len(t) for t in wl.tables))
    log(f"[bench] workload: {wl.n_seq} sequences, lengths {wl.seq_lens.tolist()}, {n_blocks0} blocks, "
        f"{args.layers} layers materialised, host pool {wl.n_objects * 2 * chunk * args.layers / 2**30:.1f} GiB")
    all_cache_slack = int(wl.n_objects - wl.resident.sum())
    n_cache_slots = int(wl.resident.sum()) + (0 if args.no_isolation else all_cache_slack)
    shared_bytes = n_cache_slots * (-(-(2 * chunk * args.layers) // 4096) * 4096) if args.shared_cache else 0

    def set_up(wl, profile):
        t0 = time.time()
        eng = HipEngine(kv=S.kv_spec(wl, cache_slack=0 if args.no_isolation else all_cache_slack, shared=args.shared_cache),
                        profile=profile, host_wgs=args.host_wgs, shared_cache_bytes=shared_bytes,
                        gather_threads=args.gather_threads, cache_planes_adjacent=args.cache_layout == "adjacent")
        run = S.KVRun(eng, wl)
        torch.cuda.synchronize()
        log(f"[bench] pools filled and {len(run.live)} blocks placed in {time.time() - t0:.1f}s")
        return eng, run, DeviceDecode(run, eng, wl, n_total, head_major=args.head_major, fetch_layers=args.fetch_layers,
                                      again=args.fetch_again)

    # Everything up to the tier times runs as callers run it.  A context with HARVEST_FLAG_PROFILE launches the two tiers of
    # a fetch apart, so that events can time them: that is a leg of its own, at the end, over the same steps.
    eng, run, dd = set_up(wl, False)

    # ---- calibration kernel of known size (for hardware byte counters) + achievable-copy ceiling ----
    cal_bytes = 2 << 30
    src = torch.empty(cal_bytes, dtype=torch.uint8, device=dev).random_(0, 256)
    dstc = torch.empty(cal_bytes, dtype=torch.uint8, device=dev)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    B.plain_copy(dstc, src, cal_bytes)
    torch.cuda.synchronize()
    ev[0].record()
    for _ in range(max(1, args.calibrate)):
        B.plain_copy(dstc, src, cal_bytes)
    ev[1].record()
    torch.cuda.synchronize()
    plain_gbs = 2 * cal_bytes * max(1, args.calibrate) / (ev[0].elapsed_time(ev[1]) * 1e-3) / 1e9
    # the two halves of a copy alone: what bounds any copy on this machine (2 / (1/read + 1/write))
    sink = torch.zeros(1, dtype=torch.int32, device=dev)
    rates = {}
    for name, fn in (("read", lambda: B.plain_read(src, cal_bytes, sink)), ("write", lambda: B.plain_write(dstc, cal_bytes, 0x5A5A5A5A))):
        fn()
        torch.cuda.synchronize()
        ev[0].record()
        for _ in range(max(1, args.calibrate)):
            fn()
        ev[1].record()
        torch.cuda.synchronize()
        rates[name] = cal_bytes * max(1, args.calibrate) / (ev[0].elapsed_time(ev[1]) * 1e-3) / 1e9
    copy_bound_gbs = 2.0 / (1.0 / rates["read"] + 1.0 / rates["write"])
    del src, dstc
    # ---- PCIe peak: 1 GiB pinned -> device DMA, median of 10 ----
    pin = torch.empty(1 << 30, dtype=torch.uint8, pin_memory=True)
    dbuf = torch.empty(1 << 30, dtype=torch.uint8, device=dev)
    ts = []
    for _ in range(11):
        torch.cuda.synchronize()
        a = time.perf_counter()
        dbuf.copy_(pin, non_blocking=True)
        torch.cuda.synchronize()
        ts.append(time.perf_counter() - a)
    pcie_peak_gbs = (1 << 30) / float(np.median(ts[1:])) / 1e9
    ts = []
    for _ in range(6):                                   # and device -> pinned host, for the write-back path
        torch.cuda.synchronize()
        a = time.perf_counter()
        pin.copy_(dbuf, non_blocking=True)
        torch.cuda.synchronize()
        ts.append(time.perf_counter() - a)
    d2h_peak_gbs = (1 << 30) / float(np.median(ts[1:])) / 1e9
    del pin, dbuf
    log(f"[bench] read only {rates['read']:.0f} GB/s, write only {rates['write']:.0f} GB/s -> no copy passes {copy_bound_gbs:.0f} GB/s")
    log(f"[bench] plain copy {plain_gbs:.0f} GB/s read+write; PCIe DMA peak {pcie_peak_gbs:.1f} GB/s to the device, "
        f"{d2h_peak_gbs:.1f} GB/s to the host")

    # ---- warm-up, then the timed region ----
    for _ in range(args.warmup):
        dd.step()
    torch.cuda.synchronize()
    c0 = kv_totals(eng.h.stats())
    torch.cuda.synchronize()
    t_start = time.perf_counter()
    for _ in range(args.steps):
        dd.step()
    torch.cuda.synchronize()
    t_end = time.perf_counter()
    c1 = kv_totals(eng.h.stats())
    d = {k: c1[k] - c0[k] for k in COUNT_KEYS}
    sec = t_end - t_start
    ms_per_step = sec * 1e3 / args.steps
    FL = args.fetch_layers                                  # requests are counted once per call, bytes move per layer
    payload = d["n_requests"] * 2 * chunk * FL              # bytes delivered into the working layout
    value = 2 * payload / sec / 1e9
    graph_replay = None
    if args.graph_steps:
        # ---- the same decode, continued, with every fetch replayed from a recorded graph ----
        dd.record_graphs()
        torch.cuda.synchronize()
        g0 = kv_totals(eng.h.stats())
        torch.cuda.synchronize()
        a = time.perf_counter()
        for _ in range(args.graph_steps):
            dd.step()
        torch.cuda.synchronize()
        gsec = time.perf_counter() - a
        g1 = kv_totals(eng.h.stats())
        dd.graphs = None
        g_payload = (g1["n_requests"] - g0["n_requests"]) * 2 * chunk
        graph_replay = {"steps": args.graph_steps, "ms_per_step": round(gsec * 1e3 / args.graph_steps, 4),
                        "value": round(2 * g_payload / gsec / 1e9, 2), "unit": "GB/s",
                        "note": "fetches replayed from HIP graphs recorded once per layer; appends, tail write-backs and "
                                "placements stay eager between the replays; included in the bit_exact check"}
        log(f"[bench] graph replay: {graph_replay['ms_per_step']:.3f} ms/step, {graph_replay['value']:.0f} GB/s")
    log(f"[bench] {args.steps} steps in {sec:.3f}s: {ms_per_step:.3f} ms/step, {value:.0f} GB/s read+write")

    # ---- bit-exactness of the timed configuration against the oracle, and the oracle's own speed ----
    bit_exact, cpu_baseline = None, None
    if not args.no_cpu_baseline:
        from oracle.engine import OracleEngine
        layer = dd.first_layer(dd.t)
        ncores = len(os.sched_getaffinity(0))
        wl1 = W.kv_decode(seed=seed, n_layers=args.layers, n_steps=n_total, shape=kv_shape, placement=args.placement)
        eo = OracleEngine(kv=S.kv_spec(wl1, cache_slack=0 if args.no_isolation else all_cache_slack), kv_layers=[layer],
                          threads=ncores)
        ro = S.KVRun(eo, wl1)
        for t in range(n_total):                         # bring the oracle to the same point of the decode
            ro.append(t)
        if args.head_major:
            table, nb = ro.table_arrays()
            final = [len(t) + len(f) for t, f in zip(wl1.tables, wl1.future_blocks)]
            want = eo.fetch_kv_head_major(layer, table, nb, ro.seq_dst_block, np.array(final, np.uint32), ro.cap,
                                          sh.n_kv_heads, sh.block_tokens)
        else:
            want = ro.fetch(layer)
        dd.fetch(layer)
        torch.cuda.synchronize()
        counts, miss, n_miss = eng.h.fetch_info(miss_cap=dd.d_table.numel())
        got_k, got_v = dd.dst[0].cpu().numpy(), dd.dst[1].cpu().numpy()
        bit_exact = bool(np.array_equal(want[0], got_k) and np.array_equal(want[1], got_v) and counts == want[3]
                         and np.array_equal(np.sort(miss), want[2]))
        log(f"[bench] layer {layer} after {n_total} steps vs oracle: bit_exact={bit_exact}")
        step_payload = want[3]["n_requests"] * 2 * chunk
        res = {}
        for threads in (1, ncores) if full else ():
            eo.threads = threads
            ro.fetch(layer)
            a = time.perf_counter()
            n = 0
            while n < 3 or time.perf_counter() - a < 6.0:
                ro.fetch(layer)
                n += 1
            res[threads] = 2 * step_payload * n / (time.perf_counter() - a) / 1e9
        if full:
            # what one core's memcpy moves on this host (read+write, as every figure here): the oracle's single-thread
            # figure is that, scattered
            big = np.ones(1 << 28, dtype=np.uint8)
            into = np.empty_like(big)
            np.copyto(into, big)
            a = time.perf_counter()
            for _ in range(8):
                np.copyto(into, big)
            memcpy_gbs = 2 * 8 * big.nbytes / (time.perf_counter() - a) / 1e9
            del big, into
            cpu_baseline = {"value": round(res[ncores], 2), "unit": "GB/s", "cores": ncores, "kind": "oracle",
                            "single_thread_value": round(res[1], 2), "host_memcpy_gbs_one_thread": round(memcpy_gbs, 2),
                            "sample": f"the same decode state, one layer's full fetch ({want[3]['n_requests']} blocks, "
                                      f"{step_payload / 2**30:.2f} GiB payload) repeated for >= 6 s per thread count, "
                                      "all tiers in host DRAM"}
            log(f"[bench] oracle: {res[1]:.1f} GB/s on 1 thread, {res[ncores]:.1f} GB/s on {ncores} threads")
        eo.close()

    # ---- isolation points: the same request list with every block in the cache tier, then every block on the host ----
    iso, write_paths = {}, {}
    if not args.no_isolation:
        closed = [b for s in range(wl.n_seq) for b in run.tables[s][:-1]]
        host_only = [b for b in closed if eng.lookup(0, b)[0] == 0]
        torch.cuda.synchronize()
        a = time.perf_counter()
        st = eng.place(0, host_only)
        torch.cuda.synchronize()
        dt = time.perf_counter() - a
        assert (st == 0).all()
        obj_bytes = 2 * chunk * sh.n_layers
        g = len(host_only) * obj_bytes / dt / 1e9
        write_paths["place"] = {"objects": len(host_only), "gbs_over_pcie": round(g, 2), "ms": round(dt * 1e3, 2),
                                "frac_of_pcie_peak": round(g / pcie_peak_gbs, 4)}
        # write-back of one layer of the longest sequence: fetch it, hand the same bytes back (state stays unchanged)
        s_long = int(np.argmax([len(t) for t in run.tables]))
        ev_ids = np.array(run.tables[s_long][:-1], dtype=np.uint32)
        dd.fetch(0)
        torch.cuda.synchronize()
        a = time.perf_counter()
        eng.h.evict(0, 0, ev_ids, dd.dst[0], dd.dst[1], int(run.seq_dst_block[s_long]) + np.arange(ev_ids.size),
                    run.cap, 0)
        torch.cuda.synchronize()
        dt = time.perf_counter() - a
        g = ev_ids.size * 2 * chunk / dt / 1e9
        write_paths["evict"] = {"objects": int(ev_ids.size), "gbs_to_host": round(g, 2), "ms": round(dt * 1e3, 2),
                                "frac_of_pcie_peak_to_host": round(g / d2h_peak_gbs, 4),
                                "note": "each block is written to its host slot and its cache slot"}
        log(f"[bench] write paths: {write_paths}")
        for name, n_it in (("all_cache", args.iso_steps), ("all_host", max(2, args.iso_steps // 4))):
            if name == "all_host":
                torch.cuda.synchronize()
                n_live = int(eng.h.stats().cache_slots_in_use[0])
                a = time.perf_counter()
                eng.revoke(0, closed)                    # nothing in flight: invalidate, publish, (empty) drain, free, callbacks
                dt = time.perf_counter() - a
                write_paths["revoke"] = {"objects": n_live, "ms": round(dt * 1e3, 3),
                                         "us_per_object": round(dt * 1e6 / max(1, n_live), 3),
                                         "note": "every cache-tier block revoked in one call, callbacks into Python included"}
                log(f"[bench] revoke: {write_paths['revoke']}")
            dd.fetch(0)
            torch.cuda.synchronize()
            counts, _, _ = eng.h.fetch_info()
            a = time.perf_counter()
            for i in range(n_it):
                dd.fetch(i % sh.n_layers)
            torch.cuda.synchronize()
            dt = time.perf_counter() - a
            iso[name] = {"ms_per_fetch": round(dt * 1e3 / n_it, 4), "objects_per_s": round(counts["n_requests"] / (dt / n_it))}
            if name == "all_cache":
                if args.graph_steps:                     # the short fetch is where launch overhead shows: replay it
                    dd.record_graphs()
                    torch.cuda.synchronize()
                    a = time.perf_counter()
                    for i in range(n_it):
                        dd.fetch(i % sh.n_layers)
                    torch.cuda.synchronize()
                    iso[name]["graph_replay_ms_per_fetch"] = round((time.perf_counter() - a) * 1e3 / n_it, 4)
                    dd.graphs = None
            log(f"[bench] isolation {name}: {iso[name]}")

    # ---- tier times: the same steps and the same isolation points in a profiled context ----
    eng.close()
    del eng, run, dd
    gc.collect()
    hbm_ms = host_ms = hbm_alg_bytes = host_bytes = hbm_gbs = host_gbs = float("nan")
    n_launches = [0, 0]
    if not args.no_profile:
        wl2 = W.kv_decode(seed=seed, n_layers=args.layers, n_steps=n_total, shape=kv_shape, placement=args.placement)
        eng, run, dd = set_up(wl2, True)
        for _ in range(args.warmup):
            dd.step()
        torch.cuda.synchronize()
        eng.h.profile()
        c0 = kv_totals(eng.h.stats())
        for _ in range(args.steps):
            dd.step()
        pr = eng.h.profile()
        c1 = kv_totals(eng.h.stats())
        p = {k: c1[k] - c0[k] for k in COUNT_KEYS}
        assert p == d
        n_launches = [int(pr.hbm_launches), int(pr.host_launches)]
        hbm_ms, host_ms = pr.hbm_ms / max(1, pr.hbm_launches), pr.host_ms / max(1, pr.host_launches)
        hbm_alg_bytes = 2 * (p["n_local"] + p["n_cache"]) * 2 * chunk * FL / max(1, pr.hbm_launches)     # read + write, per launch
        host_bytes = p["n_host"] * 2 * chunk * FL / max(1, pr.host_launches)
        hbm_gbs = hbm_alg_bytes / (hbm_ms * 1e-3) / 1e9
        host_gbs = host_bytes / (host_ms * 1e-3) / 1e9
        log(f"[bench] profiled: HBM-tier kernel {hbm_ms:.3f} ms ({hbm_gbs:.0f} GB/s), host-tier kernel {host_ms:.3f} ms "
            f"({host_gbs:.1f} GB/s)")
        if not args.no_isolation:
            closed = [b for s in range(wl2.n_seq) for b in run.tables[s][:-1]]
            assert (eng.place(0, [b for b in closed if eng.lookup(0, b)[0] == 0]) == 0).all()
            for name, n_it in (("all_cache", args.iso_steps), ("all_host", max(2, args.iso_steps // 4))):
                if name == "all_host":
                    eng.revoke(0, closed)
                dd.fetch(0)
                torch.cuda.synchronize()
                counts, _, _ = eng.h.fetch_info()
                eng.h.profile()
                for i in range(n_it):
                    dd.fetch(i % sh.n_layers)
                pr = eng.h.profile()
                if name == "all_cache":
                    k_ms, pay = pr.hbm_ms / pr.hbm_launches, counts["n_requests"] * 2 * chunk
                    g = 2 * pay / (k_ms * 1e-3) / 1e9
                    iso[name] |= {"kernel_ms": round(k_ms, 4), "hbm_gbs_read_write": round(g, 1),
                                  "frac_of_hbm_peak": round(g / HBM_PEAK_GBS, 4)}
                else:
                    k_ms = pr.host_ms / pr.host_launches
                    g = counts["n_host"] * 2 * chunk / (k_ms * 1e-3) / 1e9
                    iso[name] |= {"kernel_ms": round(k_ms, 4), "pcie_gbs": round(g, 2), "frac_of_pcie_peak": round(g / pcie_peak_gbs, 4)}
                log(f"[bench] profiled isolation {name}: {iso[name]}")
        eng.close()

    # Hardware byte counters cannot be read from inside this process: `traffic` is what two rocprofv3 --pmc passes over
    # this same command measured, kept with their command lines in the file named below - a stored figure of the
    # configuration (seed 0, default layout), not a measurement of this run; null when the file is not there or this run
    # is another configuration.
    traffic, traffic_source = None, None
    tf = os.path.join(ROOT, "profiles", "gather_hbm_kv_decode_pmc.txt")
    default_config = (seed == 0 and not args.head_major and not args.shared_cache and args.cache_layout == "adjacent"
                      and args.kv_elt_bytes == 2 and args.fetch_layers == 1 and args.placement == "shuffled")
    if os.path.exists(tf) and default_config:
        m = re.search(r"traffic_bytes_per_launch\s*=\s*([0-9.eE+]+)", open(tf).read())
        if m:
            traffic = float(m.group(1))
            traffic_source = ("profiles/gather_hbm_kv_decode_pmc.txt: rocprofv3 --pmc FETCH_SIZE and --pmc WRITE_SIZE passes over "
                              "this command, scaled by the same counters' reading of a 2 GiB plain copy; stored, not measured "
                              "by this run")
    alone = iso.get("all_cache", {}).get("hbm_gbs_read_write")        # none with --no-profile or --no-isolation

    out = {
        "metric": "fetch GB/s (read+write) and % of HBM/PCIe peak; objects/s; bit-exact vs oracle",
        "value": round(value, 2), "unit": "GB/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 4), "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "u8", "data": "synthetic",
        "config": {"workload": "configs[1]: long-context KV decode fetch, Llama-3-8B-shaped (32 layers, 8 KV heads x 128, "
                               "bf16, block 16), 4 sequences U[32K,128K] tokens, 70% HBM cache tier / 30% host, one layer "
                               "gathered per step, one token appended per step"
                               + ("" if args.kv_elt_bytes == 2 else f" -- VARIANT: {args.kv_elt_bytes}-byte KV elements, "
                                  f"{chunk // 1024} KiB blocks"),
                   "working_layout": "head-major" if args.head_major else "token-major",
                   "layers_per_fetch": args.fetch_layers, "placement": args.placement,
                   **({"fetch_again": True} if args.fetch_again else {}),
                   "cache_tier": "shared pool of best-fit segments" if args.shared_cache else
                                 ("equal-size slots, one pool [layer][slot][K|V][chunk]" if args.cache_layout == "adjacent"
                                  else "equal-size slots, a K pool and a V pool [layer][slot][chunk]"),
                   "seed": seed, "layers_materialised": args.layers, "blocks_per_step": d["n_requests"] // args.steps,
                   "blocks_per_step_mean_of_config": 20480,
                   "blocks_per_step_note": "4 lengths ~U[32K,128K] tokens: 8192..32768 blocks, mean 20480; this seed's draw is "
                                           f"{n_blocks0}",
                   "payload_bytes_per_step": payload // args.steps},
        "objects_per_s": round(d["n_requests"] * args.fetch_layers / sec),
        "bit_exact": bit_exact,
        "graph_replay": graph_replay,
        "served": {k: v // args.steps for k, v in d.items()},
        "roofline": {"bound": "hbm", "kernel": ("gather_hm<2>" if args.head_major else
                                                "gather<%d,2,%s,false>" % (args.gather_threads or 64, "true" if args.shared_cache or
                                                                     args.cache_layout == "adjacent" else "false"))
                                               + " (HBM-tier workgroups)", "achieved": round(hbm_gbs, 1),
                     "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": round(hbm_gbs / HBM_PEAK_GBS, 4), "traffic": traffic,
                     "traffic_source": traffic_source,
                     "launches": n_launches[0], "avg_launch_ms": round(hbm_ms, 5),
                     "algorithmic_bytes_per_launch": hbm_alg_bytes if math.isnan(hbm_alg_bytes) else round(hbm_alg_bytes), "plain_copy_gbs": round(plain_gbs, 1),
                     "frac_of_plain_copy": round(hbm_gbs / plain_gbs, 4),
                     "read_only_gbs": round(rates["read"], 1), "write_only_gbs": round(rates["write"], 1),
                     "copy_bound_gbs": round(copy_bound_gbs, 1),
                     "copy_bound_note": "a copy moves half its bytes each way over the same memory interface: 2 / (1/read_only + "
                                        "1/write_only), both measured in this run (one 16-byte access per thread; 1024-thread workgroups for the reads, 256 for the writes: one-wavefront workgroups with a single access each are bound by the dispatcher, not by memory)",
                     "note": "achieved / frac: a leg of the same steps in a profiled context, which launches the tiers apart so that "
                             "events can time them (the timed steps launch both in one kernel, unprofiled), the host tier "
                             "reading over PCIe beside it; alone: the same request list with every block in the cache tier "
                             "(isolation.all_cache, its kernel figures from that context too)",
                     "achieved_alone": alone, "frac_alone": round(alone / HBM_PEAK_GBS, 4) if alone else None},
        "host_tier": {"bound": "pcie", "kernel": ("gather_hm<2>" if args.head_major else "gather<64,2>") + " (host-tier workgroups, zero-copy over PCIe)",
                      "achieved": round(host_gbs, 2), "peak": round(pcie_peak_gbs, 2), "unit": "GB/s",
                      "frac": round(host_gbs / pcie_peak_gbs, 4), "launches": n_launches[1],
                      "avg_launch_ms": round(host_ms, 5), "bytes_per_launch": host_bytes if math.isnan(host_bytes) else round(host_bytes),
                      "peak_source": "1 GiB pinned->device hipMemcpyAsync, median of 10, same run"},
        "overlap": {"max_kernel_ms_over_step_ms": round(max(hbm_ms, host_ms) / ms_per_step, 4)},
        "isolation": iso,
        "write_paths": write_paths,
        "cpu_baseline": cpu_baseline,
    }
    return out


if __name__ == "__main__":
    main()
