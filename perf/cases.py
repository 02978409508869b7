"""The work a user of the library has it do, as cases that can be timed and checked.

Every case goes through the Python binding of libharvest.so, as an inference engine calls it: a context with its pools and
directory stands, the block tables, routing ids and destinations are on the device, and one pass is the calls of one step.
Shapes are those of the repository's workloads (``workloads/``, ``bench.py``): KV blocks of 16 tokens x 8 heads x 128 in
bf16 (32 KiB of K and of V) or fp8 (16 KiB), sequences from a few blocks to 128K tokens, experts of 3 x 2048 x 1408 bf16.
Payloads are bf16 normals (N(0, 1) for KV, N(0, 0.02) for weights), seen as 32-bit words: a fetch moves bytes, so every
output is compared exactly.

Tables of device addresses (the expert pointer table) are not among the outputs: they differ from process to process.
"""
import math

import numpy as np
import torch

from paper_2602_00328_amd import binding as B

KV, EXPERT = B.KV, B.EXPERT


def listed():
    return [
        # One request resumes with a handful of blocks offloaded: what a single small fetch costs (launch latency).
        kv("kv_few_blocks", n_seq=1, lo=8, hi=8, cached=1.0),
        # 16 sequences x 256 tokens, 60 % of the blocks in the cache tier, the rest on the host: a small fetch of both tiers.
        kv("kv_small_both_tiers", n_seq=16, lo=16, hi=16, cached=0.6),
        # A short context reloaded into every layer of the model in one call.
        kv("kv_all_layers", entry="layers", n_seq=1, lo=16, hi=16, layers=32, cached=1.0),
        # Continuous batching: 24 sequences of 512 to 8K tokens in a padded block table, walked layer by layer; everything is
        # in the cache tier (the setting the cache is there for).
        kv("kv_ragged_batch", entry="again", n_seq=24, lo=32, hi=512, layers=2, cached=1.0, tails=True),
        # A smaller batch into a head-major working layout (each head's tokens in one run).
        kv("kv_head_major", entry="head_major", n_seq=8, lo=64, hi=768, cached=1.0, tails=True),
        # fp8 KV cache (16 KiB blocks) through the entry point that allocates nothing, with its counters and miss list.
        kv("kv_static_fp8", entry="static", n_seq=7, lo=37, hi=411, elt_bytes=1, cached=0.97),
        # Long-context decode, 4 sequences of 32K to 128K tokens, all blocks in the cache tier: bound by HBM.
        kv("kv_long_cached", n_seq=4, lo=2048, hi=4608, cached=1.0, tails=True, adjacent=True),
        # The same with 30 % of the blocks on the host: bound by the PCIe link.
        kv("kv_long_both_tiers", n_seq=4, lo=2048, hi=4608, cached=0.7, tails=True, adjacent=True),
        # MoE decode of a few tokens: the routed experts of one layer from the cache tier.
        experts("experts_decode", tokens=4, cached=1.0),
        # MoE prefill: every expert is routed; the cache tier holds 40 %, two are local, the rest comes from the host.
        experts("experts_prefill", tokens=2048, cached=0.4, n_local=2),
        # Blocks that a step has fetched are put into the cache tier from the working buffers, and revoked again when the
        # owner of the memory wants it back.
        move("place_and_revoke", entry="place", n=64, layers=32),
        # Blocks that have filled up are written through to the host and to their cache slots, all layers.
        move("write_back", entry="evict", n=8, layers=32, cached=0.5),
    ]


def draw(rng):
    """One more case of the listed kinds; the payload stays below the largest listed case's and so does the time on the link."""
    kind = rng.choice(["kv", "kv", "kv", "experts", "move"])
    if kind == "kv":
        entry = rng.choice(["fetch", "fetch", "again", "layers", "head_major", "static"])
        elt = rng.choice([2, 2, 1])
        layers = log_int(rng, 2, 32) if entry == "layers" else (2 if entry == "again" else 1)
        most = 8192 * 2 // elt // layers                             # blocks
        blocks = log_int(rng, 1, most)
        n_seq = log_int(rng, 1, max(1, min(64, blocks)))
        hi = max(1, math.ceil(2 * blocks / (n_seq + 1)) if n_seq > 1 else blocks)
        lo = log_int(rng, 1, hi)
        if n_seq > 1 and n_seq * (lo + hi) // 2 > blocks:
            lo = max(1, 2 * blocks // n_seq - hi)
        cached = rng.choice([1.0, 1.0, 1.0, 0.97, 0.85, 0.7, 0.6])
        return kv(None, entry=entry, n_seq=n_seq, lo=min(lo, hi), hi=hi, layers=layers, cached=cached, elt_bytes=elt,
                  tails=rng.random() < 0.5, adjacent=rng.random() < 0.5)
    if kind == "experts":
        tokens = log_int(rng, 1, 2048)
        return experts(None, tokens=tokens, top_k=rng.choice([2, 4]), n_experts=rng.choice([16, 60, 64, 128]) if tokens < 8 else rng.choice([16, 32, 60]),
                       d_model=rng.choice([1024, 2048]), d_ff=rng.choice([704, 768, 1408]),
                       cached=rng.choice([1.0, 1.0, 0.7, 0.45]), n_local=rng.choice([0, 0, 2]))
    if rng.random() < 0.5:
        layers = rng.choice([1, 8, 32])
        return move(None, entry="place", n=log_int(rng, 1, 2048 // layers), layers=layers, elt_bytes=rng.choice([1, 2]))
    layers = rng.choice([1, 8, 32])
    return move(None, entry="evict", n=log_int(rng, 1, 512 // layers), layers=layers, elt_bytes=rng.choice([1, 2]),
                cached=rng.choice([0.0, 0.5, 1.0]))


def prepare(case, seed):
    return {"kv": prepare_kv, "experts": prepare_experts, "move": prepare_move}[case["kind"]](case, seed)


def run(state):
    return state["run"]()


def work(case):
    """Each byte fetched, placed or written back is read once and written once to each place that it goes to."""
    if case["kind"] == "kv":
        n = sum(lengths(case))
        return {"bytes": 2 * n * 2 * kv_chunk(case) * case["layers"], "flops": 0}
    if case["kind"] == "experts":
        routed = np.unique(routed_ranks(case))
        return {"bytes": 2 * int((routed >= case["n_local"]).sum()) * expert_chunk(case), "flops": 0}
    copies = 2.0 if case["entry"] == "place" else 2.0 + round(case["cached"] * case["n"]) / case["n"]
    return {"bytes": copies * case["n"] * 2 * kv_chunk(case) * case["layers"], "flops": 0}


def tolerance(case):
    return "exact"


def exact(case, seed):
    """What run() returns, from the inputs alone: indexing, no library."""
    if case["kind"] == "kv":
        return exact_kv(case, seed)
    if case["kind"] == "experts":
        return exact_experts(case, seed)
    return exact_move(case, seed)


# ---- cases ----------------------------------------------------------------------------------------------------------

def kv(name, entry="fetch", n_seq=1, lo=1, hi=1, layers=1, cached=1.0, elt_bytes=2, tails=False, adjacent=False):
    """n_seq sequences of lo to hi blocks; `cached` of the closed blocks in the cache tier, the others on the host; with
    `tails` the last block of each sequence is local; `adjacent`: K and V of a cached block side by side."""
    c = dict(kind="kv", entry=entry, n_seq=n_seq, lo=lo, hi=hi, layers=layers, cached=cached, elt_bytes=elt_bytes,
             tails=tails, adjacent=adjacent)
    return dict(c, name=name) if name else c


def experts(name, tokens=1, top_k=4, n_experts=60, d_model=2048, d_ff=1408, cached=1.0, n_local=0):
    """One layer's routed experts; by popularity the first n_local are local, then `cached` of the others in the cache tier."""
    c = dict(kind="experts", tokens=tokens, top_k=top_k, n_experts=n_experts, d_model=d_model, d_ff=d_ff, cached=cached,
             n_local=n_local)
    return dict(c, name=name) if name else c


def move(name, entry="place", n=1, layers=1, elt_bytes=2, cached=0.0):
    c = dict(kind="move", entry=entry, n=n, layers=layers, elt_bytes=elt_bytes, cached=cached)
    return dict(c, name=name) if name else c


def log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


BLOCK_TOKENS, HEADS, HEAD_DIM = 16, 8, 128


def kv_chunk(case):
    return BLOCK_TOKENS * HEADS * HEAD_DIM * case["elt_bytes"]


def expert_chunk(case):
    return 3 * case["d_model"] * case["d_ff"] * 2


def lengths(case):
    """Blocks per sequence, spread over [lo, hi]: the longest is hi.  They belong to the case, not to the seed."""
    n, lo, hi = case["n_seq"], case["lo"], case["hi"]
    return [hi if i == n - 1 else lo + int((hi - lo + 1) * ((i + 1) * 0.6180339887 % 1.0)) for i in range(n)]


def routed_ranks(case):
    """Routing in ranks of popularity [tokens][top_k], Zipf(1): which ranks are hit belongs to the case."""
    g = np.random.RandomState(7)
    e = case["n_experts"]
    keys = -np.log(g.random_sample((case["tokens"], e))) * np.arange(1, e + 1)      # exponential races: k distinct of each row
    return np.argsort(keys, axis=1)[:, :case["top_k"]]


def generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def normals(shape_bytes, scale, gen):
    """bf16 normals as bytes, of the given shape (last axis in bytes)."""
    t = torch.randn((*shape_bytes[:-1], shape_bytes[-1] // 2), dtype=torch.bfloat16, device="cuda", generator=gen)
    if scale != 1.0:
        t.mul_(scale)
    return t.view(torch.uint8)


def words(t):
    return t.view(torch.int32)


def fill_host(h, cls, host_slots, planes):
    """planes[p]: [layers][objects][chunk] on the device -> the pinned host pool, object i in slot host_slots[i]."""
    to = torch.from_numpy(np.argsort(host_slots)).cuda()             # slot -> object
    for p, x in enumerate(planes):
        pool = torch.from_numpy(h.host_plane(cls, p))
        for layer in range(x.shape[0]):
            pool[layer].copy_(x[layer].index_select(0, to))


# ---- KV fetches -----------------------------------------------------------------------------------------------------

def kv_inputs(case, seed):
    """Closed blocks are objects 0..C-1 in a random order over the tables, tails C..; `order`: the cached ones as placed."""
    g = np.random.RandomState(seed % (1 << 31))
    n = lengths(case)
    tails = case["n_seq"] if case["tails"] else 0
    closed = sum(n) - tails
    perm = g.permutation(closed)
    width = case["hi"]
    table = np.full((case["n_seq"], width), -1, dtype=np.int32)
    at = 0
    for s, k in enumerate(n):
        body = k - (1 if tails else 0)
        table[s, :body] = perm[at:at + body]
        at += body
        if tails:
            table[s, body] = closed + s
    order = g.permutation(closed)[:int(round(case["cached"] * closed))]
    total = closed + tails
    host_slots = g.permutation(total).astype(np.int64)
    gen = generator(seed)
    planes = [normals((case["layers"], total, kv_chunk(case)), 1.0, gen) for _ in range(2)]
    return n, closed, table, order, host_slots, planes


def prepare_kv(case, seed):
    n, closed, table, order, host_slots, planes = kv_inputs(case, seed)
    tails, layers, chunk = sum(n) - closed, case["layers"], kv_chunk(case)
    spec = B.ClassSpec(n_layers=layers, n_planes=2, chunk_bytes=chunk, max_objects=sum(n), n_host_slots=sum(n),
                       n_cache_slots=max(1, len(order)), n_local_slots=tails)
    h = B.Harvest(kv=spec, flags=B.FLAG_CACHE_PLANES_ADJACENT if case["adjacent"] else 0)
    fill_host(h, KV, host_slots, planes)
    h.register(KV, closed, host_slots[:closed])
    if tails:
        h.register(KV, tails, host_slots[closed:], tier=B.LOCAL)
        for p in range(2):
            h.dev_plane(KV, B.LOCAL, p).copy_(planes[p][:, closed:])
    if len(order):
        h.place(KV, order)
    del planes
    cap = sum(n)
    head_major = case["entry"] == "head_major"
    s = {
        "h": h,
        "table": torch.from_numpy(table).cuda(),
        "n_blocks": torch.tensor(n, dtype=torch.int32, device="cuda"),
        "seq_dst": torch.tensor(np.cumsum([0] + n[:-1]), dtype=torch.int64, device="cuda"),
        "k": torch.zeros(layers * cap * chunk, dtype=torch.uint8, device="cuda"),
        "v": torch.zeros(layers * cap * chunk, dtype=torch.uint8, device="cuda"),
    }
    out = [words(s["k"]), words(s["v"])]
    stride = cap * chunk

    def fetch(table):
        h.fetch_kv(0, table, s["n_blocks"], s["k"], s["v"], s["seq_dst"], cap)
        return out

    def again(table):                       # the block table of a step serves every layer
        k, v = s["k"].data_ptr(), s["v"].data_ptr()
        h.fetch_kv(0, table, s["n_blocks"], k, v, s["seq_dst"], cap)
        for layer in range(1, layers):
            h.fetch_kv_again(layer, k + layer * stride, v + layer * stride)
        return out

    def all_layers(table):
        h.fetch_kv_layers(0, layers, table, s["n_blocks"], s["k"], s["v"], stride, s["seq_dst"], cap)
        return out

    if head_major:
        caps = torch.tensor(n, dtype=torch.int32, device="cuda")

    def to_head_major(table):
        h.fetch_kv_head_major(0, table, s["n_blocks"], s["k"], s["v"], s["seq_dst"], caps, cap, HEADS, BLOCK_TOKENS)
        return out

    info = torch.zeros(8, dtype=torch.int32, device="cuda")
    miss = torch.zeros(table.size, dtype=torch.int32, device="cuda")

    def static(table):
        h.fetch_kv_static(0, table, s["n_blocks"], s["k"], s["v"], s["seq_dst"], cap, info, miss)
        return [*out, info, miss]

    call = {"fetch": fetch, "again": again, "layers": all_layers, "head_major": to_head_major, "static": static}[case["entry"]]
    # The context has served an earlier step, with another table, before this one.
    earlier = s["table"].clone()
    earlier[earlier >= 0] = (earlier[earlier >= 0] + 1) % sum(n)
    call(earlier)
    s["k"].zero_(), s["v"].zero_(), info.zero_(), miss.zero_()
    torch.cuda.synchronize()
    s["run"] = lambda: call(s["table"])
    return s


def exact_kv(case, seed):
    n, closed, table, order, _, planes = kv_inputs(case, seed)
    flat = np.concatenate([table[i, :k] for i, k in enumerate(n)])
    at = torch.from_numpy(flat.astype(np.int64)).cuda()
    out = []
    for x in planes:
        y = x.index_select(1, at)                                    # [layers][blocks][chunk]
        if case["entry"] == "head_major":                            # per sequence [head][token][head bytes]
            parts, first = [], 0
            for k in n:
                z = y[0, first:first + k].reshape(k * BLOCK_TOKENS, HEADS, -1)
                parts.append(z.transpose(0, 1).reshape(-1))
                first += k
            y = torch.cat(parts)
        out.append(words(y.reshape(-1).contiguous()))
    if case["entry"] != "static":
        return out
    cached = np.zeros(sum(n), dtype=bool)
    cached[order] = True
    local = np.zeros(sum(n), dtype=bool)
    local[closed:] = True
    cells = np.flatnonzero(table.reshape(-1) >= 0)
    missed = cells[~(cached | local)[table.reshape(-1)[cells]]]
    miss = np.zeros(table.size, dtype=np.int32)
    miss[:len(missed)] = missed
    info = np.array([len(flat), local[flat].sum(), cached[flat].sum(), len(missed), 0, 0, len(missed), 0], dtype=np.int32)
    return [*out, torch.from_numpy(info), torch.from_numpy(miss)]


# ---- expert fetches -------------------------------------------------------------------------------------------------

def expert_inputs(case, seed):
    g = np.random.RandomState(seed % (1 << 31))
    e = case["n_experts"]
    expert_of_rank = g.permutation(e).astype(np.int32)
    topk = expert_of_rank[routed_ranks(case)]
    host_slots = g.permutation(e).astype(np.int64)
    weights = normals((1, e, expert_chunk(case)), 0.02, generator(seed))
    return expert_of_rank, topk, host_slots, weights


def prepare_experts(case, seed):
    expert_of_rank, topk, host_slots, weights = expert_inputs(case, seed)
    e, chunk, n_local = case["n_experts"], expert_chunk(case), case["n_local"]
    cached = expert_of_rank[n_local:n_local + int(case["cached"] * (e - n_local))]
    local = np.isin(np.arange(e), expert_of_rank[:n_local])
    h = B.Harvest(expert=B.ClassSpec(n_layers=1, n_planes=1, chunk_bytes=chunk, max_objects=e, n_host_slots=e,
                                     n_cache_slots=max(1, len(cached)), n_local_slots=n_local, n_experts=e))
    fill_host(h, EXPERT, host_slots, [weights])
    slot = 0
    for i in range(e):                       # object numbers are expert numbers: registered one by one, by tier
        h.register(EXPERT, 1, host_slots[i:i + 1], tier=B.LOCAL if local[i] else B.HOST)
        if local[i]:
            h.dev_plane(EXPERT, B.LOCAL, 0)[0, slot].copy_(weights[0, i])
            slot += 1
    h.place(EXPERT, cached)
    del weights
    staging = torch.zeros(e * chunk, dtype=torch.uint8, device="cuda")
    pointers = torch.zeros(e, dtype=torch.int64, device="cuda")
    d_topk = torch.from_numpy(np.ascontiguousarray(topk)).cuda()
    out = [words(staging)]

    def call(ids):
        h.fetch_experts(0, ids, staging, e, pointers)
        return out

    call((d_topk + 1) % e)                   # an earlier step's routing
    staging.zero_()
    torch.cuda.synchronize()
    return {"h": h, "run": lambda: call(d_topk), "keep": (pointers, d_topk)}


def exact_experts(case, seed):
    expert_of_rank, topk, _, weights = expert_inputs(case, seed)
    local = set(expert_of_rank[:case["n_local"]].tolist())
    staged = [i for i in np.unique(topk).tolist() if i not in local]
    staging = torch.zeros((case["n_experts"], expert_chunk(case)), dtype=torch.uint8, device="cuda")
    staging[:len(staged)] = weights[0].index_select(0, torch.tensor(staged, device="cuda", dtype=torch.int64))
    return [words(staging.reshape(-1))]


# ---- placement, revocation, write-back ------------------------------------------------------------------------------

def move_inputs(case, seed):
    """n blocks in the library and, for both planes, the caller's working buffers [layers][n + 3][chunk] that hold block i
    (write-back: its new contents) at src_block[i]."""
    g = np.random.RandomState(seed % (1 << 31))
    n = case["n"]
    host_slots = g.permutation(n).astype(np.int64)
    ids = g.permutation(n).astype(np.uint32)
    src_block = g.permutation(n + 3)[:n].astype(np.uint64)
    gen = generator(seed)
    src = [normals((case["layers"], n + 3, kv_chunk(case)), 1.0, gen) for _ in range(2)]
    return host_slots, ids, src_block, src


def prepare_move(case, seed):
    host_slots, ids, src_block, src = move_inputs(case, seed)
    n, layers, chunk = case["n"], case["layers"], kv_chunk(case)
    h = B.Harvest(kv=B.ClassSpec(n_layers=layers, n_planes=2, chunk_bytes=chunk, max_objects=n, n_host_slots=n,
                                 n_cache_slots=n, n_local_slots=0))
    h.register(KV, n, host_slots)
    for i in range(n):                       # this program has nothing to do when a block is revoked
        h.register_cb(KV, i, enabled=False)
    k, v = src
    cache = [h.dev_plane(KV, B.CACHE, p) for p in range(2)]
    if case["entry"] == "place":
        out = [words(c) for c in cache]

        def call():
            h.place_from(KV, ids, k, v, src_block, n + 3)
            h.revoke(KV, ids)
            return out
    else:
        n_cached = int(round(case["cached"] * n))
        h.place(KV, ids[:n_cached])
        out = [words(c[:, :max(1, n_cached)]) for c in cache] + [h.host_plane(KV, p).view(np.int32) for p in range(2)]

        def call():
            h.evict(KV, -1, ids, k, v, src_block, n + 3)
            return out

    call()                                   # an earlier step's move; then the pools are as they were
    torch.cuda.synchronize()
    for p in range(2):
        cache[p].zero_()
        h.host_plane(KV, p)[:] = 0
    torch.cuda.synchronize()
    return {"h": h, "run": call, "keep": (src, ids, src_block)}


def exact_move(case, seed):
    host_slots, ids, src_block, src = move_inputs(case, seed)
    n, layers, chunk = case["n"], case["layers"], kv_chunk(case)
    order = torch.from_numpy(src_block.astype(np.int64)).cuda()
    moved = [x.index_select(1, order) for x in src]                  # [layers][i][chunk], i as in ids
    if case["entry"] == "place":                                     # slots are handed out in the order of the call
        return [words(x) for x in moved]
    n_cached = int(round(case["cached"] * n))
    cache = [x[:, :n_cached] if n_cached else torch.zeros((layers, 1, chunk), dtype=torch.uint8, device="cuda") for x in moved]
    where = torch.from_numpy(host_slots[ids]).cuda()                 # host slot of block ids[i]
    host = []
    for x in moved:
        y = torch.zeros((layers, n, chunk), dtype=torch.uint8, device="cuda")
        y[:, where] = x
        host.append(words(y))
    return [words(c.contiguous()) for c in cache] + host
