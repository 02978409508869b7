// fetch_kv_small on a CPU, with a directory that changes while it runs.  A workgroup's lanes are fibers that meet at barriers and
// ballots; workgroups run one after the other, which is one of the orders a GPU may take, and each sees the versions of the
// directory at barriers of its own (`when`), which is what workgroups that run at the same time and at different speeds see.
#include <hip/hip_runtime.h>
#include "kernels.h"

#include <ucontext.h>
#include <cstddef>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <vector>

dim3 threadIdx, blockIdx, gridDim;
const char *kernel_arguments;
uint32_t __shfl_xor(uint32_t, int) { abort(); }
void __threadfence_system() {}

namespace {
enum State { READY, AT_BALLOT, AT_BARRIER, DONE };          // (a lane that reads another's register meets the others as at a ballot)
struct Lane { ucontext_t ctx; State state; bool pred; uint32_t value; uint64_t mask; std::vector<char> stack; };
std::vector<Lane> g_lanes(256);
ucontext_t g_scheduler;
uint32_t g_current = 0;
bool g_fibers = false;
std::function<void()> g_kernel;

void wait(State s)
{
    if (!g_fibers) { fprintf(stderr, "a tile workgroup met a barrier\n"); abort(); }
    Lane &l = g_lanes[g_current];
    const dim3 me = threadIdx;
    l.state = s;
    swapcontext(&l.ctx, &g_scheduler);
    threadIdx = me;
}
void lane_main()
{
    g_kernel();
    g_lanes[g_current].state = DONE;
    swapcontext(&g_lanes[g_current].ctx, &g_scheduler);
}
// Runs the workgroup blockIdx of n threads; at_barrier(k) is called when all have met for the k-th time, and with 0 before they start.
// ballots: the ballots of any of its wavefronts count as well.
void run_workgroup(uint32_t n, const std::function<void(uint32_t)> &at_barrier, bool ballots = false)
{
    g_fibers = true;
    for (uint32_t i = 0; i < n; ++i) {
        Lane &l = g_lanes[i];
        l.stack.resize(128 << 10);
        getcontext(&l.ctx);
        l.ctx.uc_stack.ss_sp = l.stack.data();
        l.ctx.uc_stack.ss_size = l.stack.size();
        l.ctx.uc_link = nullptr;
        makecontext(&l.ctx, lane_main, 0);
        l.state = READY;
    }
    uint32_t barriers = 0;
    at_barrier(0);
    for (;;) {
        bool progress = false;
        for (uint32_t i = 0; i < n; ++i)
            if (g_lanes[i].state == READY) {
                progress = true;
                g_current = i;
                threadIdx = { i, 0, 0 };
                swapcontext(&g_scheduler, &g_lanes[i].ctx);
            }
        uint32_t done = 0, met = 0;
        for (uint32_t w = 0; w < n; w += 64) {
            uint64_t mask = 0;
            uint32_t there = 0;
            for (uint32_t i = w; i < w + 64; ++i) {
                const Lane &l = g_lanes[i];
                if (l.state == AT_BALLOT) { there++; mask |= (uint64_t)l.pred << (i - w); }
                done += l.state == DONE;
                met += l.state == AT_BARRIER;
            }
            if (there == 64) {
                for (uint32_t i = w; i < w + 64; ++i) { g_lanes[i].mask = mask; g_lanes[i].state = READY; progress = true; }
                if (ballots) at_barrier(++barriers);
            }
        }
        if (done == n) return;
        if (met && met + done == n) {
            at_barrier(++barriers);
            for (uint32_t i = 0; i < n; ++i) if (g_lanes[i].state == AT_BARRIER) g_lanes[i].state = READY;
            progress = true;
        }
        if (!progress) { fprintf(stderr, "lanes wait for each other\n"); abort(); }
    }
}
}  // namespace

void __syncthreads() { wait(AT_BARRIER); }
uint64_t __ballot(bool pred)
{
    g_lanes[g_current].pred = pred;
    wait(AT_BALLOT);
    return g_lanes[g_current].mask;
}

uint32_t read_lane(uint32_t x, uint32_t k)
{
    g_lanes[g_current].value = x;
    wait(AT_BALLOT);                                     // all have said theirs
    const uint32_t got = g_lanes[(g_current & ~63u) + k].value;
    wait(AT_BALLOT);                                     // all have read it
    return got;
}

uint32_t __shfl_up(uint32_t x, int o)
{
    g_lanes[g_current].value = x;
    wait(AT_BALLOT);
    const uint32_t got = (g_current & 63u) >= (uint32_t)o ? g_lanes[g_current - o].value : x;
    wait(AT_BALLOT);
    return got;
}

extern "C" {
// The entries idx[0 .. n) of the host's list, one after the other, by one wavefront: counts[n_seg] of its segments, recs[n_seg][seg_cells].
int host_list(const uint32_t *counts, uint32_t n_seg, uint32_t seg_cells, const hv::Rec *recs, const uint32_t *idx, uint32_t n, hv::Rec *out)
{
    using namespace hv;
    GatherRest rest{};
    rest.host_recs = recs; rest.counts = counts; rest.n_seg = n_seg; rest.seg_cells = seg_cells;
    uint32_t total = 0;
    g_kernel = [&] {
        HostList list(*(k_GatherRest *)(const __attribute__((address_space(4))) char *)(const char *)&rest);
        if (threadIdx.x == 0) total = list.sums.total;
        for (uint32_t i = 0; i < n; ++i) {
            const Rec x = list[idx[i]];
            if (threadIdx.x == 0 || (x.src != out[i].src || x.dst != out[i].dst)) out[i] = x;      // (lane 0 runs first: another's answer would show)
        }
    };
    run_workgroup(64, [](uint32_t) {});
    return (int)total;
}

struct Fetch {
    uint32_t n_planes, nthr, head_major, n_layers, n_objects, n_seq, max_blocks, n_host, lg_groups, seen, n_versions, n_heads, block_tokens, n_slots;
    uint32_t unrolled, pad;                      // two loads a thread in the tiles' workgroups
    uint64_t chunk_bytes, dst_cap, dst_step;
    uint64_t pool[3][2], dst[2];                 // [tier][plane]: pools [layer][slot][chunk]; destinations [layer][dst_cap][chunk]
    const int32_t *table, *n_blocks;
    const uint64_t *seq_dst;
    const uint32_t *seq_cap;
    const uint64_t *versions;                    // [n_versions][n_objects]: directories, from the one that `seen` stands for on
    const uint32_t *when;                        // [head or tile workgroup][n_versions - 1]: at which barrier each next one is seen
    uint32_t *cnt, *miss;
};

// Workgroups in the order of `when`: n_host that read the host, the one with the books, the tiles (x, then plane, then layer).
int run_fetch(const Fetch *f)
{
    using namespace hv;
    std::vector<uint64_t> dir(f->versions, f->versions + f->n_objects);
    const uint32_t total = f->n_seq * f->max_blocks;
    struct { const void *pointers[3]; SmallArgs a; SmallWalk w; } arguments{};
    static_assert(offsetof(decltype(arguments), w) == SMALL_WALK_AT);
    kernel_arguments = (const char *)&arguments;
    SmallArgs &a = arguments.a;
    SmallWalk &w = arguments.w;
    a.dst_cap = f->dst_cap; a.dir = dir.data(); a.chunk_bytes = f->chunk_bytes;
    a.max_blocks = f->max_blocks; a.n_objects = f->n_objects; a.n_rep = f->n_layers;
    const uint32_t tile = f->nthr * 16 * (f->unrolled ? 2 : 1);
    a.tiles_per_chunk = (uint32_t)((f->chunk_bytes + tile - 1) / tile);
    a.hbm_wgs = total * a.tiles_per_chunk;
    a.dst_base[0] = f->dst[0]; a.dst_base[1] = f->dst[1]; a.dst_step = f->dst_step;
    auto tier = [&](int t) { return SmallTier{ { f->pool[t][0], f->pool[t][1] }, f->n_slots * f->chunk_bytes, f->chunk_bytes }; };
    a.cache = tier(T_CACHE); a.local = tier(T_LOCAL); w.host = tier(T_HOST);
    a.n_cache_slots = a.n_local_slots = w.n_host_slots = f->n_slots;
    w.total = total; w.seen = f->seen; a.n_host = f->n_host; w.host_lg_groups = f->lg_groups;
    deal_out_host_pieces(a, w, f->n_planes, f->nthr);
    SmallHm<true> h{};
    if (f->head_major) {
        h.n_heads = f->n_heads;
        h.upr = (uint32_t)(f->chunk_bytes / (f->n_heads * f->block_tokens) / 16);
        h.ups = h.upr * f->block_tokens;
        h.seq_cap_blocks = f->seq_cap;
    }
    std::vector<unsigned long long> totals(C_N);
    alignas(16) Report report;
    w.n_seq = f->n_seq; w.miss_idx = f->miss; w.cnt = f->cnt; w.totals = totals.data(); w.report = &report;
    auto call = [&](auto plain, auto with_hm) {
        if (f->head_major) g_kernel = [&, with_hm] { with_hm(f->table, f->n_blocks, f->seq_dst, a, w, h); };
        else g_kernel = [&, plain] { plain(f->table, f->n_blocks, f->seq_dst, a, w, SmallHm<false>{}); };
    };
    if (f->unrolled && f->n_planes == 2) call(fetch_kv_small<2, 256, false, 2>, fetch_kv_small<2, 256, true, 2>);
    else if (f->unrolled) call(fetch_kv_small<1, 256, false, 2>, fetch_kv_small<1, 256, true, 2>);
    else if (f->n_planes == 2 && f->nthr == 64) call(fetch_kv_small<2, 64, false>, fetch_kv_small<2, 64, true>);
    else if (f->n_planes == 2) call(fetch_kv_small<2, 256, false>, fetch_kv_small<2, 256, true>);
    else if (f->nthr == 64) call(fetch_kv_small<1, 64, false>, fetch_kv_small<1, 64, true>);
    else call(fetch_kv_small<1, 256, false>, fetch_kv_small<1, 256, true>);

    const bool sliced = f->n_layers > 1;
    const uint32_t head = a.n_host + 1;
    gridDim = { sliced ? (a.hbm_wgs > head ? a.hbm_wgs : head) : a.hbm_wgs + head, f->n_planes, sliced ? f->n_layers + 1 : 1 };
    const uint32_t *when = f->when;
    uint32_t shown = 0;
    auto show = [&](uint32_t version) {
        if (version != shown) memcpy(dir.data(), f->versions + (uint64_t)version * f->n_objects, f->n_objects * 8);
        shown = version;
    };
    auto versions_at = [&](uint32_t barrier) {
        uint32_t v = 0;
        while (v + 1 < f->n_versions && when[v] <= barrier) v++;
        show(v);
    };
    for (uint32_t x = 0; x < head; ++x, when += f->n_versions - 1) {
        blockIdx = { x, 0, 0 };
        run_workgroup(f->nthr, versions_at);
    }
    g_fibers = false;
    for (uint32_t z = 0; z < f->n_layers; ++z)
        for (uint32_t p = 0; p < f->n_planes; ++p)
            for (uint32_t t = 0; t < a.hbm_wgs; ++t, when += f->n_versions - 1) {
                versions_at(0);
                blockIdx = { sliced ? t : t + head, p, sliced ? z + 1 : 0 };
                for (uint32_t i = 0; i < f->nthr; ++i) { threadIdx = { i, 0, 0 }; g_kernel(); }
            }
    return 0;
}

struct Experts {
    uint32_t n_experts, n_known, n_ids, n_staging, n_host, hbm_wgs, seen, n_versions, n_slots, pad;
    uint64_t chunk_bytes, pool[2], staging;      // [tier]: host, cache
    const int32_t *topk;
    const uint64_t *versions;                    // [n_versions][n_experts]
    const uint32_t *when;                        // [workgroup][n_versions - 1]: at which of its ballots or barriers
    uint64_t *expert_ptr;
    uint32_t *cnt, *miss;
};
int run_experts(const Experts *f)
{
    using namespace hv;
    std::vector<uint64_t> dir(f->versions, f->versions + f->n_experts);
    struct { RoutedArgs a; RoutedBooks b; } arguments{};
    kernel_arguments = (const char *)&arguments;
    RoutedArgs &a = arguments.a;
    RoutedBooks &b = arguments.b;
    a.topk = f->topk; a.dir = (k_entry *)dir.data(); a.chunk_bytes = f->chunk_bytes; a.staging = f->staging;
    a.cache_base = f->pool[1]; a.host_base = f->pool[0]; a.cache_stride = a.host_stride = f->chunk_bytes;
    a.n_experts = f->n_experts; a.n_known = f->n_known; a.n_cache_slots = a.n_host_slots = f->n_slots;
    a.n_ids = f->n_ids; a.n_staging = f->n_staging; a.n_host = f->n_host; a.hbm_wgs = f->hbm_wgs; a.seen = f->seen;
    a.tiles_per_chunk = (uint32_t)((f->chunk_bytes + WG * 32 - 1) / (WG * 32));
    std::vector<unsigned long long> totals(C_N);
    alignas(16) Report report;
    b.c.dir = dir.data(); b.c.n_objects = f->n_known; b.c.chunk_bytes = f->chunk_bytes;
    b.c.n_slots[T_HOST] = b.c.n_slots[T_CACHE] = f->n_slots;
    b.expert_ptr = f->expert_ptr; b.miss_idx = f->miss; b.cnt = f->cnt; b.totals = totals.data(); b.report = &report;
    g_kernel = [&] { fetch_experts_small<WG, 2>(a, b); };
    gridDim = { f->n_host + 1 + f->hbm_wgs, 1, 1 };
    const uint32_t *when = f->when;
    for (uint32_t x = 0; x < gridDim.x; ++x, when += f->n_versions - 1) {
        blockIdx = { x, 0, 0 };
        auto versions_at = [&](uint32_t met) {
            uint32_t v = 0;
            while (v + 1 < f->n_versions && when[v] <= met) v++;
            memcpy(dir.data(), f->versions + (uint64_t)v * f->n_experts, f->n_experts * 8);
        };
        run_workgroup(WG, versions_at, true);
    }
    return (int)report.hbm;
}
}  // extern "C"
