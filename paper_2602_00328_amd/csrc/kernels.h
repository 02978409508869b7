// Device code of the tiered cache fetch for gfx950 (CDNA4, wave64).
//
// Everything here is byte movement plus a few integers of metadata: no floating point, no MFMA.
//
//   classify_kv              : directory lookup (paper Section 5.2: the extended KV block table), classification of
//                              every request by tier, and an ORDER-PRESERVING compaction: into one HBM list whose places follow
//                              from the block table alone, and per segment of the table into the host's requests and the misses:
//                              wavefront ballots rank the lanes, LDS carries the wave totals.  Keeping the
//                              lists in request order makes the gather's writes one ascending stream, worth ~6% of
//                              HBM bandwidth over lists ordered by racing atomics.
//                              Tables of very many rows get a pass in front (sum_rows) that adds up groups of row lengths.
//   fetch_kv_small           : small block tables - the whole fetch in one launch: a workgroup per tile of HBM-tier payload that
//                              resolves its own cell, a couple of dozen that find the host tier's cells, one for the books.
//   resolve_experts          : the same for expert weights (Section 4.3: residency map) - one workgroup forms the
//                              distinct set of routed experts and walks it in ascending order (very large batches of
//                              routing ids are marked by many workgroups first: mark_experts).
//   fetch_experts_small      : a few routing ids - the whole expert fetch in one launch.
//   gather                   : the copy itself, both tiers in one launch.  HBM tier: one wavefront per workgroup and 1 KiB
//                              tile, one 16-byte non-temporal load and store per thread, as many workgroups as tiles; plane K
//                              before plane V, or - where the cache tier keeps them side by side, in chunks of 32 KiB or
//                              more - both planes of a request in one pass (measured on MI355X: short workgroups beat deep unrolling and persistent
//                              grids by ~15%, one-wavefront workgroups beat four-wavefront ones by 2-5%, non-temporal
//                              accesses are worth ~11%, 64 KiB source runs 4-5% over 32 KiB ones).  Host tier: the
//                              launch's first workgroups, 96 or 48 wavefronts that stay, with two or four loads in
//                              flight per thread: enough compute units to keep the PCIe link full, and no more host reads
//                              in flight than the link absorbs, because the rest would only stand in the HBM tier's way.
//   gather_hm                : the same into a head-major working layout.
//   move_pcie, move_hbm, fill_items, dir_write : placement, write-back (one source, up to two destinations), slot poisoning
//                              after revocation, directory publication, from lists made on the host.  What crosses PCIe runs
//                              as a dozen persistent workgroups whose tiles are counted out one at a time, and they stand
//                              back while a fetch has announced that it needs the link (link_announce, yield_link).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hv {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int WG = 256;                         // 4 wavefronts
constexpr int WAVES = WG / 64;
constexpr uint32_t TILE_4K = WG * 16;           // 4 KiB: one 16-byte access per thread of a 256-thread workgroup
constexpr int HBM_WG = 64;                      // the HBM-tier gather runs one wavefront per workgroup (see gather)
constexpr int UNROLL_HOST = 8;
constexpr uint32_t TILE_HOST = WG * 16 * UNROLL_HOST;   // 32 KiB tiles of fill_items
constexpr int HOST_PAGE = 4;                    // 16-byte loads a thread of the host-tier gather makes for one page, see host_tier

// directory entry: [1:0] tier, [31:2] slot in that tier (host slot for HOST), [63:32] number of the edit that wrote it
constexpr uint64_t TIER_MASK = 3;
__host__ __device__ inline uint32_t entry_tier(uint64_t e) { return (uint32_t)(e & TIER_MASK); }
__host__ __device__ inline uint32_t entry_slot(uint64_t e) { return (uint32_t)(e >> 2) & 0x3FFFFFFFu; }
__host__ __device__ inline uint64_t make_entry(uint32_t tier, uint32_t slot, uint32_t edit)
{
    return (uint64_t)tier | ((uint64_t)(slot & 0x3FFFFFFFu) << 2) | ((uint64_t)edit << 32);
}
// Written by an edit that the fetch is not known to come after (`seen`: the latest that it does): another workgroup of the same
// launch may have read the entry before it.
__device__ inline bool entry_young(uint64_t e, uint32_t seen) { return (int32_t)((uint32_t)(e >> 32) - seen) > 0; }
enum { T_HOST = 0, T_CACHE = 1, T_LOCAL = 2, T_NONE = 3 };

// One request of a fetch, the same for every plane of its class:
//   src = byte offset of the chunk inside its tier's plane pool, tier in bits [1:0] (offsets are multiples of 16);
//   dst = byte offset of the chunk inside the destination plane.
struct Rec { uint64_t src, dst; };
// A host-built list names chunks by absolute address (slot poisoning) ...
struct Item { uint64_t dst; };
// ... or whole objects (placement, write-back), whose chunks - every plane, every layer of the move - the kernel finds by itself:
// byte offsets of plane 0, first layer of the move, from the bases in MoveArgs.  dst1 has its tier in bits [1:0].
constexpr uint64_t NOWHERE = ~0ull;
struct MoveRec { uint64_t src, dst0, dst1; };
struct MoveArgs {
    uint64_t src_base[2], host_base[2], cache_base[2], local_base[2];      // [plane], at the first layer of the move
    uint64_t src_layer, host_layer, cache_layer, local_layer;              // layer strides
    uint64_t chunk_bytes;
    uint32_t n_planes, n_layers, n_obj, tiles_per_chunk, n_tiles;
    uint32_t order;                                                        // ORDER_*: which chunk comes after which
    const MoveRec *recs;                                                   // null: the list travels with the launch (MoveList)
    unsigned long long *next;                                              // tile counter of the copies over PCIe
    const unsigned long long *lease;
};
// The order in which a move takes its chunks follows the layout of the cache tier, so that the writes to slots that were handed
// out together are one ascending stream: [plane][layer][slot], [layer][slot][plane], or one segment per object (64 blocks of
// 32 layers from a staged copy, placed and revoked, in one run: 66.0 us object after object, 60.9 this way).
enum { ORDER_PLANE_LAYER_OBJ = 0, ORDER_LAYER_OBJ_PLANE, ORDER_OBJ_LAYER_PLANE };
// Lists of up to this many objects / entries are kernel arguments; longer ones are copied to the device first, which costs a call
// 7-8 us more whatever their length (32 KiB per object placed from a staged copy and revoked: 17 objects 34.4 us against 41.5 with
// the list on the device, 80: 51.8 against 60.4; 81 objects, beyond the line, 59.4).  The room itself costs a short list nothing (one
// object with room for 16, 80 and 160: 31.6, 33.0 and 31.6 us).  80 and 128 fill half of the 4 KiB that kernel arguments may take; nothing
// that was measured says that they must not fill more.
#ifdef HARVEST_FAULT_INJECTION
constexpr uint32_t MOVE_INLINE = 2, DIR_INLINE = 2;      // the CPU tests' lists are short: they are to walk both ways
#else
constexpr uint32_t MOVE_INLINE = 80, DIR_INLINE = 128;
#endif
struct MoveList { MoveRec r[MOVE_INLINE]; };
struct DirList { uint64_t entry[DIR_INLINE]; uint32_t id[DIR_INLINE]; };

// per-fetch counters (uint32) and running totals (uint64) share these indices
enum { C_REQ = 0, C_LOCAL, C_CACHE, C_HOST, C_LOST, C_INVALID, C_HBM_REQ, C_HOST_REQ, C_MISS, C_LIST, C_N = 16 };

struct ClassDev {
    const uint64_t *dir;
    uint32_t n_objects, n_planes;
    uint64_t chunk_bytes;
    uint64_t pool[3][2];      // [tier HOST/CACHE/LOCAL][plane] base address as the GPU sees it
    uint32_t n_slots[3];      // slot numbers a directory entry may carry, per tier
    uint32_t pad;
    // chunk (layer, slot) of a tier's plane sits at  layer * layer_stride + slot * slot_stride  from the plane's base:
    // [layer][slot][chunk] pools have (n_slots * chunk, chunk); segments of the shared cache pool, [layer][plane][chunk]
    // from granule number `slot` on, have (n_planes * chunk, granule)
    uint64_t layer_stride[3];
    uint64_t slot_stride[3];
};

struct GatherArgs {
    uint64_t src_base[3][2];  // [tier][plane]
    uint64_t dst_base[2];     // [plane]
    uint64_t chunk_bytes;
    uint32_t tiles_per_chunk;
    // consecutive layers gathered from the same lists (an object has the same slot in every layer): repetition r reads
    // layer_stride[tier] * r further and writes dst_step * r further
    uint64_t layer_stride[3];
    uint64_t dst_step;
    uint32_t n_rep;
    // the launch's first n_host workgroups serve the host tier, the next hbm_wgs (per plane, unless the planes are folded)
    // the HBM tier; either may be 0
    uint32_t n_host, hbm_wgs;
    uint32_t pages_per_chunk;            // of the host tier, see host_tier
    uint32_t host_loads;                 // 2 or HOST_PAGE: loads a thread of the host tier keeps in flight
};
// In pinned memory, one per class and stream: requests of either tier of the latest fetch whose kernels have run - hints for the
// next launch - and the rows and columns of the block table they were asked for with (experts: zero).
struct Report { uint32_t hbm, host, n_seq, max_blocks; };
// The table cells of a KV fetch are resolved in up to SEGS segments of consecutive cells, by a workgroup each, which leaves its
// requests to the host and its misses at the start of its own stretch of a list and says in counts[SC_* * SEGS + segment] how many
// there are.  (Four segments to a lane: a wavefront that reads the counts can say which segment has the n-th request without
// touching memory again, see HostList.)
constexpr uint32_t SEGS = 256;
enum { SC_HOST = 0, SC_MISS, SC_REQ, SC_LOCAL, SC_INVALID, SC_N };
constexpr uint32_t ROW_GROUP = 4096;     // rows whose lengths sum_rows adds up
// What only the host tier's workgroups and the one that keeps the books need.  They read it where they need it: as an ordinary argument
// it would be loaded at the start of every workgroup.
enum { BOOKS_NONE = 0, BOOKS_COUNTED, BOOKS_AGAIN, BOOKS_RESOLVED };
struct GatherRest {
    const Rec *host_recs;
    const uint32_t *counts;              // of the segments
    uint32_t n_seg, seg_cells;
    uint32_t n_seq, max_blocks;          // for the report
    unsigned long long *lease;           // see link_announce
    Report *report;
    uint32_t *listed;                    // KV, beside the report: how many entries the HBM list had
    // Books, by the first BOOK_WGS workgroups of the HBM tier (a segment's misses each) once they have copied their tiles.  BOOKS_COUNTED: *cnt is there, report it.
    // BOOKS_AGAIN: and add it to the running totals, for a fetch repeated from older lists.  BOOKS_RESOLVED: the segments' counts make
    // up *cnt, the running totals and the caller's copy (info, may be null), and their misses one list.
    uint32_t books, pad;
    uint32_t *cnt, *info, *miss_idx;
    const uint32_t *seg_miss;
    unsigned long long *totals;
};
constexpr uint32_t BOOK_WGS = SEGS;
typedef const __attribute__((address_space(4))) GatherRest k_GatherRest;
template <uint32_t AT> __device__ inline k_GatherRest &gather_rest()       // AT: where it is among the kernel's arguments
{
    return *(k_GatherRest *)((const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr() + AT);
}

__device__ inline uint32_t lane_id() { return __lane_id(); }

// A value that all lanes of the wavefront have, for the scalar registers.
__device__ inline uint32_t uniform(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ inline uint64_t uniform(uint64_t x) { return (uint64_t)uniform((uint32_t)(x >> 32)) << 32 | uniform((uint32_t)x); }
// These values are in registers from here on.  An argument is loaded where it is used, and every such load is a wait; a tile's workgroup
// has to wait for its directory entry anyway and gets its addresses meanwhile (300 blocks 9.77 us without, 9.69 with).
template <typename A, typename B, typename C, typename D> __device__ inline void in_registers(A a, B b, C c, D d)
{
#ifdef __HIP_DEVICE_COMPILE__
    asm volatile("" ::"s"(a), "s"(b), "s"(c), "s"(d));
#endif
}

// Selects instead of indexing: a variable index into a kernel-argument struct would send it to scratch memory.
template <typename C> __device__ inline uint32_t slots_of(const C &c, int tier)
{
    return tier == T_HOST ? c.n_slots[T_HOST] : (tier == T_CACHE ? c.n_slots[T_CACHE] : c.n_slots[T_LOCAL]);
}
template <typename C> __device__ inline uint64_t chunk_offset(const C &c, int tier, uint32_t layer, uint32_t slot)
{
    uint64_t ls = tier == T_HOST ? c.layer_stride[T_HOST] : (tier == T_CACHE ? c.layer_stride[T_CACHE] : c.layer_stride[T_LOCAL]);
    uint64_t ss = tier == T_HOST ? c.slot_stride[T_HOST] : (tier == T_CACHE ? c.slot_stride[T_CACHE] : c.slot_stride[T_LOCAL]);
    return (uint64_t)layer * ls + (uint64_t)slot * ss;
}
__device__ inline bool in_hbm(uint32_t tier) { return (tier + 1) & 2; }        // T_CACHE or T_LOCAL
__device__ inline uint64_t src_base_of(const GatherArgs &a, uint32_t tier, uint32_t plane)
{
    uint64_t h = plane ? a.src_base[T_HOST][1] : a.src_base[T_HOST][0];
    uint64_t k = plane ? a.src_base[T_CACHE][1] : a.src_base[T_CACHE][0];
    uint64_t l = plane ? a.src_base[T_LOCAL][1] : a.src_base[T_LOCAL][0];
    return tier == T_HOST ? h : (tier == T_CACHE ? k : l);
}
__device__ inline uint64_t layer_stride_of(const GatherArgs &a, uint32_t tier)
{
    return tier == T_HOST ? a.layer_stride[T_HOST] : (tier == T_CACHE ? a.layer_stride[T_CACHE] : a.layer_stride[T_LOCAL]);
}

// Exclusive rank of this lane among the lanes of its wavefront for which pred holds, and the wave total.
__device__ inline uint32_t wave_rank(bool pred, uint32_t &total)
{
    unsigned long long m = __ballot(pred);
    total = (uint32_t)__popcll(m);
    return (uint32_t)__popcll(m & ((1ull << lane_id()) - 1ull));
}

// The value that lane k of the wavefront has, k the same in all of them.
__device__ inline uint32_t lane_value(uint32_t x, uint32_t k) { return __builtin_amdgcn_readlane(x, k); }
__device__ inline uint64_t lane_value(uint64_t x, uint32_t k) { return (uint64_t)lane_value((uint32_t)(x >> 32), k) << 32 | lane_value((uint32_t)x, k); }
// The bits that any lane of the wavefront has, in all of them.
__device__ inline uint32_t wave_or(uint32_t x)
{
#ifdef __HIP_DEVICE_COMPILE__
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, true);      // row_shr:1, 2, 4, 8: lane 15 of each row has the row's
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, true);
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, true);
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, true);
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, true);      // row_bcast:15 into rows 1 and 3, row_bcast:31 into 2 and 3
    x |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, true);
    return lane_value(x, 63);
#else
    uint32_t all = 0;
    for (uint32_t k = 0; k < 32; ++k) all |= __ballot(x >> k & 1) ? 1u << k : 0u;
    return all;
#endif
}
template <uint32_t N> struct Count { static constexpr uint32_t value = N; };

__device__ inline uint32_t wave_sum(uint32_t v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// What cell r of the block table asks for: -1 nothing (beyond the row's length), 0..3 the tier of its block, 4 an invalid
// request (unknown block, or a destination that does not fit).  For tiers 0..2 rec names source and destination.  The loads
// wait for nothing but their addresses - row length, block number and destination go out together, then the directory
// entry of block 0 if the cell names none - so a cell costs two memory latencies, not four.
struct Ask { uint32_t n, s, j; int32_t b; };     // the sequence's length and number; column; block
__device__ inline Ask ask_cell(const int32_t *__restrict__ table, const int32_t *__restrict__ n_blocks, uint32_t max_blocks, uint32_t r,
                               uint32_t total)
{
    const bool there = r < total;
    if (!there) r = total - 1;
    const uint32_t s = r / max_blocks;
    const int32_t n = n_blocks[s];
    return { there && n > 0 ? (uint32_t)n : 0u, s, r - s * max_blocks, table[r] };
}
__device__ inline int resolve_cell(const ClassDev &c, uint32_t layer, const int32_t *__restrict__ table,
                                   const int32_t *__restrict__ n_blocks, uint32_t max_blocks,
                                   const uint64_t *__restrict__ seq_dst_block, uint64_t dst_cap,
                                   const uint32_t *__restrict__ seq_cap_blocks, uint64_t strip_bytes, uint32_t r, Rec &rec)
{
    const Ask x = ask_cell(table, n_blocks, max_blocks, r, r + 1);
    const uint64_t first = seq_dst_block[x.s], cap = seq_cap_blocks ? seq_cap_blocks[x.s] : 0, dst_chunk = first + x.j;
    const bool asked = x.j < x.n;
    const bool fits = seq_cap_blocks ? first + cap <= dst_cap && x.j < cap && cap < 65536 : dst_chunk < dst_cap;
    const bool known = asked && x.b >= 0 && (uint32_t)x.b < c.n_objects;
    const uint64_t e = c.dir[known ? (uint32_t)x.b : 0u];
    const int tier = (int)entry_tier(e);
    rec.dst = seq_cap_blocks ? first * c.chunk_bytes + (uint64_t)x.j * strip_bytes : dst_chunk * c.chunk_bytes;
    if (tier != T_NONE) rec.src = chunk_offset(c, tier, layer, entry_slot(e)) | (uint64_t)tier | (cap << 48);
    if (!asked) return -1;
    if (!known || !fits) return 4;
    return tier != T_NONE && entry_slot(e) >= slots_of(c, tier) ? 4 : tier;     // never for a directory the library wrote
}

// ---------------------------------------------------------------------------------------------------------
// KV: every (sequence, block-table column) looks its block up, once.  The HBM list has an entry for every request, in request order; one
// that HBM does not serve is marked T_NONE and the gather passes over it.  So the place of an entry follows from the block table alone -
// the lengths of the rows before it - and no workgroup has to know what another found in the directory: one launch, where counting the
// tiers first and placing the entries second took two.  A chain of a few memory latencies bounds it, and the way between kernels that
// fill the device: a fetch costs 4.9 us more than the same one repeated from its lists, 7.8 with the second launch (3 536 blocks of
// 2 x 32 KiB into the head-major layout 86.7 us before, 83.9 now; 15 125 token-major 315.1 and 311.7).
// What the host serves, and the misses, stay in the segment's own stretch; the gather's workgroups put the stretches together while
// the HBM tier is on its way (HostList, keep_books).  Nothing is accumulated with atomics and nothing needs zeroing, so a fetch can be
// replayed from a captured graph as it is.
// ---------------------------------------------------------------------------------------------------------
__device__ inline uint32_t row_requests(int32_t n, uint32_t max_blocks) { return n <= 0 ? 0u : (uint32_t)n < max_blocks ? (uint32_t)n : max_blocks; }

struct KvLists {
    Rec *hbm, *host;
    uint32_t *miss, *counts, *cnt;       // misses and counts of the segments; of the fetch's counters, C_LIST is written here
    const uint32_t *row_groups;          // from sum_rows, or null: few rows
    uint32_t seg_cells;                  // a multiple of the workgroup's threads
};

template <int NTHR>
__global__ __launch_bounds__(NTHR) void classify_kv(ClassDev c, uint32_t layer, const int32_t *__restrict__ table,
                                                    const int32_t *__restrict__ n_blocks, uint32_t total, uint32_t max_blocks,
                                                    const uint64_t *__restrict__ seq_dst_block, uint64_t dst_cap, KvLists l,
                                                    const uint32_t *__restrict__ seq_cap_blocks, uint64_t strip_bytes)
{
    // seq_cap_blocks != nullptr selects the head-major working layout: sequence s owns seq_cap_blocks[s] destination
    // blocks, laid out [head][token][head_bytes]; strip_bytes = block_tokens * head_bytes is what one block adds to
    // one head's strip.  The record then carries the sequence's capacity (in blocks) in bits [63:48] of src.
    constexpr uint32_t WAVES_N = NTHR / 64;
    __shared__ uint32_t s_before[WAVES_N], s_sum[2][SC_N][WAVES_N];
    const uint32_t tid = threadIdx.x, wave = tid >> 6;
    const uint32_t first = blockIdx.x * l.seg_cells, end = total - first < l.seg_cells ? total : first + l.seg_cells;
    const uint32_t s0 = first / max_blocks, j0 = first - s0 * max_blocks;
    // requests of the rows before the segment, and of its first row before its first cell
    uint32_t before = 0, s = 0;
    if (l.row_groups) {
        s = s0 / ROW_GROUP * ROW_GROUP;
        for (uint32_t g = tid; g < s0 / ROW_GROUP; g += NTHR) before += l.row_groups[g];
    }
    for (s += tid; s < s0; s += NTHR) before += row_requests(n_blocks[s], max_blocks);
    if (tid == 0) before += row_requests(n_blocks[s0], j0);
    uint32_t run[SC_N] = { 0, 0, 0, 0, 0 };               // of the segment so far
    uint32_t turn = 0;
    for (uint32_t r0 = first; r0 < end; r0 += NTHR, turn ^= 1) {
        const uint32_t r = r0 + tid;
        int tier = -1;                                    // -1 no request, 0..3 tier, 4 invalid
        Rec rec = { 0, 0 };
        if (r < end)
            tier = resolve_cell(c, layer, table, n_blocks, max_blocks, seq_dst_block, dst_cap, seq_cap_blocks, strip_bytes, r, rec);
        const bool is[SC_N] = { tier == T_HOST, tier == T_HOST || tier == T_NONE, tier >= 0, tier == T_LOCAL, tier == 4 };
        uint32_t rank[SC_N];
#pragma unroll
        for (int k = 0; k < SC_N; ++k) {
            uint32_t in_wave;
            rank[k] = wave_rank(is[k], in_wave);
            if (lane_id() == 0) s_sum[turn][k][wave] = in_wave;
        }
        if (r0 == first) {
            before = wave_sum(before);
            if (lane_id() == 0) s_before[wave] = before;
        }
        __syncthreads();                                  // (two sets of sums in turn: nobody reads the one that is written next)
        if (r0 == first) {
            before = 0;
#pragma unroll
            for (uint32_t w = 0; w < WAVES_N; ++w) before += s_before[w];
        }
#pragma unroll
        for (int k = 0; k < SC_N; ++k) {
            rank[k] += run[k];
#pragma unroll
            for (uint32_t w = 0; w < WAVES_N; ++w) {
                const uint32_t n = s_sum[turn][k][w];
                rank[k] += w < wave ? n : 0;
                run[k] += n;
            }
        }
        if (is[SC_HOST]) l.host[first + rank[SC_HOST]] = rec;
        if (is[SC_MISS]) l.miss[first + rank[SC_MISS]] = r;
        if (tier != T_LOCAL && tier != T_CACHE) rec = { T_NONE, 0 };
        if (is[SC_REQ]) l.hbm[before + rank[SC_REQ]] = rec;
    }
    if (tid < SC_N) l.counts[tid * SEGS + blockIdx.x] = tid == SC_HOST ? run[SC_HOST] : tid == SC_MISS ? run[SC_MISS] : tid == SC_REQ ? run[SC_REQ]
                                                      : tid == SC_LOCAL ? run[SC_LOCAL] : run[SC_INVALID];
    if (blockIdx.x == gridDim.x - 1 && tid == 0) l.cnt[C_LIST] = before + run[SC_REQ];
}

// Block tables of many rows: what each ROW_GROUP of them asks for, so that a segment need not add up all rows before it.
__global__ __launch_bounds__(WG) void sum_rows(const int32_t *__restrict__ n_blocks, uint32_t n_seq, uint32_t max_blocks, uint32_t *__restrict__ row_groups)
{
    __shared__ uint32_t s_wave[WAVES];
    uint32_t sum = 0;
    for (uint32_t i = threadIdx.x; i < ROW_GROUP; i += WG) {
        const uint64_t s = (uint64_t)blockIdx.x * ROW_GROUP + i;
        if (s < n_seq) sum += row_requests(n_blocks[s], max_blocks);
    }
    sum = wave_sum(sum);
    if (lane_id() == 0) s_wave[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x) return;
    for (int w = 1; w < WAVES; ++w) sum += s_wave[w];
    row_groups[blockIdx.x] = sum;
}

// One row of the segments' counts in a wavefront's registers, as running sums: lane i has segments 4 i to 4 i + 3.
struct SegSums {
    uint32_t upto[4], before, total;
    template <typename P> __device__ inline SegSums(P counts, uint32_t n_seg)
    {
        const uint32_t at = lane_id() * 4;
        uint32_t n[4];
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) n[i] = counts[at + i < n_seg ? at + i : 0];
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) upto[i] = (i ? upto[i ? i - 1 : 0] : 0) + (at + i < n_seg ? n[i] : 0);
        uint32_t all = upto[3];
#pragma unroll
        for (uint32_t o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(all, o);
            if (lane_id() >= o) all += y;
        }
        before = all - upto[3];
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) upto[i] += before;
        total = lane_value(all, 63);
    }
    // The segment that has number idx of the list (idx < total, the same in all lanes), and the numbers that it has: from first up to end.
    __device__ inline uint32_t find(uint32_t idx, uint32_t &first, uint32_t &end) const
    {
        const uint32_t k = (uint32_t)__popcll(__ballot(upto[3] <= idx));
        const uint32_t u0 = lane_value(upto[0], k), u1 = lane_value(upto[1], k), u2 = lane_value(upto[2], k);
        first = idx >= u2 ? u2 : idx >= u1 ? u1 : idx >= u0 ? u0 : lane_value(before, k);
        end = idx < u0 ? u0 : idx < u1 ? u1 : idx < u2 ? u2 : lane_value(upto[3], k);
        return 4 * k + (idx >= u0) + (idx >= u1) + (idx >= u2);
    }
};
// The host's requests in request order.  (Constant address space: the entries come by scalar loads, which wait for none of the
// payload's accesses; as vector loads behind the stores 402 MB beside another stream's copy took 8.7 ms instead of 7.6.)
typedef const __attribute__((address_space(4))) Rec k_Rec;
struct HostList {
    k_Rec *recs;
    uint32_t seg_cells;
    SegSums sums;
    // Of the segment that had the last entry asked for: a workgroup's next one mostly is of the same (12 000 blocks of 2 x 2 KiB, head-major,
    // 905.5 us with a search for each, 891.4 this way; of 2 x 64 bytes 211.5 and 204.7).
    uint32_t first = 0, end = 0;
    k_Rec *from = nullptr;
    __device__ inline HostList(k_GatherRest &r) : recs((k_Rec *)(uint64_t)r.host_recs), seg_cells(r.seg_cells), sums(r.counts + SC_HOST * SEGS, r.n_seg) {}
    __device__ inline Rec operator[](uint32_t idx)
    {
        if (idx < first || idx >= end) from = recs + (uint64_t)sums.find(idx, first, end) * seg_cells;
        k_Rec &x = from[idx - first];
        return { x.src, x.dst };
    }
};

// Who gets the PCIe link.  A fetch that reads from the host announces, in a word of device memory, until when it
// expects to need the link (link_announce: now + its host-tier bytes at the link's rate, on the device's constant 100 MHz
// clock); the copies that cross the link outside a fetch - placements, write-backs - look at that word before they take
// their next tile and stand back while the time has not come (yield_link), though never for longer than YIELD_TICKS per
// 32 KiB, whatever their tiles measure, so that they always get on (12 workgroups: 6.5 GB/s, a ninth of the link, when fetches
// never pause).  A miss is on the
// critical path and a placement is best effort (paper Sections 2.2 and 3.1).  An estimate instead of an exact begin /
// end: nothing has to be counted or taken back, and a word that is stale means no more than "nobody is fetching".  The
// estimate is on the short side (the rate of an undisturbed fetch, no margin): a copy that follows the fetch on the same
// stream, which cannot run beside it anyway, must not be kept waiting for a fetch that is already over.
constexpr uint64_t LINK_BYTES_PER_TICK = 575;      // 57.5 GB/s at 100 MHz
constexpr uint64_t YIELD_TICKS = 6000;             // 60 us
__device__ inline void link_announce(unsigned long long *lease, uint64_t host_bytes)
{
    if (!lease || !host_bytes) return;
    atomicMax(lease, (unsigned long long)(wall_clock64() + host_bytes / LINK_BYTES_PER_TICK));
}
template <uint32_t TILE>
__device__ inline void yield_link(const unsigned long long *lease)
{
    if (!lease) return;
    const uint64_t t0 = wall_clock64();
    for (;;) {
        const uint64_t now = wall_clock64();
        if (now - t0 >= YIELD_TICKS * TILE / 32768 || now >= __hip_atomic_load(lease, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
        __builtin_amdgcn_s_sleep(127);
    }
}

// ---------------------------------------------------------------------------------------------------------
// Experts: one workgroup forms the distinct set of the routed expert numbers (bitmap in LDS), then walks the
// experts in ascending order so that staging ranks are the ranks among the staged members of the set.
// ---------------------------------------------------------------------------------------------------------
constexpr uint32_t MAX_EXPERTS = 8192;

// Large batches only: many workgroups mark the routed experts - each in a bitmap of its own in LDS, merged into
// g_bitmap with one atomic per non-zero word - so that the single workgroup of resolve_experts need not read every
// routing id itself (half a million ids cost it 0.4 ms).  g_bitmap and g_invalid are zero on entry; resolve_experts
// takes their contents and leaves them zero again, so nothing has to be cleared between fetches or graph replays.
__global__ __launch_bounds__(WG) void mark_experts(const int32_t *__restrict__ topk, uint32_t n_ids, uint32_t n_experts,
                                                   uint32_t *g_bitmap, uint32_t *g_invalid)
{
    __shared__ uint32_t bm[MAX_EXPERTS / 32];
    __shared__ uint32_t inval;
    uint32_t tid = threadIdx.x, words = (n_experts + 31) / 32;
    for (uint32_t i = tid; i < words; i += WG) bm[i] = 0;
    if (tid == 0) inval = 0;
    __syncthreads();
    for (uint64_t i = (uint64_t)blockIdx.x * WG + tid; i < n_ids; i += (uint64_t)gridDim.x * WG) {
        int32_t e = topk[i];
        if (e < 0 || (uint32_t)e >= n_experts) atomicAdd(&inval, 1u);
        else atomicOr(&bm[e >> 5], 1u << (e & 31));
    }
    __syncthreads();
    for (uint32_t i = tid; i < words; i += WG)
        if (bm[i]) atomicOr(&g_bitmap[i], bm[i]);
    if (tid == 0 && inval) atomicAdd(g_invalid, inval);
}

template <typename C>              // ClassDev, as an argument or where the arguments are
__device__ inline void resolve_routed(const C &c, uint32_t layer, uint32_t n_experts, const int32_t *__restrict__ topk, uint32_t n_ids,
                                      uint64_t staging, uint32_t n_staging, uint64_t *__restrict__ expert_ptr, Rec *__restrict__ hbm_recs,
                                      Rec *__restrict__ host_recs, uint32_t *__restrict__ miss_idx, uint32_t *cnt, unsigned long long *totals,
                                      uint32_t *g_bitmap, uint32_t *g_invalid, Report *report, unsigned long long *lease)
{
    // hbm_recs == nullptr: the caller has no use for the lists, but for a report and the lease (see link_announce).
    // g_bitmap != nullptr: mark_experts has already formed the routed set; it is taken from there (and cleared).
    __shared__ uint32_t bitmap[MAX_EXPERTS / 32];
    __shared__ uint32_t s_cnt[C_N];
    __shared__ uint32_t wave_tot[WG / 64];
    __shared__ uint32_t running;
    uint32_t tid = threadIdx.x;
    for (uint32_t i = tid; i < MAX_EXPERTS / 32; i += WG) {
        uint32_t w = 0;
        if (g_bitmap && i < (n_experts + 31) / 32) { w = g_bitmap[i]; g_bitmap[i] = 0; }
        bitmap[i] = w;
    }
    if (tid < C_N) s_cnt[tid] = 0;
    if (tid == 0) running = 0;
    __syncthreads();
    if (g_bitmap) {
        if (tid == 0) { s_cnt[C_INVALID] = *g_invalid; *g_invalid = 0; }
    } else {
        // Eight ids a thread on their way together, and a bit that is there is not set again: of a batch most are.  (8 192 ids of 16
        // experts 32.9 us, the call, with an id at a time; 29.7 this way.)
        constexpr uint32_t AT_ONCE = 8;
        for (uint32_t i0 = tid; i0 < n_ids; i0 += WG * AT_ONCE) {
            int32_t id[AT_ONCE];
#pragma unroll
            for (uint32_t k = 0; k < AT_ONCE; ++k) id[k] = topk[i0 + k * WG < n_ids ? i0 + k * WG : i0];
#pragma unroll
            for (uint32_t k = 0; k < AT_ONCE; ++k) {
                if (i0 + k * WG >= n_ids) continue;
                if (id[k] < 0 || (uint32_t)id[k] >= n_experts) atomicAdd(&s_cnt[C_INVALID], 1u);
                else if (!(bitmap[id[k] >> 5] >> (id[k] & 31) & 1u)) atomicOr(&bitmap[id[k] >> 5], 1u << (id[k] & 31));
            }
        }
    }
    __syncthreads();
    for (uint32_t base = 0; base < n_experts; base += WG) {
        uint32_t e = base + tid;
        bool sel = e < n_experts && ((bitmap[e >> 5] >> (e & 31)) & 1u);
        int tier = -1;
        uint32_t slot = 0;
        if (sel) {
            uint64_t id = (uint64_t)layer * n_experts + e;
            if (id >= c.n_objects) tier = 4;
            else {
                uint64_t en = c.dir[id];
                tier = (int)entry_tier(en);
                slot = entry_slot(en);
                if (tier != T_NONE && slot >= slots_of(c, tier)) tier = 4;
            }
        }
        bool staged = tier == T_CACHE || tier == T_HOST;
        uint32_t wtot;
        uint32_t rank = wave_rank(staged, wtot);
        if (lane_id() == 0) wave_tot[tid >> 6] = wtot;
        __syncthreads();
        uint32_t before = running;
        for (uint32_t w = 0; w < (tid >> 6); ++w) before += wave_tot[w];
        rank += before;
        uint64_t ptr = 0;
        if (sel) {
            atomicAdd(&s_cnt[C_REQ], 1u);
            if (tier == T_LOCAL) {
                ptr = c.pool[T_LOCAL][0] + (uint64_t)slot * c.chunk_bytes;
                atomicAdd(&s_cnt[C_LOCAL], 1u);
            } else if (staged) {
                if (rank >= n_staging) {
                    atomicAdd(&s_cnt[C_INVALID], 1u);
                } else {
                    ptr = staging + (uint64_t)rank * c.chunk_bytes;
                    Rec it;                 // few, large objects: their order in the lists does not matter
                    it.src = chunk_offset(c, tier, 0, slot) | (uint64_t)tier;
                    it.dst = (uint64_t)rank * c.chunk_bytes;
                    const uint32_t at = atomicAdd(&s_cnt[tier == T_CACHE ? C_HBM_REQ : C_HOST_REQ], 1u);
                    if (hbm_recs) (tier == T_CACHE ? hbm_recs : host_recs)[at] = it;
                    if (tier == T_CACHE) {
                        atomicAdd(&s_cnt[C_CACHE], 1u);
                    } else {
                        miss_idx[atomicAdd(&s_cnt[C_MISS], 1u)] = e;
                        atomicAdd(&s_cnt[C_HOST], 1u);
                    }
                }
            } else if (tier == T_NONE) {
                miss_idx[atomicAdd(&s_cnt[C_MISS], 1u)] = e;
                atomicAdd(&s_cnt[C_LOST], 1u);
            } else {
                atomicAdd(&s_cnt[C_INVALID], 1u);
            }
        }
        if (e < n_experts) expert_ptr[e] = ptr;
        __syncthreads();
        if (tid == 0) {
            uint32_t t = 0;
            for (uint32_t w = 0; w < WG / 64; ++w) t += wave_tot[w];
            running += t;
        }
        __syncthreads();
    }
    if (tid < C_N) {
        cnt[tid] = s_cnt[tid == C_LIST ? C_HBM_REQ : tid];
        if (tid <= C_INVALID && s_cnt[tid]) atomicAdd(&totals[tid], (unsigned long long)s_cnt[tid]);
    }
    if (hbm_recs || tid) return;
    const u32x4 r = { s_cnt[C_HBM_REQ], s_cnt[C_HOST_REQ], 0, 0 };
    *reinterpret_cast<u32x4 *>(report) = r;
    link_announce(lease, (uint64_t)s_cnt[C_HOST_REQ] * c.chunk_bytes);
}

__global__ __launch_bounds__(WG) void resolve_experts(ClassDev c, uint32_t layer, uint32_t n_experts, const int32_t *__restrict__ topk, uint32_t n_ids,
                                                      uint64_t staging, uint32_t n_staging, uint64_t *__restrict__ expert_ptr, Rec *__restrict__ hbm_recs,
                                                      Rec *__restrict__ host_recs, uint32_t *__restrict__ miss_idx, uint32_t *cnt,
                                                      unsigned long long *totals, uint32_t *g_bitmap, uint32_t *g_invalid)
{
    resolve_routed(c, layer, n_experts, topk, n_ids, staging, n_staging, expert_ptr, hbm_recs, host_recs, miss_idx, cnt, totals, g_bitmap, g_invalid,
                   nullptr, nullptr);
}

// ---------------------------------------------------------------------------------------------------------
// The gather.
// ---------------------------------------------------------------------------------------------------------
// Every payload access names the global address space: an address computed as an integer would otherwise compile to
// flat_load / flat_store, which pay for an aperture check on each access; global_load / global_store do not.
typedef __attribute__((address_space(1))) u32x4 g_u32x4;

template <bool NT>
__device__ inline u32x4 ld16(const u32x4 *p)
{
    const g_u32x4 *g = (const g_u32x4 *)(uint64_t)p;
    if (NT) return __builtin_nontemporal_load(g);
    return *g;
}
template <bool NT>
__device__ inline void st16(u32x4 *p, u32x4 v)
{
    g_u32x4 *g = (g_u32x4 *)(uint64_t)p;
    if (NT) __builtin_nontemporal_store(v, g);
    else *g = v;
}

// One tile of NTHR * 16 * UNROLL bytes (or the first len bytes of it) by a workgroup of NTHR threads.
template <int NTHR, int UNROLL, bool NT>
__device__ inline void copy_tile(uint64_t src, uint64_t dst, uint64_t len, uint32_t tid)
{
    constexpr uint32_t TILE = NTHR * 16 * UNROLL;
    const u32x4 *s = reinterpret_cast<const u32x4 *>(src);
    u32x4 *d = reinterpret_cast<u32x4 *>(dst);
    if (len >= TILE) {
        u32x4 v[UNROLL];
#pragma unroll
        for (int i = 0; i < UNROLL; ++i) v[i] = ld16<NT>(s + tid + i * NTHR);
#pragma unroll
        for (int i = 0; i < UNROLL; ++i) st16<NT>(d + tid + i * NTHR, v[i]);
    } else {
        uint32_t n_vec = (uint32_t)(len >> 4);
        for (uint32_t i = tid; i < n_vec; i += NTHR) st16<NT>(d + i, ld16<NT>(s + i));
    }
}

// ---------------------------------------------------------------------------------------------------------
// The gathers: both tiers of a fetch in one launch.
// ---------------------------------------------------------------------------------------------------------
// The first n_host workgroups read the host list over PCIe, the others copy the HBM list; both lists' lengths live on
// the device.  One launch, because two cost more than they bring: on one stream an (often empty) host-tier launch took
// 4.4 us in front of the HBM one, and on two streams the fork and the join cost about 15 us each.  The host-tier workgroups
// come first in the grid, so the long PCIe transfer starts before the compute units fill up, and hold their slots
// until it is done while the HBM tier's one-tile workgroups pass through the others.
//
// Host tier.  What the link needs (measured on MI355X): one compute unit sustains about 12.8 GB/s of reads from host
// memory however many loads its threads have outstanding, so the rate is set by how many CUs take part (5 saturate the
// 57 GB/s link) - and every host read in flight beyond what the link can absorb only queues in the memory pipeline the HBM
// tier is using at the same time (8 x 256 threads with 16 loads per thread cost it 12 %, 24 x 256 with 2 loads 8 %).  Hence
// 192 KiB in flight (host_grid * 8 KiB), in 96 wavefronts with two 16-byte loads per thread or in 48 with four.  Each wavefront waits
// for its own loads and for its stores to be taken, so while the memory is busy 48 of them let the link idle and 96 do not.  That
// decides: a fetch that is bound by the link gets 96 (402 MB from the host beside another stream's copy: 7.62 ms against
// 9.68 with 48, alone 7.02; 12 000 blocks, 3 % of them on the host: 424 us against 433), one that is bound by HBM, whose host
// reads have time, gets 48 and an HBM tier that they disturb less (1.5 % on the host: 256 us against 273; none: 252).
//
// Work is cut into pages of HOST_PAGE loads per thread (4 KiB for one-wavefront workgroups), numbered through the whole list
// (request * pages per chunk + position), so the bytes in flight do not depend on the chunk size.  A workgroup takes a whole
// page - of both planes, half of the loads of a step each, if there are two: one-wavefront workgroups that took 1 KiB pieces in
// turn, so that four of them shared a page of host memory, ran at 57.36 (one plane, 16 MiB chunks), 57.14 and 57.02 GB/s (two
// planes, 32 and 16 KiB chunks), with whole pages it was 57.51, 57.45 and 57.36; pages of two loads change nothing (15 125
// blocks, 30 % of them on the host: 5 187 us, whole pages 5 185).  Each load is issued as soon as its list entry has arrived.  Lanes beyond a chunk's end re-read
// the chunk's first bytes and store nothing: loads stay free of branches.
template <int NTHR, int PLANES, int LOADS>
__device__ inline void host_page(const GatherArgs &a, uint64_t src, uint64_t dst, uint32_t page, uint32_t tid)
{
    constexpr int L = LOADS / PLANES;                     // loads per thread, plane and step
    const uint32_t chunk_units = (uint32_t)(a.chunk_bytes >> 4);
#pragma unroll
    for (int s = 0; s < HOST_PAGE; s += L) {
        const uint32_t u0 = (page * HOST_PAGE + s) * NTHR;
        if (u0 >= chunk_units) break;
        u32x4 v0[L], v1[L];
        uint32_t u[L];
#pragma unroll
        for (int i = 0; i < L; ++i) {
            u[i] = u0 + i * NTHR + tid;
            const uint64_t at = src + (u[i] < chunk_units ? (uint64_t)u[i] * 16 : 0);
            v0[i] = ld16<false>(reinterpret_cast<const u32x4 *>(a.src_base[T_HOST][0] + at));
            if (PLANES == 2) v1[i] = ld16<false>(reinterpret_cast<const u32x4 *>(a.src_base[T_HOST][1] + at));
        }
#pragma unroll
        for (int i = 0; i < L; ++i) {
            if (u[i] >= chunk_units) continue;
            const uint64_t d = dst + (uint64_t)u[i] * 16;
            st16<true>(reinterpret_cast<u32x4 *>(a.dst_base[0] + d), v0[i]);
            if (PLANES == 2) st16<true>(reinterpret_cast<u32x4 *>(a.dst_base[1] + d), v1[i]);
        }
    }
}

// Pages of all layers are one sequence, so that every workgroup has its share of them also where a layer has fewer than there are
// workgroups (2 x 32 KiB blocks of 32 layers: 5 of 140 on the host 206.9 us layer after layer, 196.1 this way; in the one-kernel
// fetch 1 of 5 52.0 and 42.9; 20 of 620 fp8 blocks of 10 layers, nearly a page for every workgroup, 126.5 and 127.9).
template <int NTHR, int PLANES, int LOADS>
__device__ inline void host_tier(HostList &recs, const GatherArgs &a, uint32_t b0)
{
    const uint32_t ppc = a.pages_per_chunk, n_pages = recs.sums.total * ppc;      // (fits: the host bounds requests times 1 KiB tiles)
    if (!n_pages) return;
    uint32_t rep = 0, g = b0, step_reps = 0, step = a.n_host, at = ~0u;
    Rec x = { 0, 0 };
    if (a.n_rep > 1) { step_reps = step / n_pages; step -= step_reps * n_pages; rep = g / n_pages; g %= n_pages; }
    for (;; rep += step_reps, g += step) {
        if (g >= n_pages) { g -= n_pages; rep++; }
        if (rep >= a.n_rep) return;
        const uint32_t idx = g / ppc, page = g - idx * ppc;
        if (idx != at) { at = idx; x = recs[idx]; }            // (a whole expert has thousands of pages: 2 727 us, 2 725 this way)
        host_page<NTHR, PLANES, LOADS>(a, (x.src & 0x0000FFFFFFFFFFFCull) + rep * a.layer_stride[T_HOST], x.dst + rep * a.dst_step, page,
                                       threadIdx.x);
    }
}

// The books of a fetch, see GatherRest: by workgroup bx of the HBM tier's n_wgs in a plane.  (Long lists of misses that no transfer hides
// are a chain of latencies: 500 224 lost blocks 197.6 us with 16 workgroups and a load at a time, 88.5 this way.)
template <int NTHR>
__device__ inline void keep_books(k_GatherRest &r, uint32_t bx, uint32_t n_wgs)
{
    const uint32_t tid = threadIdx.x, lane = lane_id();
    if (bx == 0 && tid < 64 && r.books) {
        uint32_t v = 0;                                   // lane i has counter i
        if (r.books == BOOKS_RESOLVED) {
            uint32_t n[SC_N];
#pragma unroll
            for (int k = 0; k < SC_N; ++k) n[k] = SegSums(r.counts + k * SEGS, r.n_seg).total;
            const uint32_t hbm = n[SC_REQ] - n[SC_MISS] - n[SC_INVALID];
            v = lane == C_REQ ? n[SC_REQ] : lane == C_LOCAL ? n[SC_LOCAL] : lane == C_CACHE ? hbm - n[SC_LOCAL] : lane == C_LOST ? n[SC_MISS] - n[SC_HOST]
              : lane == C_INVALID ? n[SC_INVALID] : lane == C_HBM_REQ ? hbm : lane == C_MISS ? n[SC_MISS] : n[SC_HOST];
            if (lane <= C_MISS) r.cnt[lane] = v;
            if (r.info && lane < 8) r.info[lane] = lane <= C_INVALID ? v : lane == 6 ? n[SC_MISS] : 0;
        } else if (lane <= C_MISS) v = r.cnt[lane];
        if (r.books != BOOKS_COUNTED && lane <= C_INVALID && v) atomicAdd(&r.totals[lane], (unsigned long long)v);
        const u32x4 report = { lane_value(v, C_HBM_REQ), lane_value(v, C_HOST_REQ), r.n_seq, r.max_blocks };
        const uint32_t listed = lane_value(v, C_REQ);
        if (lane == 0) *reinterpret_cast<u32x4 *>(r.report) = report;
        if (lane == 0 && r.listed) *r.listed = listed;
    }
    if (r.books != BOOKS_RESOLVED) return;
    const uint32_t n_books = n_wgs < BOOK_WGS ? n_wgs : BOOK_WGS;
    const SegSums missed(r.counts + SC_MISS * SEGS, r.n_seg);
    if (!missed.total) return;
    for (uint32_t seg = bx; seg < r.n_seg; seg += n_books) {
        const uint32_t lane_of = seg >> 2, i = seg & 3;
        const uint32_t before = lane_value(i == 0 ? missed.before : i == 1 ? missed.upto[0] : i == 2 ? missed.upto[1] : missed.upto[2], lane_of);
        const uint32_t n = lane_value(i == 0 ? missed.upto[0] : i == 1 ? missed.upto[1] : i == 2 ? missed.upto[2] : missed.upto[3], lane_of) - before;
        const uint32_t *from = r.seg_miss + (uint64_t)seg * r.seg_cells;
        constexpr uint32_t AT_ONCE = 4;
        for (uint32_t k0 = tid; k0 < n; k0 += NTHR * AT_ONCE) {
            uint32_t cell[AT_ONCE];
#pragma unroll
            for (uint32_t k = 0; k < AT_ONCE; ++k) cell[k] = from[k0 + k * NTHR < n ? k0 + k * NTHR : k0];
#pragma unroll
            for (uint32_t k = 0; k < AT_ONCE; ++k) if (k0 + k * NTHR < n) r.miss_idx[before + k0 + k * NTHR] = cell[k];
        }
    }
}

// The next of the tiles t, t + gx, t + 2 gx, ... whose request HBM serves, or one beyond the last tile.  Where a grid is short most of the list
// may be of other tiers, lost or invalid, and to look at them one by one is a memory latency each: after two in a row 64 are looked at
// together (12 000 lost blocks of 2 x 32 KiB 53.2 us one by one, 12.5 this way).
__device__ inline uint64_t next_in_hbm(const Rec *__restrict__ recs, uint64_t t, uint32_t gx, uint64_t n_tiles, uint32_t tpr)
{
    for (; t < n_tiles; t += 64 * (uint64_t)gx) {
        const uint64_t mine = t + lane_id() * (uint64_t)gx;
        const uint64_t there = __ballot(mine < n_tiles && in_hbm((uint32_t)recs[mine < n_tiles ? (uint32_t)mine / tpr : 0].src & 3));
        if (there) return t + (uint32_t)__builtin_ctzll(there) * (uint64_t)gx;
    }
    return t;
}

// HBM tier.  NTHR threads per workgroup, one 16-byte load and store each: a tile is NTHR * 16 bytes, and the launch has about
// as many workgroups as tiles; a smaller grid loops.  The list length is written to pinned host memory: the
// host sizes the next launch from it, because workgroups that find no tile are not free (about 0.2 ns each on MI355X) while a
// grid somewhat short of the tile count costs little.
//
// Measured on MI355X (768 MiB gathered from scattered runs, read+write): one-wavefront workgroups (1 KiB tiles) move 6.29 TB/s
// from 32 KiB runs and 6.57 TB/s from 64 KiB runs, 256-thread workgroups 6.12 and 6.40 - a wavefront that is its own
// workgroup frees its slot the moment it is done instead of waiting for three others.  Two or four loads per thread lose
// (5.9 and 5.6-5.9 against 6.2-6.5 TB/s), shifts in place of the division change nothing (6.29 against 6.30): the memory
// system's queues are full.
//
// FOLD: the planes of a request are taken in one pass - tile numbers run through plane 0, then plane 1, of each
// request - instead of plane after plane over the whole list.  Where the cache tier keeps the planes of an
// object next to each other this turns two 32 KiB source runs into one 64 KiB run, the length from which scattered
// runs read as fast as a contiguous buffer (6.29 -> 6.57 TB/s in the measurement above); where the planes live in
// pools of their own, plane after plane is the faster order (6.24 against 6.11 TB/s), and where chunks are shorter than 32 KiB too
// (two planes' destinations take turns every 16 KiB: 16 384 blocks 182.2 us against 178.4).
//
// blockIdx.y is the plane (unless folded), blockIdx.z the layer (MULTI): what a workgroup that lives for one load and one store
// has to work out first is kept to a division.
template <int NTHR, int PLANES, bool FOLD, bool MULTI>
__global__ __launch_bounds__(NTHR) void gather(const Rec *__restrict__ hbm_recs, const uint32_t *__restrict__ cnt, GatherArgs a, GatherRest)
{
    constexpr uint32_t TILE = NTHR * 16;
    constexpr uint32_t REST = 2 * sizeof(void *) + sizeof(GatherArgs);
    if (blockIdx.x < a.n_host) {
        if (blockIdx.y | blockIdx.z) return;               // the host tier's workgroups walk all planes and layers themselves
        k_GatherRest &rest = gather_rest<REST>();
        HostList recs(rest);
        if (blockIdx.x == 0 && threadIdx.x == 0) link_announce(rest.lease, (uint64_t)recs.sums.total * a.chunk_bytes * PLANES * a.n_rep);
        if (a.host_loads == HOST_PAGE) host_tier<NTHR, PLANES, HOST_PAGE>(recs, a, blockIdx.x);
        else host_tier<NTHR, PLANES, 2>(recs, a, blockIdx.x);
        return;
    }
    const uint32_t bx = blockIdx.x - a.n_host, gx = a.hbm_wgs, plane_y = FOLD ? 0 : blockIdx.y, rep = MULTI ? blockIdx.z : 0;
    // The first tile's list entry is fetched before the length is known, so that the two scalar loads overlap: a
    // workgroup lives for one load and one store, and every dependent load in front of them costs bandwidth.  The
    // host never launches more workgroups (per plane) than the list has room for tiles, so the early read stays inside
    // the list; it also guarantees capacity * tiles per request < 2^32, so tile numbers fit 32-bit division.
    uint32_t tpc = a.tiles_per_chunk;
    uint32_t tpr = FOLD ? tpc * PLANES : tpc;              // tiles per request in this plane's tile numbers
    uint64_t t = bx;
    uint32_t idx = (uint32_t)t / tpr;
    Rec x = hbm_recs[idx];
    uint32_t n_req = cnt[C_LIST];
    in_registers(x.src, x.dst, n_req, tpr);
    uint64_t n_tiles = (uint64_t)n_req * tpr;
    while (t < n_tiles) {
        uint32_t k = (uint32_t)t - idx * tpr;
        uint32_t plane = FOLD ? (k >= tpc ? 1u : 0u) : plane_y;
        uint64_t off = (uint64_t)(FOLD ? k - plane * tpc : k) * TILE;
        uint32_t tier = (uint32_t)(x.src & 3);
        if (in_hbm(tier)) {
            uint64_t src = src_base_of(a, tier, plane) + (x.src & ~(uint64_t)3) + off;
            uint64_t dst = (plane ? a.dst_base[1] : a.dst_base[0]) + x.dst + off;
            if (MULTI) { src += rep * layer_stride_of(a, tier); dst += rep * a.dst_step; }
            copy_tile<NTHR, 1, true>(src, dst, a.chunk_bytes - off, threadIdx.x);
        }
        t += gx;
        if (t >= n_tiles) break;
        idx = (uint32_t)t / tpr;
        x = hbm_recs[idx];
        if (!in_hbm(tier) && !in_hbm((uint32_t)x.src & 3)) {
            t = next_in_hbm(hbm_recs, t + gx, gx, n_tiles, tpr);
            if (t >= n_tiles) break;
            idx = (uint32_t)t / tpr;
            x = hbm_recs[idx];
        }
    }
    if (bx < BOOK_WGS && plane_y == 0 && rep == 0) keep_books<NTHR>(gather_rest<REST>(), bx, gx);
}

// A head-major working layout: a pool block is [token][head][head_bytes], the destination of a sequence [head][token][head_bytes].
struct HmArgs {
    uint32_t n_heads;
    uint32_t upr;             // 16-byte units per head row (head_bytes / 16)
    uint32_t ups;             // units one block adds to one head strip (block_tokens * upr)
    uint32_t pad;
    // unit number u of a block in destination order: where it is in the block, in units, and where it goes from the sequence's
    // first row of this block on, in bytes (cap: destination blocks of the sequence)
    __device__ inline void by_destination(uint32_t u, uint64_t cap, uint32_t &unit, uint64_t &to) const
    {
        const uint32_t head = u / ups, rem = u - head * ups, tok = rem / upr, col = rem - tok * upr;
        unit = (tok * n_heads + head) * upr + col;
        to = head * (cap * ups * 16) + (uint64_t)rem * 16;
    }
    // ... and of unit number u in source order, where it goes
    __device__ inline uint64_t by_source(uint32_t u, uint64_t cap) const
    {
        const uint32_t row_units = n_heads * upr, tok = u / row_units, rem = u - tok * row_units, head = rem / upr, col = rem - head * upr;
        return head * (cap * ups * 16) + (uint64_t)(tok * upr + col) * 16;
    }
};

// The whole KV fetch in one kernel, for small block tables.  A fetch of a few blocks is made of launch
// gaps, not of bytes.  blockIdx.y is the plane, blockIdx.z counts consecutive layers (an object has the same slot in every
// layer): layer + z is read, dst_step * z further into the destination is written.  NTHR is 256, or 64 for tables of up to 64 *
// ROUND cells, which a single wavefront walks at once and whose tiles are a little faster as workgroups of one (16 blocks of 32
// layers: 14.5 us with 256, 13.1 with 64, before a microsecond of event behind it).  blockIdx.x says what a workgroup does:
//
//   the first n_host  walk the table, list the host's cells in LDS and read them over PCIe, all planes and layers, two loads in
//                     flight per thread (see host_tier for why so few): 102 of 256 blocks of 2 x 32 KiB from the host take
//                     122.7 us, the call.  When every host tile was read at once, by a workgroup of its own, 6.7 MB of reads queued
//                     on the link together: 134 us.
//                     A table that takes several rounds to walk is shared out: workgroup b belongs to group b modulo their number, and a
//                     group walks its own share of the cells (shared_cell) and reads what it finds.  A round of a walk
//                     costs its workgroup a microsecond of waits in which it reads nothing: 2 877 cells of 2 x 16 KiB, 52 of them
//                     on the host, take 37.1-37.8 us in two groups and took 39.6-40.9 when every workgroup walked all six rounds.
//   the next one      walks the table too and keeps the books: counters, and the miss list in request order.  No atomics on
//                     shared counters (a thousand of them on one address take longer than the copy), nothing to zero.
//   the others        copy a tile of 16 bytes a thread, or twice that (U), if their cell's block is in HBM: nothing is compacted, so the grid
//                     covers the padded table - which is why this is for small tables only.  Resolving the cell in every workgroup costs
//                     little bandwidth (1 750 blocks of 2 x 16 KiB: 5.77 TB/s against 6.00 from a list, whose making
//                     takes longer than that saves).  Non-temporal accesses: on blocks that are in no cache 1 000 take 23.4 us
//                     against 27.1 for plain ones, 2 000 43.7 against 51.3.
//
// Nothing makes the directory hold still meanwhile: a revocation publishes its entries while fetches are in flight, and a placement
// on another stream when its copy has ended.  So workgroups may read different entries of a cell.  Two rules see to it that every byte
// is copied all the same.  An entry that may have changed under the launch (entry_young) is copied by whoever reads it, from where the
// entry says: of a cell's tile workgroup and its reader in the host's groups, whichever saw the older entry, the other then sees the
// younger one or copies anyway (4 096 blocks fetched from the cache tier and revoked by the next call: without it up to all of them were
// missing in the destination).  And which member of a group reads which piece of a cell follows from the cell's number alone
// (first_piece), whatever else that member has listed: were the list dealt out by position, members that had listed one cell more or
// less than others would leave pieces of cells that nobody has edited to each other.  (Objects without a host copy can leave nothing to
// copy from: with any around, fetches resolve in one place, on the general path.)
//
// HM: into the head-major layout.  Tiles of the HBM tier are taken in destination order, the host's in source order, as in gather_hm
// and host_tier_hm.  8 x 16 blocks of 2 x 32 KiB take 7.8 us, 1 024 blocks 25.4 (28.5 from a list), 4 096 98.3 (99.3; every head's
// strip 16 MiB from the next).
//
// A walk goes ROUND * NTHR cells at a time; the next round's row lengths and block numbers are on their way while this one's directory
// entries and destinations are, so a round costs one memory latency, not two.  The code of the walk is kept short on
// purpose: it runs once, and one wavefront doing the books with everything unrolled took 7 us for a table of 8 cells.
struct SmallTier { uint64_t base[2], layer_stride, slot_stride; };     // [plane], at the fetch's first layer
// What every workgroup is told ...
struct SmallArgs {
    uint64_t dst_cap;
    const uint64_t *dir;
    uint64_t chunk_bytes;
    uint32_t max_blocks, n_objects, n_rep, tiles_per_chunk, n_host, hbm_wgs;
    uint32_t n_cache_slots, n_local_slots;
    uint64_t dst_base[2], dst_step;      // [plane]; from one layer to the next
    SmallTier cache, local;
};
// ... and what only those need that walk the table, and tiles of blocks that are just changing.  They read it where they need it: as
// an ordinary argument all of it would be loaded at the start of the kernel and spilled to be out of the way (23 to 34 registers are
// spilled in the token-major forms, two of them by a tile's workgroup; 57 to 100, 38 of them there, in one argument: 16 blocks of 32 layers 15.7 us
// instead of 14.1, 300 blocks 10.8 instead of 9.7).
struct SmallWalk {
    SmallTier host;
    uint32_t n_host_slots, total;
    uint32_t n_seq, seen;                // the latest directory edit that the fetch comes after ...
    const uint32_t *snap;                // ... or where that is kept
    // the host's readers: the walk for the host's cells is cut into 1 << host_lg_groups shares, and what a workgroup reads of a cell at a
    // time is 1 << host_lg_run KiB, a piece: this many to a plane and layer, to a cell; of a cell at most so many are a workgroup's;
    // see first_piece
    uint32_t host_lg_groups, host_lg_run, host_ppc, host_pieces, host_per_cell, host_starts, host_step, pad;
    uint32_t *miss_idx, *cnt, *info;     // the books; info may be null
    unsigned long long *totals;
    Report *report;
    unsigned long long *lease;
};
typedef const __attribute__((address_space(4))) SmallWalk k_SmallWalk;
constexpr uint32_t SMALL_WALK_AT = 3 * sizeof(void *) + sizeof(SmallArgs);      // among the kernel's arguments
static_assert(sizeof(SmallArgs) % 8 == 0, "SmallWalk follows in the kernel's arguments");
template <bool HM> struct SmallHm { __device__ uint64_t by_source(uint32_t, uint64_t) const { return 0; } };
template <> struct SmallHm<true> : HmArgs { const uint32_t *seq_cap_blocks; };

constexpr uint32_t ROUND = 2;            // cells a thread looks up at a time when a workgroup walks the table
constexpr uint64_t SRC_MASK = 0x0000FFFFFFFFFFFCull;      // of a record's source: without tier and capacity

// Cell number i of group q's share, of 1 << lg_groups shares: one of the cells i << lg_groups and on, every group another one.
// Which one changes from i to i by a hash: with q itself, blocks on the host that recur with the period of the groups - every
// other row's, say - would all fall to one group.
__device__ inline uint32_t shared_cell(uint32_t i, uint32_t q, uint32_t lg_groups)
{
    return (i << lg_groups) + ((q ^ (i * 0x9E3779B1u >> 16)) & ((1u << lg_groups) - 1u));
}
// What a group's members read of cell number i of its share: its `pieces` - 1 << host_lg_run KiB of one plane and layer, plane after
// plane, layer after layer - are dealt out in turn, and this is the first one that `member` gets; every members-th from there on is its
// too.  The cell's first piece goes to a member that a hash of i names (top bits of the product: cells that follow each other are
// spread evenly, as are most that are a fixed distance apart), one of host_starts that are host_step apart.
__host__ __device__ inline uint32_t first_piece(uint32_t i, uint32_t member, uint32_t members, uint32_t starts, uint32_t step)
{
    const uint32_t at = ((i * 0x9E3779B1u >> 16) * starts >> 16) * step;
    return member >= at ? member - at : member + members - at;
}

// The numbers that follow from n_host, host_lg_groups, chunk_bytes and n_rep.  A piece is 4 KiB, a page of host memory, which the four
// wavefronts of a workgroup read side by side, or half or a quarter of that where a cell would not have one for every member otherwise:
// members whose loads are uneven leave the link idle at the end (102 of 256 blocks of 2 x 32 KiB from the host 123.6 us, 124.0 with 4 KiB
// in any case; 300 of 2 000 of 2 x 16 KiB 178.9 and 179.7).
inline void deal_out_host_pieces(SmallArgs &a, SmallWalk &w, uint32_t n_planes, uint32_t nthr)
{
    a.n_host &= ~((1u << w.host_lg_groups) - 1u);                // groups of the same size
    const uint32_t members = a.n_host >> w.host_lg_groups;
    auto cut = [&](uint32_t lg_run) {
        w.host_lg_run = lg_run;
        w.host_ppc = (uint32_t)((a.chunk_bytes + (1024ull << lg_run) - 1) >> (10 + lg_run));
        w.host_pieces = w.host_ppc * n_planes * a.n_rep;
    };
    cut(nthr == 64 ? 0 : 2);
    while (w.host_lg_run && w.host_pieces < members) cut(w.host_lg_run - 1);
    if (!members) return;
    w.host_per_cell = (w.host_pieces + members - 1) / members;
    const bool in_runs = members % w.host_pieces == 0;
    w.host_starts = in_runs ? members / w.host_pieces : members;
    w.host_step = in_runs ? w.host_pieces : 1;
}

template <int PLANES, int NTHR, bool HM, int U = 1>
__global__ __launch_bounds__(NTHR, 8) void fetch_kv_small(const int32_t *__restrict__ table, const int32_t *__restrict__ n_blocks,
                                                        const uint64_t *__restrict__ seq_dst_block, SmallArgs a, SmallWalk, SmallHm<HM> h)
{
    k_SmallWalk &w = *(k_SmallWalk *)((const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr() + SMALL_WALK_AT);
    const uint32_t tpc = a.tiles_per_chunk, tid = threadIdx.x, max_blocks = a.max_blocks;
    // several layers: blockIdx.z == 0 is a slice of its own for the head workgroups, not n_host + 1 idle ones in every layer
    const bool sliced = a.n_rep > 1, head = sliced ? blockIdx.z == 0 : blockIdx.x <= a.n_host;
    if (!head) {
        const uint32_t t = sliced ? blockIdx.x : blockIdx.x - a.n_host - 1, z = sliced ? blockIdx.z - 1 : 0;
        if (t >= a.hbm_wgs) return;                                // (several layers, and the head slice is the wider one)
        const uint32_t r = t / tpc, k = t - r * tpc, plane = blockIdx.y;
        const uint32_t s = r / max_blocks, j = r - s * max_blocks;
        const int32_t nb = n_blocks[s], b = table[r];
        const uint64_t first = seq_dst_block[s], dst_chunk = first + j;
        uint64_t cap = 0;
        bool fits;
        if constexpr (HM) { cap = h.seq_cap_blocks[s]; fits = (first + cap <= a.dst_cap) & (j < cap) & (cap < 65536); }
        else fits = dst_chunk < a.dst_cap;
        // as resolve_cell; one condition, so that the loads before it are on their way together
        if (!(fits & (nb > 0) & (j < (uint32_t)nb) & (b >= 0) & ((uint32_t)b < a.n_objects))) return;
        const uint64_t e = a.dir[b];
        const uint64_t dst_plane = (plane ? a.dst_base[1] : a.dst_base[0]) + (sliced ? z * a.dst_step : 0);
        const uint64_t cache = plane ? a.cache.base[1] : a.cache.base[0], local = plane ? a.local.base[1] : a.local.base[0];
        in_registers(cache, local, a.cache.slot_stride, a.n_cache_slots);
        const int tier = (int)entry_tier(e);
        const uint64_t off = (uint64_t)k * (NTHR * 16 * U);
        const uint64_t slot = entry_slot(e);
        uint64_t src;
        if (tier == T_CACHE || tier == T_LOCAL) {
            const bool cached = tier == T_CACHE;
            if (slot >= (cached ? a.n_cache_slots : a.n_local_slots)) return;
            src = (cached ? cache : local) + slot * (cached ? a.cache.slot_stride : a.local.slot_stride);
            if (sliced) src += z * (cached ? a.cache.layer_stride : a.local.layer_stride);
        } else {
            if (tier != T_HOST || !entry_young(e, w.snap ? *w.snap : w.seen) || slot >= w.n_host_slots) return;
            src = (plane ? w.host.base[1] : w.host.base[0]) + slot * w.host.slot_stride + z * w.host.layer_stride;
        }
        if constexpr (HM) {
            const uint64_t dst = dst_plane + first * a.chunk_bytes + (uint64_t)j * h.ups * 16;
            if (off + tid * 16 >= a.chunk_bytes) return;
            u32x4 v[U];
            uint64_t to[U];
            bool there[U];
#pragma unroll
            for (int i = 0; i < U; ++i) {                          // (a load of every turn, so that they are on their way together)
                const uint32_t u = (k * U + i) * NTHR + tid;
                uint32_t unit;
                there[i] = i == 0 || (uint64_t)u * 16 < a.chunk_bytes;
                h.by_destination(there[i] ? u : k * U * NTHR + tid, cap, unit, to[i]);
                v[i] = ld16<true>(reinterpret_cast<const u32x4 *>(src) + unit);
            }
#pragma unroll
            for (int i = 0; i < U; ++i) if (there[i]) st16<true>(reinterpret_cast<u32x4 *>(dst + to[i]), v[i]);
        } else {
            copy_tile<NTHR, U, true>(src + off, dst_plane + dst_chunk * a.chunk_bytes + off, a.chunk_bytes - off, tid);
        }
        return;
    }
    if (blockIdx.y || blockIdx.x > a.n_host) return;
    constexpr uint32_t WAVES_N = NTHR / 64;
    const bool keeper = blockIdx.x == a.n_host;
    const uint32_t wave = tid >> 6, seen = w.snap ? *w.snap : w.seen;
    const uint32_t lg = keeper ? 0 : w.host_lg_groups, last = (1u << lg) - 1u;         // the keeper's share is the whole table
    const uint32_t group = blockIdx.x & last, member = blockIdx.x >> lg, members = a.n_host >> lg, share = (w.total + last) >> lg;
    __shared__ Rec s_list[NTHR * ROUND];               // the round's cells on the host of which this workgroup reads something
    __shared__ uint32_t s_first[NTHR * ROUND];         // ... its first piece of each
    __shared__ uint32_t s_sum[ROUND * WAVES_N];
    __shared__ uint32_t s_cnt[C_N];
    uint32_t n[6] = { 0, 0, 0, 0, 0, 0 };            // requests, local, cache, host, lost, invalid, of this wavefront
    uint32_t n_miss = 0;
    if (tid < C_N) s_cnt[tid] = 0;
    auto ask = [&](uint32_t i) { return ask_cell(table, n_blocks, max_blocks, shared_cell(i, group, lg), w.total); };
    Ask next[ROUND];
#pragma unroll
    for (uint32_t i = 0; i < ROUND; ++i) next[i] = ask(i * NTHR + tid);
    for (uint32_t first = 0; first < share; first += NTHR * ROUND) {
        int tier[ROUND];
        Ask now[ROUND];
        uint64_t e[ROUND], to0[ROUND];               // directory entry; the sequence's first destination block
        uint32_t cap[ROUND];                         // ... and how many it has (head-major)
#pragma unroll
        for (uint32_t i = 0; i < ROUND; ++i) {
            now[i] = next[i];
            to0[i] = seq_dst_block[now[i].s];
            cap[i] = 0;
            if constexpr (HM) cap[i] = h.seq_cap_blocks[now[i].s];
            e[i] = a.dir[now[i].n > now[i].j && now[i].b >= 0 && (uint32_t)now[i].b < a.n_objects ? now[i].b : 0];
        }
#pragma unroll
        for (uint32_t i = 0; i < ROUND; ++i) next[i] = ask(first + (ROUND + i) * NTHR + tid);
        uint32_t piece0[ROUND];
#pragma unroll
        for (uint32_t i = 0; i < ROUND; ++i) piece0[i] = first_piece(first + i * NTHR + tid, member, members, w.host_starts, w.host_step);
        uint32_t rank[ROUND];                        // among the round's listed cells, in cell order: the host's, or the missed ones
        bool lists[ROUND];
#pragma unroll
        for (uint32_t i = 0; i < ROUND; ++i) {
            // (Without branches.  They cost more than what they skip; and written with && and ||, the compiler once left out the very
            // assignment of 4.)
            const int t = (int)entry_tier(e[i]);
            const bool known = (now[i].b >= 0) & ((uint32_t)now[i].b < a.n_objects), asked = now[i].n > now[i].j;
            const bool fits = HM ? (to0[i] + cap[i] <= a.dst_cap) & (now[i].j < cap[i]) & (cap[i] < 65536) : to0[i] + now[i].j < a.dst_cap;
            const bool there = (t == T_NONE) | (entry_slot(e[i]) < (t == T_HOST ? w.n_host_slots : t == T_CACHE ? a.n_cache_slots : a.n_local_slots));
            tier[i] = asked ? ((known & fits & there) ? t : 4) : -1;
            const bool young = ((tier[i] == T_CACHE) | (tier[i] == T_LOCAL)) & entry_young(e[i], seen);
            lists[i] = (tier[i] == T_HOST) | (keeper ? tier[i] == T_NONE : young);
            lists[i] &= keeper | (piece0[i] < w.host_pieces);
            uint32_t in_wave;
            rank[i] = wave_rank(lists[i], in_wave);
            if (lane_id() == 0) s_sum[i * WAVES_N + wave] = in_wave;
        }
        __syncthreads();
        uint32_t listed = 0;
#pragma unroll
        for (uint32_t k = 0; k < ROUND * WAVES_N; ++k) {
            if ((k & (WAVES_N - 1)) == wave) rank[k / WAVES_N] += listed;
            listed += s_sum[k];
        }
        listed = uniform(listed);
        if (!keeper && listed) {
#pragma unroll
            for (uint32_t i = 0; i < ROUND; ++i) {
                if (!lists[i]) continue;
                uint64_t src = entry_slot(e[i]) * w.host.slot_stride, dst = to0[i] * a.chunk_bytes;
                if (tier[i] != T_HOST)               // (T_HOST is 0)
                    src = entry_slot(e[i]) * (tier[i] == T_CACHE ? a.cache.slot_stride : a.local.slot_stride) | (uint64_t)tier[i];
                if constexpr (HM) { src |= (uint64_t)cap[i] << 48; dst += (uint64_t)now[i].j * h.ups * 16; }
                else dst += now[i].j * a.chunk_bytes;
                s_list[rank[i]] = { src, dst };
                s_first[rank[i]] = piece0[i];
            }
            __syncthreads();
            // A piece is read by 1 << lg_run wavefronts, a kilobyte each; the workgroup's other wavefronts are at other pieces meanwhile.
            // The lanes work out 64 pieces at a time, which all of them then read one after the other, two in flight (four where there
            // are single wavefronts).
            const uint32_t chunk_units = (uint32_t)(a.chunk_bytes >> 4), lg_run = NTHR == 64 ? 0 : w.host_lg_run, sets = WAVES_N >> lg_run;
            const uint32_t set = uniform(wave >> lg_run), sub = uniform(wave & ((1u << lg_run) - 1u));
            const uint32_t n_slots = listed * w.host_per_cell;
            for (uint32_t slot0 = set; slot0 < n_slots; slot0 += 64 * sets) {
                const uint32_t slot = slot0 + lane_id() * sets;
                bool there = slot < n_slots;
                uint32_t idx = there ? slot : 0, later = 0, rep = 0;
                if (w.host_per_cell > 1) { idx /= w.host_per_cell; later = (slot - idx * w.host_per_cell) * members; }
                const Rec x = s_list[idx];
                uint32_t piece = s_first[idx] + later;
                if (piece >= w.host_pieces) { there = false; piece = 0; }
                if (a.n_rep > 1) { rep = piece / (w.host_ppc * PLANES); piece -= rep * (w.host_ppc * PLANES); }
                const uint32_t plane = PLANES == 2 && piece >= w.host_ppc;
                const uint32_t from = (uint32_t)(x.src & 3);
                const uint32_t unit = there ? (((piece - plane * w.host_ppc) << lg_run) + sub) * 64 : chunk_units, cap_of = HM ? (uint32_t)(x.src >> 48) : 0;
                // (the second plane as a difference, or every lane would load its pool's address from the arguments by itself)
                uint64_t src = w.host.base[0] + (plane ? w.host.base[1] - w.host.base[0] : 0);
                uint64_t dst = a.dst_base[0] + (plane ? a.dst_base[1] - a.dst_base[0] : 0) + x.dst;
                if (a.n_rep > 1) { src += rep * w.host.layer_stride; dst += rep * a.dst_step; }
                if (__ballot(from != T_HOST)) {      // rare
                    const SmallTier &x1 = a.cache, &x2 = a.local;
                    if (from == T_CACHE) src = (plane ? x1.base[1] : x1.base[0]) + rep * x1.layer_stride;
                    if (from == T_LOCAL) src = (plane ? x2.base[1] : x2.base[0]) + rep * x2.layer_stride;
                }
                src += x.src & (HM ? SRC_MASK : ~(uint64_t)3);
                const uint64_t whole = __ballot(unit + 64 <= chunk_units), any = __ballot(there);
                auto to_at = [&](uint32_t k, uint32_t u) {
                    const uint64_t to = lane_value(dst, k);
                    return reinterpret_cast<u32x4 *>(to + (HM ? h.by_source(u, lane_value(cap_of, k)) : (uint64_t)u * 16));
                };
                auto from_at = [&](uint32_t k, uint32_t u) { return reinterpret_cast<const u32x4 *>(lane_value(src, k)) + u; };
                auto unit_at = [&](uint32_t k) { return lane_value(unit, k) + lane_id(); };
                auto read = [&](uint32_t k, auto count) {        // whole pieces: with a condition on a load the next one would wait for it
                    constexpr uint32_t N = decltype(count)::value;
                    u32x4 v[N];
#pragma unroll
                    for (uint32_t i = 0; i < N; ++i) v[i] = ld16<false>(from_at(k + i, unit_at(k + i)));
#pragma unroll
                    for (uint32_t i = 0; i < N; ++i) st16<true>(to_at(k + i, unit_at(k + i)), v[i]);
                    return N;
                };
                for (uint32_t k = 0; k < 64 && any >> k;) {
                    if (NTHR == 64 && (whole >> k & 15) == 15) k += read(k, Count<4>{});
                    else if ((whole >> k & 3) == 3) k += read(k, Count<2>{});
                    else {                           // the last of them, or a chunk's last piece
                        const uint32_t u = unit_at(k);
                        const u32x4 *from = from_at(k, u);
                        u32x4 *to = to_at(k, u);
                        if (u < chunk_units) st16<true>(to, ld16<false>(from));
                        k++;
                    }
                }
            }
        }
        if (keeper) {
#pragma unroll
            for (uint32_t i = 0; i < ROUND; ++i) {
                if (tier[i] == T_HOST || tier[i] == T_NONE) w.miss_idx[n_miss + rank[i]] = first + i * NTHR + tid;
                const bool pred[6] = { tier[i] >= 0, tier[i] == T_LOCAL, tier[i] == T_CACHE, tier[i] == T_HOST, tier[i] == T_NONE, tier[i] == 4 };
#pragma unroll
                for (int k = 0; k < 6; ++k) n[k] += (uint32_t)__popcll(__ballot(pred[k]));
            }
            n_miss += listed;
        }
        __syncthreads();                             // s_sum and s_list are written again
    }
    if (!keeper) return;
    if (lane_id() == 0) {
        const int to[6] = { C_REQ, C_LOCAL, C_CACHE, C_HOST, C_LOST, C_INVALID };
#pragma unroll
        for (int k = 0; k < 6; ++k) if (n[k]) atomicAdd(&s_cnt[to[k]], n[k]);
    }
    __syncthreads();
    if (tid <= C_INVALID) {
        const uint32_t x = s_cnt[tid];
        w.cnt[tid] = x;
        if (x) atomicAdd(&w.totals[tid], (unsigned long long)x);
        if (w.info) w.info[tid] = x;
    }
    if (tid == 0) {
        const uint32_t hbm = s_cnt[C_LOCAL] + s_cnt[C_CACHE], host = s_cnt[C_HOST];
        w.cnt[C_HBM_REQ] = hbm;
        w.cnt[C_HOST_REQ] = host;
        w.cnt[C_MISS] = n_miss;
        if (w.info) { w.info[6] = n_miss; w.info[7] = 0; }
        const u32x4 r = { hbm, host, w.n_seq, max_blocks };        // one store
        *reinterpret_cast<u32x4 *>(w.report) = r;
        link_announce(w.lease, (uint64_t)host * a.chunk_bytes * PLANES * a.n_rep);
    }
}

// A whole expert fetch in one kernel, for a few routing ids: what resolve_experts and the gather do in two launches, the first of which
// is a chain of latencies and a boundary between kernels.  Every workgroup forms the routed set for itself: a wavefront loads the ids at once and
// ors their bits together (by LDS atomics instead, 240 ids of 16 experts took 57 us against 42; by scalar loads and instructions the scalar unit,
// one for 32 wavefronts, becomes the bound).  Of experts that no cache holds, 4 of 17.3 MB take 25.4 us (27.6 in two launches), 11 59.7 (62.1), 14 74.8 (77.1), 8 of
// 4.3 MB 15.3 (19.3), 64 87.8 (97.8).  Two loads a thread, in 256 threads: 11 experts fetched again and again 60.5, and with one load, when the
// way to it takes too much of a workgroup's life, 65.5; four are more bytes in flight than the memory takes (63.2); 64 and 128 threads with
// two: 60.3, 60.5.  256 ids of 16
// experts of 4.3 MB 27.1 in two launches and 24.7; with room for 512 ids 24.9, and 512 of them 25.0, but 32 ids 45.3 instead of 45.1 and 11
// experts 60.6 instead of 60.4.
//
// The rank of an expert, its place in the staging buffer, is its rank in the set, whatever the directory says: the caller sees to it that
// all registered experts are in the cache tier or on the host.  A directory that changes under the fetch is met as in fetch_kv_small: an entry
// that is younger than `seen` is copied by whoever reads it, and which of the host's readers reads which tile of an expert follows from
// its rank alone.
//
// The first n_host workgroups read the host's experts (24 of them, 192 KiB in flight, see host_tier), the next one keeps the books, the others
// copy a tile each, or several of them where the grid is short.
constexpr uint32_t ROUTED_IDS = 256, ROUTED_EXPERTS = 128;      // routing ids and experts that the one kernel takes
typedef const __attribute__((address_space(4))) uint64_t k_entry;      // (by scalar loads)
struct RoutedArgs {
    const int32_t *topk;
    k_entry *dir;                        // of the layer
    uint64_t chunk_bytes, staging;
    uint64_t cache_base, cache_stride, host_base, host_stride;
    uint32_t n_experts, n_known;         // known: registered
    uint32_t n_cache_slots, n_host_slots;
    uint32_t n_ids, n_staging, tiles_per_chunk, n_host, hbm_wgs, seen;
};
struct RoutedBooks {
    ClassDev c;
    uint64_t *expert_ptr;
    uint32_t *miss_idx, *cnt;
    unsigned long long *totals, *lease;
    Report *report;
    uint32_t layer, pad;
};
typedef const __attribute__((address_space(4))) RoutedBooks k_RoutedBooks;
// The set of the routed experts, the same in all lanes.
struct Routed { uint64_t lo, hi; };      // experts 0 to 63, 64 to 127
__device__ inline Routed routed_set(const RoutedArgs &a)
{
    const uint32_t n = a.n_known < a.n_experts ? a.n_known : a.n_experts, lane = lane_id();
    uint32_t id[ROUTED_IDS / 64], bits[ROUTED_EXPERTS / 32] = { 0, 0, 0, 0 };
#pragma unroll
    for (uint32_t i = 0; i < ROUTED_IDS / 64; ++i) {
        id[i] = ~0u;
        if (i * 64 < a.n_ids) id[i] = (uint32_t)a.topk[i * 64 + lane < a.n_ids ? i * 64 + lane : 0];
    }
#pragma unroll
    for (uint32_t i = 0; i < ROUTED_IDS / 64; ++i)
#pragma unroll
        for (uint32_t k = 0; k < ROUTED_EXPERTS / 32; ++k) bits[k] |= id[i] < n && id[i] >> 5 == k ? 1u << (id[i] & 31) : 0u;
    Routed set = { (uint64_t)wave_or(bits[1]) << 32 | wave_or(bits[0]), 0 };
    if (a.n_experts > 64) set.hi = (uint64_t)wave_or(bits[3]) << 32 | wave_or(bits[2]);
    return set;
}
// Number r of the set, or ~0.
__device__ inline uint32_t routed_expert(const Routed &set, uint32_t r)
{
    const uint32_t n_lo = (uint32_t)__popcll(set.lo);
    const bool low = r < n_lo;
    const uint64_t m = low ? set.lo : set.hi;
    if (!low) r -= n_lo;
    // lane i: is expert i in the set, and the r-th of it
    const uint64_t it = __ballot((m >> lane_id() & 1) && (uint32_t)__popcll(m & ((1ull << lane_id()) - 1)) == r);
    if (!it) return ~0u;
    return (uint32_t)__builtin_ctzll(it) + (low ? 0 : 64);
}
template <int NTHR, int U>
__global__ __launch_bounds__(NTHR) void fetch_experts_small(RoutedArgs a, RoutedBooks)
{
    constexpr uint32_t TILE = NTHR * 16 * U;
    const uint32_t tid = threadIdx.x;
    if (blockIdx.x == a.n_host) {
        k_RoutedBooks &b = *(k_RoutedBooks *)((const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr() + sizeof(RoutedArgs));
        resolve_routed(b.c, b.layer, a.n_experts, a.topk, a.n_ids, a.staging, a.n_staging, b.expert_ptr, nullptr, nullptr, b.miss_idx,
                       b.cnt, b.totals, nullptr, nullptr, b.report, b.lease);
        return;
    }
    const Routed set = routed_set(a);
    if (blockIdx.x < a.n_host) {
        // tiles are numbered through the set, and every n_host-th one is this workgroup's
        const uint32_t tpc = a.tiles_per_chunk;
        uint32_t piece = blockIdx.x;     // of expert number r
        for (uint32_t r = 0; r < a.n_staging; ++r) {
            const uint32_t x = routed_expert(set, r);
            if (x == ~0u) return;
            const uint64_t e = a.dir[x], slot = entry_slot(e), dst = a.staging + (uint64_t)r * a.chunk_bytes;
            const bool host = entry_tier(e) == T_HOST, young = entry_tier(e) == T_CACHE && entry_young(e, a.seen);
            if ((host && slot < a.n_host_slots) || (young && slot < a.n_cache_slots)) {
                const uint64_t src = host ? a.host_base + slot * a.host_stride : a.cache_base + slot * a.cache_stride;
                for (; piece < tpc; piece += a.n_host)
                    copy_tile<NTHR, U, false>(src + (uint64_t)piece * TILE, dst + (uint64_t)piece * TILE, a.chunk_bytes - (uint64_t)piece * TILE, tid);
            } else if (piece < tpc) piece += (tpc - piece + a.n_host - 1) / a.n_host * a.n_host;
            piece -= tpc;
        }
        return;
    }
    for (uint32_t t = blockIdx.x - a.n_host - 1;; t += a.hbm_wgs) {
        const uint32_t r = t / a.tiles_per_chunk;
        if (r >= a.n_staging) return;
        const uint32_t x = routed_expert(set, r);
        if (x == ~0u) return;
        const uint64_t e = a.dir[x], slot = entry_slot(e), off = (uint64_t)(t - r * a.tiles_per_chunk) * TILE;
        const bool cached = entry_tier(e) == T_CACHE;
        if (cached ? slot < a.n_cache_slots : entry_tier(e) == T_HOST && entry_young(e, a.seen) && slot < a.n_host_slots) {
            const uint64_t src = cached ? a.cache_base + slot * a.cache_stride : a.host_base + slot * a.host_stride;
            copy_tile<NTHR, U, true>(src + off, a.staging + (uint64_t)r * a.chunk_bytes + off, a.chunk_bytes - off, tid);
        }
    }
}

// Host tier, WG threads, one load per plane in flight and twice as many threads as host_tier's (24 workgroups: 57.5 GB/s at
// 32 KiB chunks).  Threads walk the block in SOURCE order, so that every wave load is one contiguous kilobyte (PCIe reads of
// 256-byte pieces reach only 22 GB/s); the stores, which go to HBM, are the ones cut into head rows.  K and V of a unit go
// to the same place in their planes: one address computation serves both.
template <int PLANES>
__device__ inline void host_tier_hm(HostList &recs, const GatherArgs &a, const HmArgs &h, uint32_t b0)
{
    const uint32_t spc = a.tiles_per_chunk;
    const uint64_t n_sub = (uint64_t)recs.sums.total * spc;
    const uint32_t chunk_units = (uint32_t)(a.chunk_bytes >> 4);
    for (uint64_t g = b0; g < n_sub; g += a.n_host) {
        const uint32_t idx = (uint32_t)g / spc;
        const Rec x = recs[idx];
        const uint32_t u = ((uint32_t)g - idx * spc) * WG + threadIdx.x, unit = u < chunk_units ? u : 0;
        const uint64_t src = (x.src & 0x0000FFFFFFFFFFFCull) + (uint64_t)unit * 16;
        u32x4 v0 = ld16<false>(reinterpret_cast<const u32x4 *>(a.src_base[T_HOST][0] + src)), v1;
        if (PLANES == 2) v1 = ld16<false>(reinterpret_cast<const u32x4 *>(a.src_base[T_HOST][1] + src));
        const uint64_t d = x.dst + h.by_source(unit, x.src >> 48);
        if (u < chunk_units) {
            st16<true>(reinterpret_cast<u32x4 *>(a.dst_base[0] + d), v0);
            if (PLANES == 2) st16<true>(reinterpret_cast<u32x4 *>(a.dst_base[1] + d), v1);
        }
    }
}

// HBM tier: threads walk the block in DESTINATION order (16-byte units), so stores are
// fully contiguous per head strip and loads come as head_bytes-long runs (256 B at the paper-shaped config: two whole
// 128-byte lines).  No LDS: nothing is reused, the permutation is pure address arithmetic.  Staging through LDS was
// measured on MI355X and lost: a whole 32 KiB block per workgroup (source-order loads, 8 strips of 4 KiB stored) moves
// 5.31 TB/s against 5.81 for this kernel (12 041 scattered blocks, alone), and tiles of 4 tokens x 4 heads (every wave
// instruction a contiguous kilobyte on both sides) 5.91 in isolation but 5.85 against 5.94 once inside the library's
// looping, feedback-sized launch.  One-wavefront workgroups (1 KiB tiles), the token-major gather's shape, are a
// wash here: 5.95 against 5.90 TB/s alone, 5.32 against 5.35 inside the step.
template <int PLANES, bool SKIP>
__global__ __launch_bounds__(WG) void gather_hm(const Rec *__restrict__ hbm_recs, const uint32_t *__restrict__ cnt, GatherArgs a, HmArgs h,
                                                GatherRest)
{
    constexpr uint32_t REST = 2 * sizeof(void *) + sizeof(GatherArgs) + sizeof(HmArgs);
    if (blockIdx.x < a.n_host) {
        if (blockIdx.y) return;
        k_GatherRest &rest = gather_rest<REST>();
        HostList recs(rest);
        if (blockIdx.x == 0 && threadIdx.x == 0) link_announce(rest.lease, (uint64_t)recs.sums.total * a.chunk_bytes * PLANES);
        host_tier_hm<PLANES>(recs, a, h, blockIdx.x);
        return;
    }
    // SKIP: next_in_hbm, for grids that are known to be far too short.  With that code in its loop, though it does not run, the usual fetch
    // takes longer (12 000 blocks 271.7 and 274.0 us).
    // plane after plane: taking both planes of a request in one pass, as gather does for a cache tier that keeps
    // them side by side, was measured to lose here (5.60 against 5.98 TB/s alone): the stores are 4 KiB strips, and with
    // two planes' strips interleaved they no longer follow each other
    const uint32_t bx = blockIdx.x - a.n_host, gx = a.hbm_wgs, plane = blockIdx.y;
    uint32_t tpr = a.tiles_per_chunk;
    uint64_t t = bx;
    uint32_t idx = (uint32_t)t / tpr;
    Rec x = hbm_recs[idx];                               // speculative, as in gather
    uint32_t n_req = cnt[C_LIST];
    in_registers(x.src, x.dst, n_req, tpr);
    uint64_t n_tiles = (uint64_t)n_req * tpr;
    uint32_t chunk_units = (uint32_t)(a.chunk_bytes >> 4);
    while (t < n_tiles) {
        uint32_t k = (uint32_t)t - idx * tpr;
        uint64_t dst_plane = plane ? a.dst_base[1] : a.dst_base[0];
        uint32_t u = k * WG + threadIdx.x;
        uint64_t cap = x.src >> 48;
        uint32_t tier = (uint32_t)(x.src & 3);
        uint64_t src = src_base_of(a, tier, plane) + (x.src & 0x0000FFFFFFFFFFFCull);
        uint64_t dst = dst_plane + x.dst;
        if (in_hbm(tier) && u < chunk_units) {
            uint32_t s_unit;
            uint64_t d_off;
            h.by_destination(u, cap, s_unit, d_off);
            st16<true>(reinterpret_cast<u32x4 *>(dst + d_off), ld16<true>(reinterpret_cast<const u32x4 *>(src) + s_unit));
        }
        t += gx;
        if (t >= n_tiles) break;
        idx = (uint32_t)t / tpr;
        x = hbm_recs[idx];
        if (SKIP && !in_hbm(tier) && !in_hbm((uint32_t)x.src & 3)) {
            t = next_in_hbm(hbm_recs, t + gx, gx, n_tiles, tpr);
            if (t >= n_tiles) break;
            idx = (uint32_t)t / tpr;
            x = hbm_recs[idx];
        }
    }
    if (bx < BOOK_WGS && plane == 0) keep_books<WG>(gather_rest<REST>(), bx, gx);
}

// ---------------------------------------------------------------------------------------------------------
// Host-built lists (absolute addresses).
// ---------------------------------------------------------------------------------------------------------
// Placement and write-back.  The list has one record per object; which chunk a tile belongs to - object, plane, layer - is
// worked out per tile.  Up to MOVE_INLINE records are kernel arguments: 64 objects of 32 layers and two planes were 4 096
// addresses before, copied to the device by a memcpy of their own in front of the kernel (about 14 us on the stream).
// A kernel argument that is indexed by a variable would be copied to scratch memory, hence the segment pointer.
typedef const __attribute__((address_space(4))) MoveRec k_MoveRec;
typedef const __attribute__((address_space(4))) DirList k_DirList;
static_assert(sizeof(MoveArgs) % 8 == 0, "MoveList follows MoveArgs in the kernel's arguments");
struct MoveChunk { uint64_t src, dst0, dst1; };         // addresses of one chunk; 0: nowhere
template <bool INLINE>
__device__ inline MoveChunk move_chunk(const MoveArgs &a, uint32_t item)
{
    const uint32_t inner = a.order == ORDER_PLANE_LAYER_OBJ ? a.n_obj : a.n_planes, mid = a.order == ORDER_LAYER_OBJ_PLANE ? a.n_obj : a.n_layers;
    const uint32_t rest = item / inner, x0 = item - rest * inner, x2 = rest / mid, x1 = rest - x2 * mid;
    const uint32_t plane = a.order == ORDER_PLANE_LAYER_OBJ ? x2 : x0;
    const uint32_t layer = a.order == ORDER_LAYER_OBJ_PLANE ? x2 : x1;
    const uint32_t obj = a.order == ORDER_PLANE_LAYER_OBJ ? x0 : a.order == ORDER_LAYER_OBJ_PLANE ? x1 : x2;
    MoveRec x;
    if (INLINE) {
        k_MoveRec *r = (k_MoveRec *)((const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr() + sizeof(MoveArgs));
        x.src = r[obj].src; x.dst0 = r[obj].dst0; x.dst1 = r[obj].dst1;
    } else x = a.recs[obj];
    MoveChunk m;
    m.src = (plane ? a.src_base[1] : a.src_base[0]) + layer * a.src_layer + x.src;
    m.dst0 = x.dst0 == NOWHERE ? 0 : (plane ? a.host_base[1] : a.host_base[0]) + layer * a.host_layer + x.dst0;
    const uint64_t base1 = (x.dst1 & 3) == T_CACHE ? (plane ? a.cache_base[1] : a.cache_base[0]) + layer * a.cache_layer
                                                   : (plane ? a.local_base[1] : a.local_base[0]) + layer * a.local_layer;
    m.dst1 = x.dst1 == NOWHERE ? 0 : base1 + (x.dst1 & ~(uint64_t)3);
    if (m.dst1 == m.src) m.dst1 = 0;                    // a source that already is the slot needs no copy
    return m;
}

// Over PCIe, either way: a few persistent workgroups (harvest_config.pcie_wgs) with U loads per thread in flight, their tiles
// counted out one at a time from a.next: when something else is using the link as well, the
// workgroups of one launch progress at very different rates (a 3.4-fold spread was measured), and with fixed shares
// the launch ends with a few workgroups working off their backlog alone - a 906 MB placement beside a stream of
// fetches took 106 ms that way.  Only the first tile is the workgroup's own, without a draw - nothing has run at any rate yet, and lists of
// no more tiles than workgroups draw none at all (8 MiB to the host 78.3 us with a draw in front, 77.8 without, 1 MiB 23.0 and 22.8, 0.5 MiB
// in tiles of 16 KiB 13.9 and 13.4).  The counter is zero at launch and again at the end: every workgroup draws one number
// beyond the tiles, and the one that draws the last puts it back.  The next number is drawn while the tile is on its way; whether
// a fetch needs the link is asked last, right before the next tile's loads go out - asked along with the draw, the answer was a tile
// old, and a fetch of 200 blocks beside a placement of 32 workgroups took 1.56 ms instead of 0.98 (alone 0.25).
//
// TO_HOST, writes to the host: stores at system scope, which the L2 passes on as they come - 16 MiB take 296.5 us in tiles of 32 KiB
// (56.6 GB/s, the DMA engine 55.3), 304 with non-temporal stores, 316 with plain ones; 64 MiB 1 177, 1 203 and 1 220 us.  They are
// acknowledged by the host, so it takes more workgroups to keep their rate beside a kernel that fills the device (launch_move).  A
// list of up to THROUGH_FROM bytes the L2 takes as a whole, and non-temporal stores are faster (1 MiB: 22.3 us, 23.1 at system scope).
enum StoreWay { PLAIN_STORES, NT_STORES, THROUGH_STORES };
constexpr uint64_t THROUGH_FROM = 2u << 20;
template <int WAY> __device__ inline void st16_to(u32x4 *p, u32x4 v)
{
    if (WAY == THROUGH_STORES) __builtin_amdgcn_global_store_b128((g_u32x4 *)(uint64_t)p, v, "");
    else st16<WAY == NT_STORES>(p, v);
}
template <bool INLINE, int U, int WAY>
__global__ __launch_bounds__(WG) void move_pcie(MoveArgs a, MoveList)
{
    constexpr uint32_t TILE = WG * 16 * U;
    constexpr int WAY1 = WAY == PLAIN_STORES ? PLAIN_STORES : NT_STORES;        // of the copy that stays in HBM
    __shared__ unsigned long long s_tile[2];
    const uint32_t tid = threadIdx.x;
    const bool drawn = a.n_tiles > gridDim.x;            // otherwise every workgroup has the one tile that it starts with
    if (tid == 0) yield_link<TILE>(a.lease);
    __syncthreads();
    uint64_t t = blockIdx.x;
    for (uint32_t turn = 1; t < a.n_tiles; turn ^= 1) {
        const uint32_t item = (uint32_t)t / a.tiles_per_chunk;
        const uint64_t off = (uint64_t)((uint32_t)t - item * a.tiles_per_chunk) * TILE;
        const MoveChunk m = move_chunk<INLINE>(a, item);
        const u32x4 *s = reinterpret_cast<const u32x4 *>(m.src + off);
        u32x4 *d0 = reinterpret_cast<u32x4 *>(m.dst0 + off), *d1 = reinterpret_cast<u32x4 *>(m.dst1 + off);
        const uint64_t len = a.chunk_bytes - off;
        if (len >= TILE) {                       // whole tile: all loads in flight, then the stores
            u32x4 v[U];
#pragma unroll
            for (int i = 0; i < U; ++i) v[i] = ld16<false>(s + tid + i * WG);
            if (drawn && tid == 0) s_tile[turn] = gridDim.x + atomicAdd(a.next, 1ull);
            if (m.dst0) {
#pragma unroll
                for (int i = 0; i < U; ++i) st16_to<WAY>(d0 + tid + i * WG, v[i]);
            }
            if (m.dst1) {
#pragma unroll
                for (int i = 0; i < U; ++i) st16_to<WAY1>(d1 + tid + i * WG, v[i]);
            }
        } else {
            if (drawn && tid == 0) s_tile[turn] = gridDim.x + atomicAdd(a.next, 1ull);
            const uint32_t n_vec = (uint32_t)(len >> 4);
            for (uint32_t i = tid; i < n_vec; i += WG) {
                u32x4 v = ld16<false>(s + i);
                if (m.dst0) st16_to<WAY>(d0 + i, v);
                if (m.dst1) st16_to<WAY1>(d1 + i, v);
            }
        }
        if (!drawn) return;
        if (tid == 0) yield_link<TILE>(a.lease);
        __syncthreads();                         // two words in turn: nobody reads the one that is written next
        t = s_tile[turn];
    }
    if (tid == 0 && t == (uint64_t)a.n_tiles + gridDim.x - 1) __hip_atomic_store(a.next, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Between HBM pools only (placement from a staged copy, demotion of lossy objects): the HBM-tier gather's shape - one wavefront
// per workgroup, one 1 KiB tile each, non-temporal accesses (measured on 17 GB of staged experts: 6.30 TB/s, 4.99 TB/s in
// the persistent form).
template <bool INLINE>
__global__ __launch_bounds__(64) void move_hbm(MoveArgs a, MoveList)
{
    constexpr uint32_t TILE = 64 * 16;
    for (uint32_t t = blockIdx.x; t < a.n_tiles; t += gridDim.x) {
        const uint32_t item = t / a.tiles_per_chunk;
        const uint64_t off = (uint64_t)(t - item * a.tiles_per_chunk) * TILE;
        const MoveChunk m = move_chunk<INLINE>(a, item);
        const uint64_t len = a.chunk_bytes - off;
        const uint32_t n_vec = (uint32_t)((len > TILE ? TILE : len) >> 4);
        if (threadIdx.x < n_vec) {
            u32x4 v = ld16<true>(reinterpret_cast<const u32x4 *>(m.src + off) + threadIdx.x);
            if (m.dst0) st16<true>(reinterpret_cast<u32x4 *>(m.dst0 + off) + threadIdx.x, v);
            if (m.dst1) st16<true>(reinterpret_cast<u32x4 *>(m.dst1 + off) + threadIdx.x, v);
        }
        if (a.n_tiles - t <= gridDim.x) break;
    }
}

__global__ __launch_bounds__(WG) void fill_items(const Item *__restrict__ items, uint32_t n_items, uint64_t chunk_bytes,
                                                 uint32_t tiles_per_chunk, uint32_t pattern)
{
    constexpr uint32_t TILE = TILE_HOST;
    uint64_t n_tiles = (uint64_t)n_items * tiles_per_chunk;
    u32x4 v = { pattern, pattern, pattern, pattern };
    for (uint64_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
        uint64_t it = t / tiles_per_chunk;
        uint64_t off = (t - it * tiles_per_chunk) * TILE;
        uint64_t len = chunk_bytes - off;
        if (len > TILE) len = TILE;
        u32x4 *d = reinterpret_cast<u32x4 *>(items[it].dst + off);
        uint32_t n_vec = (uint32_t)(len >> 4);
        for (uint32_t i = threadIdx.x; i < n_vec; i += WG) st16<false>(d + i, v);
    }
}

// The same with the gather's shape: one wavefront per workgroup, one 1 KiB tile each.  Tile numbers are 32-bit: the host
// checks n_items * tiles_per_chunk.
template <int NTHR>
__global__ __launch_bounds__(NTHR) void fill_items_hbm(const Item *__restrict__ items, uint32_t n_items,
                                                       uint64_t chunk_bytes, uint32_t tiles_per_chunk, uint32_t pattern)
{
    constexpr uint32_t TILE = NTHR * 16;
    uint32_t n_tiles = n_items * tiles_per_chunk;
    u32x4 v = { pattern, pattern, pattern, pattern };
    for (uint32_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
        uint32_t it = t / tiles_per_chunk;
        uint64_t off = (uint64_t)(t - it * tiles_per_chunk) * TILE;
        uint64_t len = chunk_bytes - off;
        uint32_t n_vec = (uint32_t)((len > TILE ? TILE : len) >> 4);
        if (threadIdx.x < n_vec) st16<true>(reinterpret_cast<u32x4 *>(items[it].dst + off) + threadIdx.x, v);
        if (n_tiles - t <= gridDim.x) break;
    }
}

// Directory edits: from a host-built list, or (up to DIR_INLINE of them) from the kernel's arguments.  Every entry carries the
// number of its edit, and `done` says which edits are complete (for fetches in recorded graphs, which learn it when they are
// replayed): done[0] is the latest, done[1] counts workgroups.  Entries are written through to where every XCD sees them and
// waited for (a barrier of the workgroup alone waits for no store) before the number is.
__device__ inline void write_entry(uint64_t *dir, uint32_t id, uint64_t entry)
{
    __hip_atomic_store(dir + id, entry, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}
__global__ __launch_bounds__(WG) void dir_write(uint64_t *dir, const uint32_t *__restrict__ ids,
                                                const uint64_t *__restrict__ entries, uint32_t n, uint32_t *done, uint32_t edit)
{
    uint32_t i = blockIdx.x * WG + threadIdx.x;
    if (i < n) write_entry(dir, ids[i], entries[i]);
    __syncthreads();
    if (threadIdx.x) return;
    if (__hip_atomic_fetch_add(done + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != gridDim.x - 1) return;
    __hip_atomic_store(done + 1, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(done, edit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
struct DirArgs { uint64_t *dir; uint32_t *done; uint32_t n, edit; };
static_assert(sizeof(DirArgs) % 8 == 0, "DirList follows DirArgs in the kernel's arguments");
__global__ __launch_bounds__(DIR_INLINE) void dir_write_inline(DirArgs a, DirList)
{
    k_DirList *l = (k_DirList *)((const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr() + sizeof(DirArgs));
    if (threadIdx.x < a.n) write_entry(a.dir, l->id[threadIdx.x], l->entry[threadIdx.x]);
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(a.done, a.edit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The latest complete edit, for the fetch behind this kernel on the stream.
__global__ void snap_edit(const uint32_t *done, uint32_t *snap)
{
    *snap = __hip_atomic_load(done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ void system_fence() { __threadfence_system(); }

// harvest_fetch_kv_static's counters for a fetch that had no table cell and ran no kernel.
__global__ void zero_info(uint32_t *__restrict__ info)
{
    if (threadIdx.x < 8) info[threadIdx.x] = 0;
}

// Plain contiguous copy with the HBM-tier inner loop (reference ceiling / counter calibration).
template <int NTHR>
__global__ __launch_bounds__(NTHR) void plain_copy(uint64_t dst, uint64_t src, uint64_t bytes)
{
    constexpr uint32_t TILE = NTHR * 16;
    uint64_t n_tiles = (bytes + TILE - 1) / TILE;
    for (uint64_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
        uint64_t off = t * TILE;
        copy_tile<NTHR, 1, true>(src + off, dst + off, bytes - off, threadIdx.x);
    }
}

// Read-only and write-only streams (one non-temporal 16-byte access per thread): what the memory system delivers in each
// direction alone, from which the bound of any copy follows.  With one-wavefront workgroups these two measure the
// dispatcher instead (one access per workgroup: 4.8 TB/s, 4.7 G workgroups/s), so the host launches them with the
// workgroup size that was measured fastest: 1024 threads for reads (7.5 TB/s), 256 for writes (6.7 TB/s).
template <int NTHR>
__global__ __launch_bounds__(NTHR) void plain_read(uint64_t src, uint64_t bytes, uint32_t *sink)
{
    constexpr uint32_t TILE = NTHR * 16;
    uint64_t n_vec = bytes >> 4;
    uint32_t acc = 0;
    for (uint64_t t = blockIdx.x; t * (TILE / 16) < n_vec; t += gridDim.x) {
        uint64_t i = t * (TILE / 16) + threadIdx.x;
        if (i < n_vec) {
            u32x4 v = ld16<true>(reinterpret_cast<const u32x4 *>(src) + i);
            acc ^= v.x ^ v.y ^ v.z ^ v.w;
        }
    }
    if (acc == 0x9E3779B9u) *sink = acc;             // never true for the calibration buffers: keeps the loads alive
}

template <int NTHR>
__global__ __launch_bounds__(NTHR) void plain_write(uint64_t dst, uint64_t bytes, uint32_t pattern)
{
    constexpr uint32_t TILE = NTHR * 16;
    uint64_t n_vec = bytes >> 4;
    u32x4 v = { pattern, pattern, pattern, pattern };
    for (uint64_t t = blockIdx.x; t * (TILE / 16) < n_vec; t += gridDim.x) {
        uint64_t i = t * (TILE / 16) + threadIdx.x;
        if (i < n_vec) st16<true>(reinterpret_cast<u32x4 *>(dst) + i, v);
    }
}

}  // namespace hv
