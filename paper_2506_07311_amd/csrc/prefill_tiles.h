// Pieces shared by the matrix-core prefill kernels (internal header): tile geometry in LDS, the swizzle, the
// launch plan, and the tile fetch that lets the load unit write K/V rows straight into LDS.
#pragma once

#include "common.h"

namespace pa {
namespace prefill {

typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef mfma_f32x16 f32x16;
typedef __attribute__((ext_vector_type(8))) float f32x8;

constexpr int kBM = 128;              // rows per workgroup of the 32-rows-per-wave kernel
constexpr int kBN = 64;               // keys per tile
constexpr int kThreads = 256;
constexpr int kPreciseKeys = 256;     // contexts up to this length use two-term bf16 weights
constexpr int kRow = 256;             // bytes per K or V row in LDS (unpadded, pieces swizzled)
constexpr int kTileBytes = kBN * kRow;   // K part of a tile buffer; the V part follows
constexpr int kBufBytes = 2 * kTileBytes;

// 16-byte piece L of LDS row r is stored at piece L ^ swz(r).
__device__ __forceinline__ int swz(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// ---------------------------------------------------------------------------------------------------
// Tile fetch.  Wave w issues, for i < 4, one load-to-LDS instruction for K and one for V that fill rows
// 16*i + 4*w .. +3 of the tile: lane l brings the 16-byte piece that belongs at position l%16 of row
// 16*i + 4*w + l/16.  UNIFORM (page size >= 16): the four rows of an instruction lie in one page, so the page
// id is a scalar load and the page base scalar arithmetic; page ids are fetched one tile earlier than the rows.
// ---------------------------------------------------------------------------------------------------
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) const void glb_void;

// 16 bytes per lane from global memory straight into LDS (lane i lands at lds_addr + 16 i; lds_addr wave-uniform),
// written as ONE OPAQUE STATEMENT.  Issued through the compiler's builtin, a load that writes LDS is booked as an
// access that may complete out of order with LDS reads, and while one is in flight -- here: for the whole tile --
// every wait for an LDS read becomes a wait for ALL of them, which drains the operand pipeline of the matrix
// instructions (reads kept four ahead) at every step.  The compiler does not look inside this statement, so its
// LDS waits count exactly; the loads are waited for by hand (wait_tile_loads) in front of the barrier that
// publishes a tile.  Two forms: scalar 64-bit base + 32-bit lane offset, and a 64-bit lane address.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"   // m0 is written on purpose: it carries the LDS address of the load
// lds = wave-uniform LDS byte address, lds_imm = compile-time constant added to it
__device__ __forceinline__ void load_to_lds16(uint32_t lds, int lds_imm, const char* base, uint32_t off)
{
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(lds), "v"(off), "s"(base), "n"(lds_imm)
                 : "memory", "m0", "scc");
}
__device__ __forceinline__ void load_to_lds16(uint32_t lds, int lds_imm, const char* addr)
{
    asm volatile("s_add_u32 m0, %0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                 :
                 : "s"(lds), "v"(addr), "n"(lds_imm)
                 : "memory", "m0", "scc");
}
#pragma clang diagnostic pop
// LDS byte address of a (wave-uniform) pointer into a __shared__ array, as a scalar
__device__ __forceinline__ uint32_t lds_address(const char* p)
{
    return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)p);
}
// This wave's loads to LDS have landed (to be followed by the workgroup barrier).  The wait is the compiler's own
// instruction, not text: it also tells the compiler's bookkeeping that none of ITS loads is pending any more
// (otherwise the query fragments loaded in front of the tile loop would be waited for again inside the loop, with
// counts that the tile loads in flight turn into waits for the next tile).
__device__ __forceinline__ void wait_tile_loads()
{
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0), the other counters left alone
}

// A fold over the wave in data-parallel-primitive moves, STEP(control, rows that receive): shifts by 1, 2, 4, 8 inside each row
// of 16 lanes, then lane 15 of a row into the next row, lane 31 into the upper half; lane 63 holds the
// result, every other lane the fold over the lanes up to it.
#define PA_WAVE_FOLD(STEP) \
    STEP(0x111, 0xF) STEP(0x112, 0xF) STEP(0x114, 0xF) STEP(0x118, 0xF) STEP(0x142, 0xA) STEP(0x143, 0xC)

// Sum over the wave without six round trips through LDS in front of a workgroup's first tile (append + prefill of one prompt,
// 32 / 8 heads: 128 tokens 11.9 -> 11.6 us, 200 13.2 -> 13.0, 500 and more the same).
__device__ __forceinline__ float wave_sum_moves(float v)
{
#define PA_SUM_STEP(CTRL, ROWS) \
    v += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), CTRL, ROWS, 0xF, true));
    PA_WAVE_FOLD(PA_SUM_STEP)
#undef PA_SUM_STEP
    return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), 63));
}

// The same for the inclusive scans and sums that find an item (a workgroup without one 4.4 -> 3.8 us; 23 sequences of up to 5465
// tokens, three with 200 queries, 62.9 -> 60.7 us a call).
__device__ __forceinline__ int32_t wave_scan_moves(int32_t v)
{
#define PA_SCAN_STEP(CTRL, ROWS) v += __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, true);
    PA_WAVE_FOLD(PA_SCAN_STEP)
#undef PA_SCAN_STEP
    return v;
}
__device__ __forceinline__ int32_t wave_total_moves(int32_t v) { return __builtin_amdgcn_readlane(wave_scan_moves(v), 63); }

// How the launch cuts the work: head packing and the context split.
struct PrefillPlan {
    int32_t log2_pack;    // query heads of one KV head packed into a row tile (1 << log2_pack divides the group size)
    int32_t group;        // query heads per KV head
    int32_t chunk;        // context tokens per workgroup (multiple of 64 and of the page size when nsplit > 1)
    int32_t nsplit;       // chunks along the grid; > 1: partials go to part_o / part_lse for the merge kernel
    int32_t skip_small;   // 1: sequences with q_len * G <= 16 are computed by the decode kernel, not here
    int32_t list_items;   // > 0: work-list mode (below); at most list_items x head groups items, the grid steps over them
    float* list_o;        // its partials: [slot][wave][16 bytes of a lane][lane]
    float* list_lse;      // [slot][row]
    int32_t list_unit;    // chunks are multiples of this many tokens (a tile and a page)
    float* part_o;        // [total_q, Hq, nsplit, head_dim]
    float* part_lse;      // [total_q, Hq, nsplit]
    ModArgs mods;         // mask / score hooks (used by the instantiations that have them)
    int32_t chunk_unit;   // > 0: chunks by each sequence's own length instead (sequence_chunk; kLengthGrid, kEitherList)
    int32_t order;        // of the grid: one of the five below
};

// All row tiles of a context chunk, then the next chunk's; the row tiles that there are, in one piece (locate_live); chunk after
// chunk from the last one on; row tile after row tile, the chunks of one beside each other, and all that is in one piece; by each
// sequence's own length (chunk_unit).
constexpr int32_t kByChunk = 0, kLiveTiles = 1, kLastChunkFirst = 2, kByTile = 3, kByLengths = 4;

PrefillPlan make_plan(const AttnArgs& a);

// ---------------------------------------------------------------------------------------------------
// Work-list mode.  A jagged call (a few chunks of long prompts among decode rows) has neither of the shapes the plain
// grid serves: most of its (tile, sequence) pairs are empty, and the host, which knows no lengths, cannot see that a
// handful of workgroups would walk the longest contexts alone (60 decode rows + 4 chunks of 512 tokens, contexts
// of 2.7k to 31k tokens: 128 workgroups of 490 tiles each set the time, 1510 us, with three quarters of the machine
// idle).  Here every wave derives the same list from cu_q_lens and seq_lens: row tiles of the live sequences only, the
// context of a sequence cut into chunks of one length, chosen so that the call has about kListTarget work items
// (two per workgroup slot; none shorter than kListMinTiles, where a workgroup's start and its partial begin to show).
// Item order: sequence, chunk, row tile from last to first, head group -- the workgroups that run together on a
// chiplet walk the same keys, so a chunk's K/V comes from HBM once per head.  Same call: prefill kernel
// 1510 -> 460 us (410 GFLOP: 0.9 PFLOP/s) + 10 us of merging; the whole call 1690 -> 655 us (560 with the few-query sequences
// beside it in the same launch).  All whole chunks come before the shorter ones that end the sequences (list_locate): an
// item is a sixth of the launch, so the last ones to start decide when it ends (574 -> 557; 64 sequences of up to
// 13000 tokens, eight with 200 queries, 276 -> 267, 24 such calls 0.98 in the mean).
// ---------------------------------------------------------------------------------------------------
constexpr int32_t kListTarget = 1024;
constexpr int32_t kListMinTiles = 32;
// ... except that chunks may be as short as kListShortTiles while all items fit the workgroup slots of the machine (two
// per compute unit up to head_dim 128): one chunk of 512 tokens on 2787 among 16 sequences 73 us against 86 with 32 tiles, but
// six chunks of 200 tokens on up to 3508, whose 728 items of 16 tiles need a second round, 134 against 123.
constexpr int32_t kListShortTiles = 16;
// At head_dim 256 one workgroup fits a compute unit (200 queries among 17 sequences of up to 8000 tokens, 32 / 8 heads, 186 -> 158
// us, two of 200 among 30 to 6000 180 -> 161, calls with more work 340 - 369 the same).  At head_dim 64 three do, but slots for
// 768 items gain nothing in the mean (60 sequences to 4500, six with 200, 95 -> 88, 40 to 12000, three with 200, 93 -> 97).
__host__ __device__ constexpr int32_t list_wg_slots(int32_t d) { return d > 128 ? 256 : 512; }
// Workgroups of the launch and of its merge (an eighth of a row tile each).  Items beyond the grid are taken by
// stepping over the list: the host can only bound the number of items, and a workgroup that finds none still costs its
// slot for the 3 us that finding out takes (60 sequences with three short chunks of 200 tokens: 147 us with a workgroup
// for every possible item and quarter, 129 like this, 131 on the plain grid).
constexpr int32_t kListGrid = 2048;
constexpr int32_t kListMergeGrid = 2048;
// The chunk unit that leaves every context whole: the list as a grid of the row tiles that exist.
constexpr int32_t kListUncut = 1 << 28;

// small_group = query heads per KV head when sequences with q_len * G <= 16 are left to the decode kernel, kNoSmallGroup
// when none is.
constexpr int32_t kNoSmallGroup = 17;

// One lane's sequence of a block of 64: row tiles (0: no queries, or left to the decode kernel) and key tiles.
struct ListSeq {
    int32_t tiles, len;
    bool few;            // left to the decode kernel
};
__device__ __forceinline__ ListSeq list_seq(const int32_t* __restrict__ cu_q_lens, const int32_t* __restrict__ seq_lens,
                                            int32_t batch, int32_t i, int32_t log2_pack, int32_t small_group)
{
    ListSeq q = {0, 0, false};
    if (i < batch) {
        const int32_t q_len = cu_q_lens[i + 1] - cu_q_lens[i];
        q.len = seq_lens[i];
        q.few = q_len > 0 && q_len * small_group <= 16;
        if (q_len > 0 && !q.few) q.tiles = ((q_len << log2_pack) + kBM - 1) / kBM;
    }
    return q;
}

// The list of a call, as one wave sees it: the chunk length (the same on every wave: fixed order of the sums) and, for
// batches of up to 64 sequences, this lane's sequence, so that finding an item needs no further load.
struct WorkList {
    int32_t chunk;
    int32_t nsplit, unit;    // BY_LENGTH with unit > 0: each sequence's chunk from its own length instead (sequence_chunk)
    int32_t small_group, log2_pack, heads, batch;
    float work;              // (row tile, key tile) pairs per head group
    int32_t few_tiles;       // 32-key tiles of the sequences left to the decode kernel
    ListSeq own;
};
// The sequences and the work of the list; cut_list completes it.
__device__ __forceinline__ WorkList scan_list(const int32_t* __restrict__ cu_q_lens,
                                              const int32_t* __restrict__ seq_lens, int32_t batch, int32_t log2_pack,
                                              int32_t small_group, int32_t heads, int lane)
{
    WorkList w;
    w.small_group = small_group;
    w.log2_pack = log2_pack;
    w.heads = heads;
    w.batch = batch;
    w.own = list_seq(cu_q_lens, seq_lens, batch, lane, log2_pack, small_group);
    float work = (float)w.own.tiles * (float)((w.own.len + kBN - 1) / kBN);   // (row tile, key tile) pairs per head group
    int32_t few = w.own.few ? (w.own.len + 31) / 32 : 0;
    for (int32_t i = lane + 64; i < batch; i += 64) {
        const ListSeq q = list_seq(cu_q_lens, seq_lens, batch, i, log2_pack, small_group);
        work += (float)q.tiles * (float)((q.len + kBN - 1) / kBN);
        few += q.few ? (q.len + 31) / 32 : 0;
    }
    w.work = wave_sum_moves(work);
    w.few_tiles = wave_total_moves(few);
    return w;
}
__device__ __forceinline__ void cut_list(WorkList& w, const int32_t* __restrict__ cu_q_lens,
                                         const int32_t* __restrict__ seq_lens, int32_t unit, int32_t d, int lane)
{
    const int32_t batch = w.batch, log2_pack = w.log2_pack, small_group = w.small_group, heads = w.heads;
    int32_t tiles = max(kListMinTiles, (int32_t)(w.work * (float)heads * (1.f / kListTarget)) + 1);
    if (tiles == kListMinTiles) {
        // little work: shorter chunks, if all items still run at once
#pragma unroll 1
        for (int32_t c = kListShortTiles; c < kListMinTiles; c += 8) {
            int32_t n = 0;
            for (int32_t i = lane; i < batch; i += 64) {
                const ListSeq q = i < 64 ? w.own : list_seq(cu_q_lens, seq_lens, batch, i, log2_pack, small_group);
                n += min(q.tiles * ((max(q.len, 1) + c * kBN - 1) / (c * kBN)), 2 * list_wg_slots(d));
            }
            n = wave_total_moves(min(n, 1 << 20));
            if ((int64_t)n * heads <= list_wg_slots(d)) {
                tiles = c;
                break;
            }
        }
        tiles = __builtin_amdgcn_readfirstlane(tiles);
    }
    w.chunk = __builtin_amdgcn_readfirstlane((min(tiles, 1 << 22) * kBN + unit - 1) / unit * unit);
}
__device__ __forceinline__ WorkList make_list(const int32_t* __restrict__ cu_q_lens,
                                              const int32_t* __restrict__ seq_lens, int32_t batch, int32_t log2_pack,
                                              int32_t small_group, int32_t heads, int32_t unit, int32_t d, int lane)
{
    WorkList w = scan_list(cu_q_lens, seq_lens, batch, log2_pack, small_group, heads, lane);
    cut_list(w, cu_q_lens, seq_lens, unit, d, lane);
    return w;
}

// Item (or, SPLIT_TILES: the idx-th row tile of the sequences that are cut) number idx of the list; false = no such item.
struct ListItem {
    int32_t s;           // sequence
    int32_t tile;        // row tile
    int32_t split;       // chunk of the context
    int32_t tiles;       // row tiles of the sequence
    int32_t chunks;      // chunks of the sequence; 1 = the item writes its rows, > 1 = a partial
    int32_t slot;        // partial of chunk 0 of the sequence's last row tile, per head group
};
template <bool BY_LENGTH>
__device__ __forceinline__ int32_t list_chunk(const WorkList& w, int32_t len)
{
    return BY_LENGTH && w.unit > 0 ? sequence_chunk(len, 0, w.nsplit, w.unit) : w.chunk;
}
template <bool SPLIT_TILES, bool BY_LENGTH = false>
__device__ __forceinline__ bool list_locate(ListItem& it, const WorkList& w, const int32_t* __restrict__ cu_q_lens,
                                            const int32_t* __restrict__ seq_lens, int32_t idx, int lane)
{
    // whole chunks, then the shorter ones: an uncut list has none of the former, contexts cut by their own lengths none of the latter
    const bool by_length = BY_LENGTH && w.unit > 0;
    int32_t items_before = 0;
    for (int32_t part = !SPLIT_TILES && !by_length && w.chunk >= kListUncut ? 1 : 0; part < (SPLIT_TILES || by_length ? 1 : 2);
         ++part) {
        int32_t slots_before = 0;
        for (int32_t blk = 0; blk < w.batch; blk += 64) {
            const ListSeq q = blk == 0 ? w.own : list_seq(cu_q_lens, seq_lens, w.batch, blk + lane, w.log2_pack, w.small_group);
            const int32_t chunk = list_chunk<BY_LENGTH>(w, q.len);
            const int32_t chunks = max((q.len + chunk - 1) / chunk, 1);
            const int32_t slots = chunks > 1 ? q.tiles * chunks : 0;
            const int32_t whole = by_length ? chunks : q.len / chunk;
            const int32_t n = SPLIT_TILES ? (chunks > 1 ? q.tiles : 0) : q.tiles * (part == 0 ? whole : chunks - whole);
            const int32_t inc = wave_scan_moves(n), sinc = wave_scan_moves(slots);
            const uint64_t hit = __ballot(items_before + inc > idx);
            if (hit) {
                const int first = __ffsll((unsigned long long)hit) - 1;
                it.s = blk + first;
                it.tiles = __builtin_amdgcn_readlane(q.tiles, first);
                it.chunks = __builtin_amdgcn_readlane(chunks, first);
                it.slot = slots_before + __builtin_amdgcn_readlane(sinc, first) - __builtin_amdgcn_readlane(slots, first);
                const int32_t rest = idx - (items_before + __builtin_amdgcn_readlane(inc, first) -
                                            __builtin_amdgcn_readlane(n, first));
                it.split = rest / it.tiles + (part == 0 ? 0 : __builtin_amdgcn_readlane(whole, first));
                it.tile = it.tiles - 1 - rest % it.tiles;
                return true;
            }
            items_before += __builtin_amdgcn_readlane(inc, 63);
            slots_before += __builtin_amdgcn_readlane(sinc, 63);
        }
    }
    return false;
}
// slot of chunk `split` of row tile `tile`, head group hg
__device__ __forceinline__ int32_t list_slot(const ListItem& it, int32_t split, int32_t heads, int32_t hg)
{
    return (it.slot + split * it.tiles + it.tiles - 1 - it.tile) * heads + hg;
}
// floats of a slot's accumulators: 128 rows x the 32-column blocks of head_dim
__host__ __device__ constexpr int32_t list_slot_floats(int32_t d) { return kBM * ((d + 31) / 32 * 32); }

struct PageIds {
    int32_t p0, p1, p2, p3;
};

template <bool UNIFORM>
__device__ __forceinline__ void load_ids(PageIds& p, const CacheView& cache, const int32_t* table, int32_t t0,
                                         int32_t row, int32_t last_key)
{
    const int32_t key = UNIFORM ? t0 : t0 + row;
    p.p0 = table[min(key, last_key) >> cache.log2_page];
    p.p1 = table[min(key + 16, last_key) >> cache.log2_page];
    p.p2 = table[min(key + 32, last_key) >> cache.log2_page];
    p.p3 = table[min(key + 48, last_key) >> cache.log2_page];
    if (UNIFORM) {
        p.p0 = __builtin_amdgcn_readfirstlane(p.p0);
        p.p1 = __builtin_amdgcn_readfirstlane(p.p1);
        p.p2 = __builtin_amdgcn_readfirstlane(p.p2);
        p.p3 = __builtin_amdgcn_readfirstlane(p.p3);
    }
}

// K row and V row of `key` (clamped to a live slot) in page `page` -> LDS rows at lds + IMM (K) and TB further (V).
template <bool UNIFORM, int IMM, int TB = kTileBytes>
__device__ __forceinline__ void fetch_rows(uint32_t lds, const CacheView& cache, int32_t page, int32_t key,
                                           int32_t last_key, uint32_t lane_off)
{
    const int32_t slot = min(key, last_key) & (cache.page_size - 1);
    if (UNIFORM) {
        // scalar page base + 32-bit lane offset: the loads take the scalar-base form and a row group costs a handful
        // of 32-bit vector operations instead of 64-bit multiply-adds per lane
        int64_t page_off = (int64_t)page * cache.page_stride * 2;
        asm volatile("" : "+s"(page_off));                 // stays in scalar registers
        const uint32_t off32 = (uint32_t)slot * (uint32_t)(cache.token_stride * 2) + lane_off;
        const char* kp = reinterpret_cast<const char*>(cache.k) + page_off;
        const char* vp = reinterpret_cast<const char*>(cache.v) + page_off;
        load_to_lds16(lds, IMM, kp, off32);
        load_to_lds16(lds, IMM + TB, vp, off32);
        return;
    }
    const int64_t off = ((int64_t)page * cache.page_stride + (int64_t)slot * cache.token_stride) * 2 + lane_off;
    load_to_lds16(lds, IMM, reinterpret_cast<const char*>(cache.k) + off);
    load_to_lds16(lds, IMM + TB, reinterpret_cast<const char*>(cache.v) + off);
}

// lds = LDS address of buffer + 4*w*kRow (this wave's first row); row = 4*w + lane/16 (this lane's row within a
// 16-row group).
template <bool UNIFORM>
__device__ __forceinline__ void fetch_tile(uint32_t lds, const PageIds& p, const CacheView& cache, int32_t t0, int32_t row,
                                           int32_t last_key, uint32_t lane_off)
{
    fetch_rows<UNIFORM, 0>(lds, cache, p.p0, t0 + row, last_key, lane_off);
    fetch_rows<UNIFORM, 16 * kRow>(lds, cache, p.p1, t0 + row + 16, last_key, lane_off);
    fetch_rows<UNIFORM, 32 * kRow>(lds, cache, p.p2, t0 + row + 32, last_key, lane_off);
    fetch_rows<UNIFORM, 48 * kRow>(lds, cache, p.p3, t0 + row + 48, last_key, lane_off);
}


// max over the GROUPS lanes that share a row (lane, lane ^ 32 and, of four, lane ^ 16) without an LDS round trip
template <int GROUPS>
__device__ __forceinline__ float row_max(float x)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    if (GROUPS == 4) {
        const auto u = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        x = fmaxf(__uint_as_float(u[0]), __uint_as_float(u[1]));
    }
    return x;
}

// Online softmax keeps a REFERENCE exponent (log2 domain) that may trail the true running max; the reference is
// raised when the weights a lane computes for a half tile (16, or 8 with 16 rows a wave) sum to more than this (fp16
// operands end at 65504).
constexpr float kWeightSumMax = 16384.f;

}  // namespace prefill
}  // namespace pa
