// C ABI of the paged-attention library: argument validation, split planning and kernel dispatch.
// Nothing here touches device memory; every check is a host check made before the first launch.
#include <string.h>

#include <atomic>
#include <mutex>
#include <string>
#include <vector>

#include "common.h"

// Scratch of paged_attention_decode_static: the split-KV partials of a decode call, for callers that cannot bring
// a workspace.  One copy per GPU, held until the process ends.  In host code this name is only a handle for
// hipGetSymbolAddress; kernels receive the address that call returns.
constexpr size_t kStaticScratchBytes = (size_t)16 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace pa {

namespace {

struct Options {
    int64_t decode_chunk_tokens = 0;
    int64_t decode_workgroups = 0;
    int64_t force_generic = 0;
    int64_t prefill_chunk_tokens = 0;
    int64_t no_small_q_route = 0;
    int64_t step_append_kernel = 0;   // 1 = paged_decode_step on the tile stream appends with a kernel of its own
                                      // (0: every decode kernel performs the step's append itself)
    int64_t decode_short = 0;      // 0 = heuristic, 1 = whenever the one-launch kernel supports the call, -1 = never
    int64_t decode_short_splits = 0;   // workgroups per (sequence, KV head) of the one-launch kernel; 0 = heuristic
};
thread_local Options g_opt;       // per host thread: a thread's knobs shape only the calls it makes itself

// Compute units of the current device (the tile-stream decode launches one workgroup per CU by default).
int32_t device_cus()
{
    static int32_t cached[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (cached[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cached[dev] = n;
    }
    return cached[dev];
}

struct ProfileRecord {
    std::string kernel;
    hipEvent_t start;
    hipEvent_t stop;
};
bool g_profile_on = false;
std::vector<ProfileRecord> g_records;
std::vector<hipEvent_t> g_spare_events;   // events of records that were reset, reused instead of created anew
std::mutex g_profile_mutex;

bool take_event(hipEvent_t* e)
{
    if (!g_spare_events.empty()) {
        *e = g_spare_events.back();
        g_spare_events.pop_back();
        return true;
    }
    return hipEventCreate(e) == hipSuccess;
}

inline int elem_bytes(pa_dtype t) { return t == PA_DTYPE_F32 ? 4 : 2; }

bool is_pow2(int32_t x) { return x > 0 && (x & (x - 1)) == 0; }

// Is `id` the kId of a user modification the library was built with?
bool user_mod_known(int32_t id)
{
#define PA_USER_CASE(U) if (id == U::kId) return true;
    PA_USER_MODS(PA_USER_CASE)
#undef PA_USER_CASE
    return false;
}

}  // namespace

pa_status check_cache(const pa_kv_cache_desc* c)
{
    if (!c || !c->k_cache || !c->v_cache) return PA_ERR_INVALID_ARG;
    if (c->dtype != PA_DTYPE_F32 && c->dtype != PA_DTYPE_BF16 && c->dtype != PA_DTYPE_F16) return PA_ERR_UNSUPPORTED;
    if (c->num_pages <= 0 || c->num_kv_heads <= 0 || c->head_dim <= 0) return PA_ERR_INVALID_ARG;
    if (!is_pow2(c->page_size)) return PA_ERR_INVALID_ARG;   // Algorithm 1 requires a power of two
    const int epv = 16 / elem_bytes(c->dtype);
    if (c->head_dim % epv != 0 || c->head_dim > 256) return PA_ERR_UNSUPPORTED;
    if (c->page_stride <= 0 || c->token_stride <= 0 || c->head_stride <= 0) return PA_ERR_INVALID_ARG;
    if (c->page_stride % epv || c->token_stride % epv || c->head_stride % epv) return PA_ERR_UNSUPPORTED;
    if (((uintptr_t)c->k_cache | (uintptr_t)c->v_cache) & 15) return PA_ERR_UNSUPPORTED;
    return PA_OK;
}

namespace {

int32_t nsplit_bound(int32_t max_seq_len)
{
    int64_t n = ((int64_t)max_seq_len + kMinChunk - 1) / kMinChunk;
    if (n < 1) n = 1;
    if (n > kMaxSplits) n = kMaxSplits;
    return (int32_t)n;
}

// Context tokens per split-KV workgroup.  Chunks are a multiple of max(P, 32) so that a chunk starts on a
// page boundary and on a 32-key MFMA tile; their number never exceeds the bound the workspace is sized by.
SplitPlan plan_decode(int32_t batch, int32_t max_seq_len, int32_t page_size)
{
    const int32_t unit = page_size > 32 ? page_size : 32;
    int64_t chunk = g_opt.decode_chunk_tokens;
    if (chunk <= 0) {
        // aim at a few thousand (sequence, chunk) work items so that 256 CUs stay busy and ragged
        // batches balance, but keep chunks long enough to amortise a workgroup's start-up
        const int64_t tokens = (int64_t)batch * max_seq_len;
        chunk = kMinChunk;
        while (chunk < 2048 && tokens / chunk > 4096) chunk *= 2;
    }
    chunk = (chunk + unit - 1) / unit * unit;
    const int32_t bound = nsplit_bound(max_seq_len);
    while (((int64_t)max_seq_len + chunk - 1) / chunk > bound) chunk *= 2;
    SplitPlan p;
    p.chunk = (int32_t)chunk;
    p.nsplit = (int32_t)(((int64_t)max_seq_len + chunk - 1) / chunk);
    if (p.nsplit < 1) p.nsplit = 1;
    return p;
}

size_t align256(size_t x) { return (x + 255) / 256 * 256; }

// Context split of the MFMA prefill kernel.  The kernel gets one workgroup per (128-row tile, head group); the
// host knows only total_q and batch, so it bounds the live tiles by total_q * pack / 128 + batch.  When that fills
// the machine there is no split; a call with few query rows over a long context (a chunk of a long prompt, a
// mixed batch that is mostly decode rows) is cut along the context into chunks of at least kPrefillMinChunk
// tokens until about kPrefillTargetWGs work items exist.  A pure function of its arguments: the workspace size is
// computed from the same rule with the largest packing.
constexpr int64_t kPrefillTargetWGs = 1024;
constexpr int64_t kPrefillFullWGs = 512;

SplitPlan plan_prefill(int32_t batch, int32_t num_q_heads, int32_t log2_pack, int32_t total_q, int32_t max_seq_len,
                       int32_t page_size)
{
    SplitPlan p;
    p.chunk = max_seq_len > 0 ? max_seq_len : 1;
    p.nsplit = 1;
    if (g_opt.prefill_chunk_tokens > 0) {
        const int64_t unit = page_size > 64 ? page_size : 64;
        int64_t chunk = (g_opt.prefill_chunk_tokens + unit - 1) / unit * unit;
        while (((int64_t)max_seq_len + chunk - 1) / chunk > kMaxSplits) chunk *= 2;
        if (chunk < max_seq_len) {
            p.chunk = (int32_t)chunk;
            p.nsplit = (int32_t)(((int64_t)max_seq_len + chunk - 1) / chunk);
        }
        return p;
    }
    const int64_t wgs = (((int64_t)total_q << log2_pack) / 128 + batch) * (num_q_heads >> log2_pack);
    if (wgs >= kPrefillFullWGs || max_seq_len < 2 * kPrefillMinChunk) return p;
    int64_t n = (kPrefillTargetWGs + wgs - 1) / wgs;
    if (n > max_seq_len / kPrefillMinChunk) n = max_seq_len / kPrefillMinChunk;
    if (n > kMaxSplits) n = kMaxSplits;
    if (n < 2) return p;
    const int64_t unit = page_size > 64 ? page_size : 64;
    int64_t chunk = ((int64_t)max_seq_len + n - 1) / n;
    chunk = (chunk + unit - 1) / unit * unit;
    if (chunk >= max_seq_len) return p;
    p.chunk = (int32_t)chunk;
    p.nsplit = (int32_t)(((int64_t)max_seq_len + chunk - 1) / chunk);
    return p;
}

// The number of chunks for a call whose contexts are much longer than its query ranges, where every workgroup walks a whole
// chunk: at most plan_prefill's (which workspaces are sized for), the one for which the fullest compute unit is done first.
// A compute unit works through the tiles of two workgroups hardly faster than through those of one after the other
// (64 keys at head_dim 128: 1.93 us two at a time, 1.05 alone; one at a time only at head_dim 256; three at head_dim 64), so
// what counts is how evenly the workgroups divide among the compute units; a chunk more costs its partials' way to memory and
// back (3.3 GB a ms in the merge, and 10 us for its launch and the workgroups' other end).  With every number of chunks measured
// for 56 calls with equal contexts this one is at most 2 % behind the best (two sequences at head_dim 256 4 and 12 %); at
// head_dim 64, two, four and eight chunks, as for two workgroups a compute unit, are behind three, six and 16 by 1 to 9 %.
// us a call with about 1024 workgroups / like this, 32 / 8 heads: 1024 tokens of a 32768-token context 514 / 511, 512 of it
// 273 / 265, 128 of it 109 / 87, 500 of 12000 125 / 109, two sequences with 128 tokens of 32768 each 184 / 154, four
// 374 / 290, 500 of 20000 at head_dim 256 488 / 363, 1024 of 32768 at 64 343 / 314.
// max_seq_len is a bound and query counts say nothing of contexts: each sequence's own length is cut on the device
// (sequence_chunk), which divides as evenly for any length (1024 workgroups and chunks of the bound / this many chunks of the
// bound / like this: 128 tokens of 8192 in a call for up to 131072 97 / 200 / 40, 1000 of 20000 for up to 32768 403 / 413 / 320).
// A batch need not be as even as its query counts: one long context among short ones has its own workgroups alone, so they
// have to fill the machine by themselves, or there are nearly as many chunks as there can be (all chunks of the bound / what is
// even for equal contexts / like this: 64 tokens of 32768 and of 1500 seven times 145 / 204 / 114, 128 of 12284 and of
// 1500 with 32 / 32 heads 58 / 67 / 56; equal contexts pay at most for chunks that only they could spare: 200 tokens of 18000
// three times 239 / 204 / 220, 256 of 20496 four times with 8 / 1 heads 120 / 103 / 113, 128 of 32768 twice 193 / 157 / 157).
SplitPlan even_prefill_split(const SplitPlan& most, int32_t batch, int64_t wgs, int64_t rows, int32_t max_seq_len,
                             int32_t page_size, int32_t d)
{
    // us that a compute unit takes for 64 keys of its first, second and third workgroup together (as many as fit it at once;
    // 32 heads' rows on 8192 and 16384 keys with one to three workgroups a compute unit)
    const double tile[3] = {d > 128 ? 2.4 : d > 112 ? 1.05 : d > 96 ? 1.6 : d > 64 ? 1.35 : 0.84,
                            d > 128 ? 4.8 : d > 112 ? 1.93 : d > 96 ? 2.75 : d > 64 ? 2.25 : 1.25, 1.75};
    const int64_t slots = d > 64 ? 2 : 3;
    const int64_t unit = page_size > 64 ? page_size : 64;
    SplitPlan best = most;
    best.unit = (int32_t)unit;
    double best_us = 1e30;
    for (int32_t n = 1; n <= most.nsplit; ++n) {
        const int64_t chunk = (((int64_t)max_seq_len + n - 1) / n + unit - 1) / unit * unit;
        if (((int64_t)max_seq_len + chunk - 1) / chunk != n) continue;
        if (batch > 1 && wgs / batch * n < device_cus() && 4 * n < 3 * most.nsplit) continue;
        const int64_t per_cu = (wgs * n + device_cus() - 1) / device_cus();
        const double us = (double)(chunk / 64) * ((per_cu / slots) * tile[slots - 1] +
                                                  (per_cu % slots ? tile[per_cu % slots - 1] : 0.0)) +
                          (n > 1 ? 10.0 + (double)rows * n * d * 4.0 / 3.3e6 : 0.0);
        if (us < best_us) {
            best_us = us;
            best.nsplit = n;
            best.chunk = n > 1 ? (int32_t)chunk : max_seq_len;
            best.unit = n > 1 ? (int32_t)unit : 0;
        }
    }
    return best;
}

// Largest number of chunks plan_prefill can choose for these sizes, whatever the packing and page size.
int32_t prefill_nsplit_bound(int32_t batch, int32_t num_q_heads, int32_t total_q, int32_t max_seq_len)
{
    if (g_opt.prefill_chunk_tokens > 0) return kMaxSplits;
    int32_t best = 1;
    for (int32_t lg = 0; lg <= 4; ++lg) {
        if (num_q_heads % (1 << lg)) break;
        const SplitPlan p = plan_prefill(batch, num_q_heads, lg, total_q, max_seq_len, 1);
        if (p.nsplit > best) best = p.nsplit;
    }
    return best;
}

// Workgroups along the tile stream for the MFMA decode kernel: one per compute unit and KV-head group, and more when
// that leaves fewer than four waves per compute unit (a workgroup holds one wave per KV head: few KV heads, as on one
// shard of a tensor-parallel model, mean small workgroups; `slices` = grid slices of 16 heads for groups above 16) --
// but never so many that a workgroup gets fewer than two 32-key tiles of the longest possible stream.
int32_t plan_stream_wgs(int32_t batch, int32_t max_seq_len, int32_t head_groups, int32_t num_kv_heads, int32_t slices)
{
    int64_t target = g_opt.decode_workgroups;
    if (target <= 0) {
        target = device_cus() / head_groups;
        const int64_t by_waves = 4LL * device_cus() / ((int64_t)num_kv_heads * (slices < 1 ? 1 : slices));
        if (by_waves > target) target = by_waves;
    }
    if (target < 1) target = 1;
    const int64_t tiles = (int64_t)batch * ((max_seq_len + 31) / 32);
    int64_t n = tiles / 2;
    if (n > target) n = target;
    if (n > kMaxDecodeWGs) n = kMaxDecodeWGs;
    if (n < 1) n = 1;
    return (int32_t)n;
}

// One launch instead of tile stream + merge: pays while a step is bound by launches and memory round trips.  A
// workgroup of the one-launch kernel streams its share of a (sequence, KV head) at about 55 GB/s, so its time is
// about 4 us + 9 us per 512 KB, against a floor of 12-16 us for tile stream + merge.  With few sequences the
// kernel puts several workgroups on a (sequence, KV head) -- as many as fill the machine once (a compute unit holds
// one workgroup of this kernel: its eight waves take the whole register file), at least 128 keys each at head_dim 128 -- which
// merge through the workspace inside the same launch; the route is taken while a workgroup's share stays within
// 512 KB of K and V rows (1024 tokens at head_dim <= 128, 512 at head_dim 256: rows twice as long).  Beyond that
// the tile stream's whole-row reads and equal split use the memory system better.  Measured, steps, 32 / 8 heads, one box,
// workgroups per (sequence, KV head): 4 x 700 tokens 8.2 us with 4, 9.9 with 2, 11.2 with one (15.0 tile stream + merge);
// 8 x 4096 26.1 with 4, 43.3 with one (29.5); 2 x 1000 at head_dim 256 11.0 with 8, 13.0 with 4 (17.9); 1 x 30000 with
// 8 / 1 heads 19.9 with 32, 25.4 with 16 (32.9).  More than 16 pay only where the units are few: 1 x 8192 with 8 KV heads
// 13.9 with 16, 15.5 with 32.  At least 16384 / head_dim keys to a workgroup, half its waves' tiles: below that the merge
// costs more than the tiles (1 x 128: 7.0 with 2, 5.2 with one; 8 x 300 with 8 / 1 heads at head_dim 64: 7.3 and 6.3).
constexpr int64_t kShortMaxRowBytes = 1024 * 512;   // context tokens x bytes of a K row and a V row (>= 512) per workgroup
// A single sequence has no lengths to balance, and its split reads at what the memory gives: the tile stream's slower start
// and second launch are worth it only beyond this many bytes of K and V (32 / 8 heads: 32768 tokens 30.0 us against 37.9,
// 65536 62.0 against 56.1; 8 / 1 heads, 131072 tokens = 67 MB, 48 against 66; 32 / 32, 16384 = 268 MB, 48.0 against 48.5).
// Nor beyond what so many workgroups read in that time: a unit has at most 32, so with one or two KV heads most of the machine
// stands by (8 / 1 heads: 131072 tokens = 2.1 MB a workgroup 48 us against 66, 300000 = 4.8 MB 94 against 77; head_dim 64,
// 600000 99 against 78); with several slices of 16 heads a unit's rows are read by all of them, from the caches at best
// (64 / 1, 30000 tokens = 0.5 MB 20.6 against 28.2, 200000 = 3.2 MB 67 against 56; 40 / 2, 100000 = 1.6 MB 40.7 against 41.9).
// head_dim 256, whose tile stream has half the waves: 8 / 1 heads, 150000 tokens = 4.8 MB 107 against 123.
constexpr int64_t kShortMaxSingleBytes = (int64_t)160 << 20;
constexpr int64_t kShortMaxSingleShare = (int64_t)3 << 20;
constexpr int64_t kShortMaxWideShare = (int64_t)5 << 20;
constexpr int64_t kShortMaxSlicedShare = (int64_t)3 << 19;
constexpr int64_t kShortMaxWGsPerCU = 2;
// Nor while every wave has at most one tile of the whole context: 1 x 256 7.3 with 2, 6.2 with one (300 tokens, two tiles a
// wave, 7.5 and 7.8); 2 x 512 at head_dim 64 8.0 and 6.7 (700: 8.2 and 8.4); 8 x 256 7.4 and 6.35.
constexpr int32_t kShortMinSplitElems = 16384;   // keys x head_dim
// The plan that paged_attention_decode_static's scratch limit is stated for (see run_attention).
constexpr int32_t kScratchMaxSplit = 16;
constexpr int32_t kScratchMinSplitKeys = 256;

int64_t short_units(const AttnArgs& a)
{
    return (int64_t)a.batch * a.cache.num_kv_heads * ((a.num_q_heads / a.cache.num_kv_heads + 15) / 16);
}

// Workgroups per (sequence, KV head, slice of 16 heads) of the one-launch kernel.
int32_t plan_short_splits(const AttnArgs& a, int32_t min_keys = 0, int32_t max_split = 0)
{
    const int64_t units = short_units(a);
    int64_t n = g_opt.decode_short_splits;
    if (n <= 0) {
        n = device_cus() / units;
        if (min_keys <= 0) min_keys = kShortMinSplitElems / a.cache.head_dim;
        if (max_split <= 0) max_split = units < 8 ? kShortMaxSplit : kScratchMaxSplit;
        const int64_t by_keys = a.max_seq_len / min_keys;
        if (n > by_keys) n = by_keys;
        if (a.max_seq_len <= decode_short_one_round(a.cache.head_dim)) n = 1;
    }
    if (max_split > 0 && n > max_split) n = max_split;
    if (n > kShortMaxSplit) n = kShortMaxSplit;
    return n < 1 ? 1 : (int32_t)n;
}

// any_share: a single sequence may give a workgroup any share (where the tile stream has no room for its partials).
bool short_decode_pays(const AttnArgs& a, int32_t nsplit, bool any_share = false)
{
    if (g_opt.decode_workgroups > 0) return false;     // the caller shapes the tile stream: keep it
    const int64_t row_bytes = 4LL * (a.cache.head_dim > 128 ? a.cache.head_dim : 128);
    const int64_t share = ((int64_t)a.max_seq_len + nsplit - 1) / nsplit;
    const int64_t share_bytes = share * 4LL * a.cache.head_dim;
    const int64_t most = a.num_q_heads / a.cache.num_kv_heads > 16 ? kShortMaxSlicedShare
                         : a.cache.head_dim > 128                  ? kShortMaxWideShare
                                                                   : kShortMaxSingleShare;
    const bool single = a.batch == 1 && nsplit > 1 &&
                        (any_share || share_bytes <= most) &&
                        4LL * a.max_seq_len * a.cache.num_kv_heads * a.cache.head_dim <= kShortMaxSingleBytes;
    return (single || share * row_bytes <= kShortMaxRowBytes) && short_units(a) * nsplit <= kShortMaxWGsPerCU * device_cus();
}

// What a split call of the one-launch kernel keeps in the workspace: the workgroups' partials (16 rows of head_dim floats
// plus maxima and sums each), then the units' arrival counters.
size_t short_split_bytes(int64_t units, int32_t nsplit, int32_t d)
{
    return align256(decode_short_part_floats(units * nsplit, d) * sizeof(float)) + arrival_bytes(units);
}

// Its bound.  The heuristic splits only while one workgroup per compute unit is not reached, so the counters fit the room
// of the second one.
size_t short_split_workspace_bytes(int32_t batch, int32_t hq, int32_t d)
{
    // units <= batch * hq (group size 1, one slice); the heuristic never exceeds two workgroups per compute unit
    if (g_opt.decode_short_splits > 1)
        return short_split_bytes((int64_t)batch * hq, (int32_t)g_opt.decode_short_splits, d);
    return align256(decode_short_part_floats(kShortMaxWGsPerCU * device_cus(), d) * sizeof(float));
}

// What a call's arrival counters count in: a scrambled call number (the 64-bit finalizer of MurmurHash3), made odd so that
// its first 2^64 multiples differ.
uint64_t next_arrival_step()
{
    static std::atomic<uint64_t> calls{0};
    uint64_t x = calls.fetch_add(1, std::memory_order_relaxed) + 0x9e3779b97f4a7c15ull;
    x = (x ^ (x >> 33)) * 0xff51afd7ed558ccdull;
    x = (x ^ (x >> 33)) * 0xc4ceb9fe1a85ec53ull;
    return (x ^ (x >> 33)) | 1;
}

// Partials and arrival counters of a split call of the fp32 decode kernel.
size_t f32_split_bytes(const AttnArgs& a, int32_t nsplit)
{
    return align256(decode_f32_part_floats(a, nsplit) * sizeof(float)) + arrival_bytes((int64_t)a.batch * a.cache.num_kv_heads);
}

// Workgroups per (sequence, KV head) of the fp32 decode kernel.  `fill`: what fills the machine, one workgroup per compute
// unit (its eight waves take the register file of one), while each slot of its waves has a tile; every sequence is cut that
// far.  `nsplit`: what a long context among others is cut into, so that no workgroup walks more than kF32MaxShare keys (40
// us and more) while the machine idles; a sequence takes as many as it has shares of `chunk` tiles.  The others leave at
// once but cost their slot for about a microsecond, so there are at most kF32MaxWGs in all: beyond that the batch itself
// averages the lengths out.  Not more than the workspace holds partials for.  us with the chunks of the portable
// kernel / with `fill` alone / like this: 32 sequences of 64 .. 32768 tokens, 32 / 8 heads, head_dim 128 1460 / 1910 / 888; 64
// of them at head_dim 64 1322 / 1099 / 842, 8 / 8 heads - / 793 / 417; 32 of 64 .. 131072 at head_dim 64 2399 / 2800 / 1718;
// 256 of 64 .. 8192, 8 / 8 heads, head_dim 64 - / 416 / 395 (with shares of 1024 keys and 8192 workgroups 445).
constexpr int64_t kF32MaxShare = 2048;
constexpr int64_t kF32MaxWGs = 4096;

void plan_f32_splits(AttnArgs& a, size_t ws_bytes)
{
    const int64_t units = (int64_t)a.batch * a.cache.num_kv_heads;
    const int64_t tiles = ((int64_t)a.max_seq_len + 15) / 16;
    auto fits = [&](int64_t n) { return n <= 1 || f32_split_bytes(a, (int32_t)n) <= ws_bytes; };
    int64_t fill = device_cus() / units;
    int64_t n = 0;
    if (g_opt.decode_chunk_tokens > 0) {
        fill = (a.max_seq_len + g_opt.decode_chunk_tokens - 1) / g_opt.decode_chunk_tokens;
    } else {
        const int64_t by_keys = tiles / decode_f32_tile_slots(a);
        if (fill > by_keys) fill = by_keys;
        if (a.batch > 1) n = (a.max_seq_len + kF32MaxShare - 1) / kF32MaxShare;
        if (n > kF32MaxWGs / units) n = kF32MaxWGs / units;
    }
    if (n < fill) n = fill;
    if (n > kF32MaxSplit) n = kF32MaxSplit;
    while (!fits(n)) --n;
    if (n < 1) n = 1;
    if (fill > n) fill = n;
    a.short_nsplit = (int32_t)n;
    a.short_fill = fill < 1 ? 1 : (int32_t)fill;
    a.short_chunk = tiles > n ? (int32_t)((tiles + n - 1) / n) : 1;
}

size_t stream_workspace_bytes(int32_t batch, int32_t hq, int32_t d, int32_t wgs)
{
    const size_t parts = (size_t)wgs + batch;
    return align256(parts * hq * d * sizeof(float)) + align256(parts * hq * sizeof(float)) +
           2 * align256((size_t)batch * sizeof(int32_t));
}

// Workgroups of the decode kernel when it runs the few-query sequences of a prefill call; its partials there take
// 16 rows per KV head, so the count is held to kSmallRouteMaxWGs and to kSmallRouteMaxHeadWGs / Hkv (a workgroup
// holds up to eight KV heads: about one workgroup per compute unit either way).
constexpr int32_t kSmallRouteMaxWGs = 256;
constexpr int32_t kSmallRouteMaxHeadWGs = 2048;

int32_t small_route_wgs_cap(int32_t num_kv_heads)
{
    const int32_t by_heads = kSmallRouteMaxHeadWGs / num_kv_heads;
    return by_heads < 1 ? 1 : by_heads < kSmallRouteMaxWGs ? by_heads : kSmallRouteMaxWGs;
}

size_t small_route_bytes(int32_t wgs, int32_t batch, int32_t num_kv_heads, int32_t d)
{
    const size_t rows = ((size_t)wgs + batch) * num_kv_heads * 16;
    return align256(rows * d * sizeof(float)) + align256(rows * sizeof(float)) +
           2 * align256((size_t)batch * sizeof(int32_t));
}

// Bound of small_route_bytes over every KV-head count that divides hq: wgs * Hkv <= kSmallRouteMaxHeadWGs, Hkv <= hq.
size_t small_route_workspace_bytes(int32_t batch, int32_t hq, int32_t d)
{
    const size_t rows = ((size_t)kSmallRouteMaxHeadWGs + (size_t)batch * hq) * 16;
    return align256(rows * d * sizeof(float)) + align256(rows * sizeof(float)) +
           2 * align256((size_t)batch * sizeof(int32_t));
}

// Largest tile-stream grid plan_stream_wgs can choose for a call with hq query heads: head_groups >= 1 and
// Hkv * slices >= hq / 16.
int32_t stream_wgs_bound(int32_t batch, int32_t hq, int32_t max_seq_len)
{
    int64_t n = g_opt.decode_workgroups;
    if (n <= 0) {
        n = device_cus();
        const int64_t by_waves = 64LL * device_cus() / hq;
        if (by_waves > n) n = by_waves;
    }
    const int64_t tiles = (int64_t)batch * ((max_seq_len + 15) / 16);
    if (n > tiles / 2) n = tiles / 2;
    if (n > kMaxDecodeWGs) n = kMaxDecodeWGs;
    return n < 1 ? 1 : (int32_t)n;
}

size_t part_o_bytes(int64_t rows, int32_t hq, int32_t d, int32_t nsplit)
{
    return align256((size_t)rows * hq * nsplit * d * sizeof(float));
}

size_t part_lse_bytes(int64_t rows, int32_t hq, int32_t nsplit)
{
    return align256((size_t)rows * hq * nsplit * sizeof(float));
}

// The number of chunks for whole prompts (and chunks of prompts on less than themselves) whose row tiles are few: the launch
// lasts as long as the longest row tile's walk while most of the machine stands by, which costs more than partials and their merge
// do.  Estimated from the sizes: t1 us for 64 keys of a workgroup alone on its compute unit, up to 1.67 times that beside another,
// `start` for its start and end, and of the row tiles of causal prompts half a walk on average; the merge 5.5 us and its partials at
// 3.3 MB a us.  us a call in one piece / in so many, 8 / 1 heads, head_dim 128: 1000 tokens 23.1 / 21.2 (4), 2000 40.0 / 34.2 (2: as
// many as the workspace holds), 4000 73.5 / 60.1 (3); with slopes 600 28.2 / 22.3 (3), 1000 42.0 / 26.2 (4); 600 and 1195 with a cap
// 39.1 / 32.9 (2); head_dim 256 1000 42.8 / 32.6 (4), 3000 110 / 75 (2).  One piece stays with 600 tokens (16.5), 32 / 8 heads and 500 at
// 256 (26.3) and 16 / 8 and 3000 (112).  With every number of chunks measured for 100 calls the one chosen is 0.9 % behind the best that
// the workspace holds, 16 % at worst (443 tokens, 4 / 1 heads, head_dim 256, documents 24.0 / 27.7); of 294 estimates eight in ten are
// within -14 .. 20 %.
SplitPlan prompt_split(const AttnArgs& a, int32_t log2_pack, const SplitPlan& given, size_t room)
{
    const int32_t d = a.cache.head_dim, heads = a.num_q_heads >> log2_pack;
    const int64_t bound = ((((int64_t)a.max_q_len << log2_pack) + 127) / 128) * a.batch;
    int64_t tiles = (((int64_t)a.total_q << log2_pack) / 128) + a.batch;
    if (tiles > bound) tiles = bound;
    const double cus = device_cus(), wgs = (double)tiles * heads;
    if (given.nsplit == 1 && wgs > cus) return given;
    const int64_t window = a.causal || a.mods.window <= 0 ? a.mods.window : 2LL * a.mods.window - 1;   // keys that a row sees
    const bool windowed = window > 0 && window < a.max_seq_len;
    double t1 = d > 128 ? 2.25 : d == 128 ? 1.05 : d > 96 ? 1.5 : d > 80 ? 1.28 : d > 64 ? 1.05 : 0.75;
    if (a.mods.alibi_slopes || a.mods.user_mod) t1 *= 2.0;
    else if (a.mods.doc_ids) t1 *= 1.5;
    if (a.mods.softcap > 0.f) t1 += 0.65;
    const double start = d > 128 ? 7.0 : 6.0, part = a.causal ? 0.5 : 1.0;
    const double walk = (double)(((windowed ? window : a.max_seq_len) + 63) / 64);      // key tiles of the longest row tile
    const double slots = d > 128 ? 1.0 : d > 64 ? 2.0 : 3.0;
    const int64_t unit = a.cache.page_size > 64 ? a.cache.page_size : 64;
    const double mb = (double)a.total_q * a.num_q_heads * d * 4e-6;
    SplitPlan best = given;
    double best_us = 1e30;
    for (int32_t n = 1; n <= 8; ++n) {
        const int64_t chunk = (((int64_t)a.max_seq_len + n - 1) / n + unit - 1) / unit * unit;
        if (n > 1 && (chunk < 256 || ((int64_t)a.max_seq_len + chunk - 1) / chunk != n)) continue;
        if (n > 1 && part_o_bytes(a.total_q, a.num_q_heads, d, n) + part_lse_bytes(a.total_q, a.num_q_heads, n) > room) break;
        // (a window's row tiles reach into two chunks)
        const double own = n == 1 || walk < (double)chunk / 64 ? walk : (double)chunk / 64;
        const double live = n == 1 ? wgs : wgs * (windowed ? 2.0 : 1.0 + (n - 1) * part);
        // (causal walks are of all lengths, so the compute units fill up evenly; without a causal bound they end together, round by
        // round: 2311 queries on 3489 keys, 16 / 8 heads, cap, 296 workgroups, one piece 138, three chunks 125; 36 such calls 0.95)
        const double beside = slots > 1.0 && live > cus ? 0.67 * (a.causal && live < 2 * cus ? live / cus - 1.0 : 1.0) : 0.0;
        const double rounds = live > slots * cus ? (a.causal ? (n > 1 ? live / (slots * cus) : 1.0) : ceil(live / (slots * cus))) : 1.0;
        double us = (start + own * t1 * (1.0 + beside)) * rounds;
        if (n > 1) {
            us += 5.5 + n * mb / 3.3;
        } else {
            const double all = wgs / cus * (walk * part * t1 * (slots > 1.0 ? 0.84 : 1.0) + start / slots);
            if (all > us) us = all;
        }
        if (n > 1) us *= 1.05;                               // (not for an estimate's margin)
        if (us < best_us) {
            best_us = us;
            best.nsplit = n;
            best.chunk = n > 1 ? (int32_t)chunk : a.max_seq_len;
            best.unit = 0;
        }
    }
    return best;
}

// Partials of the prefill kernel's work-list mode.
size_t list_bytes(int32_t d)
{
    return align256(prefill_list_slots() * prefill_list_slot_floats(d) * sizeof(float)) +
           align256((size_t)prefill_list_slots() * 128 * sizeof(float));
}

// Can a call of these sizes take the work-list mode?  (More than one sequence, a context long enough to cut.)
bool list_possible(int32_t batch, int32_t total_q, int32_t max_seq_len)
{
    return g_opt.prefill_chunk_tokens == 0 && batch > 1 && total_q > batch && max_seq_len >= prefill_list_min_context() &&
           max_seq_len < (1 << 28);
}

// The work-list mode replaces the plain grid where that is unbalanced: sequences with different query counts, contexts at
// least twice as long as the longest query range (chunks of long prompts, not whole prompts, whose heaviest-first grid
// balances itself: 4 x 2048 loses 2-3 % in sequence order), and too few row tiles to average the lengths out --
// estimated as if the queries sat in as few sequences as max_q_len allows, since the host knows no lengths.
// Every workgroup scans all sequences 64 at a time, several times over: with many of them it pays only while the sequences
// with queries are few, whose grid cannot balance itself (us plain / list, sequences of 64 .. 4300 tokens: 1000 of which 32
// bring 100 tokens, 32 / 8 heads 1198 / 960, 16 / 2 481 / 413; 900 of which 100 bring 20 767 / 783, 16 / 2 326 / 353, 8 / 1
// 247 / 273; 700 of which 100 bring 40 755 / 755, 8 / 1 217 / 222; 500 of 64 .. 5000 of which 167 bring 60, 8 / 1 215 / 217).
constexpr int64_t kListMaxWGs = 2048;
constexpr int32_t kListScanBatch = 512;
constexpr int64_t kListScanLive = 64;

bool list_pays(const AttnArgs& a, int32_t log2_pack)
{
    if (!list_possible(a.batch, a.total_q, a.max_seq_len) || !prefill_list_supported(a)) return false;
    if ((int64_t)a.batch * a.max_q_len == a.total_q || a.max_seq_len / 2 < a.max_q_len) return false;
    const int64_t live = (a.total_q + a.max_q_len - 1) / (a.max_q_len > 0 ? a.max_q_len : 1);
    if (a.batch > kListScanBatch && live > kListScanLive) return false;
    return ((((int64_t)a.total_q << log2_pack) / 128) + live) * (a.num_q_heads >> log2_pack) < kListMaxWGs;
}

// Jagged calls whose contexts are too short for the list with slots take it all the same where one launch then holds it and the
// few-query stream: the plain grid is row tiles of every sequence, most of them of decode rows and empty, and the stream waits
// behind it.  What the plain grid would cut (from 2048 keys on, while row tiles do not fill the machine) the list cuts as well,
// by each context's own length: the longest one may be a decode row's.  us plain / uncut / like this, 32 / 8 heads: 2 sequences of
// 4000 keys with 200 queries and one 64 / 90 / 47 (8 / 4 heads 49 / 87 / 42), 40 to 3900, two with 128, 85 / 93 / 50, 32 to 3212,
// two with 200 on 81 and 3076 104 / 80 / 50, 33 to 2232, four with 200, 86 / 63 / 59; where nothing needs a cut: 21 to 2917, three
// with up to 512 on 136 .. 525 62 / 32 / 35, 56 to 3500, four with 512 214 / 100 / 101 and 39 to 1500, five with 200
// 69 / 51 / 52.  Of 114 such calls none is slower than 0.89 of the plain grid's time, nor than 1.1 of the uncut list's.
bool jagged_short_list_pays(const AttnArgs& a, int32_t log2_pack)
{
    const int64_t live = (a.total_q + a.max_q_len - 1) / (a.max_q_len > 0 ? a.max_q_len : 1);
    return jagged_mfma_stream_wgs(a, device_cus()) > 0 && a.batch > 1 && a.batch <= kListScanBatch &&
           (int64_t)a.batch * a.max_q_len != a.total_q && a.max_seq_len / 2 >= a.max_q_len &&
           a.max_seq_len < prefill_list_min_context() && g_opt.prefill_chunk_tokens == 0 &&
           ((((int64_t)a.total_q << log2_pack) / 128) + live) * (a.num_q_heads >> log2_pack) < kListMaxWGs;
}

// What a call's workspace has to hold.  (paged_attention_workspace_bytes adds the room of the prefill kernel's
// work-list mode, an optimisation that a smaller workspace does without.)
size_t required_workspace_bytes(int32_t batch, int32_t num_q_heads, int32_t head_dim, int32_t total_q,
                                int32_t max_seq_len)
{
    if (batch <= 0 || num_q_heads <= 0 || head_dim <= 0 || total_q <= 0) return 256;
    if (total_q <= batch) {
        // decode: partials of the portable kernel's chunks, or of the tile stream's workgroups
        const int32_t ns = nsplit_bound(max_seq_len);
        const size_t chunked = part_o_bytes(batch, num_q_heads, head_dim, ns) + part_lse_bytes(batch, num_q_heads, ns);
        const size_t stream = stream_workspace_bytes(batch, num_q_heads, head_dim,
                                                     stream_wgs_bound(batch, num_q_heads, max_seq_len));
        const size_t split = short_split_workspace_bytes(batch, num_q_heads, head_dim);
        const size_t need = chunked > stream ? chunked : stream;
        return need > split ? need : split;
    }
    // prefill: partials of the context split, when the sizes make it split, and of the few-query route
    const int32_t np = prefill_nsplit_bound(batch, num_q_heads, total_q, max_seq_len);
    const size_t split = np > 1 ? part_o_bytes(total_q, num_q_heads, head_dim, np) + part_lse_bytes(total_q, num_q_heads, np)
                                : 0;
    return split + small_route_workspace_bytes(batch, num_q_heads, head_dim);
}

// The workspace of a call.  The public entry points promise the bound paged_attention_workspace_bytes() and are
// checked against it (bound = true); the entry point that brings its own scratch array is checked against what the
// call's plan really uses.
struct Workspace {
    void* ptr;
    size_t bytes;
    bool bound;
};

pa_status run_attention(const pa_kv_cache_desc* cache, const void* q, void* out, float* lse,
                        const int32_t* cu_q_lens, int32_t total_q, int32_t max_q_len, const int32_t* block_table,
                        const int32_t* seq_lens, int32_t batch, int32_t num_q_heads, int32_t max_blocks,
                        int32_t max_seq_len, float scale, int32_t causal, const pa_attn_mods* mods,
                        const Workspace& ws, void* stream, bool decode, const void* k_new = nullptr,
                        const void* v_new = nullptr)
{
    pa_status st = check_cache(cache);
    if (st != PA_OK) return st;
    if (batch < 0 || total_q < 0 || max_blocks < 0 || max_seq_len < 0 || max_q_len < 0) return PA_ERR_INVALID_ARG;
    if (num_q_heads <= 0 || num_q_heads % cache->num_kv_heads != 0) return PA_ERR_INVALID_ARG;
    if (batch == 0 || total_q == 0) return PA_OK;
    if (!q || !out || !block_table || !seq_lens || (!decode && !cu_q_lens)) return PA_ERR_INVALID_ARG;
    if (((uintptr_t)q | (uintptr_t)out) & 15) return PA_ERR_UNSUPPORTED;
    if ((int64_t)max_blocks * cache->page_size < max_seq_len) return PA_ERR_INVALID_ARG;
    if (!(scale == scale)) return PA_ERR_INVALID_ARG;
    ModArgs m = {0, 0.f, nullptr, nullptr, 0, 0, nullptr};
    if (mods) {
        if (mods->window < 0 || !(mods->softcap >= 0.f) || mods->softcap > 3.0e38f) return PA_ERR_INVALID_ARG;
        if (mods->doc_ids && mods->doc_stride < max_seq_len) return PA_ERR_INVALID_ARG;
        if (mods->user_mod != 0 && !user_mod_known(mods->user_mod)) return PA_ERR_INVALID_ARG;
        m.user_mod = mods->user_mod;
        m.user_data = mods->user_mod ? mods->user_data : nullptr;
        m.window = mods->window;
        m.softcap = mods->softcap;
        m.alibi_slopes = mods->alibi_slopes;
        m.doc_ids = mods->doc_ids;
        m.doc_stride = mods->doc_ids ? mods->doc_stride : 0;
    }
    if (ws.bound) {
        const size_t need = required_workspace_bytes(batch, num_q_heads, cache->head_dim, total_q, max_seq_len);
        if (!ws.ptr || ws.bytes < need) return PA_ERR_WORKSPACE_TOO_SMALL;
    }
    if ((uintptr_t)ws.ptr & 255) return PA_ERR_INVALID_ARG;
    // a prefill call whose every sequence brings exactly one query is a decode call (its causal bound is the length
    // mask: the query sits at the last position)
    if (!decode && max_q_len == 1 && total_q == batch) decode = true;

    AttnArgs a;
    a.cache = make_view(cache);
    a.dtype = cache->dtype;
    a.q = q;
    a.out = out;
    a.lse = lse;
    a.cu_q_lens = decode ? nullptr : cu_q_lens;
    a.block_table = block_table;
    a.seq_lens = seq_lens;
    a.batch = batch;
    a.total_q = total_q;
    a.max_q_len = max_q_len;
    a.num_q_heads = num_q_heads;
    a.max_blocks = max_blocks;
    a.max_seq_len = max_seq_len;
    a.scale = scale;
    a.causal = causal ? 1 : 0;
    a.plan.chunk = max_seq_len > 0 ? max_seq_len : 1;
    a.plan.nsplit = 1;
    a.part_o = nullptr;
    a.part_lse = nullptr;
    a.stream_split = 0;
    a.num_wgs = 0;
    a.seg_first = a.seg_last = nullptr;
    a.rows_o = a.rows_lse = nullptr;
    a.list_items = 0;
    a.list_o = a.list_lse = nullptr;
    a.skip_small = 0;
    a.mods = m;
    a.has_mods = m.window > 0 || m.softcap > 0.f || m.alibi_slopes || m.doc_ids || m.user_mod != 0;
    a.k_new = k_new;
    a.v_new = v_new;
    a.short_nsplit = a.short_fill = 1;
    a.short_chunk = 0;
    a.short_part = nullptr;
    a.short_arrive = nullptr;
    a.short_step = 0;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    char* const base = reinterpret_cast<char*>(ws.ptr);
    const int32_t d = cache->head_dim;

    // tile-stream partials of the decode kernel at `p`: outputs, LSEs, first / last workgroup per sequence
    auto place_stream = [&](AttnArgs& b, char* p, size_t rows) {
        b.part_o = reinterpret_cast<float*>(p);
        p += align256(rows * d * sizeof(float));
        b.part_lse = reinterpret_cast<float*>(p);
        p += align256(rows * sizeof(float));
        b.seg_first = reinterpret_cast<int32_t*>(p);
        p += align256((size_t)batch * sizeof(int32_t));
        b.seg_last = reinterpret_cast<int32_t*>(p);
    };

    // a split call of a one-launch kernel: partials from the start of the workspace, counters at the end of `bytes`
    auto place_split = [&](size_t bytes, int64_t units) {
        a.short_part = reinterpret_cast<float*>(base);
        a.short_arrive = reinterpret_cast<uint64_t*>(base + bytes - arrival_bytes(units));
        a.short_step = next_arrival_step();
    };

    const bool f32 = !g_opt.force_generic && attention_f32_supported(a);
    auto plan_stream = [&]() -> int32_t {
        const int32_t head_groups = cache->num_kv_heads / decode_mfma_heads_per_wg(cache->num_kv_heads, d);
        return plan_stream_wgs(batch, max_seq_len, head_groups, cache->num_kv_heads, (num_q_heads / cache->num_kv_heads + 15) / 16);
    };
    auto tile_stream_bytes = [&]() { return stream_workspace_bytes(batch, num_q_heads, d, plan_stream()); };

    if (decode) {
        if (!g_opt.force_generic && g_opt.decode_short >= 0 && decode_short_supported(a)) {
            const int32_t nsplit = plan_short_splits(a);
            const bool cramped = !ws.bound && g_opt.decode_short == 0 && ws.bytes < tile_stream_bytes();
            if (g_opt.decode_short > 0 || short_decode_pays(a, nsplit, cramped)) {
                // A call that the static scratch array was too small for stays refused, although this kernel now takes it with
                // less: the limit is that of the tile stream wherever a split of 16 or of 256 keys would have left it that.
                if (cramped && !short_decode_pays(a, plan_short_splits(a, kScratchMinSplitKeys, kScratchMaxSplit), true))
                    return PA_ERR_WORKSPACE_TOO_SMALL;
                a.short_nsplit = nsplit;
                if (nsplit > 1) {
                    const size_t need = short_split_bytes(short_units(a), nsplit, d);
                    if (ws.bytes < need) return PA_ERR_WORKSPACE_TOO_SMALL;
                    place_split(need, short_units(a));
                }
                return launch_decode_short(a, s);          // with k_new / v_new: the append happens in this launch
            }
        }
        const bool stream_route = !g_opt.force_generic && decode_mfma_supported(a);
        if (stream_route) {
            a.stream_split = 1;
            a.num_wgs = plan_stream();
            if (ws.bytes < tile_stream_bytes()) return PA_ERR_WORKSPACE_TOO_SMALL;
            place_stream(a, base, ((size_t)a.num_wgs + batch) * num_q_heads);
            if (a.k_new && g_opt.step_append_kernel) {     // append as a launch of its own, then attend
                st = launch_kv_append_last(cache, k_new, v_new, seq_lens, block_table, batch, max_blocks, s);
                if (st != PA_OK) return st;
                a.k_new = a.v_new = nullptr;
            }                                              // (otherwise the decode kernel appends by itself)
            st = launch_decode_mfma(a, s);
            if (st != PA_OK) return st;
            return launch_merge(a, s);
        }
        a.plan = plan_decode(batch, max_seq_len, cache->page_size);
        const size_t po = part_o_bytes(batch, num_q_heads, d, a.plan.nsplit);
        if (a.plan.nsplit > 1 && ws.bytes < po + part_lse_bytes(batch, num_q_heads, a.plan.nsplit))
            return PA_ERR_WORKSPACE_TOO_SMALL;
        // (behind the check above: a workspace or scratch array that was too small for the chunks' partials stays too small)
        if (f32 && decode_f32_supported(a)) {
            plan_f32_splits(a, ws.bytes);
            if (a.short_nsplit > 1)
                place_split(f32_split_bytes(a, a.short_nsplit), (int64_t)batch * cache->num_kv_heads);
            return launch_decode_f32(a, s);
        }
        a.part_o = reinterpret_cast<float*>(base);
        a.part_lse = reinterpret_cast<float*>(base + po);
        // (With one or two KV heads and room on the machine for every (row, head, chunk) the portable kernel was never slower
        // than one matrix tile for a group's heads, at head_dim 128 by up to 8 %: us portable / matrix, 16 / 1 heads, 1 x 256
        // 16.2 / 17.2, 1 x 1000 20.1 / 21.8, 8 x 300 20.3 / 20.9; 32 / 2, 1 x 1000 20.3 / 22.0, 1 x 4000, 512 workgroups, 36.7 /
        // 27.6; 16 / 1 at head_dim 64, 1 x 1000 14.6 / 15.0; one tile a wave, 1 x 128, 7.9 / 7.6; 40 / 8 heads, 1 x 600 22.6 / 20.2.)
        const bool few = cache->num_kv_heads <= 2 && max_seq_len > 192 &&
                         (int64_t)batch * num_q_heads * a.plan.nsplit <= device_cus();
        st = f32 && !few ? launch_attention_f32(a, s) : launch_attention_generic(a, s);
        if (st != PA_OK) return st;
        if (a.plan.nsplit > 1) st = launch_merge(a, s);
        return st;
    }
    if (!g_opt.force_generic && prefill_mfma_supported(a)) {
        // Jagged batch: sequences with few queries (q_len * G <= 16: decode rows, a few speculative tokens) are
        // bound by streaming their context once, which the decode kernel's equal-work tile stream does best; the
        // others go to the prefill kernel.  Both kernels decide per sequence from cu_q_lens on the device; the
        // host only skips a launch that cannot find work.
        const int32_t G = num_q_heads / cache->num_kv_heads;
        // Where it cannot pay, its two launches are left out.  That is when no sequence can have so few queries (the others
        // have at most max_q_len), and when the call is whole prompts in the main (no context longer than the longest
        // query range, half of that range on average): a few-query sequence among those walks no more keys than the
        // longest prompt's last row tile does beside it.  Append + prefill, with / without: 2 prompts of 300 .. 900 tokens
        // 31.1 / 27.5 us, 16 of 60 .. 170 with 8 / 1 heads 17.3 / 13.1, 4 of 700 .. 2000 122 / 118; 24 prompts of 300 ..
        // 1000 among 8 single queries 240 / 234.  Below that average it does pay: one prompt of 2048 tokens among 15 single
        // queries on 1000 .. 2048 keys 175 / 186, one of 4000 among 7 447 / 495.
        const int64_t least_q = (int64_t)total_q - (int64_t)(batch - 1) * max_q_len;
        const bool whole_prompts = max_seq_len <= max_q_len && 2LL * total_q >= (int64_t)batch * max_q_len;
        bool may_have_small = !g_opt.no_small_q_route && decode_mfma_supported(a) && G <= 16 && least_q * G <= 16 &&
                              !whole_prompts;
        const int32_t lg = prefill_mfma_log2_pack(num_q_heads, cache->num_kv_heads);
        SplitPlan pp = plan_prefill(batch, num_q_heads, lg, total_q, max_seq_len, cache->page_size);
        // (a workspace that holds what is required and not the list's partials as well keeps the plain grid)
        int64_t list_items = 0;
        if (list_pays(a, lg) &&
            ws.bytes >= required_workspace_bytes(batch, num_q_heads, d, total_q, max_seq_len) + list_bytes(d))
            list_items = prefill_list_items(a);
        if (list_items * (num_q_heads >> lg) > 0x7fffffffLL) list_items = 0;
        const bool list_cuts = list_items > 0;
        if (prefill_padded_dim(d) && !list_cuts && prefill_grid_mostly_empty(a)) {
            // These head_dims came from the portable kernel, whose grid has no empty workgroups.  The list without cuts has none
            // either; it pays beyond one round of the machine's slots while one wave sees all sequences at once, and where
            // empty workgroups cost more than its scans (plain grid / list, D = 96: 64 sequences of up to 2048 tokens, four
            // with 300 queries 100 / 74 us, 8 prompts of 33 .. 900 with 8 / 2 heads, 464 workgroups 30.4 / 31.0; 256 sequences,
            // four with 300 queries, 20480 workgroups 68 / 89, one with 2048, 131072 155 / 181).  A few rows on a long
            // context, which the plain grid cuts, go back to the portable kernel where the empty ones cost as much as it does.
            const double wgs = prefill_grid_workgroups(a, pp.nsplit);
            if (pp.nsplit == 1 && max_seq_len < (1 << 28) && prefill_list_supported(a) && wgs > 512.0 &&
                (batch <= 64 || wgs > 262144.0) && prefill_list_items(a) * (num_q_heads >> lg) <= 0x7fffffffLL)
                list_items = prefill_list_items(a);
            else if (wgs > 262144.0 || (pp.nsplit > 1 && wgs > 65536.0))
                return launch_attention_generic(a, s);
        }
        // (a ragged call's row tiles are few and unequal, its bound on them loose: 33 sequences of up to 2232 tokens, four with 200
        // queries, 85 us with the two chunks of plan_prefill, 89 with the one that this would choose)
        if (pp.nsplit > 1 && g_opt.prefill_chunk_tokens == 0 && m.window == 0 && max_seq_len / 2 >= max_q_len &&
            (int64_t)batch * max_q_len == total_q) {
            const int64_t tiles = (((int64_t)max_q_len << lg) + 127) / 128 * batch;
            pp = even_prefill_split(pp, batch, tiles * (num_q_heads >> lg), (int64_t)total_q * num_q_heads, max_seq_len,
                                    cache->page_size, d);
        }
        if (!may_have_small && list_items == 0 && g_opt.prefill_chunk_tokens == 0 && max_seq_len / 2 < max_q_len) {
            // (as many as the whole bound holds, or else what is required, also in a larger workspace: the same call gives the same
            // bits.  Two prompts of 4200 tokens, 4 / 1 heads, head_dim 64, slopes: 5 chunks in the bound 75 us, 4 in what is required 81)
            const size_t bound = paged_attention_workspace_bytes(batch, num_q_heads, d, total_q, max_seq_len);
            pp = prompt_split(a, lg, pp, ws.bytes >= bound ? bound : required_workspace_bytes(batch, num_q_heads, d, total_q, max_seq_len));
        }
        int32_t small_wgs = 0;
        if (may_have_small) {
            const int32_t head_groups = cache->num_kv_heads / decode_mfma_heads_per_wg(cache->num_kv_heads, d);
            small_wgs = plan_stream_wgs(batch, max_seq_len, head_groups, cache->num_kv_heads, 1);
            const int32_t cap = small_route_wgs_cap(cache->num_kv_heads);
            if (small_wgs > cap) small_wgs = cap;
        }
        const size_t small_bytes = may_have_small ? small_route_bytes(small_wgs, batch, cache->num_kv_heads, d) : 0;
        // Jagged calls on shorter contexts than the list has slots for: the list for the sake of the launch that it shares with
        // the few-query stream, uncut where the plain grid is, else cut by each context's own length into the plain grid's
        // partials (if the workspace holds the stream's as well: the list alone would only lose the plain order).
        size_t split_bytes =
            pp.nsplit > 1 ? part_o_bytes(total_q, num_q_heads, d, pp.nsplit) + part_lse_bytes(total_q, num_q_heads, pp.nsplit)
                          : 0;
        const bool list_short = list_items == 0 && may_have_small && ws.bytes >= split_bytes + small_bytes &&
                                jagged_short_list_pays(a, lg);
        if (list_short) list_items = prefill_list_items(a);
        if (list_short && pp.nsplit > 1) pp.unit = cache->page_size > 64 ? cache->page_size : 64;
        if (list_cuts) {
            pp.chunk = max_seq_len;
            pp.nsplit = 1;
            split_bytes = list_bytes(d);
        }
        // The route is an optimisation: a workspace without room for its partials (a call with total_q == batch is promised the
        // decode bound only) keeps those sequences on the prefill kernel.
        if (ws.bytes < split_bytes + small_bytes) may_have_small = false;
        const bool may_have_large = (int64_t)max_q_len * G > 16 || !may_have_small;
        if (ws.bytes < split_bytes) return PA_ERR_WORKSPACE_TOO_SMALL;
        if (may_have_large) {
            AttnArgs b = a;
            b.skip_small = may_have_small ? 1 : 0;
            b.plan = pp;
            b.part_o = reinterpret_cast<float*>(base);
            b.part_lse = reinterpret_cast<float*>(base + part_o_bytes(total_q, num_q_heads, d, pp.nsplit));
            b.list_items = (int32_t)list_items;
            if (list_cuts) {
                a.list_items = b.list_items;
                a.list_o = b.list_o = reinterpret_cast<float*>(base);
                a.list_lse = b.list_lse = reinterpret_cast<float*>(
                    base + align256(prefill_list_slots() * prefill_list_slot_floats(d) * sizeof(float)));
                a.skip_small = b.skip_small;
            }
            const int32_t beside = (list_cuts || list_short) && may_have_small ? jagged_mfma_stream_wgs(b, device_cus()) : 0;
            if (beside > 0) {                              // both in one launch, their pieces merged by one
                AttnArgs c = a;
                c.stream_split = 1;
                c.num_wgs = beside < small_wgs ? beside : small_wgs;
                place_stream(c, base + split_bytes, ((size_t)c.num_wgs + batch) * cache->num_kv_heads * 16);
                if (pp.nsplit > 1) {
                    c.plan = pp;
                    c.rows_o = b.part_o;
                    c.rows_lse = b.part_lse;
                }
                st = launch_jagged_mfma(b, c, device_cus(), s);
                return st != PA_OK ? st : launch_merge(c, s);
            }
            st = launch_prefill_mfma(b, device_cus(), s);
            if (st != PA_OK) return st;
            if (list_cuts && !may_have_small) return launch_merge(a, s);
        }
        if (may_have_small) {
            AttnArgs b = a;
            b.stream_split = 1;
            b.num_wgs = small_wgs;
            place_stream(b, base + split_bytes, ((size_t)small_wgs + batch) * cache->num_kv_heads * 16);
            st = launch_decode_mfma(b, s);
            if (st != PA_OK) return st;
            st = launch_merge(b, s);
        }
        return st;
    }
    // (A few query rows on a short context: the portable kernel has a workgroup for each and was never slower than one matrix
    // tile for all, at head_dim 128 by up to 8 %: us portable / matrix, 8 / 8 heads, 16 queries on 250 keys 18.6 / 20.2, on
    // 500 30.1 / 31.4, on 1000 53.2 / 53.0; 32 on 250 19.3 / 20.3, on 500 31.1 / 31.5; 64 on 250 22.7 / 20.4.  At head_dim
    // 64 2 % and less: 16 on 250 13.3 / 13.5, on 500 19.0 / 19.3, on 1000 31.1 / 31.6; 32 on 250 13.7 / 13.6.)
    const bool few = batch == 1 && (int64_t)total_q * num_q_heads <= (d > 64 ? 256 : 128) && max_seq_len >= 128 && max_seq_len <= 768;
    return f32 && !few ? launch_attention_f32(a, s) : launch_attention_generic(a, s);
}

// Device address of this GPU's copy of `scratch`, looked up once per device with that device current.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

pa_status static_scratch(void** ptr)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return PA_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return PA_ERR_HIP;
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return PA_OK;
}

}  // namespace


void profile_begin(const char* kernel, hipStream_t stream)
{
    if (!g_profile_on) return;
    std::lock_guard<std::mutex> lock(g_profile_mutex);
    ProfileRecord r;
    r.kernel = kernel;
    if (!take_event(&r.start)) return;
    if (!take_event(&r.stop)) {
        g_spare_events.push_back(r.start);
        return;
    }
    (void)hipEventRecord(r.start, stream);
    g_records.push_back(r);
}

void profile_end(hipStream_t stream)
{
    if (!g_profile_on) return;
    std::lock_guard<std::mutex> lock(g_profile_mutex);
    if (!g_records.empty()) (void)hipEventRecord(g_records.back().stop, stream);
}

}  // namespace pa

using namespace pa;

extern "C" {

pa_status paged_kv_append(const pa_kv_cache_desc* cache, const void* k_new, const void* v_new,
                          const int32_t* seq_ids, const int32_t* positions, int32_t T, const int32_t* block_table,
                          int32_t batch, int32_t max_blocks, void* stream)
{
    pa_status st = check_cache(cache);
    if (st != PA_OK) return st;
    if (T < 0 || batch < 0 || max_blocks < 0) return PA_ERR_INVALID_ARG;
    if (T == 0) return PA_OK;
    if (!k_new || !v_new || !seq_ids || !positions || !block_table || batch == 0 || max_blocks == 0)
        return PA_ERR_INVALID_ARG;
    if (((uintptr_t)k_new | (uintptr_t)v_new) & 15) return PA_ERR_UNSUPPORTED;
    return launch_kv_append(cache, k_new, v_new, seq_ids, positions, T, block_table, max_blocks,
                            reinterpret_cast<hipStream_t>(stream));
}

pa_status paged_kv_gather(const pa_kv_cache_desc* cache, void* out_k, void* out_v, const int32_t* block_table,
                          const int32_t* seq_lens, const int32_t* cu_seq_lens, int32_t batch, int32_t max_blocks,
                          int32_t max_seq_len, void* stream)
{
    pa_status st = check_cache(cache);
    if (st != PA_OK) return st;
    if (batch < 0 || max_blocks < 0 || max_seq_len < 0) return PA_ERR_INVALID_ARG;
    if (batch == 0 || max_seq_len == 0) return PA_OK;
    if (!out_k || !out_v || !block_table || !seq_lens || !cu_seq_lens) return PA_ERR_INVALID_ARG;
    if ((int64_t)max_blocks * cache->page_size < max_seq_len) return PA_ERR_INVALID_ARG;
    if (((uintptr_t)out_k | (uintptr_t)out_v) & 15) return PA_ERR_UNSUPPORTED;
    return launch_kv_gather(cache, out_k, out_v, block_table, seq_lens, cu_seq_lens, batch, max_blocks, max_seq_len,
                            reinterpret_cast<hipStream_t>(stream));
}

pa_status pa_debug_check(const pa_kv_cache_desc* cache, const int32_t* block_table, const int32_t* seq_lens,
                         int32_t batch, int32_t max_blocks, const int32_t* seq_ids, const int32_t* positions, int32_t T,
                         void* scratch, int64_t* counts, void* stream)
{
    pa_status st = check_cache(cache);
    if (st != PA_OK) return st;
    if (batch < 0 || max_blocks < 0 || T < 0 || !counts || !scratch) return PA_ERR_INVALID_ARG;
    if (((uintptr_t)scratch & 7) || (batch > 0 && (!block_table || !seq_lens)) || (T > 0 && (!seq_ids || !positions)))
        return PA_ERR_INVALID_ARG;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    st = launch_debug_check(cache, block_table, seq_lens, batch, max_blocks, seq_ids, positions, T, scratch, s);
    if (st != PA_OK) return st;
    unsigned long long host[4] = {0, 0, 0, 0};
    if (hipMemcpyAsync(host, scratch, sizeof(host), hipMemcpyDeviceToHost, s) != hipSuccess) return PA_ERR_HIP;
    if (hipStreamSynchronize(s) != hipSuccess) return PA_ERR_HIP;
    for (int i = 0; i < 3; ++i) counts[i] = (int64_t)host[i];
    return PA_OK;
}

size_t paged_attention_workspace_bytes(int32_t batch, int32_t num_q_heads, int32_t head_dim, int32_t total_q,
                                       int32_t max_seq_len)
{
    const size_t need = required_workspace_bytes(batch, num_q_heads, head_dim, total_q, max_seq_len);
    // (dtype, hooks, page size and the query lengths' spread, which also decide, are not known here)
    const bool sized = batch > 0 && num_q_heads > 0 && prefill_list_dim(head_dim) && total_q > 0;
    return need + (sized && list_possible(batch, total_q, max_seq_len) ? list_bytes(head_dim) : 0);
}

pa_status paged_attention_decode(const pa_kv_cache_desc* cache, const void* q, void* out, float* lse,
                                 const int32_t* block_table, const int32_t* seq_lens, int32_t batch,
                                 int32_t num_q_heads, int32_t max_blocks, int32_t max_seq_len, float scale,
                                 void* workspace, size_t workspace_bytes, void* stream)
{
    return run_attention(cache, q, out, lse, nullptr, batch, 1, block_table, seq_lens, batch, num_q_heads, max_blocks,
                         max_seq_len, scale, 0, nullptr, Workspace{workspace, workspace_bytes, true}, stream, true);
}

pa_status paged_attention_decode_mod(const pa_kv_cache_desc* cache, const void* q, void* out, float* lse,
                                     const int32_t* block_table, const int32_t* seq_lens, int32_t batch,
                                     int32_t num_q_heads, int32_t max_blocks, int32_t max_seq_len, float scale,
                                     const pa_attn_mods* mods, void* workspace, size_t workspace_bytes, void* stream)
{
    return run_attention(cache, q, out, lse, nullptr, batch, 1, block_table, seq_lens, batch, num_q_heads, max_blocks,
                         max_seq_len, scale, 0, mods, Workspace{workspace, workspace_bytes, true}, stream, true);
}

pa_status paged_attention_decode_static(const pa_kv_cache_desc* cache, const void* q, void* out, float* lse,
                                        const int32_t* block_table, const int32_t* seq_lens, int32_t batch,
                                        int32_t num_q_heads, int32_t max_blocks, int32_t max_seq_len, float scale,
                                        void* stream)
{
    void* ptr = nullptr;
    if (batch > 0) {
        const pa_status st = static_scratch(&ptr);
        if (st != PA_OK) return st;
    }
    const pa_status st = run_attention(cache, q, out, lse, nullptr, batch, 1, block_table, seq_lens, batch, num_q_heads,
                                       max_blocks, max_seq_len, scale, 0, nullptr,
                                       Workspace{ptr, kStaticScratchBytes, false}, stream, true);
    return st == PA_ERR_WORKSPACE_TOO_SMALL ? PA_ERR_SCRATCH_LIMIT : st;
}

pa_status paged_decode_step(const pa_kv_cache_desc* cache, const void* k_new, const void* v_new, const void* q,
                            void* out, float* lse, const int32_t* block_table, const int32_t* seq_lens, int32_t batch,
                            int32_t num_q_heads, int32_t max_blocks, int32_t max_seq_len, float scale,
                            const pa_attn_mods* mods, void* workspace, size_t workspace_bytes, void* stream)
{
    if (batch > 0 && (!k_new || !v_new)) return PA_ERR_INVALID_ARG;
    if (((uintptr_t)k_new | (uintptr_t)v_new) & 15) return PA_ERR_UNSUPPORTED;
    return run_attention(cache, q, out, lse, nullptr, batch, 1, block_table, seq_lens, batch, num_q_heads, max_blocks,
                         max_seq_len, scale, 0, mods, Workspace{workspace, workspace_bytes, true}, stream, true, k_new, v_new);
}

pa_status paged_attention_prefill_mod(const pa_kv_cache_desc* cache, const void* q, void* out, float* lse,
                                      const int32_t* cu_q_lens, int32_t total_q, int32_t max_q_len,
                                      const int32_t* block_table, const int32_t* seq_lens, int32_t batch,
                                      int32_t num_q_heads, int32_t max_blocks, int32_t max_seq_len, float scale,
                                      int32_t causal, const pa_attn_mods* mods, void* workspace,
                                      size_t workspace_bytes, void* stream)
{
    return run_attention(cache, q, out, lse, cu_q_lens, total_q, max_q_len, block_table, seq_lens, batch, num_q_heads,
                         max_blocks, max_seq_len, scale, causal, mods, Workspace{workspace, workspace_bytes, true}, stream, false);
}

pa_status paged_attention_prefill(const pa_kv_cache_desc* cache, const void* q, void* out, float* lse,
                                  const int32_t* cu_q_lens, int32_t total_q, int32_t max_q_len,
                                  const int32_t* block_table, const int32_t* seq_lens, int32_t batch,
                                  int32_t num_q_heads, int32_t max_blocks, int32_t max_seq_len, float scale,
                                  int32_t causal, void* workspace, size_t workspace_bytes, void* stream)
{
    return run_attention(cache, q, out, lse, cu_q_lens, total_q, max_q_len, block_table, seq_lens, batch, num_q_heads,
                         max_blocks, max_seq_len, scale, causal, nullptr, Workspace{workspace, workspace_bytes, true}, stream, false);
}

const char* pa_status_string(pa_status status)
{
    switch (status) {
        case PA_OK: return "ok";
        case PA_ERR_INVALID_ARG: return "invalid argument";
        case PA_ERR_UNSUPPORTED: return "unsupported dtype, shape or alignment";
        case PA_ERR_WORKSPACE_TOO_SMALL: return "workspace too small";
        case PA_ERR_HIP: return "HIP call failed";
        case PA_ERR_OUT_OF_PAGES: return "page pool exhausted";
        case PA_ERR_SCRATCH_LIMIT: return "the call's split-KV partials exceed the 16 MiB static scratch array";
    }
    return "unknown status";
}

pa_status pa_set_option(const char* name, int64_t value)
{
    if (!name) return PA_ERR_INVALID_ARG;
    if (!strcmp(name, "decode_chunk_tokens")) {
        if (value < 0 || value > (1 << 24)) return PA_ERR_INVALID_ARG;
        g_opt.decode_chunk_tokens = value;
        return PA_OK;
    }
    if (!strcmp(name, "decode_workgroups")) {
        if (value < 0 || value > kMaxDecodeWGs) return PA_ERR_INVALID_ARG;
        g_opt.decode_workgroups = value;
        return PA_OK;
    }
    if (!strcmp(name, "prefill_chunk_tokens")) {
        if (value < 0 || value > (1 << 24)) return PA_ERR_INVALID_ARG;
        g_opt.prefill_chunk_tokens = value;
        return PA_OK;
    }
    if (!strcmp(name, "no_small_q_route")) {
        if (value != 0 && value != 1) return PA_ERR_INVALID_ARG;
        g_opt.no_small_q_route = value;
        return PA_OK;
    }
    if (!strcmp(name, "step_append_kernel")) {
        if (value != 0 && value != 1) return PA_ERR_INVALID_ARG;
        g_opt.step_append_kernel = value;
        return PA_OK;
    }
    if (!strcmp(name, "decode_short")) {
        if (value < -1 || value > 1) return PA_ERR_INVALID_ARG;
        g_opt.decode_short = value;
        return PA_OK;
    }
    if (!strcmp(name, "decode_short_splits")) {
        if (value < 0 || value > 16) return PA_ERR_INVALID_ARG;
        g_opt.decode_short_splits = value;
        return PA_OK;
    }
    if (!strcmp(name, "force_generic")) {
        if (value != 0 && value != 1) return PA_ERR_INVALID_ARG;
        g_opt.force_generic = value;
        return PA_OK;
    }
    return PA_ERR_INVALID_ARG;
}

pa_status pa_stream_read(const void* a, const void* b, size_t bytes_each, void* sink, void* stream)
{
    if (!a || !b || !sink || (((uintptr_t)a | (uintptr_t)b | (uintptr_t)sink) & 15)) return PA_ERR_INVALID_ARG;
    return launch_stream_read(a, b, bytes_each, sink, reinterpret_cast<hipStream_t>(stream));
}

pa_status pa_profile_enable(int32_t on)
{
    std::lock_guard<std::mutex> lock(g_profile_mutex);
    g_profile_on = on != 0;
    return PA_OK;
}

pa_status pa_profile_reset(void)
{
    std::lock_guard<std::mutex> lock(g_profile_mutex);
    for (auto& r : g_records) {
        (void)hipEventSynchronize(r.stop);
        g_spare_events.push_back(r.start);
        g_spare_events.push_back(r.stop);
    }
    g_records.clear();
    return PA_OK;
}

pa_status pa_profile_read(const char* kernel_prefix, int32_t* launches, double* total_ms)
{
    if (!kernel_prefix || !launches || !total_ms) return PA_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lock(g_profile_mutex);
    const size_t n = strlen(kernel_prefix);
    int32_t count = 0;
    double sum = 0.0;
    for (auto& r : g_records) {
        if (r.kernel.compare(0, n, kernel_prefix) != 0) continue;
        if (hipEventSynchronize(r.stop) != hipSuccess) return PA_ERR_HIP;
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, r.start, r.stop) != hipSuccess) return PA_ERR_HIP;
        sum += ms;
        ++count;
    }
    *launches = count;
    *total_ms = sum;
    return PA_OK;
}

}  // extern "C"
