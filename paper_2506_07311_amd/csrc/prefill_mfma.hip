// Paged prefill on the matrix cores: support check, launch plan, dispatch over head_dim, and the head_dim 128
// kernels.
#include "prefill_mfma_impl.h"

namespace pa {

using namespace prefill;

template pa_status launch_prefill_mfma_dim<128>(const AttnArgs&, const PrefillPlan&, int64_t, int64_t, hipStream_t);
extern template pa_status launch_prefill_mfma_dim<64>(const AttnArgs&, const PrefillPlan&, int64_t, int64_t,
                                                      hipStream_t);
extern template pa_status launch_prefill_mfma_dim<256>(const AttnArgs&, const PrefillPlan&, int64_t, int64_t,
                                                       hipStream_t);

extern template pa_status launch_prefill_mfma_dim<80>(const AttnArgs&, const PrefillPlan&, int64_t, int64_t,
                                                      hipStream_t);
extern template pa_status launch_prefill_mfma_dim<96>(const AttnArgs&, const PrefillPlan&, int64_t, int64_t,
                                                      hipStream_t);
extern template pa_status launch_prefill_mfma_dim<112>(const AttnArgs&, const PrefillPlan&, int64_t, int64_t,
                                                       hipStream_t);

bool prefill_mfma_supported(const AttnArgs& a)
{
    if (a.dtype != PA_DTYPE_BF16 && a.dtype != PA_DTYPE_F16) return false;
    const int32_t d = a.cache.head_dim;
    // head_dims 80, 96, 112 without hooks, pages of 16 tokens and more: faster than the portable kernel at every size
    // (append + prefill, portable / this kernel): 1 x 8 tokens 8.6 / 7.2 us, 1 x 100 with 32 heads 20.1 / 9.7, 2 x 300
    // 138 / 13.0, 2 prompts of 700 and 950 tokens with 32 / 32 heads at D = 96 1075 / 36; 2 rows behind 4000 cached
    // tokens 83.5 / 33.3.  Hooks and smaller pages stay on the portable kernel: instantiations for them do not exist.
    const bool odd = prefill_padded_dim(d) && !a.has_mods && a.cache.page_size >= 16;
    if (d != 128 && d != 64 && !(d == 256 && a.cache.page_size >= 16) && !odd) return false;
    if (!(a.scale > 0.f)) return false;   // the kernel takes the max before scaling
    // the tile fetch keeps a row's byte offset inside its page (slot, KV head, piece) in 32 bits
    const int64_t in_page = (int64_t)(a.cache.page_size - 1) * a.cache.token_stride * 2 +
                            (int64_t)(a.cache.num_kv_heads - 1) * a.cache.head_stride * 2 + 512;
    if (in_page > 0xffffffffLL) return false;
    return true;
}

int32_t prefill_mfma_log2_pack(int32_t num_q_heads, int32_t num_kv_heads)
{
    // all heads of a group when the group size is a power of two (up to 16), else no packing
    const int32_t g = num_q_heads / num_kv_heads;
    int32_t lg = 0;
    while ((1 << (lg + 1)) <= g && lg < 4) ++lg;
    return (1 << lg) == g ? lg : 0;
}

int32_t prefill_list_slots() { return 2 * kListTarget; }
size_t prefill_list_slot_floats(int32_t head_dim) { return list_slot_floats(head_dim); }
int32_t prefill_list_min_context() { return 2 * kListMinTiles * kBN; }

// (the work list has no instantiations with hooks or for pages below 16 tokens)
bool prefill_list_supported(const AttnArgs& a) { return !a.has_mods && a.cache.page_size >= 16; }

// Items: every chunk holds at least 1 / kListTarget of the call's work, plus one rounded-up chunk per row tile.
int64_t prefill_list_items(const AttnArgs& a)
{
    const int32_t lg = prefill_mfma_log2_pack(a.num_q_heads, a.cache.num_kv_heads);
    return kListTarget / (a.num_q_heads >> lg) + (((int64_t)a.total_q << lg) / kBM) +
           (a.batch < a.total_q ? a.batch : a.total_q) + 1;
}

static int64_t plain_row_tiles(const AttnArgs& a)
{
    return (((int64_t)a.max_q_len << prefill_mfma_log2_pack(a.num_q_heads, a.cache.num_kv_heads)) + kBM - 1) / kBM;
}
bool prefill_grid_mostly_empty(const AttnArgs& a)
{
    const int32_t lg = prefill_mfma_log2_pack(a.num_q_heads, a.cache.num_kv_heads);
    return plain_row_tiles(a) * a.batch > 2 * ((((int64_t)a.total_q << lg) / kBM) + a.batch);
}
double prefill_grid_workgroups(const AttnArgs& a, int32_t nsplit)
{
    const int32_t lg = prefill_mfma_log2_pack(a.num_q_heads, a.cache.num_kv_heads);
    return (double)plain_row_tiles(a) * nsplit * (a.num_q_heads >> lg) * a.batch;
}

PrefillPlan prefill::make_plan(const AttnArgs& a)
{
    PrefillPlan plan;
    plan.list_items = a.list_items;
    plan.list_o = a.list_o;
    plan.list_lse = a.list_lse;
    plan.list_unit = !a.list_o ? kListUncut : a.cache.page_size > kBN ? a.cache.page_size : kBN;
    plan.log2_pack = prefill_mfma_log2_pack(a.num_q_heads, a.cache.num_kv_heads);
    plan.group = a.num_q_heads / a.cache.num_kv_heads;
    plan.chunk = a.plan.chunk;
    plan.chunk_unit = a.plan.unit;
    plan.order = kByTile;
    plan.nsplit = a.plan.nsplit;
    plan.skip_small = a.skip_small;
    plan.part_o = a.part_o;
    plan.part_lse = a.part_lse;
    plan.mods = a.mods;
    return plan;
}

// Workgroups go to the eight chiplets in turn and on each to its four shader engines in turn, 32 places in all.  How often do
// workgroups that come every `every` of them fall on another place before they are back at the first?
static int64_t turns(int64_t every)
{
    int64_t n = 32;
    while (n > 1 && every % 2 == 0) {
        n /= 2;
        every /= 2;
    }
    return n;
}
// Do `own` workgroups in a row that come every `every` fall on all places alike?
static bool goes_round(int64_t every, int64_t own) { return turns(every) * own % 32 == 0; }

// Chunk after chunk, the first row tiles of causal prompts, which have no keys in the later chunks, leave no gaps among the others;
// tile after tile the workgroups that are handed out last have the least to do.  The latter is better where the
// gaps go round (as with an odd number of chunks on a sequence's one head group) and there is a queue at all.  us chunk after chunk /
// tile after tile, three chunks, 8 / 1 heads: 4000 tokens at head_dim 64 47.4 / 42.4, with slopes 89 / 72.5, 5000 60 / 55, 2366 at
// head_dim 256 with documents 83 / 68.5; without a queue 2700 with a cap 43.0 / 44.4, 2500 29.4 / 30.8; where the gaps stay, four
// chunks of 4000 45 / 56, two of 3131 at head_dim 256 77 / 111.
static bool prefill_chunks_by_tile(const AttnArgs& a, int32_t nsplit, int32_t cus)
{
    const int32_t lg = prefill_mfma_log2_pack(a.num_q_heads, a.cache.num_kv_heads), heads = a.num_q_heads >> lg;
    const int64_t most = (((int64_t)a.total_q << lg) / kBM) + a.batch, tiles = plain_row_tiles(a) * a.batch;
    const double live = (double)(tiles < most ? tiles : most) * heads * (1.0 + (nsplit - 1) * (a.causal ? 0.5 : 1.0));
    const bool equal = (int64_t)a.batch * a.max_q_len == a.total_q;
    return live > (a.cache.head_dim > 128 ? 1.0 : 1.7) * cus &&
           goes_round((int64_t)a.batch * heads * nsplit, (int64_t)heads * (equal ? a.batch : 1));
}

pa_status launch_prefill_mfma(const AttnArgs& a, int32_t cus, hipStream_t stream)
{
    PrefillPlan plan = make_plan(a);
    if (plan.nsplit > 1 && (plan.chunk % kBN != 0 || plan.chunk % a.cache.page_size != 0)) return PA_ERR_INVALID_ARG;
    const int64_t tiles = (((int64_t)a.max_q_len << plan.log2_pack) + kBM - 1) / kBM;
    if (tiles <= 0) return PA_OK;
    const int32_t heads = a.num_q_heads >> plan.log2_pack;
    int64_t row_tiles = tiles * a.batch;
    // Sequences with fewer queries than the longest leave gaps in a grid of the longest's row tiles.  Gaps that fall on the
    // same shader engines again and again (goes_round) leave their compute units idle while the others have a queue
    // (locate_live); without gaps a workgroup starts 0.5 us later, which shows where the longest walk is a few tiles and is all there
    // is to see where the gaps go round.  us with gaps / without, attention alone, 32 / 8 heads: 4 prompts of up to 1546 tokens at
    // head_dim 256 224 / 106, of up to 2436 500 / 420, 8 of up to 727 with a cap 48 / 41, 16 of up to 738 92 / 84, 4 of up to 838 with
    // 64 / 8 heads 60 / 34; where they go round, 5 of up to 1359 at head_dim 64 29.1 / 30.9, 3 of up to 3519 with 16 / 2 80 / 84, 15
    // of up to 675 with 40 / 8 56 / 60.  Of 150 ragged calls 30 lost (1 % in the mean) where the gaps go round, and 56 gained 10 %
    // elsewhere; the rule still loses with 24 / 8 heads, 4 of up to 1261 at head_dim 64 22.9 / 24.3, and gives up 3 of up to 827 with
    // 40 / 8 19.9 / 17.4.  (Up to 64 sequences: a lane for each finds its row tiles.)
    // Where most of the grid would be gaps, in a call that is mostly decode rows above all, leaving them out is worth it wherever they
    // fall (queries fill as few sequences as the longest allows: `few` row tiles): 13 sequences, four with 512 queries, 16 / 2
    // heads, head_dim 64, window and cap, 55 / 41, 49 of which 19 bring up to 512, 8 / 1 heads at 256, 152 / 125, 43 of which two bring
    // 179, 40 / 8 heads with a cap 44 / 39; 60 such calls 0.973 in the mean, 1.02 at worst.
    // So it is where a row tile's keys take long (head_dim 256, a score hook, document masks) unless a sequence has all 32 places: 11 prompts
    // of up to 989 tokens, 8 / 2 heads, head_dim 256, 69 / 61, 5 of up to 786 with 24 / 8 and a cap 35 / 32, 15 of up to 587 with 8 / 8,
    // slopes, 256 55 / 50; 48 such calls 0.970 in the mean, 1.02 at worst, 42 others where gaps go round 1.013.
    const bool costly = (a.cache.head_dim > 128 || a.mods.alibi_slopes || a.mods.user_mod || a.mods.softcap > 0.f ||
                         a.mods.doc_ids) && heads % 32 != 0;
    int64_t window = a.mods.window;
    if (!a.causal && window > 0) window = 2 * window - 1;    // keys that a row sees
    const int64_t walk = window > 0 && window < a.max_seq_len ? window : a.max_seq_len;
    const int64_t full = ((int64_t)a.total_q << plan.log2_pack) / kBM, most = full + a.batch;
    const int64_t few = full + (a.total_q + a.max_q_len - 1) / a.max_q_len;
    if (plan.list_items == 0 && plan.chunk_unit == 0 && plan.nsplit == 1 && a.batch > 1 && a.batch <= 64 &&
        (int64_t)a.batch * a.max_q_len != a.total_q && row_tiles * heads > cus && walk >= 8 * kBN &&
        (row_tiles > 2 * few || (most < row_tiles && (!goes_round((int64_t)a.batch * heads, heads) || costly)))) {
        plan.order = kLiveTiles;
        if (row_tiles > most) row_tiles = most;
    } else if (plan.nsplit > 1 && plan.chunk_unit == 0) {
        // A window's keys are in one or two chunks, most of them the last ones of contexts, and the workgroups of all others end at
        // once: in front of those with keys they only cost their time.  us tile after tile / chunk after chunk / from the last one
        // on: 500 queries on 4589 keys, window 256, 64 / 8 heads 70 / 52 / 44.5, 1000 on 12406, window 1024, 16 / 8 at head_dim 64
        // 43.0 / 45.4 / 40.3, 256 on 30669 four times, window 256, 8 / 1 56 / 66 / 57 (40 calls in the mean 1 / 0.97 / 0.89).  Where
        // query counts differ the chunks stay beside each other while a sequence's row tiles then meet half of the 32 places: eight
        // sequences of up to 13760 keys, 8 / 1 heads, window 1000, one place, 155 / 68 / 82, four of up to 11738 with 32 / 8 at head_dim
        // 256, window 2000, cap, eight, 189 / 225 / 147; five of up to 7824 with 8 / 1, window 128, all, 37.3 / 39.9 / 40.6, five of up to
        // 8838 with 16 / 8, all, 40.6 / 43.9 / 43.0.  50 such calls with fewer places 1 / 0.95 / 0.92, 57 with more 1 / 1.02 / 1.01.
        if (window > 0 && window < a.max_seq_len) {
            if ((int64_t)a.batch * a.max_q_len == a.total_q || turns((int64_t)a.batch * heads * plan.nsplit) * heads < 16)
                plan.order = kLastChunkFirst;
        } else if (!prefill_chunks_by_tile(a, plan.nsplit, cus)) {
            plan.order = kByChunk;
        }
    } else if (plan.chunk_unit > 0) {
        plan.order = kByLengths;
    }
    int64_t blocks = plan.list_items > 0 ? (int64_t)plan.list_items * heads : row_tiles * plan.nsplit * heads;
    if (plan.list_items > 0 && blocks > kListGrid) blocks = kListGrid;
    if (blocks > 0x7fffffffLL) return PA_ERR_UNSUPPORTED;
    {
        static const char* const kOrders[] = {nullptr, "paged_prefill_mfma_kernel_live", "paged_prefill_mfma_kernel_last_chunk_first",
                                              "paged_prefill_mfma_kernel_by_tile", nullptr};
        const char* const variant = plan.order == kByTile && plan.nsplit == 1 ? nullptr : kOrders[plan.order];
        ProfileScope prof("paged_prefill_mfma_kernel", stream, variant);
        pa_status st;
        switch (a.cache.head_dim) {
            case 64: st = launch_prefill_mfma_dim<64>(a, plan, blocks, tiles, stream); break;
            case 80: st = launch_prefill_mfma_dim<80>(a, plan, blocks, tiles, stream); break;
            case 96: st = launch_prefill_mfma_dim<96>(a, plan, blocks, tiles, stream); break;
            case 112: st = launch_prefill_mfma_dim<112>(a, plan, blocks, tiles, stream); break;
            case 256: st = launch_prefill_mfma_dim<256>(a, plan, blocks, tiles, stream); break;
            default: st = launch_prefill_mfma_dim<128>(a, plan, blocks, tiles, stream); break;
        }
        if (st != PA_OK || plan.nsplit == 1) return st;    // (a work list is merged by launch_merge)
    }
    return launch_merge(a, stream);
}

}  // namespace pa
