// Split-KV merge: combines the per-chunk softmax partials of one (query row, head) exactly.
// With partial c holding the normalised output o_c and lse_c = log sum_j exp(score_j) over its keys,
//   M = max_c lse_c,  w_c = exp(lse_c - M),  out = sum_c w_c o_c / sum_c w_c,  lse = M + log sum_c w_c.
// Only the ceil(n_keys / chunk) chunks that hold keys are read; a row without keys gets out = 0, lse = -inf.
// A chunk whose scores held a NaN says so by a NaN for its LSE, and the row becomes NaN: only LSEs of -inf mean no key.
#include "prefill_tiles.h"

namespace pa {

namespace {

// An LSE as the maximum over the chunks takes it: a NaN, which fmaxf would drop, as +inf (and its weight is exp(NaN - inf)).
__device__ __forceinline__ float max_term(float lse) { return lse == lse ? lse : INFINITY; }

// OUT: element type of `out` as a pa_dtype value.
template <int OUT>
__device__ __forceinline__ void store_out(void* out, int64_t i, float r)
{
    if (OUT == PA_DTYPE_BF16)
        reinterpret_cast<uint16_t*>(out)[i] = (uint16_t)float_to_bf16_bits(r);
    else if (OUT == PA_DTYPE_F16)
        reinterpret_cast<uint16_t*>(out)[i] = (uint16_t)float_to_f16_bits(r);
    else
        reinterpret_cast<float*>(out)[i] = r;
}

// Four consecutive output elements of one row.
template <int OUT>
__device__ __forceinline__ void store_out4(void* out, int64_t i, float4 r)
{
    if (OUT == PA_DTYPE_F32) {
        *reinterpret_cast<float4*>(reinterpret_cast<float*>(out) + i) = r;
    } else {
        uint2 w;
        if (OUT == PA_DTYPE_BF16) {
            w.x = float_to_bf16_bits(r.x) | (float_to_bf16_bits(r.y) << 16);
            w.y = float_to_bf16_bits(r.z) | (float_to_bf16_bits(r.w) << 16);
        } else {
            w.x = float_to_f16_bits(r.x) | (float_to_f16_bits(r.y) << 16);
            w.y = float_to_f16_bits(r.z) | (float_to_f16_bits(r.w) << 16);
        }
        *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(out) + i) = w;
    }
}

// A workgroup of 256 threads merges kMergePairs (query row, head) pairs: 32 lanes per pair, four consecutive output
// columns per lane and pass (head_dim is a multiple of 4 for every supported element type), 16-byte loads of the
// partial rows.  (One small workgroup per pair, as this kernel once was, is bound by the rate at which workgroups are
// dispatched: 65536 of them for a 2048-token prompt with 32 heads.)
constexpr int kMergePairs = 8;

// Partials by (query row, head): `nsplit` slots each, filled as sequence_chunk cuts the row's context.
struct RowMerge {
    const float* part_o;
    const float* part_lse;
    int64_t pairs;
    int32_t blocks;          // of the launch, where it merges other partials too; 0 = none
    int32_t batch, causal, chunk, nsplit, unit;
    int32_t final_group;     // > 0: what a list beside the few-query stream wrote itself is left alone: rows of sequences with
                             // q_len * final_group <= 16 (the stream's) and of contexts in one piece
};

template <int OUT>
__device__ __forceinline__ void merge_rows(const RowMerge& p, int64_t o_idx, void* __restrict__ out, float* __restrict__ lse,
                                           const int32_t* __restrict__ cu_q_lens, const int32_t* __restrict__ seq_lens,
                                           int32_t num_q_heads, int32_t d)
{
    if (o_idx >= p.pairs) return;
    const int lane = threadIdx.x & 31;
    const int32_t row = (int32_t)(o_idx / num_q_heads);
    const RowInfo ri = locate_row(cu_q_lens, seq_lens, p.batch, row, p.causal);
    if (ri.pos >= ri.len) return;                        // behind the last sequence: rows that pad the buffers
    const int32_t own = sequence_chunk(ri.len, p.chunk, p.nsplit, p.unit);
    if (p.final_group > 0 && (ri.q_len * p.final_group <= 16 || own >= ri.len)) return;
    const int32_t n = (ri.n_keys + own - 1) / own;       // chunks that hold keys
    const float* pl = p.part_lse + o_idx * p.nsplit;
    const float* po = p.part_o + o_idx * p.nsplit * d;

    float M = -INFINITY;
    for (int32_t c = 0; c < n; ++c) M = fmaxf(M, max_term(pl[c]));
    const bool none = M == -INFINITY;            // no chunk holds a visible key (masks can empty every chunk)
    float wsum = 0.f;
    for (int32_t c = 0; c < n && !none; ++c) wsum += expf(pl[c] - M);
    for (int e = 4 * lane; e < d; e += 128) {
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int32_t c = 0; c < n && !none; ++c) {
            const float w = expf(pl[c] - M);
            const float4 v = *reinterpret_cast<const float4*>(po + (int64_t)c * d + e);
            acc.x = fmaf(w, v.x, acc.x);
            acc.y = fmaf(w, v.y, acc.y);
            acc.z = fmaf(w, v.z, acc.z);
            acc.w = fmaf(w, v.w, acc.w);
        }
        const float4 r = none ? make_float4(0.f, 0.f, 0.f, 0.f)
                              : make_float4(acc.x / wsum, acc.y / wsum, acc.z / wsum, acc.w / wsum);
        store_out4<OUT>(out, o_idx * d + e, r);
    }
    if (lse && lane == 0) lse[o_idx] = !none ? M + logf(wsum) : -INFINITY;
}

template <int OUT>
__global__ __launch_bounds__(256) void paged_attention_merge_kernel(
    RowMerge rows, void* __restrict__ out, float* __restrict__ lse, const int32_t* __restrict__ cu_q_lens,
    const int32_t* __restrict__ seq_lens, int32_t num_q_heads, int32_t d)
{
    merge_rows<OUT>(rows, (int64_t)blockIdx.x * kMergePairs + (threadIdx.x >> 5), out, lse, cu_q_lens, seq_lens, num_q_heads, d);
}

// Tile-stream layout: sequence s was cut by the workgroups seg_first[s] .. seg_last[s]; workgroup w left its
// partial at index (w + s).  seg_first[s] < 0 means one workgroup held the whole sequence and wrote the final
// result itself.  One workgroup merges one (sequence, head): the partial LSEs are fetched by as many threads at
// once and reduced through LDS, then every thread owns one output column and sums the weighted partial rows
// with independent loads (eight in flight), so the kernel costs a few memory latencies, not one per partial.
constexpr int kMergeThreads = 128;

// Partials of the prefill kernel's work list (prefill_tiles.h): blocks [0, blocks) of the launch.
struct ListMerge {
    const float* part_o;
    const float* part_lse;
    int32_t blocks;          // a multiple of 8; 0 = no work list
    int32_t batch, heads, log2_pack, small_group, unit, causal;
};

// Eight workgroups of two waves share a row tile of a sequence that is cut: 32 rows each and every second pair of a lane's
// 16-byte accumulator pieces, so that a few hundred tiles fill the machine; consecutive lanes read consecutive 16 bytes.
// Bound by reading the partials once (21 us for the 67 MB of four 512-token chunks on 2.7k to 31k tokens).
template <int OUT>
__device__ void merge_list(const ListMerge& p, int32_t block, void* __restrict__ out, float* __restrict__ lse,
                           const int32_t* __restrict__ cu_q_lens, const int32_t* __restrict__ seq_lens,
                           int32_t num_q_heads, int32_t d)
{
    using namespace prefill;
    const int lane = threadIdx.x & 63;
    const int32_t quarter = block & 3, piece = (block >> 1 & 2) + (int32_t)(threadIdx.x >> 6);
    const int32_t lg = p.log2_pack, T = (d + 31) / 32;
    const WorkList list = make_list(cu_q_lens, seq_lens, p.batch, lg, p.small_group, p.heads, p.unit, d, lane);
    for (int32_t index = block >> 3;; index += p.blocks >> 3) {
        const int32_t hg = index % p.heads;
        ListItem it;
        if (!list_locate<true>(it, list, cu_q_lens, seq_lens, index / p.heads, lane)) return;
        const int32_t q_begin = cu_q_lens[it.s], q_len = cu_q_lens[it.s + 1] - q_begin, len = seq_lens[it.s];
        const int32_t n_rows = q_len << lg, m0 = it.tile * kBM;
        const int32_t row = m0 + 32 * quarter + (lane & 31);
        // the chunks that hold keys of this row tile (the others left nothing behind)
        int32_t nk = len;
        if (p.causal) nk = min(len, len - q_len + ((min(m0 + kBM, n_rows) - 1) >> lg) + 1);
        const int32_t n = (max(nk, 0) + list.chunk - 1) / list.chunk;
        if (row >= n_rows) continue;                          // (nothing below is shared between lanes)
        const float* pl = p.part_lse + 32 * quarter + (lane & 31);
        float M = -INFINITY;
        for (int32_t c = 0; c < n; ++c) M = fmaxf(M, max_term(pl[(int64_t)list_slot(it, c, p.heads, hg) * kBM]));
        const bool none = M == -INFINITY;
        float wsum = 0.f;
        for (int32_t c = 0; c < n && !none; ++c) wsum += expf(pl[(int64_t)list_slot(it, c, p.heads, hg) * kBM] - M);
        const int64_t o_row = (int64_t)(q_begin + (row >> lg)) * num_q_heads + (hg << lg) + (row & ((1 << lg) - 1));
        const float4* po = reinterpret_cast<const float4*>(p.part_o) + quarter * (T * 256) + piece * 64 + lane;
        for (int32_t t = 0; t < T; ++t) {
            const int32_t col = 32 * t + 8 * piece + 4 * (lane >> 5);
            if (col >= d) break;
            float4 acc = float4{0.f, 0.f, 0.f, 0.f};
            for (int32_t c = 0; c < n && !none; ++c) {
                const int64_t slot = list_slot(it, c, p.heads, hg);
                const float w = expf(pl[slot * kBM] - M);
                const float4 v = po[slot * (T * 1024) + t * 256];
                acc.x = fmaf(w, v.x, acc.x);
                acc.y = fmaf(w, v.y, acc.y);
                acc.z = fmaf(w, v.z, acc.z);
                acc.w = fmaf(w, v.w, acc.w);
            }
            const float4 r = none ? float4{0.f, 0.f, 0.f, 0.f}
                                  : float4{acc.x / wsum, acc.y / wsum, acc.z / wsum, acc.w / wsum};
            store_out4<OUT>(out, o_row * d + col, r);
        }
        if (lse && piece == 0 && lane < 32) lse[o_row] = none ? -INFINITY : M + logf(wsum);
    }
}

// RAGGED (the few-query sequences of a prefill call): one workgroup per (sequence, KV head, column); column
// c of the 16 is query c / G, head c % G of the group; partials are 16 rows per KV head; sequences that did not
// take that path (q_len * G > 16) are skipped.
template <int OUT, bool RAGGED>
__global__ __launch_bounds__(kMergeThreads) void paged_attention_merge_stream_kernel(
    const float* __restrict__ part_o, const float* __restrict__ part_lse, void* __restrict__ out,
    float* __restrict__ lse, const int32_t* __restrict__ seq_lens, const int32_t* __restrict__ seg_first,
    const int32_t* __restrict__ seg_last, int32_t num_q_heads, int32_t d, const int32_t* __restrict__ cu_q_lens,
    int32_t num_kv_heads, ListMerge list, RowMerge by_row)
{
    if (RAGGED && (int32_t)blockIdx.x < list.blocks) {
        merge_list<OUT>(list, blockIdx.x, out, lse, cu_q_lens, seq_lens, num_q_heads, d);
        return;
    }
    int32_t block = RAGGED ? (int32_t)blockIdx.x - list.blocks : (int32_t)blockIdx.x;
    if (RAGGED && block < by_row.blocks) {
        merge_rows<OUT>(by_row, (int64_t)block * (kMergeThreads / 32) + (threadIdx.x >> 5), out, lse, cu_q_lens, seq_lens,
                        num_q_heads, d);
        return;
    }
    if (RAGGED) block -= by_row.blocks;
    __shared__ float w_s[kMaxDecodeWGs + 1];
    __shared__ float red[4];
    const int32_t rows = RAGGED ? num_kv_heads * 16 : num_q_heads;   // partial rows per (workgroup, sequence)
    const int32_t s = block / rows;
    const int32_t h = block % rows;
    int64_t o_idx = block;
    if (RAGGED) {
        const int32_t G = num_q_heads / num_kv_heads;
        const int32_t q_len = cu_q_lens[s + 1] - cu_q_lens[s];
        const int32_t col = h & 15;
        if (q_len < 1 || q_len * G > 16 || col >= q_len * G) return;
        o_idx = (int64_t)(cu_q_lens[s] + col / G) * num_q_heads + (h >> 4) * G + col % G;
    }
    const int tid = threadIdx.x;
    const int32_t len = seq_lens[s];
    const int32_t first = seg_first[s];
    const int32_t last = seg_last[s];
    if (len > 0 && first < 0) return;                  // already final
    const int32_t n = len > 0 ? last - first + 1 : 0;
    const int64_t p0 = (int64_t)(first + s) * rows + h;            // partial c sits `rows` rows further each

    // weights exp(lse_c - M) into LDS
    float mx = -INFINITY;
    for (int32_t c = tid; c < n; c += kMergeThreads) {
        const float v = part_lse[p0 + (int64_t)c * rows];
        w_s[c] = v;
        mx = fmaxf(mx, max_term(v));
    }
    mx = wave_max(mx);
    if ((tid & 63) == 0) red[tid >> 6] = mx;
    __syncthreads();
    float M = fmaxf(red[0], red[1]);
    const bool no_keys = M == -INFINITY;               // RAGGED: a row whose causal bound excludes every key
    if (no_keys) M = 0.f;
    float ws = 0.f;
    for (int32_t c = tid; c < n; c += kMergeThreads) {
        const float wgt = expf(w_s[c] - M);
        w_s[c] = wgt;
        ws += wgt;
    }
    ws = wave_sum(ws);
    if ((tid & 63) == 0) red[2 + (tid >> 6)] = ws;
    __syncthreads();
    const float wsum = red[2] + red[3];

    for (int e = tid; e < d; e += kMergeThreads) {
        const float* po = part_o + p0 * d + e;
        const int64_t step = (int64_t)rows * d;
        float acc = 0.f;
        int32_t c = 0;
        for (; c + 8 <= n; c += 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = po[(int64_t)(c + u) * step];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc = fmaf(w_s[c + u], v[u], acc);
        }
        for (; c < n; ++c) acc = fmaf(w_s[c], po[(int64_t)c * step], acc);
        const float r = (n > 0 && !no_keys) ? acc / wsum : 0.f;
        store_out<OUT>(out, o_idx * d + e, r);
    }
    if (lse && tid == 0) lse[o_idx] = (n > 0 && !no_keys) ? M + logf(wsum) : -INFINITY;
}

RowMerge row_merge(const AttnArgs& a, const float* part_o, const float* part_lse, int64_t pairs)
{
    return {part_o, part_lse, pairs, 0, a.batch, a.causal, a.plan.chunk, a.plan.nsplit, a.plan.unit, 0};
}

}  // namespace

pa_status launch_merge(const AttnArgs& a, hipStream_t stream)
{
    const int64_t blocks = (int64_t)a.total_q * a.num_q_heads;
    if (blocks > 0x7fffffffLL) return PA_ERR_UNSUPPORTED;
    ProfileScope prof(a.list_items > 0 ? "paged_attention_merge_list_kernel" : "paged_attention_merge_kernel", stream);
    if (a.stream_split || a.list_items > 0) {
        // tile-stream partials of the MFMA decode kernel (16-bit pools only); with cu_q_lens: the few-query
        // sequences of a prefill call
        const bool ragged = a.cu_q_lens != nullptr;
        // (stream and list partials of one call are merged by one launch: 4 us less than two on a mixed batch)
        ListMerge list = {};
        if (a.list_items > 0) {
            const int32_t G = a.num_q_heads / a.cache.num_kv_heads;
            list.part_o = a.list_o;
            list.part_lse = a.list_lse;
            list.batch = a.batch;
            list.log2_pack = prefill_mfma_log2_pack(a.num_q_heads, a.cache.num_kv_heads);
            list.heads = a.num_q_heads >> list.log2_pack;
            list.small_group = a.skip_small ? G : prefill::kNoSmallGroup;
            list.unit = a.cache.page_size > prefill::kBN ? a.cache.page_size : prefill::kBN;
            list.causal = a.causal;
            // row tiles of the sequences that are cut: each has more keys than a chunk
            const int64_t most = prefill::kListTarget / list.heads + 1;
            const int64_t eighths = 8 * list.heads * (most < a.list_items ? most : a.list_items);
            list.blocks = (int32_t)(eighths < prefill::kListMergeGrid ? eighths : prefill::kListMergeGrid);
        }
        RowMerge by_row = {};
        if (a.rows_o) {
            by_row = row_merge(a, a.rows_o, a.rows_lse, blocks);
            by_row.blocks = (int32_t)((blocks + kMergeThreads / 32 - 1) / (kMergeThreads / 32));
            by_row.final_group = a.num_q_heads / a.cache.num_kv_heads;
        }
        const int64_t sblocks = (int64_t)list.blocks + by_row.blocks +
                                (!a.stream_split ? 0 : ragged ? (int64_t)a.batch * a.cache.num_kv_heads * 16 : blocks);
        if (sblocks > 0x7fffffffLL || a.dtype == PA_DTYPE_F32) return PA_ERR_UNSUPPORTED;
        auto kern = a.dtype == PA_DTYPE_BF16
                        ? (ragged ? paged_attention_merge_stream_kernel<PA_DTYPE_BF16, true>
                                  : paged_attention_merge_stream_kernel<PA_DTYPE_BF16, false>)
                        : (ragged ? paged_attention_merge_stream_kernel<PA_DTYPE_F16, true>
                                  : paged_attention_merge_stream_kernel<PA_DTYPE_F16, false>);
        hipLaunchKernelGGL(kern, dim3((uint32_t)sblocks), dim3(kMergeThreads), 0, stream, a.part_o, a.part_lse, a.out,
                           a.lse, a.seq_lens, a.seg_first, a.seg_last, a.num_q_heads, a.cache.head_dim, a.cu_q_lens,
                           a.cache.num_kv_heads, list, by_row);
        return launch_status();
    }
    auto kern = a.dtype == PA_DTYPE_BF16  ? paged_attention_merge_kernel<PA_DTYPE_BF16>
                : a.dtype == PA_DTYPE_F16 ? paged_attention_merge_kernel<PA_DTYPE_F16>
                                          : paged_attention_merge_kernel<PA_DTYPE_F32>;
    if (a.cache.head_dim % 4 != 0) return PA_ERR_UNSUPPORTED;   // (16-byte rows: every supported element type has it)
    hipLaunchKernelGGL(kern, dim3((uint32_t)((blocks + kMergePairs - 1) / kMergePairs)), dim3(256), 0, stream,
                       row_merge(a, a.part_o, a.part_lse, blocks), a.out, a.lse, a.cu_q_lens, a.seq_lens, a.num_q_heads,
                       a.cache.head_dim);
    return launch_status();
}

}  // namespace pa
