// A jagged prefill call in ONE attention launch (head_dim 128): the work list of its chunks of prompts, bound by the matrix
// cores, beside the tile stream of its few-query sequences, bound by HBM.
#include "decode_mfma_impl.h"
#include "prefill_mfma_impl.h"

namespace pa {

using namespace prefill;

namespace {

// The stream's side of the launch.
struct StreamPart {
    float* part_o;
    float* part_lse;
    int32_t* seg_first;
    int32_t* seg_last;
    int32_t wgs;          // workgroups along the stream, at most
    int32_t head_groups;  // of four KV heads, a wave each
    int32_t cus;
};

// Workgroups of the stream, a compute unit each (the first workgroups of a launch go to different ones).  Behind the stream's
// rows a list workgroup's tile loads come back late whatever HBM has to do elsewhere (2.7 us a tile beside a stream workgroup,
// 1.05 alone), so the stream gets as few compute units as let it end with the list: n (stream tiles a us and workgroup) = its
// share of the time in which the others' two list workgroups and the n that are left beside the stream do the list.
// Measured with every number of workgroups for eleven calls, this one is within 2 % of the best: 60 sequences with four
// chunks of 512 tokens on 2.7k .. 31k keys 605 us with all compute units, 565 with 96, 588 with 144; 64 on up to 7451, eight
// with 200 queries, 130 and 116 with 160; 53 on 20510 with three short chunks 131 with all, 168 with 160.
constexpr float kStreamRate = 0.46f;     // 32 keys of four KV heads, a us
constexpr float kListRate = 1.1f, kListRateBeside = 0.37f;   // key tiles a us: two list workgroups, one beside a stream
__device__ __forceinline__ int32_t stream_workgroups(const StreamPart& p, const WorkList& list)
{
    const int32_t most = p.wgs * p.head_groups;
    const float us = (float)list.few_tiles * (float)p.head_groups / kStreamRate;
    const float n = (float)p.cus * kListRate * us / (list.work * (float)list.heads + (kListRate - kListRateBeside) * us + 1.f);
    const int32_t unit = max(p.cus / 8, 1);                 // (rounded up: a stream that ends last leaves the machine idle)
    int32_t c = min(((int32_t)fminf(n, (float)most) + unit - 1) / unit * unit, most);
    c = max(c / p.head_groups, 1) * p.head_groups;
    return __builtin_amdgcn_readfirstlane(c);
}

// Run one after the other, the prefill kernel leaves HBM idle (60 decoding sequences with four chunks of 512 tokens on 2.7k ..
// 31k keys: 460 us) and the decode kernel the matrix cores (180 us).  Both are held to two waves a SIMD by their registers, so
// a workgroup of either fits a slot of the other: the first workgroups walk the stream with four waves (one a KV head: half of
// what the decode kernel has in flight), all others step over the list.  The whole call 655 -> 557 us; 18 with two of 512 on up
// to 8192 keys 51 -> 38, 63 on 16384 with one chunk of 64 774 -> 760 (40 with 32 / 32 heads 1802 -> 1812).  Two stream workgroups
// on half as many compute units are as good as one a compute unit (581 us on 64, 592 on 96), but the second of them gets less
// and ends late, and a call that is mostly stream wants all compute units.
template <typename E>
__global__ __launch_bounds__(kThreads, 2) void paged_jagged_mfma_kernel(
    CacheView cache, const uint16_t* __restrict__ q, uint16_t* __restrict__ out, float* __restrict__ lse,
    const int32_t* __restrict__ cu_q_lens, const int32_t* __restrict__ block_table,
    const int32_t* __restrict__ seq_lens, int32_t batch, int32_t num_q_heads, int32_t max_blocks, float scale,
    int32_t causal, PrefillPlan plan, StreamPart stream)
{
    __shared__ __attribute__((aligned(1024))) char buf0[RowGeo<128>::kBufB];
    __shared__ __attribute__((aligned(1024))) char buf1[RowGeo<128>::kBufB];
    WorkList list = scan_plan_list(plan, cu_q_lens, seq_lens, batch, num_q_heads);
    const int32_t n = stream_workgroups(stream, list);
    const int32_t block = (int32_t)blockIdx.x;
    if (block < n) {
        decode::stream_body<4, true, true, E, NoMods, decode::Geo<128>>(
            cache, q, out, lse, block_table, seq_lens, batch, num_q_heads, max_blocks, scale, stream.part_o, stream.part_lse,
            stream.seg_first, stream.seg_last, cu_q_lens, causal, plan.mods, nullptr, nullptr, block / stream.head_groups,
            n / stream.head_groups, block % stream.head_groups, 0);
        return;
    }
    list_body<true, kEitherList, E, NoMods, 128>(buf0, buf1, nullptr, nullptr, cache, q, out, lse, cu_q_lens, block_table, seq_lens,
                                    batch, num_q_heads, max_blocks, scale, causal, plan, list,
                                    (uint32_t)(block - n), gridDim.x - (uint32_t)n);
}

}  // namespace

// Workgroups along the stream (each of four KV heads), 0: the call takes two launches.
int32_t jagged_mfma_stream_wgs(const AttnArgs& a, int32_t cus)
{
    if (a.cache.head_dim != 128 || a.cache.num_kv_heads % 4 != 0 || !prefill_list_supported(a)) return 0;
    const int32_t n = cus / (a.cache.num_kv_heads / 4);
    return n > 1 ? n : 1;
}

// a: the work list; s: the stream (partials, segments and num_wgs).
pa_status launch_jagged_mfma(const AttnArgs& a, const AttnArgs& s, int32_t cus, hipStream_t stream)
{
    const PrefillPlan plan = make_plan(a);
    const StreamPart part = {s.part_o, s.part_lse, s.seg_first, s.seg_last, s.num_wgs, a.cache.num_kv_heads / 4, cus};
    int64_t blocks = (int64_t)plan.list_items * (a.num_q_heads >> plan.log2_pack);
    if (blocks > kListGrid) blocks = kListGrid;
    blocks += (int64_t)part.wgs * part.head_groups;
    if (blocks > 0x7fffffffLL) return PA_ERR_UNSUPPORTED;
    ProfileScope prof("paged_jagged_mfma_kernel", stream);
    auto kern = a.dtype == PA_DTYPE_BF16 ? paged_jagged_mfma_kernel<ElemBf16> : paged_jagged_mfma_kernel<ElemF16>;
    hipLaunchKernelGGL(kern, dim3((uint32_t)blocks), dim3(kThreads), 0, stream, a.cache, (const uint16_t*)a.q,
                       (uint16_t*)a.out, a.lse, a.cu_q_lens, a.block_table, a.seq_lens, a.batch, a.num_q_heads, a.max_blocks,
                       a.scale, a.causal, plan, part);
    return launch_status();
}

}  // namespace pa
