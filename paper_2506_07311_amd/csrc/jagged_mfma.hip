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
    int32_t wgs;          // workgroups along the stream
    int32_t head_groups;  // of four KV heads, a wave each
};

// Run one after the other, the prefill kernel leaves HBM idle (60 decoding sequences with four chunks of 512 tokens on 2.7k ..
// 31k keys: 460 us) and the decode kernel the matrix cores (180 us).  Both are held to two waves a SIMD by their registers, so
// a workgroup of either fits a slot of the other: the first workgroups, one a compute unit, walk the stream with four
// waves (one a KV head: half of what the decode kernel has in flight, which costs it little beside a neighbour that wants
// nothing from HBM), all others step over the list, and a compute unit has one of each until the stream ends.  The whole call
// 655 -> 600 us; 56 with eight chunks of 200 495 -> 445, 18 with two of 512 on up to 8192 keys 51 -> 38, 63 on 16384 with
// one chunk of 64 774 -> 762 (40 with 32 / 32 heads 1746 -> 1757, the only one of twenty-one that lost).  Stream workgroups on every second compute unit 587, 479, -, 1199 us, on three of four 603, 429,
// -, 878, two a compute unit (a second round of them behind the first 512 workgroups) 616, 450, 42, 772.
template <typename E>
__global__ __launch_bounds__(kThreads, 2) void paged_jagged_mfma_kernel(
    CacheView cache, const uint16_t* __restrict__ q, uint16_t* __restrict__ out, float* __restrict__ lse,
    const int32_t* __restrict__ cu_q_lens, const int32_t* __restrict__ block_table,
    const int32_t* __restrict__ seq_lens, int32_t batch, int32_t num_q_heads, int32_t max_blocks, float scale,
    int32_t causal, PrefillPlan plan, StreamPart stream)
{
    __shared__ __attribute__((aligned(1024))) char buf0[RowGeo<128>::kBufB];
    __shared__ __attribute__((aligned(1024))) char buf1[RowGeo<128>::kBufB];
    const uint32_t streaming = (uint32_t)(stream.wgs * stream.head_groups);
    if (blockIdx.x < streaming) {
        const int32_t b = (int32_t)blockIdx.x;
        decode::stream_body<4, true, true, E, NoMods, decode::Geo<128>>(
            cache, q, out, lse, block_table, seq_lens, batch, num_q_heads, max_blocks, scale, stream.part_o, stream.part_lse,
            stream.seg_first, stream.seg_last, cu_q_lens, causal, plan.mods, nullptr, nullptr, b / stream.head_groups,
            stream.wgs, b % stream.head_groups, 0);
        return;
    }
    list_body<true, kEitherList, E, NoMods, 128>(buf0, buf1, nullptr, nullptr, cache, q, out, lse, cu_q_lens, block_table, seq_lens,
                                    batch, num_q_heads, max_blocks, scale, causal, plan, blockIdx.x - streaming,
                                    gridDim.x - streaming);
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
pa_status launch_jagged_mfma(const AttnArgs& a, const AttnArgs& s, hipStream_t stream)
{
    const PrefillPlan plan = make_plan(a);
    const StreamPart part = {s.part_o, s.part_lse, s.seg_first, s.seg_last, s.num_wgs, a.cache.num_kv_heads / 4};
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
