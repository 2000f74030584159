"""GPU parity of the matrix-core kernels at head_dims whose rows do not fill their tiles (80, 96, 112): padded column
blocks, padded score steps, repeated row pieces."""
import pytest
import torch

from paper_2506_07311_amd import workloads as W
from tests import parity

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def pa():
    import paper_2506_07311_amd as pa_mod
    pa_mod.load_library()
    return pa_mod


@pytest.mark.parametrize("d", [80, 96, 112])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("Hq,Hkv,P,causal,chunk", [(4, 4, 16, True, 0), (8, 2, 32, True, 0), (6, 2, 16, False, 0),
                                                   (16, 1, 128, True, 64), (4, 4, 16, False, 128)])
def test_prefill_at_padded_head_dims(pa, oracle, d, dtype, Hq, Hkv, P, causal, chunk):
    """Prompts, chunks and single rows around the 64-key and 128-row tile edges, with and without a context split;
    unused slots hold NaN.  Tolerances of tests/parity.py: the output's rounding and nothing else (the weights carry two
    16-bit terms)."""
    from paper_2506_07311_amd import binding
    lens = [1, 63, 64, 65, 300, 0, 129, 517]
    q_lens = [1, 63, 64, 65, 128, 0, 1, 33]
    w = W.make_workload("t", seq_lens=lens, q_lens=q_lens, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, page_size=P,
                        dtype=dtype, causal=causal, seed=201, device=DEV)
    binding.pa_set_option("prefill_chunk_tokens", chunk)
    binding.pa_profile_reset()
    binding.pa_profile_enable(True)
    try:
        parity.check_step(pa, oracle, w, f"prefill d={d} {dtype}")
        assert binding.pa_profile_read("paged_prefill_mfma")[0] == 1
    finally:
        binding.pa_profile_enable(False)
        binding.pa_profile_reset()
        binding.pa_set_option("prefill_chunk_tokens", 0)


@pytest.mark.parametrize("d", [80, 96, 112])
def test_prefill_at_padded_head_dims_equals_the_portable_kernel(pa, d):
    """Token-major and head-major pools against the portable kernel on the same bits.  Both round the same fp32 result
    to bf16, so they differ by at most one rounding step of the larger value plus the fp32 error of their sums."""
    from paper_2506_07311_amd import binding
    w = W.make_workload("t", seq_lens=[700, 33, 150], q_lens=[700, 33, 20], num_q_heads=8, num_kv_heads=4, head_dim=d,
                        page_size=16, dtype=torch.bfloat16, causal=True, seed=202, device=DEV)
    pa.paged_kv_append(w.k_cache, w.v_cache, w.k_new, w.v_new, w.seq_ids, w.positions, w.block_table)
    outs = []
    for generic in (1, 0):
        for head_major in (False, True):
            k, v = w.k_cache, w.v_cache
            if head_major:
                k, v = k.transpose(1, 2).contiguous(), v.transpose(1, 2).contiguous()
            lse = torch.empty((w.total_q, 8), dtype=torch.float32, device=DEV)
            binding.pa_set_option("force_generic", generic)
            try:
                out = pa.paged_attention_prefill(k, v, w.q, w.cu_q_lens, w.max_q_len, w.block_table, w.seq_lens,
                                                 w.max_seq_len, w.scale, True, lse=lse, head_major=head_major)
            finally:
                binding.pa_set_option("force_generic", 0)
            outs.append((out.float(), lse))
    ref, ref_lse = outs[0]
    for out, lse in outs[1:]:
        assert ((out - ref).abs() <= 2.0 ** -7 * ref.abs() + 1e-4).all()
        assert (lse - ref_lse).abs().max() <= 2e-5
