"""GPU parity of the prefill kernel's work-list mode: jagged calls whose long contexts are cut into chunks on the device."""
import numpy as np
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


# chunks of 2048 keys at the least: contexts on, one below and one above its multiples; sequences without queries, without
# keys, left to the decode kernel, not cut; more sequences than lanes
LENS = [4096, 2048, 0, 4097, 6143, 70, 2049, 300, 1]
Q_LENS = [130, 64, 0, 1, 257, 33, 40, 0, 1]
CASES = [  # lens, q_lens, Hq, Hkv, d, P, dtype, causal, hooks
    (LENS, Q_LENS, 8, 2, 128, 16, torch.bfloat16, True, None),
    (LENS, Q_LENS, 6, 2, 64, 128, torch.float16, False, None),
    (LENS, Q_LENS, 2, 2, 256, 16, torch.bfloat16, True, None),
    (LENS, Q_LENS, 2, 1, 96, 16, torch.bfloat16, True, None),
    (LENS, Q_LENS, 4, 4, 128, 4, torch.bfloat16, True, dict(alibi=True, softcap=30.0)),
    ([40] * 70 + LENS + [9], [1] * 70 + Q_LENS + [9], 4, 1, 128, 16, torch.bfloat16, True, None),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"Hq{c[2]}-Hkv{c[3]}-d{c[4]}-P{c[5]}-n{len(c[0])}")
def test_jagged_calls_with_long_contexts(pa, oracle, case):
    from paper_2506_07311_amd import binding
    from tests.test_gpu_parity import build_mods
    lens, q_lens, Hq, Hkv, d, P, dtype, causal, hooks = case
    w = W.make_workload("t", seq_lens=lens, q_lens=q_lens, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, page_size=P,
                        dtype=dtype, causal=causal, seed=211, device=DEV)
    mods = build_mods(hooks, Hq, lens) if hooks else None
    binding.pa_profile_reset()
    binding.pa_profile_enable(True)
    try:
        parity.check_step(pa, oracle, w, f"{case[2:]}", mods=mods)
        listed = hooks is None and P >= 16                    # (hooks and smaller pages keep the plain grid)
        assert binding.pa_profile_read("paged_attention_merge_list")[0] == (1 if listed else 0)
    finally:
        binding.pa_profile_enable(False)
        binding.pa_profile_reset()


@pytest.mark.parametrize("Hq,Hkv,P,dtype,causal,extra", [
    (16, 4, 16, torch.bfloat16, True, []),                    # one group of four KV heads
    (32, 8, 128, torch.float16, True, []),                    # two
    (12, 12, 16, torch.bfloat16, False, []),                  # three; no grouping, no causal bound
    (64, 4, 32, torch.bfloat16, True, []),                    # 16 heads a group: single queries alone are few
    (8, 4, 16, torch.float16, True, [40] * 70 + [2000, 1])])  # more sequences than lanes, most of a tile or two
def test_chunks_and_single_queries_in_one_launch(pa, oracle, Hq, Hkv, P, dtype, causal, extra):
    """The list's workgroups and the stream's in one launch: sequences that either side takes, of one tile, of none, cut by
    workgroup boundaries and by chunks; a second call on the same workspace gives the same bits."""
    from paper_2506_07311_amd import binding
    lens, q_lens = extra + LENS, [1] * len(extra) + Q_LENS
    w = W.make_workload("t", seq_lens=lens, q_lens=q_lens, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=128, page_size=P,
                        dtype=dtype, causal=causal, seed=215, device=DEV)
    binding.pa_profile_reset()
    binding.pa_profile_enable(True)
    try:
        parity.check_step(pa, oracle, w, f"{Hq} {Hkv} {dtype} {causal}")
        counts = [binding.pa_profile_read(k)[0] for k in ("paged_jagged_mfma", "paged_decode_mfma", "paged_prefill_mfma",
                                                          "paged_attention_merge_list")]
        assert counts == [1, 0, 0, 1]
    finally:
        binding.pa_profile_enable(False)
        binding.pa_profile_reset()
    ws = torch.full((pa.paged_attention_workspace_bytes(w.batch, Hq, 128, w.total_q, w.max_seq_len),), 0xFF,
                    dtype=torch.uint8, device=DEV)
    outs = [pa.paged_attention_prefill(w.k_cache, w.v_cache, w.q, w.cu_q_lens, w.max_q_len, w.block_table, w.seq_lens,
                                       w.max_seq_len, w.scale, causal, workspace=ws) for _ in range(2)]
    assert torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("Hq,Hkv", [(8, 4), (32, 8), (12, 12)])
@pytest.mark.parametrize("lens,q_lens", [
    ([5000] * 6 + [33], [200] * 6 + [1]),                     # the stream is two tiles of one sequence
    ([6100] * 12 + [4096], [1] * 12 + [33]),                  # nearly all of the call
    ([4100, 9000, 6200, 2048], [130, 1, 70, 200])])           # whole chunks and remainders of one key and more
def test_the_streams_share_of_the_machine(pa, oracle, lens, q_lens, Hq, Hkv):
    """The stream's workgroups are counted on the device from both sides' work, from one a head group to all there is room for;
    chunks that are whole come before those that are not."""
    w = W.make_workload("t", seq_lens=lens, q_lens=q_lens, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=128, page_size=16,
                        dtype=torch.bfloat16, causal=True, seed=219, device=DEV)
    parity.check_step(pa, oracle, w, f"{lens} {q_lens} {Hq} {Hkv}")


@pytest.mark.parametrize("lens,q_lens,Hq,Hkv,P,dtype,causal", [
    ([2100, 0, 700, 1, 1500, 64, 65], [130, 0, 1, 1, 129, 2, 17], 16, 4, 16, torch.bfloat16, True),
    ([4095, 300, 33], [33, 1, 1], 8, 8, 64, torch.float16, False),            # one key short of the list that is cut
    ([40] * 70 + [600, 500], [1] * 70 + [250, 3], 4, 4, 32, torch.float16, True),
    ([500, 700, 900], [100, 101, 102], 8, 4, 16, torch.bfloat16, True)])      # nothing for the stream, and may be
def test_uncut_chunks_and_single_queries_in_one_launch(pa, oracle, lens, q_lens, Hq, Hkv, P, dtype, causal):
    """Contexts below the length that the list has slots for: row tiles beside the stream, no partials by slot."""
    from paper_2506_07311_amd import binding
    w = W.make_workload("t", seq_lens=lens, q_lens=q_lens, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=128, page_size=P,
                        dtype=dtype, causal=causal, seed=217, device=DEV)
    may_be_small = (w.total_q - (w.batch - 1) * w.max_q_len) * (Hq // Hkv) <= 16
    binding.pa_profile_reset()
    binding.pa_profile_enable(True)
    try:
        parity.check_step(pa, oracle, w, f"{lens} {q_lens}")
        counts = [binding.pa_profile_read(k)[0] for k in ("paged_jagged_mfma", "paged_decode_mfma", "paged_prefill_mfma",
                                                          "paged_attention_merge_list")]
        assert counts == ([1, 0, 0, 0] if may_be_small else [0, 0, 1, 0])
    finally:
        binding.pa_profile_enable(False)
        binding.pa_profile_reset()


@pytest.mark.parametrize("lens,q_lens,Hq,Hkv,d,P,dtype,causal", [
    ([4096], [128], 8, 8, 128, 16, torch.bfloat16, True),     # chunks of 1024 keys, the last one ends the diagonal
    ([2049], [129], 4, 2, 64, 128, torch.float16, True),      # one key in the last page, one row in the last tile
    ([3000, 3000], [64, 64], 16, 4, 128, 64, torch.bfloat16, False),
    ([2500], [130], 4, 4, 96, 16, torch.bfloat16, True),
    ([5000], [33], 2, 1, 256, 32, torch.float16, True),
    ([3000, 2000], [70, 64], 4, 4, 256, 16, torch.bfloat16, True)])
def test_chunks_of_prompts_on_long_contexts(pa, oracle, lens, q_lens, Hq, Hkv, d, P, dtype, causal):
    """Contexts cut into as many chunks as the workspace holds partials for, at each kernel's head_dims."""
    w = W.make_workload("t", seq_lens=lens, q_lens=q_lens, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, page_size=P,
                        dtype=dtype, causal=causal, seed=216, device=DEV)
    parity.check_step(pa, oracle, w, f"{lens} {q_lens} {Hq} {Hkv} {d}")


def _reference(w):
    """Attention of every row over the gathered pages in fp32, one KV head at a time."""
    out = torch.zeros(w.q.shape, device=DEV)
    G = w.num_q_heads // w.num_kv_heads
    row = 0
    for s, (n, nq) in enumerate(zip(w.seq_lens_host, w.q_lens_host)):
        pages = w.block_table[s, :-(-n // w.page_size)].long()
        hidden = torch.arange(n, device=DEV)[None, :] > torch.arange(n - nq, n, device=DEV)[:, None]
        for g in range(w.num_kv_heads):
            k, v = (c[pages, :, g].reshape(-1, w.head_dim)[:n].float() for c in (w.k_cache, w.v_cache))
            for h in range(g * G, g * G + G):
                x = w.q[row:row + nq, h].float() @ k.t() * w.scale
                if w.causal:
                    x.masked_fill_(hidden, float("-inf"))
                out[row:row + nq, h] = torch.softmax(x, dim=1) @ v
        row += nq
    return out


@pytest.mark.parametrize("lens,q,bound,Hq,Hkv,d,P,dtype,causal,chunks", [
    ([32768], 1024, 32768, 32, 8, 128, 16, torch.bfloat16, True, [2]),               # of four possible ones
    ([32768, 32768], 128, 32768, 32, 8, 128, 16, torch.bfloat16, True, [8, 8]),      # of 13
    ([32768], 1024, 32768, 32, 8, 64, 16, torch.bfloat16, True, [3]),                # three workgroups a compute unit
    ([8192], 256, 8192, 32, 8, 96, 16, torch.float16, True, [8]),
    ([2048], 1024, 2048, 32, 8, 128, 16, torch.bfloat16, True, [1]),                 # of two
    ([8192], 128, 131072, 32, 8, 128, 16, torch.bfloat16, True, [8]),                # a bound far from the length
    ([700], 128, 131072, 32, 8, 128, 64, torch.float16, True, [1]),
    ([32768, 16000, 900], 128, 32768, 32, 8, 128, 16, torch.bfloat16, False, [8, 8, 1]),
    ([2000] * 3 + [32768] + [2000] * 4, 64, 32768, 32, 8, 128, 32, torch.float16, True, [2] * 3 + [6] + [2] * 4),
    ([9000, 1100, 64], 64, 10000, 8, 8, 64, 128, torch.bfloat16, True, [9, 2, 1]),
    ([5000, 4999], 33, 9000, 8, 2, 256, 32, torch.bfloat16, True, [5, 5])])
def test_chunks_follow_the_compute_units_and_each_context(pa, lens, q, bound, Hq, Hkv, d, P, dtype, causal, chunks):
    """The number of chunks that the rule picks on 256 compute units, and that a sequence is cut by its own length whatever the
    bound and the other sequences: counted by the partials that the call leaves in its workspace."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the expected chunks are those of 256 compute units")
    w = W.make_workload("t", seq_lens=lens, q_lens=[q] * len(lens), num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, page_size=P,
                        dtype=dtype, causal=causal, seed=218, device=DEV)
    pa.paged_kv_append(w.k_cache, w.v_cache, w.k_new, w.v_new, w.seq_ids, w.positions, w.block_table)
    table = torch.nn.functional.pad(w.block_table, (0, max(0, -(-bound // P) - w.block_table.shape[1])), value=-1)
    nbytes = pa.paged_attention_workspace_bytes(w.batch, Hq, d, w.total_q, bound)
    ws = torch.full((-(-nbytes // 4),), -1, dtype=torch.int32, device=DEV)       # (a NaN as a float)
    out = pa.paged_attention_prefill(w.k_cache, w.v_cache, w.q, w.cu_q_lens, q, table, w.seq_lens, bound, w.scale, causal,
                                     workspace=ws)
    parity.assert_close(parity.to_f64(out), parity.to_f64(_reference(w)), dtype, f"{lens} {q}")
    written = int((ws != -1).sum())
    if len(lens) == 1 and chunks == [1] and bound == lens[0]:
        assert written == 0                                   # uncut: no partials at all
    else:
        assert written == q * Hq * (d + 1) * sum(chunks)


def test_chunks_of_each_context_with_score_hooks(pa, oracle):
    from tests.test_gpu_parity import build_mods
    lens, q_lens = [5000, 2100, 70], [40, 40, 40]
    w = W.make_workload("t", seq_lens=lens, q_lens=q_lens, num_q_heads=4, num_kv_heads=2, head_dim=128, page_size=16,
                        dtype=torch.bfloat16, causal=True, seed=219, device=DEV)
    parity.check_step(pa, oracle, w, "hooks", mods=build_mods(dict(alibi=True, softcap=30.0), 4, lens))


@pytest.mark.parametrize("d,chunks", [(256, 4), (128, 8)])
def test_chunks_of_the_list_fill_the_workgroups_that_fit_at_once(pa, d, chunks):
    """58 row tiles and heads' items of 1024 keys are one round of two workgroups a compute unit, and more than one of the single
    one at head_dim 256, which takes chunks of 2048 keys instead; counted by the partials that are left."""
    w = W.make_workload("t", seq_lens=[8192, 300, 300], q_lens=[200, 20, 20], num_q_heads=32, num_kv_heads=8, head_dim=d,
                        page_size=16, dtype=torch.bfloat16, causal=True, seed=222, device=DEV)
    pa.paged_kv_append(w.k_cache, w.v_cache, w.k_new, w.v_new, w.seq_ids, w.positions, w.block_table)
    nbytes = pa.paged_attention_workspace_bytes(w.batch, 32, d, w.total_q, w.max_seq_len)
    ws = torch.full((-(-nbytes // 4),), -1, dtype=torch.int32, device=DEV)
    out = pa.paged_attention_prefill(w.k_cache, w.v_cache, w.q, w.cu_q_lens, w.max_q_len, w.block_table, w.seq_lens,
                                     w.max_seq_len, w.scale, True, workspace=ws)
    parity.assert_close(parity.to_f64(out), parity.to_f64(_reference(w)), torch.bfloat16, f"{d}")
    assert int((ws != -1).sum()) == 200 * 32 * (d + 1) * chunks


@pytest.mark.parametrize("lens,q_lens,Hq,Hkv,P,dtype,causal,nsplit,chunks", [
    ([4000, 4000], [200, 1], 32, 8, 16, torch.bfloat16, True, 3, [3, 0]),
    ([4095, 1300, 900, 300, 33, 0], [64, 64, 64, 1, 1, 0], 8, 8, 128, torch.float16, True, 3, [3, 2, 0, 0, 0, 0]),
    ([2100, 1060, 200], [500, 300, 1], 8, 4, 16, torch.bfloat16, False, 2, [2, 2, 0]),
    ([40] * 70 + [3000], [1] * 70 + [90], 4, 4, 32, torch.bfloat16, True, 2, [0] * 70 + [2]),
    ([1900, 300], [300, 1], 8, 4, 16, torch.bfloat16, True, 1, [0, 0])])
def test_short_jagged_calls_cut_each_context_by_its_length(pa, lens, q_lens, Hq, Hkv, P, dtype, causal, nsplit, chunks):
    """The list beside the stream cuts what the plain grid would: counted by the partials that it leaves, none of them of
    contexts in one piece or of the stream's sequences.  A second call on the same workspace gives the same bits."""
    from paper_2506_07311_amd import binding
    w = W.make_workload("t", seq_lens=lens, q_lens=q_lens, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=128, page_size=P,
                        dtype=dtype, causal=causal, seed=220, device=DEV)
    pa.paged_kv_append(w.k_cache, w.v_cache, w.k_new, w.v_new, w.seq_ids, w.positions, w.block_table)
    nbytes = pa.paged_attention_workspace_bytes(w.batch, Hq, 128, w.total_q, w.max_seq_len)
    ws = torch.full((-(-nbytes // 4),), -1, dtype=torch.int32, device=DEV)
    lse = torch.full((w.total_q, Hq), float("nan"), device=DEV)
    outs = []
    for _ in range(2):
        binding.pa_profile_reset()
        binding.pa_profile_enable(True)
        try:
            outs.append(pa.paged_attention_prefill(w.k_cache, w.v_cache, w.q, w.cu_q_lens, w.max_q_len, w.block_table,
                                                   w.seq_lens, w.max_seq_len, w.scale, causal, lse=lse, workspace=ws))
            torch.cuda.synchronize()
            counts = [binding.pa_profile_read(k)[0] for k in ("paged_jagged_mfma", "paged_attention_merge_kernel")]
            assert counts == [1, 1]
        finally:
            binding.pa_profile_enable(False)
            binding.pa_profile_reset()
    assert torch.equal(outs[0], outs[1])
    parity.assert_close(parity.to_f64(outs[0]), parity.to_f64(_reference(w)), dtype, f"{lens} {q_lens}")
    assert torch.isfinite(lse).all()
    if nsplit > 1:
        rows = ws[:w.total_q * Hq * nsplit * 128]
        assert int((rows != -1).sum()) == 128 * Hq * sum(n * c for n, c in zip(q_lens, chunks))


def test_a_short_jagged_call_without_room_for_the_stream_keeps_its_chunks(pa, oracle):
    """A call with no more queries than sequences is promised the decode bound, which does not hold the stream's partials:
    without the stream there is no reason for the list either."""
    from paper_2506_07311_amd import binding
    w = W.make_workload("t", seq_lens=[4000] + [50] * 39, q_lens=[36, 1, 1, 1] + [0] * 36, num_q_heads=32, num_kv_heads=8,
                        head_dim=128, page_size=16, dtype=torch.bfloat16, causal=True, seed=221, device=DEV)
    binding.pa_profile_reset()
    binding.pa_profile_enable(True)
    try:
        parity.check_step(pa, oracle, w, "no room")
        counts = [binding.pa_profile_read(k)[0] for k in ("paged_jagged_mfma", "paged_decode_mfma", "paged_prefill_mfma",
                                                          "paged_attention_merge_kernel")]
        assert counts == [0, 0, 1, 1]
    finally:
        binding.pa_profile_enable(False)
        binding.pa_profile_reset()


def test_a_workspace_of_the_smaller_size_is_accepted_and_keeps_the_plain_grid(pa):
    """The list's partials are room on top of what a call requires: without it the plain grid runs, with the same results
    up to the merge's rounding (bf16 outputs one step apart at most)."""
    from paper_2506_07311_amd import binding
    w = W.make_workload("t", seq_lens=LENS, q_lens=Q_LENS, num_q_heads=8, num_kv_heads=2, head_dim=128, page_size=16,
                        dtype=torch.bfloat16, causal=True, seed=212, device=DEV)
    pa.paged_kv_append(w.k_cache, w.v_cache, w.k_new, w.v_new, w.seq_ids, w.positions, w.block_table)
    full = pa.paged_attention_workspace_bytes(w.batch, 8, 128, w.total_q, w.max_seq_len)
    outs = []
    for nbytes in (full, full - 256):
        ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device=DEV)
        binding.pa_profile_reset()
        binding.pa_profile_enable(True)
        try:
            out = pa.paged_attention_prefill(w.k_cache, w.v_cache, w.q, w.cu_q_lens, w.max_q_len, w.block_table,
                                             w.seq_lens, w.max_seq_len, w.scale, True, workspace=ws)
            torch.cuda.synchronize()
            assert binding.pa_profile_read("paged_attention_merge_list")[0] == (1 if nbytes == full else 0)
        finally:
            binding.pa_profile_enable(False)
            binding.pa_profile_reset()
        outs.append(out.float())
    assert ((outs[0] - outs[1]).abs() <= 2.0 ** -7 * outs[1].abs() + 2e-3).all()


@pytest.mark.parametrize("batch,live,listed", [(600, 70, 0), (600, 60, 1), (512, 70, 1)])
def test_many_sequences_with_queries_keep_the_plain_grid(pa, oracle, batch, live, listed):
    from paper_2506_07311_amd import binding
    lens = [4096] + [70] * (batch - 1)
    q_lens = [20 if s < live else 0 for s in range(batch)]
    w = W.make_workload("t", seq_lens=lens, q_lens=q_lens, num_q_heads=4, num_kv_heads=2, head_dim=64, page_size=16,
                        dtype=torch.bfloat16, causal=True, seed=214, device=DEV)
    binding.pa_profile_reset()
    binding.pa_profile_enable(True)
    try:
        parity.check_step(pa, oracle, w, f"{batch} {live}")
        assert binding.pa_profile_read("paged_attention_merge_list")[0] == listed
    finally:
        binding.pa_profile_enable(False)
        binding.pa_profile_reset()


@pytest.mark.parametrize("q_lens,launches", [([200, 1, 150, 190], 0),     # whole prompts in the main: one launch, all sequences
                                             ([200, 5, 1, 3], 1),         # mostly few queries: they take the decode kernel
                                             ([200, 20], 0)])             # no sequence can have few queries
def test_the_few_query_launches_are_left_out_of_ragged_prompts(pa, oracle, q_lens, launches):
    from paper_2506_07311_amd import binding
    w = W.make_workload("t", seq_lens=[200, 133, 150, 190][:len(q_lens)], q_lens=q_lens, num_q_heads=8, num_kv_heads=2, head_dim=128,
                        page_size=16, dtype=torch.bfloat16, causal=True, seed=213, device=DEV)
    binding.pa_profile_reset()
    binding.pa_profile_enable(True)
    try:
        parity.check_step(pa, oracle, w, f"{q_lens}")
        assert binding.pa_profile_read("paged_decode_mfma")[0] == launches
    finally:
        binding.pa_profile_enable(False)
        binding.pa_profile_reset()


@pytest.mark.parametrize("lens,q_lens,Hq,Hkv,d,P,dtype,causal,hooks", [
    # prompts of all tiles, of one row, of none, one row beyond a tile; a lane for every tile index
    ([700, 33, 0, 545, 129, 1], [700, 33, 0, 513, 129, 1], 32, 8, 128, 16, torch.bfloat16, True, None),
    ([700, 600, 520], [641, 64, 65], 16, 8, 256, 32, torch.float16, True, dict(window=520, softcap=30.0)),
    ([600] * 3 + [90] * 20, [257] * 3 + [70] * 20, 16, 8, 64, 16, torch.bfloat16, False, None),   # more than 16 sequences
    ([1100, 600, 70], [1100, 33, 64], 16, 2, 64, 16, torch.float16, True, dict(alibi=True)),      # more than 64 tile indexes
    ([900, 800, 700, 600], [180, 1, 2, 150], 32, 8, 128, 64, torch.bfloat16, True, dict(window=600)),  # some are the stream's
    ([600, 700, 70, 650], [600, 20, 70, 300], 12, 12, 128, 16, torch.bfloat16, True, dict(docs=True))])
def test_a_grid_of_the_row_tiles_that_there_are(pa, oracle, lens, q_lens, Hq, Hkv, d, P, dtype, causal, hooks):
    """Ragged batches whose grid leaves out what shorter sequences do not have, in the order of the full grid."""
    from tests.test_gpu_parity import build_mods
    w = W.make_workload("t", seq_lens=lens, q_lens=q_lens, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, page_size=P,
                        dtype=dtype, causal=causal, seed=221, device=DEV)
    parity.check_step(pa, oracle, w, f"{lens} {q_lens} {d}", mods=build_mods(hooks, Hq, lens) if hooks else None)


@pytest.mark.parametrize("lens,q_lens,Hq,Hkv,d,P,dtype,causal,hooks", [
    # prompts of all tiles, of one row, of none, one row beyond a tile; a lane for every tile index
    ([700, 33, 0, 545, 129, 1], [700, 33, 0, 513, 129, 1], 32, 8, 128, 16, torch.bfloat16, True, None),
    ([700, 600, 520, 9], [641, 64, 65, 0], 16, 8, 256, 32, torch.float16, True, dict(window=520, softcap=30.0)),
    ([600] * 3 + [90] * 21, [257] * 3 + [70] * 21, 16, 8, 64, 16, torch.bfloat16, False, None),   # more than 16 sequences
    ([1100, 600, 70, 5], [1100, 33, 64, 1], 16, 2, 64, 16, torch.float16, True, dict(alibi=True)),      # more than 64 tile indexes
    ([900, 800, 700, 600], [300, 1, 2, 250], 32, 8, 128, 64, torch.bfloat16, True, dict(window=600)),  # some are the stream's
    ([900, 600], [900, 300], 32, 8, 128, 16, torch.float16, False, dict(window=400)),    # a window to both sides: 799 keys
    ([700, 700, 70, 650], [700, 20, 70, 300], 12, 12, 128, 16, torch.bfloat16, True, dict(docs=True)),
    ([700, 133, 600, 1], [700, 133, 600, 1], 32, 8, 96, 16, torch.bfloat16, True, None),
    ([700, 133, 600, 64], [700, 133, 600, 64], 32, 8, 128, 16, torch.bfloat16, True, dict(prefix=True)),
    # gaps that go round, where a row tile takes long
    ([900, 400, 300], [900, 400, 300], 32, 8, 64, 16, torch.float16, True, dict(softcap=30.0)),
    ([900, 700, 1, 400, 300], [900, 700, 1, 400, 300], 16, 8, 256, 16, torch.bfloat16, True, None)])
def test_a_grid_without_gaps_by_its_name(pa, oracle, lens, q_lens, Hq, Hkv, d, P, dtype, causal, hooks):
    """Ragged batches whose grid leaves out what shorter sequences do not have, which its launch says."""
    from paper_2506_07311_amd import binding
    from tests.test_gpu_parity import build_mods
    w = W.make_workload("t", seq_lens=lens, q_lens=q_lens, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, page_size=P,
                        dtype=dtype, causal=causal, seed=221, device=DEV)
    mods = build_mods(hooks, Hq, lens) if hooks else None
    if hooks and "prefix" in hooks:                           # a user modification
        mods = dict(prefix_lens=np.array([n // 2 for n in lens], dtype=np.int32), prefix_bias=0.5)
    binding.pa_profile_reset()
    binding.pa_profile_enable(True)
    try:
        parity.check_step(pa, oracle, w, f"{lens} {q_lens} {d}", mods=mods)
        assert binding.pa_profile_read("paged_prefill_mfma_kernel_live")[0] == 1
    finally:
        binding.pa_profile_enable(False)
        binding.pa_profile_reset()


@pytest.mark.parametrize("lens,Hq,Hkv,live", [
    ([900, 400], 32, 8, 1),                                    # 8 head groups: every second shader engine
    ([900, 400, 400], 32, 8, 0),                               # 24 a tile index: each sequence meets all four in turn
    ([900, 400, 400, 300], 32, 8, 1),                          # always the same one
    ([900, 400, 400, 300, 300], 32, 8, 0),
    ([900, 400, 400, 300, 300, 300], 32, 8, 1),
    ([900, 400], 32, 32, 0),                                   # all of them in every sequence
    ([900, 400, 300], 16, 2, 0),
    ([900, 400, 300, 300], 16, 2, 1),
    ([900, 897], 32, 8, 0)])                                   # no gaps
def test_gaps_that_go_round_stay_in_the_grid(pa, lens, Hq, Hkv, live):
    """A grid without gaps costs its workgroups a later start: only where the gaps would keep the same shader engines idle.  The
    same bits in either grid, here against one in which 70 sequences without queries keep the full grid."""
    from paper_2506_07311_amd import binding
    w = W.make_workload("t", seq_lens=lens, q_lens=lens, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=64, page_size=16,
                        dtype=torch.bfloat16, causal=True, seed=227, device=DEV)
    pa.paged_kv_append(w.k_cache, w.v_cache, w.k_new, w.v_new, w.seq_ids, w.positions, w.block_table)
    pad = torch.nn.functional.pad
    more = (pad(w.cu_q_lens, (0, 70), value=w.total_q), pad(w.block_table, (0, 0, 0, 70)), pad(w.seq_lens, (0, 70)))
    res = []
    for cu, table, n in ((w.cu_q_lens, w.block_table, w.seq_lens), more):
        binding.pa_profile_reset()
        binding.pa_profile_enable(True)
        binding.pa_set_option("no_small_q_route", 1)
        try:
            lse = torch.empty((w.total_q, Hq), device=DEV)
            out = pa.paged_attention_prefill(w.k_cache, w.v_cache, w.q, cu, w.max_q_len, table, n, w.max_seq_len, w.scale, True,
                                             lse=lse)
            torch.cuda.synchronize()
            counts = [binding.pa_profile_read(k)[0] for k in ("paged_prefill_mfma_kernel_live", "paged_prefill_mfma_kernel",
                                                              "paged_attention_merge")]
            assert counts == [live if cu is w.cu_q_lens else 0, 1, 0]
        finally:
            binding.pa_set_option("no_small_q_route", 0)
            binding.pa_profile_enable(False)
            binding.pa_profile_reset()
        res.append((out, lse))
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])
    parity.assert_close(parity.to_f64(res[0][0]), parity.to_f64(_reference(w)), torch.bfloat16, f"{lens}")


@pytest.mark.parametrize("window,cap,causal,d", [(0, 0.0, True, 128), (700, 0.0, True, 128), (700, 0.0, False, 64),
                                                 (0, 0.0, False, 64), (0, 30.0, True, 256)])
def test_the_two_term_rule_is_one_rule_in_both_grids(pa, window, cap, causal, d):
    """Which rows carry two-term weights follows from the harmonic mean of the rows' keys, which the two grids' kernels each compute
    for themselves: prompts around that mean, bit for bit."""
    from paper_2506_07311_amd import binding
    lens, q_lens = [1500, 1100, 700, 400], [1000, 1100, 300, 400]
    w = W.make_workload("t", seq_lens=lens, q_lens=q_lens, num_q_heads=16, num_kv_heads=8, head_dim=d, page_size=16,
                        dtype=torch.bfloat16, causal=causal, seed=228, device=DEV)
    pa.paged_kv_append(w.k_cache, w.v_cache, w.k_new, w.v_new, w.seq_ids, w.positions, w.block_table)
    pad = torch.nn.functional.pad
    more = (pad(w.cu_q_lens, (0, 61), value=w.total_q), pad(w.block_table, (0, 0, 0, 61)), pad(w.seq_lens, (0, 61)))
    outs = []
    for live, (cu, table, n) in ((1, (w.cu_q_lens, w.block_table, w.seq_lens)), (0, more)):
        binding.pa_profile_reset()
        binding.pa_profile_enable(True)
        binding.pa_set_option("no_small_q_route", 1)
        try:
            outs.append(pa.paged_attention_prefill_mod(w.k_cache, w.v_cache, w.q, cu, w.max_q_len, table, n, w.max_seq_len, w.scale,
                                                       causal, window=window, softcap=cap))
            torch.cuda.synchronize()
            counts = [binding.pa_profile_read(k)[0] for k in ("paged_prefill_mfma_kernel_live", "paged_attention_merge")]
            assert counts == [live, 0]
        finally:
            binding.pa_set_option("no_small_q_route", 0)
            binding.pa_profile_enable(False)
            binding.pa_profile_reset()
    assert torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("lens,q_lens,Hq,Hkv,d,P,dtype,causal,hooks", [
    ([1025], [1025], 8, 1, 128, 16, torch.bfloat16, True, None),                # the last chunk holds one key
    ([1000], [900], 8, 1, 128, 128, torch.float16, False, None),                # every row tile reaches into every chunk
    ([1100, 640], [1100, 640], 8, 1, 64, 16, torch.bfloat16, True, dict(alibi=True)),
    ([1000], [1000], 8, 1, 256, 32, torch.float16, True, dict(softcap=30.0)),
    ([1900], [1900], 8, 1, 128, 16, torch.bfloat16, True, dict(window=1500, softcap=30.0)),     # windows begin in a later chunk
    ([1300], [1000], 4, 1, 96, 16, torch.bfloat16, True, None),
    ([1200], [1200], 8, 1, 128, 16, torch.bfloat16, True, dict(docs=True))])
def test_prompts_of_few_row_tiles_in_chunks(pa, oracle, lens, q_lens, Hq, Hkv, d, P, dtype, causal, hooks):
    """Whole prompts that leave most of the machine idle are cut along their keys; with the workspace's bound and not more."""
    from paper_2506_07311_amd import binding
    from tests.test_gpu_parity import build_mods
    w = W.make_workload("t", seq_lens=lens, q_lens=q_lens, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, page_size=P,
                        dtype=dtype, causal=causal, seed=223, device=DEV)
    binding.pa_profile_reset()
    binding.pa_profile_enable(True)
    try:
        parity.check_step(pa, oracle, w, f"{lens} {d}", mods=build_mods(hooks, Hq, lens) if hooks else None)
        assert binding.pa_profile_read("paged_attention_merge_kernel")[0] == 1
    finally:
        binding.pa_profile_enable(False)
        binding.pa_profile_reset()


@pytest.mark.parametrize("lens,q_lens,Hq,Hkv,d,dtype,kernel", [
    ([1000], [1000], 8, 1, 128, torch.bfloat16, "paged_attention_merge_kernel"),               # a whole prompt in chunks
    ([8192], [128], 8, 2, 64, torch.float16, "paged_attention_merge_kernel"),                  # a chunk of a long one
    ([300, 70, 4000], [1, 1, 200], 32, 8, 128, torch.bfloat16, "paged_jagged_mfma_kernel"),    # by row, beside the stream
    ([4096, 300], [130, 1], 8, 2, 128, torch.bfloat16, "paged_attention_merge_list_kernel")])
def test_rows_behind_the_last_sequence_are_left_alone(pa, lens, q_lens, Hq, Hkv, d, dtype, kernel):
    """A query buffer longer than its sequences' queries (as a captured call has): the merge of a context that is cut writes what
    the kernels in one piece write."""
    from paper_2506_07311_amd import binding
    w = W.make_workload("t", seq_lens=lens, q_lens=q_lens, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, page_size=16,
                        dtype=dtype, causal=True, seed=224, device=DEV)
    pa.paged_kv_append(w.k_cache, w.v_cache, w.k_new, w.v_new, w.seq_ids, w.positions, w.block_table)
    n, pad = w.total_q, 37
    q = torch.cat([w.q, torch.zeros((pad, Hq, d), dtype=dtype, device=DEV)])
    out = torch.full_like(q, 7.0)
    lse = torch.full((n + pad, Hq), 7.0, device=DEV)
    ws = torch.full((pa.paged_attention_workspace_bytes(w.batch, Hq, d, n + pad, w.max_seq_len),), 0xFF, dtype=torch.uint8,
                    device=DEV)
    binding.pa_profile_reset()
    binding.pa_profile_enable(True)
    try:
        pa.paged_attention_prefill(w.k_cache, w.v_cache, q, w.cu_q_lens, w.max_q_len, w.block_table, w.seq_lens, w.max_seq_len,
                                   w.scale, True, out=out, lse=lse, workspace=ws)
        torch.cuda.synchronize()
        assert binding.pa_profile_read(kernel)[0] == 1
    finally:
        binding.pa_profile_enable(False)
        binding.pa_profile_reset()
    parity.assert_close(parity.to_f64(out[:n]), parity.to_f64(_reference(w)), dtype, f"{lens}")
    assert torch.isfinite(lse[:n]).all()
    assert (out[n:] == 7.0).all() and (lse[n:] == 7.0).all()


@pytest.mark.parametrize("lens,q_lens,Hq,Hkv,d,dtype,kernel", [
    ([1000], [1000], 8, 1, 128, torch.bfloat16, "paged_attention_merge_kernel"),               # a whole prompt in chunks
    ([2000], [2000], 8, 1, 64, torch.float16, "paged_attention_merge_kernel"),
    ([1000], [1000], 8, 1, 256, torch.bfloat16, "paged_attention_merge_kernel"),
    ([1300], [1000], 4, 1, 96, torch.bfloat16, "paged_attention_merge_kernel"),
    ([8192], [128], 8, 2, 128, torch.bfloat16, "paged_attention_merge_kernel"),                # a chunk of a long one
    ([300, 70, 4000], [1, 1, 200], 32, 8, 128, torch.bfloat16, "paged_jagged_mfma_kernel"),    # by row, beside the stream
    ([4096, 6000], [130, 1], 8, 2, 64, torch.float16, "paged_attention_merge_list_kernel"),
    ([4096, 6000], [130, 1], 8, 4, 128, torch.bfloat16, "paged_jagged_mfma_kernel"),
    ([20000, 9000, 70, 300], [1, 1, 1, 1], 32, 8, 128, torch.bfloat16, "paged_decode_mfma_kernel"),      # the tile stream
    ([900, 700, 70, 300], [1, 1, 1, 1], 32, 8, 128, torch.bfloat16, "paged_decode_short_kernel"),        # one launch, split
    ([500, 300], [500, 300], 32, 8, 128, torch.bfloat16, "paged_prefill_mfma_kernel")])                  # in one piece
@pytest.mark.parametrize("where", ["q", "k"])
def test_a_nan_reaches_the_rows_that_see_it_through_every_merge(pa, lens, q_lens, Hq, Hkv, d, dtype, kernel, where):
    """A NaN in a query makes its row NaN, LSE included, and one in K the rows that see the key: chunks whose scores are all NaN
    are not taken for chunks without a visible key, nor is the NaN of one chunk lost beside the others."""
    from paper_2506_07311_amd import binding
    w = W.make_workload("t", seq_lens=lens, q_lens=q_lens, append_lens=lens, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, page_size=16,
                        dtype=dtype, causal=True, seed=225, device=DEV)
    s = max(range(len(lens)), key=lambda i: q_lens[i])
    cu, G = w.cu_q_lens.tolist(), Hq // Hkv
    bad = torch.zeros((w.total_q, Hq), dtype=torch.bool, device=DEV)
    if where == "q":
        rows = {cu[s], cu[s + 1] - 1, cu[0], cu[-1] - 1}      # (among them a sequence's only row)
        for r in rows:
            w.q[r, Hq - 1, 5] = float("nan")
            bad[r, Hq - 1] = True
    else:
        at = lens[s] - q_lens[s] // 2 - 1                     # the half of the queries behind it, on one KV head
        w.k_new[sum(lens[:s]) + at, 0, 5] = float("nan")
        bad[cu[s] + max(at - (lens[s] - q_lens[s]), 0):cu[s + 1], :G] = True
    pa.paged_kv_append(w.k_cache, w.v_cache, w.k_new, w.v_new, w.seq_ids, w.positions, w.block_table)
    out, lse = torch.zeros_like(w.q), torch.zeros((w.total_q, Hq), device=DEV)
    ws = torch.full((pa.paged_attention_workspace_bytes(w.batch, Hq, d, w.total_q, w.max_seq_len),), 0x3F, dtype=torch.uint8,
                    device=DEV)
    binding.pa_profile_reset()
    binding.pa_profile_enable(True)
    try:
        pa.paged_attention_prefill(w.k_cache, w.v_cache, w.q, w.cu_q_lens, w.max_q_len, w.block_table, w.seq_lens, w.max_seq_len,
                                   w.scale, True, out=out, lse=lse, workspace=ws)
        torch.cuda.synchronize()
        assert binding.pa_profile_read(kernel)[0] == 1
    finally:
        binding.pa_profile_enable(False)
        binding.pa_profile_reset()
    assert torch.equal(lse.isnan(), bad)
    assert torch.equal(out.isnan(), bad[..., None].expand_as(out))
    ref = _reference(w)
    ref[bad] = 0.0
    out[bad] = 0.0
    assert torch.isfinite(lse[~bad]).all()
    parity.assert_close(parity.to_f64(out), parity.to_f64(ref), dtype, f"{lens}")


@pytest.mark.parametrize("lens,q_lens,Hq,Hkv,d,dtype", [
    ([2000], [2000], 8, 1, 128, torch.bfloat16),              # the workspace's bound holds two chunks, the GPU has room for four
    ([1700], [1600], 8, 1, 128, torch.float16),
    ([3000], [3000], 8, 1, 256, torch.bfloat16)])
def test_chunks_of_a_prompt_do_not_depend_on_the_workspace(pa, lens, q_lens, Hq, Hkv, d, dtype):
    """A workspace that was sized for a larger call gives the same bits as one of the call's own size."""
    w = W.make_workload("t", seq_lens=lens, q_lens=q_lens, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, page_size=16, dtype=dtype,
                        causal=True, seed=226, device=DEV)
    pa.paged_kv_append(w.k_cache, w.v_cache, w.k_new, w.v_new, w.seq_ids, w.positions, w.block_table)
    nbytes = pa.paged_attention_workspace_bytes(w.batch, Hq, d, w.total_q, w.max_seq_len)
    res = []
    for room in (0, 256 << 20):
        ws = torch.full((nbytes + room,), 0xFF, dtype=torch.uint8, device=DEV)
        lse = torch.empty((w.total_q, Hq), device=DEV)
        out = pa.paged_attention_prefill(w.k_cache, w.v_cache, w.q, w.cu_q_lens, w.max_q_len, w.block_table, w.seq_lens,
                                         w.max_seq_len, w.scale, True, lse=lse, workspace=ws)
        res.append((out, lse, int((ws.view(torch.int32) != -1).sum())))
    assert res[0][2] == res[1][2] > 0                         # as many words of partials
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])


@pytest.mark.parametrize("lens,q_lens,Hq,Hkv,d,P,causal,hooks,order", [
    ([2366], [2366], 8, 1, 256, 16, True, dict(docs=True), "by_tile"),                         # three chunks, one head group
    ([4589], [500], 64, 8, 128, 16, True, dict(window=256), "last_chunk_first"),               # four, most without keys
    ([6000] * 2, [300] * 2, 8, 1, 128, 64, False, dict(window=700), "last_chunk_first"),        # windows to both sides
    ([5000, 2100, 33], [64] * 2 + [33], 16, 8, 256, 16, True, dict(window=1024, softcap=30.0), "last_chunk_first"),     # unequal queries, few places
    ([3500, 2100, 700], [130, 1, 70], 8, 8, 64, 16, True, dict(window=900, alibi=True), "by_tile")])           # some the stream's
def test_orders_of_chunks(pa, oracle, lens, q_lens, Hq, Hkv, d, P, causal, hooks, order):
    """The three orders in which a grid hands out row tiles and chunks; the fourth has the cases of prompts in chunks."""
    from paper_2506_07311_amd import binding
    from tests.test_gpu_parity import build_mods
    w = W.make_workload("t", seq_lens=lens, q_lens=q_lens, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, page_size=P,
                        dtype=torch.bfloat16, causal=causal, seed=229, device=DEV)
    binding.pa_profile_reset()
    binding.pa_profile_enable(True)
    try:
        parity.check_step(pa, oracle, w, f"{lens} {d}", mods=build_mods(hooks, Hq, lens) if hooks else None)
        assert binding.pa_profile_read("paged_prefill_mfma_kernel_" + order)[0] == 1
    finally:
        binding.pa_profile_enable(False)
        binding.pa_profile_reset()


@pytest.mark.parametrize("lens,Hq,Hkv,d,causal,hooks,n", [
    ([700, 4500], 4, 1, 64, True, dict(alibi=True), 8),       # more than what is required of a workspace holds
    ([33, 4200], 4, 1, 128, True, dict(softcap=30.0), 6),
    ([1000], 8, 1, 128, False, dict(window=700), 4),          # a window to both sides: all 1000 keys for most rows
    ([2085, 645], 8, 1, 128, False, dict(softcap=30.0), 1),   # without a causal bound: one round in one piece, a second in two
    ([900], 8, 1, 128, True, dict(prefix=True), 4),           # a user modification
    ([1025], 8, 1, 128, True, {}, 3)])                        # four are estimated within a margin behind three
def test_the_number_of_chunks_of_prompts(pa, oracle, lens, Hq, Hkv, d, causal, hooks, n):
    """How many chunks prompts get with the bound's workspace: the last row, which sees all of them, ends what is written to it."""
    from paper_2506_07311_amd import binding
    from tests.test_gpu_parity import alibi, build_mods
    w = W.make_workload("t", seq_lens=lens, q_lens=lens, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, page_size=16,
                        dtype=torch.bfloat16, causal=causal, seed=230, device=DEV)
    mods = build_mods(hooks, Hq, lens) if hooks else None
    kw = {k: v for k, v in hooks.items() if k not in ("alibi", "prefix")}
    if "prefix" in hooks:
        mods = dict(prefix_lens=np.array([m // 2 for m in lens], dtype=np.int32), prefix_bias=0.5)
        prefix = torch.tensor(mods["prefix_lens"], dtype=torch.int32, device=DEV)
        kw = dict(user_mod=binding.PA_MOD_PREFIX_LM, user_data=binding.prefix_lm_data(prefix, mods["prefix_bias"]))
    parity.check_step(pa, oracle, w, f"{lens} {d}", mods=mods)
    if "alibi" in hooks:
        kw["alibi_slopes"] = torch.tensor(alibi(Hq), dtype=torch.float32, device=DEV)
    ws = torch.full((pa.paged_attention_workspace_bytes(w.batch, Hq, d, w.total_q, w.max_seq_len),), 0xFF, dtype=torch.uint8,
                    device=DEV)
    pa.paged_attention_prefill_mod(w.k_cache, w.v_cache, w.q, w.cu_q_lens, w.max_q_len, w.block_table, w.seq_lens, w.max_seq_len,
                                   w.scale, causal, workspace=ws, **kw)
    part_o = -(-w.total_q * Hq * n * d * 4 // 256) * 256
    written = (ws.view(torch.int32) != -1).nonzero()
    end = int(written.max()) + 1 if written.numel() else 0
    assert end == (part_o // 4 + w.total_q * Hq * n if n > 1 else 0)


@pytest.mark.parametrize("lens,q_lens,Hq,Hkv,d,dtype,causal,hooks", [
    ([300, 700, 90] * 3 + [650, 600, 400, 310], [1] * 9 + [300, 1, 33, 310], 16, 2, 64, torch.bfloat16, True, dict(window=600)),
    ([600, 33, 5] * 9, [1, 3, 1] * 8 + [179, 33, 5], 40, 8, 128, torch.float16, True, dict(softcap=30.0)),
    ([700] * 5, [1, 0, 700, 0, 2], 16, 2, 256, torch.bfloat16, False, None)])      # one sequence has them all
def test_a_grid_of_mostly_gaps(pa, oracle, lens, q_lens, Hq, Hkv, d, dtype, causal, hooks):
    """Gaps that go round the shader engines are left out all the same where most of the grid would be gaps."""
    from paper_2506_07311_amd import binding
    from tests.test_gpu_parity import build_mods
    w = W.make_workload("t", seq_lens=lens, q_lens=q_lens, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, page_size=16,
                        dtype=dtype, causal=causal, seed=231, device=DEV)
    binding.pa_profile_reset()
    binding.pa_profile_enable(True)
    try:
        parity.check_step(pa, oracle, w, f"{lens} {d}", mods=build_mods(hooks, Hq, lens) if hooks else None)
        assert binding.pa_profile_read("paged_prefill_mfma_kernel_live")[0] == 1
    finally:
        binding.pa_profile_enable(False)
        binding.pa_profile_reset()


@pytest.mark.parametrize("lens,q_lens,Hq,Hkv,d,kernel", [
    ([769], [769], 8, 1, 256, "paged_attention_merge_kernel"),                     # a prompt in chunks of 256 keys
    ([4097, 300], [130, 1], 8, 4, 128, "paged_attention_merge_list_kernel"),      # the list: of 1024 keys
    ([4097, 4097], [64, 64], 8, 2, 64, "paged_attention_merge_kernel")])
def test_a_last_chunk_of_one_key(pa, oracle, lens, q_lens, Hq, Hkv, d, kernel):
    """Contexts one key longer than their chunks are."""
    from paper_2506_07311_amd import binding
    w = W.make_workload("t", seq_lens=lens, q_lens=q_lens, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, page_size=16,
                        dtype=torch.bfloat16, causal=True, seed=232, device=DEV)
    binding.pa_profile_reset()
    binding.pa_profile_enable(True)
    try:
        parity.check_step(pa, oracle, w, f"{lens} {d}")
        assert binding.pa_profile_read(kernel)[0] == 1
    finally:
        binding.pa_profile_enable(False)
        binding.pa_profile_reset()


@pytest.mark.parametrize("lens,q_lens,Hq,Hkv,d,dtype", [
    ([3000, 70], [1, 1], 8, 8, 64, torch.float32),
    ([600, 70], [600, 70], 8, 8, 64, torch.float32),
    ([3000, 70], [1, 1], 8, 2, 96, torch.bfloat16),
    ([700, 70], [64, 1], 8, 2, 96, torch.float16),
    ([3000, 70], [1, 1], 8, 2, 128, torch.bfloat16),
    ([3000, 70], [130, 1], 8, 2, 128, torch.bfloat16),
    ([1000], [1000], 8, 1, 64, torch.float16),
    ([1000], [1000], 8, 1, 256, torch.bfloat16)])
@pytest.mark.parametrize("docs", [True, False])
def test_a_nan_in_a_query_beside_document_masks(pa, lens, q_lens, Hq, Hkv, d, dtype, docs):
    """Scores that are all NaN or hidden are not taken for a row without a visible key, by any of the kernels."""
    from tests.test_gpu_parity import doc_ids
    w = W.make_workload("t", seq_lens=lens, q_lens=q_lens, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, page_size=16,
                        dtype=dtype, causal=True, seed=233, device=DEV)
    bad = torch.zeros((w.total_q, Hq), dtype=torch.bool, device=DEV)
    for r in (0, w.total_q - 1):
        w.q[r, Hq - 1, 5] = float("nan")
        bad[r, Hq - 1] = True
    pa.paged_kv_append(w.k_cache, w.v_cache, w.k_new, w.v_new, w.seq_ids, w.positions, w.block_table)
    lse = torch.zeros((w.total_q, Hq), device=DEV)
    ids = torch.tensor(doc_ids(lens, 7), dtype=torch.int32, device=DEV) if docs else None
    out = pa.paged_attention_prefill_mod(w.k_cache, w.v_cache, w.q, w.cu_q_lens, w.max_q_len, w.block_table, w.seq_lens,
                                         w.max_seq_len, w.scale, True, lse=lse, doc_ids=ids)
    assert torch.equal(lse.isnan(), bad)
    assert torch.equal(out.isnan(), bad[..., None].expand_as(out))
    assert torch.isfinite(lse[~bad]).all()
