"""GPU parity of the matrix-core kernels at head_dims whose rows do not fill their tiles (80, 96, 112): padded column
blocks, padded score steps, repeated row pieces; and at head_dim 256, whose waves hold 16 rows."""
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


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("causal,chunk", [(True, 0), (False, 0), (True, 128)])
@pytest.mark.parametrize("case", [None, dict(window=1), dict(window=70), dict(softcap=2.0), dict(window=33, softcap=5.0),
                                  dict(window=70, softcap=5.0, alibi=True)],
                         ids=["plain", "window1", "window70", "cap", "window_cap", "window_cap_alibi"])
def test_prefill_at_head_dim_256(pa, oracle, dtype, causal, chunk, case):
    """Row counts around the 16 rows of a wave and the 128 of a workgroup (two heads a row tile), contexts around the
    64-key tile, windows that cut a tile's first keys, and each of the kernels a call's hooks choose between."""
    from paper_2506_07311_amd import binding
    lens = [1, 15, 16, 17, 0, 64, 65, 129, 300, 191]
    q_lens = [1, 7, 8, 9, 0, 63, 64, 65, 128, 33]
    w = W.make_workload("t", seq_lens=lens, q_lens=q_lens, num_q_heads=4, num_kv_heads=2, head_dim=256, page_size=32,
                        dtype=dtype, causal=causal, seed=211, device=DEV)
    mods = None
    if case:
        mods = {k: v for k, v in case.items() if k != "alibi"}
        if case.get("alibi"):
            mods["alibi_slopes"] = [2.0 ** -(i + 1) for i in range(4)]
    binding.pa_set_option("prefill_chunk_tokens", chunk)
    binding.pa_profile_reset()
    binding.pa_profile_enable(True)
    try:
        parity.check_step(pa, oracle, w, f"prefill d=256 {dtype} {case}", mods=mods)
        assert binding.pa_profile_read("paged_prefill_mfma")[0] == 1
    finally:
        binding.pa_profile_enable(False)
        binding.pa_profile_reset()
        binding.pa_set_option("prefill_chunk_tokens", 0)


# ----------------------------------------------------------------------------- fp32 pools on the fp64 matrix cores
F32_CASES = [  # lens, q_lens (None: decode), Hq, Hkv, d, P, causal
    ([1, 15, 16, 17, 0, 129, 777, 33], [1, 15, 16, 17, 0, 100, 200, 33], 4, 4, 64, 16, True),
    ([1, 15, 16, 300], [1, 15, 16, 50], 6, 2, 128, 32, True),
    ([40, 200], [7, 33], 40, 2, 64, 64, False),                  # 20 heads a group: row tiles that straddle queries
    ([1, 16, 0, 129, 2049, 255], None, 32, 4, 64, 16, False),    # 2049 keys: chunks of 256 and the merge kernel
    ([700, 3, 128], None, 40, 2, 128, 128, False),
]


@pytest.mark.parametrize("case", F32_CASES, ids=lambda c: f"Hq{c[2]}-Hkv{c[3]}-d{c[4]}-P{c[5]}-{'prefill' if c[1] else 'decode'}")
def test_fp32_on_the_matrix_cores(pa, oracle, case):
    """Against the fp64 oracle at 2e-6 max-abs / 1e-5 max-rel: fp64 products and sums leave the exponential (one fp32 ulp, 6e-8
    of a weight), the fp32 partials (6e-8) and the output's rounding (6e-8) of values below 4."""
    from paper_2506_07311_amd import binding
    lens, q_lens, Hq, Hkv, d, P, causal = case
    w = W.make_workload("t", seq_lens=lens, q_lens=q_lens or [1] * len(lens), append_lens=q_lens or [min(n, 1) for n in lens],
                        num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, page_size=P, dtype=torch.float32, causal=causal,
                        seed=203, device=DEV)
    binding.pa_profile_reset()
    binding.pa_profile_enable(True)
    try:
        parity.check_step(pa, oracle, w, f"fp32 {case[2:]}", tol=(2e-6, 1e-5), step_call=q_lens is None)
        assert binding.pa_profile_read("paged_attention_f32_kernel")[0] == 1
        assert binding.pa_profile_read("paged_attention_merge_kernel")[0] == (0 if q_lens else 1)
    finally:
        binding.pa_profile_enable(False)
        binding.pa_profile_reset()


@pytest.mark.parametrize("d,dtype", [(64, torch.float32), (128, torch.float32), (80, torch.bfloat16), (96, torch.float16),
                                     (112, torch.bfloat16), (80, torch.float16)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("where", ["v", "k"])
@pytest.mark.parametrize("n,new,chunk", [(150, 150, 0), (700, 700, 0), (700, 60, 256)], ids=["edge", "inside", "cut"])
def test_values_that_are_not_finite_do_what_they_did_on_the_portable_kernel(pa, d, dtype, bad, where, n, new, chunk):
    """A NaN or an infinity in V or K reaches the queries that see it as what it was on the portable kernel, which takes every
    product in one term, and no other query: on the tile at a row's causal edge, on full tiles, and through a merge."""
    from paper_2506_07311_amd import binding
    at = 70
    eps = 2e-6 if dtype == torch.float32 else 4e-3 if dtype == torch.float16 else 3e-2     # one rounding step of values below 4
    w = W.make_workload("t", seq_lens=[n], q_lens=[new], append_lens=[n], num_q_heads=4, num_kv_heads=2, head_dim=d, page_size=16,
                        dtype=dtype, causal=True, seed=204, device=DEV)
    (w.v_new if where == "v" else w.k_new)[at, :, 3] = bad
    pa.paged_kv_append(w.k_cache, w.v_cache, w.k_new, w.v_new, w.seq_ids, w.positions, w.block_table)
    res = []
    for generic in (1, 0):
        binding.pa_set_option("force_generic", generic)
        binding.pa_set_option("prefill_chunk_tokens", chunk)
        lse = torch.empty((new, 4), device=DEV)
        try:
            out = pa.paged_attention_prefill(w.k_cache, w.v_cache, w.q, w.cu_q_lens, w.max_q_len, w.block_table, w.seq_lens, n,
                                             w.scale, True, lse=lse)
            torch.cuda.synchronize()
        finally:
            binding.pa_set_option("force_generic", 0)
            binding.pa_set_option("prefill_chunk_tokens", 0)
        res.append((out.float(), lse))
    for ref, got, tol in ((res[0][0], res[1][0], eps), (res[0][1], res[1][1], 1e-4)):
        assert torch.equal(got.isnan(), ref.isnan())
        assert torch.equal(got.isinf(), ref.isinf()) and torch.equal(got[got.isinf()] > 0, ref[ref.isinf()] > 0)
        assert ((got - ref)[ref.isfinite()].abs() <= tol).all()
    first = max(at - (n - new), 0)                                # the first query that sees the value
    assert first == 0 or res[1][0][:first].isfinite().all()
    assert not res[1][0][first:].isfinite().all()


@pytest.mark.parametrize("d,Hq", [(64, 2), (64, 8), (128, 8)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("where", ["v", "k"])
def test_fp32_decode_of_values_that_are_not_finite(pa, d, Hq, bad, where):
    """As above for the decode kernel: one sequence that holds the value, at its last key, one that does not."""
    from paper_2506_07311_amd import binding
    w = W.make_workload("t", seq_lens=[2049, 300, 77], num_q_heads=Hq, num_kv_heads=2, head_dim=d, page_size=16,
                        dtype=torch.float32, seed=210, device=DEV)
    (w.v_new if where == "v" else w.k_new)[0::2, :, 3] = bad
    pa.paged_kv_append(w.k_cache, w.v_cache, w.k_new, w.v_new, w.seq_ids, w.positions, w.block_table)
    res = []
    for generic in (1, 0):
        binding.pa_set_option("force_generic", generic)
        binding.pa_set_option("decode_chunk_tokens", generic << 20)   # (its merge takes a chunk that is all NaN for an empty one)
        lse = torch.empty((3, Hq), device=DEV)
        try:
            res.append((pa.paged_attention_decode(w.k_cache, w.v_cache, w.q, w.block_table, w.seq_lens, 2049, w.scale, lse=lse), lse))
            torch.cuda.synchronize()
        finally:
            binding.pa_set_option("force_generic", 0)
            binding.pa_set_option("decode_chunk_tokens", 0)
    assert res[1][0][1].isfinite().all()
    for ref, got, tol in ((res[0][0], res[1][0], 2e-6), (res[0][1], res[1][1], 1e-5)):
        assert torch.equal(got.isnan(), ref.isnan())
        assert torch.equal(got.isinf(), ref.isinf()) and torch.equal(got[got.isinf()] > 0, ref[ref.isinf()] > 0)
        assert ((got - ref)[ref.isfinite()].abs() <= tol).all()


F32_DECODES = [  # lens, Hq, Hkv, d, P
    ([1, 15, 16, 17, 0, 129, 2049, 33], 8, 8, 64, 16),           # no groups: one row a wave
    ([300, 0, 2049, 128, 129], 8, 4, 64, 32),                    # two heads a group
    ([300, 2049, 257, 1], 12, 4, 64, 16),                        # three heads on four rows
    ([2049, 64, 1000], 16, 4, 64, 128),
    ([1, 300, 0, 2049, 511], 8, 8, 128, 16),
    ([300, 2049, 17], 12, 4, 128, 64),
    ([2049, 64, 1000], 16, 4, 128, 16),
    ([5000, 1, 63] + [40, 129] * 16, 32, 8, 64, 16),             # more (sequence, KV head) units than compute units: only the
    ([3000] + [20] * 64, 8, 8, 128, 16),                         # long contexts are cut
    ([9000], 4, 4, 64, 16),                                      # more workgroups than a round of tiles each
]


@pytest.mark.parametrize("case", F32_DECODES, ids=lambda c: f"n{len(c[0])}-Hq{c[1]}-Hkv{c[2]}-d{c[3]}-P{c[4]}")
@pytest.mark.parametrize("room", ["workspace", "static array"])
def test_fp32_decode_on_the_vector_unit(pa, oracle, case, room):
    """The one-launch fp32 decode kernel, up to four heads a group: its cuts by the real lengths, with the whole workspace and
    through the entry point whose workspace is the static array; tolerance as above."""
    from paper_2506_07311_amd import binding
    lens, Hq, Hkv, d, P = case
    w = W.make_workload("t", seq_lens=lens, q_lens=[1] * len(lens), append_lens=[min(n, 1) for n in lens], num_q_heads=Hq,
                        num_kv_heads=Hkv, head_dim=d, page_size=P, dtype=torch.float32, seed=205, device=DEV)
    k, v, o_ref, lse_ref = parity.oracle_step(oracle, w)
    pa.paged_kv_append(w.k_cache, w.v_cache, w.k_new, w.v_new, w.seq_ids, w.positions, w.block_table)
    lse = torch.full((w.batch, Hq), float("nan"), device=DEV)
    out = torch.full_like(w.q, float("nan"))
    binding.pa_profile_reset()
    binding.pa_profile_enable(True)
    try:
        if room == "workspace":
            ws = torch.full((pa.paged_attention_workspace_bytes(w.batch, Hq, d, w.batch, w.max_seq_len),), 0xFF,
                            dtype=torch.uint8, device=DEV)
            pa.paged_attention_decode(w.k_cache, w.v_cache, w.q, w.block_table, w.seq_lens, w.max_seq_len, w.scale, out=out,
                                      lse=lse, workspace=ws)
        else:
            pa.paged_attention_decode_static(w.k_cache, w.v_cache, w.q, w.block_table, w.seq_lens, w.max_seq_len, w.scale,
                                             out=out, lse=lse)
        torch.cuda.synchronize()
        assert binding.pa_profile_read("paged_decode_f32_kernel")[0] == 1
        assert binding.pa_profile_read("paged_attention")[0] == 0
    finally:
        binding.pa_profile_enable(False)
        binding.pa_profile_reset()
    parity.assert_close(parity.to_f64(out), o_ref, torch.float32, "out", tol=(2e-6, 1e-5))
    got, empty = parity.to_f64(lse), ~torch.tensor(lse_ref).isfinite().numpy()
    assert (got[empty] == float("-inf")).all() and abs(got[~empty] - lse_ref[~empty]).max() <= 1e-5


@pytest.mark.parametrize("Hq,Hkv,d", [(4, 4, 64), (8, 2, 64), (4, 4, 128), (8, 2, 128)])
@pytest.mark.parametrize("n", [40, 2049])
def test_fp32_decode_of_large_values(pa, Hq, Hkv, d, n):
    """Values whose mean fits fp32 and whose weighted sum relative to an early key's score would not: every first key of a tile
    scores 0 and the others e^10, which is as far as the kernel's softmax reference may trail (2^16).  Every value is the
    same, so the output is that value up to the rounding of the partials (a few ulp)."""
    w = W.make_workload("t", seq_lens=[n], num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, page_size=16, dtype=torch.float32,
                        identity_pages=True, poison=False, seed=206, device=DEV)
    w.q.fill_(1.0)
    w.k_cache.fill_(10.0 / d)
    w.k_cache[:, 0] = 0.0
    w.v_cache.fill_(1e35)
    lse = torch.empty((1, Hq), device=DEV)
    out = pa.paged_attention_decode(w.k_cache, w.v_cache, w.q, w.block_table, w.seq_lens, n, 1.0, lse=lse)
    assert ((out.double() / 1e35 - 1.0).abs() <= 4e-7).all()
    firsts = (n + 15) // 16
    ref = torch.log(torch.tensor(firsts + (n - firsts) * float(torch.exp(torch.tensor(10.0, dtype=torch.float64)))))
    assert (lse.cpu() - ref).abs().max() <= 1e-5


@pytest.mark.parametrize("lens,q_lens", [([300] + [40] * 70, [200] + [1] * 70),           # one prompt among single queries
                                         ([40, 0, 33, 64, 16, 17, 5], [40, 0, 3, 16, 0, 17, 1]),
                                         ([16] * 5000 + [100], [0, 1] * 2500 + [90])],    # more than 64 x 64 sequences
                         ids=lambda v: f"n{len(v)}")
@pytest.mark.parametrize("max_q_len", [0, 1 << 30])
def test_fp32_prefill_with_mostly_empty_row_tiles(pa, oracle, lens, q_lens, max_q_len):
    """max_q_len is an upper bound: however loose, the call runs, and gives what the tight one gives."""
    from paper_2506_07311_amd import binding
    for Hq, Hkv, d in ((3, 1, 64), (2, 2, 128)):
        w = W.make_workload("t", seq_lens=lens, q_lens=q_lens, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, page_size=16,
                            dtype=torch.float32, causal=True, seed=207, device=DEV)
        _, _, o_ref, lse_ref = parity.oracle_step(oracle, w)
        pa.paged_kv_append(w.k_cache, w.v_cache, w.k_new, w.v_new, w.seq_ids, w.positions, w.block_table)
        lse = torch.full((w.total_q, Hq), float("nan"), device=DEV)
        binding.pa_profile_reset()
        binding.pa_profile_enable(True)
        try:
            out = pa.paged_attention_prefill(w.k_cache, w.v_cache, w.q, w.cu_q_lens, max_q_len or w.max_q_len, w.block_table,
                                             w.seq_lens, w.max_seq_len, w.scale, True, lse=lse)
            torch.cuda.synchronize()
            assert binding.pa_profile_read("paged_attention_f32_kernel")[0] == 1
        finally:
            binding.pa_profile_enable(False)
            binding.pa_profile_reset()
        parity.assert_close(parity.to_f64(out), o_ref, torch.float32, "out", tol=(2e-6, 1e-5))
        assert abs(parity.to_f64(lse) - lse_ref).max() <= 1e-5


@pytest.mark.parametrize("lens,q_lens", [([300] + [40] * 70, [200] + [1] * 70),
                                         ([400, 0, 33, 64, 16, 17, 5], [140, 0, 3, 16, 0, 17, 1]),
                                         ([2500], [3])],                                   # cut along the context
                         ids=lambda v: f"n{len(v)}")
@pytest.mark.parametrize("d", [80, 96, 112])
def test_padded_head_dims_with_mostly_empty_row_tiles(pa, oracle, d, lens, q_lens):
    """As above: the bound on the query lengths may be loose, up to where the plain grid has more workgroups than a launch."""
    for max_q_len in (max(q_lens), 1 << 20, 1 << 30):
        w = W.make_workload("t", seq_lens=lens, q_lens=q_lens, num_q_heads=8, num_kv_heads=2, head_dim=d, page_size=16,
                            dtype=torch.bfloat16, causal=True, seed=208, device=DEV)
        _, _, o_ref, lse_ref = parity.oracle_step(oracle, w)
        pa.paged_kv_append(w.k_cache, w.v_cache, w.k_new, w.v_new, w.seq_ids, w.positions, w.block_table)
        lse = torch.full((w.total_q, 8), float("nan"), device=DEV)
        out = pa.paged_attention_prefill(w.k_cache, w.v_cache, w.q, w.cu_q_lens, max_q_len, w.block_table, w.seq_lens,
                                         w.max_seq_len, w.scale, True, lse=lse)
        parity.assert_close(parity.to_f64(out), o_ref, torch.bfloat16, f"out {max_q_len}")
        assert abs(parity.to_f64(lse) - lse_ref).max() <= 1e-3


@pytest.mark.parametrize("n,new,Hq,Hkv,d,portable", [(250, 16, 8, 8, 128, True), (500, 32, 8, 8, 128, True), (250, 33, 8, 8, 128, False),
                                                     (1000, 16, 8, 8, 128, False), (250, 16, 8, 8, 64, True), (250, 17, 8, 8, 64, False),
                                                     (100, 4, 32, 8, 64, False), (500, 4, 32, 8, 64, True)])
def test_fp32_prefill_of_few_rows_on_a_short_context(pa, oracle, n, new, Hq, Hkv, d, portable):
    from paper_2506_07311_amd import binding
    w = W.make_workload("t", seq_lens=[n], q_lens=[new], num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, page_size=16,
                        dtype=torch.float32, causal=True, seed=209, device=DEV)
    binding.pa_profile_reset()
    binding.pa_profile_enable(True)
    try:
        parity.check_step(pa, oracle, w, "few rows")
        assert binding.pa_profile_read("paged_attention_generic_kernel")[0] == (1 if portable else 0)
        assert binding.pa_profile_read("paged_attention_f32_kernel")[0] == (0 if portable else 1)
    finally:
        binding.pa_profile_enable(False)
        binding.pa_profile_reset()


@pytest.mark.parametrize("d", [80, 96, 112])
def test_fp16_weights_far_below_the_largest_are_not_lost(pa, d):
    """One key leads 8000 others by e^15: each of those weighs less than 2^-21 of it, all of them together 2e-3.  The output is
    their values' share to the rounding of fp16 (2^-11 of values up to 4e-3, subnormal below 6e-5 only)."""
    n, at = 8000, 100
    w = W.make_workload("t", seq_lens=[n], q_lens=[64], num_q_heads=2, num_kv_heads=2, head_dim=d, page_size=16,
                        dtype=torch.float16, causal=True, identity_pages=True, poison=False, seed=220, device=DEV)
    w.q.fill_(1.0)
    w.k_cache.zero_()
    w.k_cache[at // 16, at % 16] = 15.0 / d
    w.v_cache.fill_(1.0)
    w.v_cache[at // 16, at % 16] = 0.0
    out = pa.paged_attention_prefill(w.k_cache, w.v_cache, w.q, w.cu_q_lens, w.max_q_len, w.block_table, w.seq_lens, n, 1.0, True)
    score = float(w.k_cache[at // 16, at % 16].double().sum(-1)[0])
    keys = torch.arange(n - 64, n, dtype=torch.float64, device=DEV)              # of the row at that position, but for `at`
    ref = keys / (keys + torch.exp(torch.tensor(score, dtype=torch.float64)))
    assert (out.double() / ref[:, None, None] - 1.0).abs().max() <= 2.0 ** -10


@pytest.mark.parametrize("d", [80, 96, 112])
def test_bf16_sums_of_large_values_stay_finite(pa, d):
    """Later keys outweigh the ones the softmax reference was taken from by 2^9: sums of finite values must not overflow."""
    n = 300
    w = W.make_workload("t", seq_lens=[n], q_lens=[n], num_q_heads=2, num_kv_heads=2, head_dim=d, page_size=16,
                        dtype=torch.bfloat16, causal=True, identity_pages=True, poison=False, seed=221, device=DEV)
    w.q.fill_(1.0)
    w.k_cache.fill_(6.25 / d)
    w.k_cache[:4] = 0.0                                                           # the first 64 keys
    w.v_cache.fill_(1e35)
    out = pa.paged_attention_prefill(w.k_cache, w.v_cache, w.q, w.cu_q_lens, w.max_q_len, w.block_table, w.seq_lens, n, 1.0, True)
    v = float(w.v_cache[0, 0, 0, 0].double())
    assert (out.double() / v - 1.0).abs().max() <= 2.0 ** -8


@pytest.mark.parametrize("lens,Hq,Hkv,portable", [([257, 1, 30], 16, 2, True), ([192, 100], 16, 2, False), ([2049], 32, 2, False),
                                                  ([257, 30], 15, 3, False), ([1000], 16, 1, True)])
@pytest.mark.parametrize("d", [64, 128])
def test_fp32_decode_of_large_groups_with_few_kv_heads(pa, oracle, lens, Hq, Hkv, portable, d):
    from paper_2506_07311_amd import binding
    w = W.make_workload("t", seq_lens=lens, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, page_size=16, dtype=torch.float32,
                        seed=211, device=DEV)
    binding.pa_profile_reset()
    binding.pa_profile_enable(True)
    try:
        parity.check_step(pa, oracle, w, f"{lens}", step_call=True)
        assert binding.pa_profile_read("paged_attention_generic_kernel")[0] == (1 if portable else 0)
        assert binding.pa_profile_read("paged_attention_f32_kernel")[0] == (0 if portable else 1)
    finally:
        binding.pa_profile_enable(False)
        binding.pa_profile_reset()
