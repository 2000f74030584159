"""One-launch decode calls that split a (sequence, KV head) over workgroups: their arrival counters live in the caller's
workspace, so whatever it holds on entry and however many calls are in flight, each call merges its own partials once."""
import pytest
import torch

from paper_2506_07311_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

SHAPES = [  # seq_lens, Hq, Hkv, d, dtype: the 16-bit kernel (with a head slice of its own, too), fp32 with and without groups
    ([2048, 1500], 32, 8, 128, torch.bfloat16),
    ([6000], 40, 2, 64, torch.float16),
    ([2048, 900], 8, 8, 64, torch.float32),
    ([1000], 24, 8, 128, torch.float32),
]
IDS = [f"Hq{s[1]}-Hkv{s[2]}-d{s[3]}-{str(s[4])[6:]}" for s in SHAPES]


@pytest.fixture(scope="module")
def pa():
    import paper_2506_07311_amd as pa_mod
    pa_mod.load_library()
    return pa_mod


def make(shape, seed):
    lens, Hq, Hkv, d, dtype = shape
    return W.make_workload("t", seq_lens=lens, num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, page_size=16, dtype=dtype,
                           seed=seed, device=DEV)


def prepare(pa, w, q, out, lse, ws, stream=None):
    return pa.prepare_decode(w.k_cache, w.v_cache, q, w.block_table, w.seq_lens, w.max_seq_len, w.scale, out=out, lse=lse,
                             workspace=ws, stream=stream)


def buffers(pa, w, n):
    """n queries, outputs, LSEs and workspaces, the workspaces holding random bytes."""
    nbytes = pa.paged_attention_workspace_bytes(w.batch, w.num_q_heads, w.head_dim, w.batch, w.max_seq_len)
    qs = [w.q + i for i in range(n)]
    outs = [torch.full_like(w.q, float("nan")) for _ in range(n)]
    lses = [torch.full((w.batch, w.num_q_heads), float("nan"), device=DEV) for _ in range(n)]
    wss = [torch.randint(0, 256, (nbytes,), dtype=torch.uint8, device=DEV) for _ in range(n)]
    return qs, outs, lses, wss


def serial(pa, w, qs):
    """The same calls one after the other, each waited for, on one clean workspace."""
    ws = torch.zeros(pa.paged_attention_workspace_bytes(w.batch, w.num_q_heads, w.head_dim, w.batch, w.max_seq_len),
                     dtype=torch.uint8, device=DEV)
    res = []
    for q in qs:
        lse = torch.empty((w.batch, w.num_q_heads), device=DEV)
        out = prepare(pa, w, q, torch.empty_like(q), lse, ws)()
        torch.cuda.synchronize()
        res.append((out, lse))
    return res


@pytest.mark.parametrize("shape", SHAPES, ids=IDS)
def test_a_workspace_may_hold_anything(pa, oracle, shape):
    from paper_2506_07311_amd import binding
    from tests import parity
    w = make(shape, 301)
    binding.pa_profile_reset()
    binding.pa_profile_enable(True)
    try:
        parity.check_step(pa, oracle, w, f"{shape}")                    # (a workspace of ones)
        launches = sum(binding.pa_profile_read(k)[0] for k in ("paged_decode_short_kernel", "paged_decode_f32_kernel"))
        assert launches == 1 and binding.pa_profile_read("paged_attention_merge")[0] == 0
    finally:
        binding.pa_profile_enable(False)
        binding.pa_profile_reset()
    ref_out, ref_lse = serial(pa, w, [w.q])[0]
    nbytes = pa.paged_attention_workspace_bytes(w.batch, w.num_q_heads, w.head_dim, w.batch, w.max_seq_len)
    for fill in ("ones", "random", "left by the call before"):
        if fill == "ones":
            ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device=DEV)
        elif fill == "random":
            ws = torch.randint(0, 256, (nbytes,), dtype=torch.uint8, device=DEV)
        lse = torch.full_like(ref_lse, float("nan"))
        out = prepare(pa, w, w.q, torch.full_like(w.q, float("nan")), lse, ws)()
        assert torch.equal(out, ref_out) and torch.equal(lse, ref_lse), fill


@pytest.mark.parametrize("shape", SHAPES, ids=IDS)
def test_many_calls_in_flight_on_several_streams(pa, shape):
    """72 calls on three streams that start one after the other, so that calls far apart in issue order run together."""
    w = make(shape, 302)
    n, streams = 72, [torch.cuda.Stream() for _ in range(3)]
    qs, outs, lses, wss = buffers(pa, w, n)
    ref = serial(pa, w, qs)
    calls = [prepare(pa, w, qs[i], outs[i], lses[i], wss[i], stream=streams[i % 3]) for i in range(n)]
    torch.cuda.synchronize()
    for s, st in enumerate(streams):
        with torch.cuda.stream(st):
            torch.cuda._sleep(1000000 * (3 - s))
    for c in calls:
        c()
    torch.cuda.synchronize()
    for i in range(n):
        assert torch.equal(outs[i], ref[i][0]) and torch.equal(lses[i], ref[i][1]), i


@pytest.mark.parametrize("shape", SHAPES, ids=IDS)
def test_captured_calls_replay_beside_each_other(pa, shape):
    """Graphs of single calls, captured one after the other and replayed three times over on two streams; between the
    replays the workspaces are filled with other bytes and eager calls run on them."""
    w = make(shape, 303)
    n, streams = 18, [torch.cuda.Stream() for _ in range(2)]
    qs, outs, lses, wss = buffers(pa, w, n)
    ref = serial(pa, w, qs)
    graphs = []
    for i in range(n):
        with torch.cuda.stream(streams[i % 2]):
            call = prepare(pa, w, qs[i], outs[i], lses[i], wss[i], stream=streams[i % 2])
            call()
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=streams[i % 2]):
                call()
            graphs.append(g)
    for rep in range(3):
        for t in outs + lses:
            t.fill_(float("nan"))
        for ws in wss[rep::3]:
            ws.random_(0, 256)
        torch.cuda.synchronize()
        for i, g in enumerate(graphs):
            with torch.cuda.stream(streams[i % 2]):
                g.replay()
        torch.cuda.synchronize()
        for i in range(n):
            assert torch.equal(outs[i], ref[i][0]) and torch.equal(lses[i], ref[i][1]), (rep, i)
        eager = prepare(pa, w, qs[rep], torch.empty_like(w.q), None, wss[rep])()
        torch.cuda.synchronize()
        assert torch.equal(eager, ref[rep][0])


@pytest.mark.parametrize("L,Hq,Hkv,d,one_launch", [(30000, 8, 1, 128, True), (300000, 8, 1, 128, False),
                                                   (600000, 8, 1, 64, False), (30000, 64, 1, 128, True),
                                                   (150000, 64, 1, 128, False), (20000, 32, 8, 128, True),
                                                   (150000, 8, 1, 256, True)])
def test_one_launch_takes_a_single_sequence_while_its_workgroups_shares_are_short(pa, L, Hq, Hkv, d, one_launch):
    """A (sequence, KV head) has at most 32 workgroups: with one KV head a long context belongs on the tile stream."""
    from paper_2506_07311_amd import binding
    w = W.make_workload("t", seq_lens=[L], num_q_heads=Hq, num_kv_heads=Hkv, head_dim=d, page_size=64,
                        dtype=torch.bfloat16, seed=304, device=DEV, poison=False, pool_factor=1.0)
    out = torch.empty_like(w.q)
    binding.pa_profile_reset()
    binding.pa_profile_enable(True)
    try:
        prepare(pa, w, w.q, out, None, buffers(pa, w, 1)[3][0])()
        torch.cuda.synchronize()
        assert binding.pa_profile_read("paged_decode_short_kernel")[0] == (1 if one_launch else 0)
        assert binding.pa_profile_read("paged_decode_mfma_kernel")[0] == (0 if one_launch else 1)
    finally:
        binding.pa_profile_enable(False)
        binding.pa_profile_reset()


@pytest.mark.parametrize("L,d,split", [(256, 128, False), (257, 128, True), (512, 64, False), (513, 64, True), (64, 256, False),
                                       (128, 256, True)])
def test_a_context_of_one_tile_a_wave_is_not_split(pa, L, d, split):
    """Two workgroups and their merge cost more than the one round of tiles they share: the workspace stays untouched."""
    w = W.make_workload("t", seq_lens=[L], num_q_heads=8, num_kv_heads=8, head_dim=d, page_size=16, dtype=torch.bfloat16,
                        seed=305, device=DEV)
    ws = buffers(pa, w, 1)[3][0]
    before = ws.clone()
    prepare(pa, w, w.q, torch.empty_like(w.q), None, ws)()
    assert torch.equal(ws, before) != split
