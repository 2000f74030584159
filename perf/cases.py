"""The workloads this library is timed on, each as a user's program calls it: a decode step (`paged_decode_step`) or a
prompt / chunk (`paged_kv_append` followed by `paged_attention_prefill[_mod]`) over pools, block tables and buffers
that the program already holds, with the arguments marshalled once as in a serving loop.

A case is a dict of plain values:
    kind        "decode" (one new token per sequence) or "prefill" (ragged packed queries, causal)
    dtype       "bf16", "fp16" or "fp32" pools
    batch, lo, hi, lens_seed   sequences; context lengths log-uniform in [lo, hi] (counting the call's own tokens)
    new         prefill: tokens each sequence brings (0 = its whole prompt); `every` = n: only each n-th sequence
                brings `new` tokens, the others decode one
    hq, hkv, d, page           query heads, KV heads, head_dim, tokens per page
    share       tokens of prefix that groups of eight sequences map to the same pages (0 = none)
    window, softcap, alibi, doc   mask / score hooks (0 = off); doc = tokens per packed document
Page tables are random permutations of a pool with twice the pages in use.
"""
import math
import random

import numpy as np
import torch

import paper_2506_07311_amd as pa

DEVICE = "cuda:0"
TORCH = {"bf16": torch.bfloat16, "fp16": torch.float16, "fp32": torch.float32}
BASE = dict(kind="decode", dtype="bf16", batch=1, lo=2048, hi=2048, lens_seed=0, new=0, every=0, hq=32, hkv=8, d=128,
            page=16, share=0, window=0, softcap=0.0, alibi=False, doc=0)


def _case(name=None, **kw):
    c = dict(BASE, **kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest step: one fp32 sequence of 128 tokens, launch and latency only.
        _case("decode_fp32_1x128", dtype="fp32", batch=1, lo=128, hi=128, hq=8, hkv=8, d=64),
        # Interactive serving: eight chats of 128 to 2048 tokens, lengths as they come.
        _case("decode_8x128to2048", batch=8, lo=128, hi=2048, lens_seed=1),
        # One user on a 32-head layer without grouping, fp16 pools with 64-token pages, at the end of a 2048-token chat.
        _case("decode_fp16_mha_1x2048", dtype="fp16", batch=1, hkv=32, page=64),
        # A busy server: 64 sequences of 64 to 32768 tokens whose groups of eight share a 1024-token system prompt.
        _case("decode_64_mixed", batch=64, lo=64, hi=32768, lens_seed=4, share=1024),
        # Long documents: 16 sequences of 131072 tokens, 8.6 GB of K and V per step.
        _case("decode_16x131072", batch=16, lo=131072, hi=131072, hq=64),
        # A batch of prompts on arrival.
        _case("prefill_4x2048", kind="prefill", batch=4),
        # One user's prompt on the 32-head layer (time to first token).
        _case("prompt_fp16_mha_1x2048", kind="prefill", dtype="fp16", batch=1, hkv=32, page=64),
        # A chat that grows: the next 1024 tokens of a 32768-token context.
        _case("prefill_chunk_1k_of_32k", kind="prefill", batch=1, lo=32768, hi=32768, new=1024),
        # Continuous batching: four 512-token chunks ride along with sixty decoding sequences in one call.
        _case("jagged_60_decode_4_chunks", kind="prefill", batch=64, lo=64, hi=32768, lens_seed=4, new=512, every=16),
        # A local-attention layer: head_dim 256, sliding window and soft-capped scores.
        _case("prefill_d256_window_softcap", kind="prefill", batch=2, lo=2000, hi=4000, lens_seed=3, hq=16, hkv=8, d=256,
              page=32, window=1024, softcap=50.0),
        # A model whose head_dim is not a power of two, odd prompt lengths.
        _case("prefill_d96_2x1000", kind="prefill", batch=2, lo=600, hi=1100, lens_seed=7, hq=32, hkv=32, d=96),
        # Full precision: the prompt in front of fp32 decode.
        _case("prompt_fp32_1x777", kind="prefill", dtype="fp32", batch=1, lo=777, hi=777, hq=8, hkv=8, d=64),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another case of the ranges above."""
    c = _case(lens_seed=rng.randrange(1 << 20))
    family = rng.choice(["decode", "decode", "decode_mixed", "decode_fp32", "prompts", "prompts", "chunk", "jagged",
                         "hooks", "odd_dim", "prompt_fp32"])
    c["dtype"] = rng.choice(["bf16", "bf16", "fp16"])
    c["hq"], c["hkv"] = rng.choice([(32, 8), (32, 8), (32, 32), (64, 8), (8, 1)])
    c["d"] = rng.choice([128, 128, 128, 64, 256])
    c["page"] = rng.choice([16, 16, 32, 64, 128])
    row = 4 * c["hkv"] * c["d"]                                   # bytes of one token's K and V at 16 bits
    if family == "decode":                                        # a few short chats up to long documents
        c["lo"] = c["hi"] = _log(rng, 100, 131072)
        if rng.random() < 0.5:
            c["lo"] = max(64, c["hi"] // rng.choice([2, 8, 30]))
        c["batch"] = max(1, min(_log(rng, 1, 64), int(4e9 // (row * c["hi"]))))
    elif family == "decode_mixed":
        c.update(lo=64, hi=_log(rng, 4096, 32768), share=rng.choice([0, 512, 1024]), d=128, hq=32, hkv=8,
                 batch=rng.randint(16, 64))
    elif family == "decode_fp32":
        c.update(dtype="fp32", batch=_log(rng, 1, 8), d=rng.choice([64, 64, 128]), page=16)
        c["hq"], c["hkv"] = rng.choice([(8, 8), (32, 8)])
        c["lo"] = c["hi"] = _log(rng, 16, 2048)
    else:
        c["kind"] = "prefill"
        if family == "prompts":                                   # single prompts and batches of them
            c["hi"] = _log(rng, 100, 4096)
            c["lo"] = c["hi"] if rng.random() < 0.5 else max(33, c["hi"] // 3)
            c["batch"] = max(1, min(rng.choice([1, 1, 2, 4, 8, 16]), 8192 // c["hi"]))
        elif family == "chunk":
            c.update(lo=_log(rng, 4096, 32768), new=rng.choice([128, 256, 500, 512, 1000, 1024]), batch=rng.choice([1, 1, 2]))
            c["hi"] = c["lo"]
        elif family == "jagged":
            c.update(lo=64, hi=_log(rng, 4096, 32768), batch=rng.randint(16, 64), new=rng.choice([200, 512]),
                     every=rng.choice([8, 16]), hq=32, hkv=8, d=128)
        elif family == "hooks":
            c.update(lo=_log(rng, 300, 1500), batch=rng.choice([1, 2, 4]))
            c["hi"] = 2 * c["lo"]
            hook = rng.choice(["window", "softcap", "both", "alibi", "doc"])
            c["window"] = rng.choice([256, 1000, 1024]) if hook in ("window", "both") else 0
            c["softcap"] = rng.choice([30.0, 50.0]) if hook in ("softcap", "both") else 0.0
            c["alibi"], c["doc"] = hook == "alibi", 300 if hook == "doc" else 0
        elif family == "odd_dim":
            c["d"] = rng.choice([80, 96, 112])
            c.update(lo=_log(rng, 100, 1000), batch=rng.choice([1, 2]))
            c["hi"] = c["lo"]
            if rng.random() < 0.4:
                c.update(kind="decode", batch=rng.randint(1, 8))
        else:
            c.update(dtype="fp32", batch=1, d=rng.choice([64, 64, 128]), page=16, lo=_log(rng, 64, 777))
            c["hq"], c["hkv"] = rng.choice([(8, 8), (8, 2)])
            c["hi"] = c["lo"]
    return c


def _lengths(case):
    """(context lengths, query lengths) of the case's sequences; the same for every seed."""
    rng = random.Random(900 + case["lens_seed"])
    lens = [_log(rng, case["lo"], case["hi"]) for _ in range(case["batch"])]
    if case["kind"] == "decode":
        return lens, [1] * len(lens)
    q = []
    for s, n in enumerate(lens):
        if case["every"] and s % case["every"] != case["every"] // 3:
            q.append(1)
        else:
            q.append(min(n, case["new"]) if case["new"] else n)
    return lens, q


def _randn(shape, dtype, gen):
    """N(0, 1) in the storage type, drawn in pieces so that no fp32 copy of a large pool exists."""
    out = torch.empty(shape, dtype=dtype, device=DEVICE)
    step = max(1, (1 << 28) // max(1, math.prod(shape[1:])))
    for i in range(0, shape[0], step):
        out[i:i + step] = torch.randn((min(step, shape[0] - i),) + tuple(shape[1:]), generator=gen, device=DEVICE)
    return out


def _inputs(case, seed):
    """Pools, tables and tokens of one call, plain torch and numpy."""
    lens, q_lens = _lengths(case)
    dtype, P, hkv, d = TORCH[case["dtype"]], case["page"], case["hkv"], case["d"]
    blocks = [-(-n // P) for n in lens]
    table = np.full((len(lens), max(blocks)), -1, dtype=np.int32)
    perm = np.random.default_rng(seed).permutation(2 * sum(blocks)).astype(np.int32)
    at = 0
    for s, nb in enumerate(blocks):
        shared = 0
        head = s - s % 8
        if case["share"] and s != head:                           # whole pages, never the page a token is appended to
            shared = min(case["share"], lens[s] - 1, lens[head] - 1) // P
            table[s, :shared] = table[head, :shared]
        table[s, shared:nb] = perm[at:at + nb - shared]
        at += nb - shared
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    pool = (len(perm), P, hkv, d)
    t = dict(k_cache=_randn(pool, dtype, gen), v_cache=_randn(pool, dtype, gen))
    n = sum(q_lens)
    t["q"] = _randn((n, case["hq"], d), dtype, gen)
    t["k_new"], t["v_new"] = _randn((n, hkv, d), dtype, gen), _randn((n, hkv, d), dtype, gen)
    if case["doc"]:                                               # packed documents, lengths about `doc`
        cut = np.random.default_rng(seed + 1).random((len(lens), max(lens))) < 1.0 / case["doc"]
        t["doc_ids"] = torch.from_numpy(np.cumsum(cut, axis=1, dtype=np.int32)).to(DEVICE)
    if case["alibi"]:
        t["alibi_slopes"] = torch.exp2(-8.0 * torch.arange(1, case["hq"] + 1, device=DEVICE) / case["hq"])

    def ints(x):
        return torch.tensor(x, dtype=torch.int32, device=DEVICE)

    t["block_table"] = torch.from_numpy(table).to(DEVICE)
    t["seq_lens"] = ints(lens)
    t["cu_q_lens"] = ints([0] + np.cumsum(q_lens).tolist())
    t["seq_ids"] = ints(np.repeat(np.arange(len(lens)), q_lens))
    t["positions"] = ints(np.concatenate([np.arange(a - b, a) for a, b in zip(lens, q_lens)]))
    return t


def prepare(case, seed):
    t = _inputs(case, seed)
    lens, q_lens = _lengths(case)
    n = sum(q_lens)
    out = torch.empty_like(t["q"])
    lse = torch.empty((n, case["hq"]), dtype=torch.float32, device=DEVICE)
    workspace = torch.empty(pa.paged_attention_workspace_bytes(len(lens), case["hq"], case["d"], n, max(lens)),
                            dtype=torch.uint8, device=DEVICE)
    scale = case["d"] ** -0.5
    k, v = t["k_cache"], t["v_cache"]
    hooks = dict(window=case["window"], softcap=case["softcap"], alibi_slopes=t.get("alibi_slopes"),
                 doc_ids=t.get("doc_ids"))
    if case["kind"] == "decode":
        calls = [pa.prepare_decode_step(k, v, t["k_new"], t["v_new"], t["q"], t["block_table"], t["seq_lens"], max(lens),
                                        scale, out=out, lse=lse, workspace=workspace, **hooks)]
    else:
        calls = [pa.prepare_kv_append(k, v, t["k_new"], t["v_new"], t["seq_ids"], t["positions"], t["block_table"])]
        args = (k, v, t["q"], t["cu_q_lens"], max(q_lens), t["block_table"], t["seq_lens"], max(lens), scale, True)
        keep = dict(out=out, lse=lse, workspace=workspace)
        if any(case[h] for h in ("window", "softcap", "alibi", "doc")):
            calls.append(lambda: pa.paged_attention_prefill_mod(*args, **keep, **hooks))
        else:
            calls.append(pa.prepare_prefill(*args, **keep))
    # the pools are the call's updated state; the two large ones would take longer to look at than to make
    pools = (k, v) if k.numel() <= 1 << 28 else ()
    return dict(calls=calls, outputs=(out, lse) + pools)


def run(state):
    for call in state["calls"]:
        call()
    return state["outputs"]


def _visible(case, n, nq):
    """(query, key) pairs and keys that one sequence's queries see."""
    w = case["window"] or n
    i = np.arange(n - nq, n, dtype=np.int64)
    per = np.minimum(i + 1, w)
    if case["doc"]:
        per = np.minimum(per, case["doc"])
    return int(per.sum()), min(n, nq - 1 + w)


def work(case):
    lens, q_lens = _lengths(case)
    e = 4 if case["dtype"] == "fp32" else 2
    pairs = keys = 0
    for s, (n, nq) in enumerate(zip(lens, q_lens)):
        p, k = _visible(case, n, nq)
        pairs += p
        head = lens[s - s % 8]
        shared = min(case["share"], n - 1, head - 1) // case["page"] * case["page"] if s % 8 else 0
        keys += max(0, k - shared)                                # a shared prefix is read once
    rows = sum(q_lens)
    kv = 2 * case["hkv"] * case["d"] * e
    return {"bytes": keys * kv + rows * (kv + 2 * case["hq"] * case["d"] * e + 4 * case["hq"]) + 4 * rows,
            "flops": 4 * case["d"] * case["hq"] * pairs}


def tolerance(case):
    # about four times the largest error against exact() over the listed and fourteen drawn cases (rel / max):
    # bf16 2.4e-3 / 1.1e-2, fp16 2.3e-4 / 1.4e-3, fp32 2.4e-7 / 1.1e-6
    return {"bf16": {"rel": 1e-2, "max": 5e-2}, "fp16": {"rel": 1e-3, "max": 6e-3},
            "fp32": {"rel": 1e-6, "max": 5e-6}}[case["dtype"]]


def exact(case, seed):
    """Attention over the gathered pages in 64 bits; the pools themselves are copies, not computed numbers."""
    t = _inputs(case, seed)
    lens, q_lens = _lengths(case)
    hq, hkv, d, P = case["hq"], case["hkv"], case["d"], case["page"]
    G = hq // hkv
    out = torch.zeros((sum(q_lens), hq, d), dtype=torch.float64, device=DEVICE)
    lse = torch.zeros((sum(q_lens), hq), dtype=torch.float64, device=DEVICE)
    row = 0
    for s, (n, nq) in enumerate(zip(lens, q_lens)):
        pages = t["block_table"][s, :-(-n // P)].long()
        new = slice(row, row + nq)
        pos = torch.arange(n - nq, n, device=DEVICE)[:, None]
        j = torch.arange(n, device=DEVICE)[None, :]
        hidden = j > pos
        if case["window"]:
            hidden |= j <= pos - case["window"]
        if case["doc"]:
            ids = t["doc_ids"][s, :n]
            hidden |= ids[None, :] != ids[n - nq:, None]
        for g in range(hkv):
            k = t["k_cache"][pages, :, g].reshape(-1, d)[:n].double()
            v = t["v_cache"][pages, :, g].reshape(-1, d)[:n].double()
            k[n - nq:], v[n - nq:] = t["k_new"][new, g].double(), t["v_new"][new, g].double()
            kt = k.t().contiguous()
            for h in range(g * G, (g + 1) * G):
                x = t["q"][new, h].double() @ kt * d ** -0.5
                if case["softcap"]:
                    x = case["softcap"] * torch.tanh(x / case["softcap"])
                if case["alibi"]:
                    x += t["alibi_slopes"][h].double() * (j - pos)
                x.masked_fill_(hidden, -math.inf)
                lse[new, h] = torch.logsumexp(x, dim=1)
                out[new, h] = torch.exp(x - lse[new, h][:, None]) @ v
        row += nq
    return (out, lse) + ((None, None) if t["k_cache"].numel() <= 1 << 28 else ())
