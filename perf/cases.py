"""Workloads that time this package through its public entry points.

A decode pass is what a serving loop does for one token of every sequence: per layer, the new tokens' hidden states are
down-projected into the paged latent cache (append_latent), then the queries attend to the cache.  A prefill pass is what
it does with new prompts: the prompts' hidden states are appended, then causal attention runs over them.  Packed factors,
page pool, block table, workspace and output buffer are what such a program keeps between passes.

Shapes are those of the paper's model table and of this repository's benchmark: the 8B layer (D 4096, 32 query / 8 KV
heads of 128), the 70B layer (D 8192, 64 / 8), the 13B layer (D 5120, 40 / 40) and the tiny layer of the smoke test.
Hidden states and queries are N(0, 1); cached latents follow the law of x A for such x: N(0, sigma_j^2) with the
power-law spectrum sigma_j ~ j^-0.7.
"""
from __future__ import annotations

import math

import torch

import lorc_inputs as gen
import paper_2410_03111_amd as lorc

PAGE = lorc.PAGE_TOKENS

SHAPES = {
    "tiny": dict(d_model=256, q_heads=4, kv_heads=2, head_dim=64, rope_base=10000.0),
    "8b": dict(d_model=4096, q_heads=32, kv_heads=8, head_dim=128, rope_base=500000.0),
    "70b": dict(d_model=8192, q_heads=64, kv_heads=8, head_dim=128, rope_base=500000.0),
    "13b": dict(d_model=5120, q_heads=40, kv_heads=40, head_dim=128, rope_base=10000.0),
}


def _case(kind, shape, rank_first, batch, context, *, rank_last=None, layers=1, ragged=False, name=None):
    """kind: "decode" (rotary, compressed), "decode_absorbed" (no rotation, key factor folded into the query),
    "decode_plain" (uncompressed layer), "prefill", "prefill_plain".  context: the longest sequence (decode) or prompt
    (prefill); ragged: the others are shorter, down to an eighth of it."""
    c = dict(kind=kind, shape=shape, rank_first=rank_first, rank_last=rank_first if rank_last is None else rank_last,
             layers=layers, batch=batch, context=context, ragged=ragged)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smoke test's layer: one short sequence, all latency
        _case("decode", "tiny", 32, 1, 128, name="decode_tiny"),
        # one interactive user of an 8B layer at half rank, an ordinary conversation length
        _case("decode", "8b", 512, 1, 1337, name="decode_8b_single_user"),
        # the headline decode step: sixteen users, 4096 positions each
        _case("decode", "8b", 512, 16, 4096, name="decode_8b_batch16"),
        # a step through the progressive-rank stack (768 -> 384), continuous batching: every user at another length
        _case("decode", "8b", 768, 32, 8192, rank_last=384, layers=8, ragged=True, name="decode_8b_rank_ramp"),
        # one layer of the 70B share with long contexts: the largest decode launch
        _case("decode", "70b", 512, 64, 32768, name="decode_70b_long"),
        # the 13B layer: multi-head attention, rank 2048
        _case("decode", "13b", 2048, 16, 4096, name="decode_13b_wide"),
        # a layer that the rank schedule leaves uncompressed
        _case("decode_plain", "8b", 1024, 16, 4096, name="decode_8b_uncompressed"),
        # a model without positional rotation: absorbed query
        _case("decode_absorbed", "8b", 512, 16, 4096, name="decode_8b_absorbed"),
        # the benchmark's prefill: four prompts of 8192 tokens
        _case("prefill", "8b", 512, 4, 8192, name="prefill_8b_4x8192"),
        # ordinary prompts that arrive together, none a multiple of anything
        _case("prefill", "8b", 576, 6, 777, ragged=True, name="prefill_8b_prompts"),
        # prompts of the 13B layer
        _case("prefill", "13b", 2048, 3, 1500, ragged=True, name="prefill_13b_prompts"),
        # a prompt of an uncompressed layer
        _case("prefill_plain", "8b", 1024, 2, 3001, name="prefill_8b_uncompressed"),
    ]


# ------------------------------------------------------------------------------------------------ sizes of a case
def _lengths(case):
    """Positions per sequence: the first has `context`; ragged ones are spread over [context / 8, context]."""
    n, out = case["context"], []
    for s in range(case["batch"]):
        short = 0.875 * ((s * 0.6180339887498949) % 1.0) if case["ragged"] else 0.0
        out.append(max(1, int(n * (1.0 - short))))
    return out


def _ranks(case):
    if case["layers"] == 1:
        return [case["rank_first"]]
    return gen.rank_ramp(case["layers"], case["rank_first"], case["rank_last"])


def work(case):
    """Latents, factors, tokens and queries read once, outputs and new latents written once.  Operations: the
    down-projection of the new tokens; per cached position the rank-r rebuild of its keys for all KV heads (not for
    uncompressed layers and absorbed queries; prefill rebuilds values as well), scores and weighted sum; the value
    up-projection of the outputs.  Causal attention counts the pairs j <= i."""
    sh = SHAPES[case["shape"]]
    D, hq, d = sh["d_model"], sh["q_heads"], sh["head_dim"]
    n = sh["kv_heads"] * d
    lens = _lengths(case)
    prefill, plain = case["kind"].startswith("prefill"), case["kind"].endswith("_plain")
    new = sum(lens) if prefill else case["batch"]
    positions = sum(lens)
    nbytes = flops = 0
    for r in _ranks(case):
        factors = 2 * D * r + (0 if plain else 2 * r * n)
        q_width = r if case["kind"] == "decode_absorbed" else d
        nbytes += 2 * (factors + new * (D + 2 * r + hq * (q_width + d)))
        flops += 2 * new * D * 2 * r
        if prefill:
            flops += 4 * hq * d * sum(L * (L + 1) // 2 for L in lens)
            if not plain:
                flops += 2 * positions * 2 * r * n
        else:
            nbytes += 2 * 2 * r * positions
            if plain:
                flops += 4 * hq * d * positions
            else:
                score_width = r if case["kind"] == "decode_absorbed" else d
                flops += 2 * hq * (score_width + r) * positions + 2 * case["batch"] * hq * r * d
                if case["kind"] == "decode":
                    flops += 2 * r * n * positions
    return {"bytes": nbytes, "flops": flops}


def draw(rng):
    largest = [max(v) for v in zip(*((w["bytes"], w["flops"]) for w in map(work, listed())))]
    log_int = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    kind = rng.choice(["decode"] * 5 + ["decode_plain", "decode_absorbed"] + ["prefill"] * 3 + ["prefill_plain"])
    layers = 1
    if kind == "decode":
        shape = rng.choice(["8b"] * 5 + ["70b", "70b", "13b", "tiny"])
    elif kind == "prefill":
        shape = rng.choice(["8b"] * 4 + ["13b", "tiny"])
    else:
        shape = "8b"
    rank = {"tiny": rng.choice([32, 64]), "8b": 32 * rng.randint(8, 24), "70b": 32 * rng.randint(12, 24),
            "13b": 32 * rng.randint(40, 64)}[shape]
    rank_last = rank
    if kind.endswith("_plain"):
        rank = rank_last = SHAPES[shape]["kv_heads"] * SHAPES[shape]["head_dim"]
    elif kind == "decode_absorbed":
        rank = rank_last = 32 * rng.randint(8, 16)
    elif kind == "decode" and shape == "8b" and rng.random() < 0.3:
        layers, rank_last = 4, max(256, rank - 128)
    batch = log_int(1, 8) if kind.startswith("prefill") else log_int(1, 64)
    context = log_int(16, 8192) if kind.startswith("prefill") else log_int(64, 32768)
    case = _case(kind, shape, rank, batch, context, rank_last=rank_last, layers=layers, ragged=rng.random() < 0.6)
    while any(w > m for w, m in zip((work(case)["bytes"], work(case)["flops"]), largest)):
        case["context"] = case["context"] * 3 // 4
    return case


# ------------------------------------------------------------------------------------------------ a pass
def _page_columns(r, keys):
    """Latent index of every element of a page's K (or V) part, in memory order (the tilings of include/lorc.h)."""
    j = torch.arange(r).view(1, r).expand(PAGE, r)
    t = torch.arange(PAGE).view(PAGE, 1).expand(PAGE, r)
    if keys:
        at = ((t // 32 * (r // 16) + j // 16) * 64 + t % 32 + 32 * (j % 16 // 8)) * 8 + j % 8
    else:
        at = ((j // 32 * 4 + t // 16) * 64 + j % 32 + 32 * (t % 16 // 8)) * 8 + t % 8
    out = torch.empty(PAGE * r, dtype=torch.int64)
    out[at.reshape(-1)] = j.reshape(-1)
    return out


def prepare(case, seed):
    dev = torch.device("cuda")
    rng = torch.Generator(device=dev).manual_seed(1000003 * (seed + 1))
    normal = lambda *shape: torch.empty(*shape, dtype=torch.bfloat16, device=dev).normal_(generator=rng)
    i32 = lambda v: torch.tensor(v, dtype=torch.int32, device=dev)
    kind, batch, lens = case["kind"], case["batch"], _lengths(case)
    prefill, plain, absorbed = kind.startswith("prefill"), kind.endswith("_plain"), kind == "decode_absorbed"
    sh = SHAPES[case["shape"]]
    D, hq, hkv, d = sh["d_model"], sh["q_heads"], sh["kv_heads"], sh["head_dim"]
    n = hkv * d
    sigma = torch.from_numpy(gen.power_law_spectrum(n)).to(dev, torch.float32)

    max_pages = (max(lens) + PAGE - 1) // PAGE
    n_pages = batch * max_pages + 3
    table = torch.randperm(n_pages, generator=torch.Generator().manual_seed(seed + 17))[:batch * max_pages]
    st = dict(kind=kind, max_len=max(lens), block_table=table.to(torch.int32).view(batch, max_pages).to(dev), layers=[])
    if prefill:
        st["slot_seq"] = torch.repeat_interleave(torch.arange(batch), torch.tensor(lens)).to(torch.int32).to(dev)
        st["slot_pos"] = torch.cat([torch.arange(L) for L in lens]).to(torch.int32).to(dev)
        st["cu_seqlens"] = i32([0] + list(torch.tensor(lens).cumsum(0)))
    else:
        st["slot_seq"], st["slot_pos"] = i32(list(range(batch))), i32([L - 1 for L in lens])
        st["ctx_len"] = i32(lens)
    tokens = sum(lens) if prefill else batch

    workspace_bytes = 256
    for r in _ranks(case):
        desc = lorc.layer_desc(D, hq, hkv, d, r, r, sh["rope_base"])
        a_scale = (sigma[:r] / math.sqrt(D)).view(1, r)
        A = [torch.randn(D, r, generator=rng, device=dev).mul_(a_scale).to(torch.bfloat16) for _ in range(2)]
        B = [None, None] if plain else [torch.randn(r, n, generator=rng, device=dev).mul_(1 / math.sqrt(n)).to(torch.bfloat16) for _ in range(2)]
        scale = torch.cat([sigma[_page_columns(r, keys).to(dev)] for keys in (True, False)]).to(torch.bfloat16)
        cache = normal(n_pages, scale.numel()).mul_(scale).view(-1).view(torch.uint8)
        q = normal(tokens, hq, d)
        if absorbed:
            per_head = B[0].float().view(r, hkv, d).permute(1, 2, 0).contiguous()
            q = torch.matmul(q.float().view(batch, hkv, hq // hkv, d), per_head).view(batch, hq, r).to(torch.bfloat16).contiguous()
        st["layers"].append(dict(desc=desc, packed=lorc.pack_factors(desc, A[0], A[1], B[0], B[1]), cache=cache, q=q,
                                 x=normal(tokens, D), out=torch.empty(tokens, hq, d, dtype=torch.bfloat16, device=dev)))
        if prefill:
            need = lorc.prefill_workspace_bytes(desc, batch, max(lens))
        else:
            size = (lorc.decode_plain_workspace_bytes if plain else
                    lorc.decode_absorbed_workspace_bytes if absorbed else lorc.decode_workspace_bytes)
            need = size(desc, batch, max(lens))
        workspace_bytes = max(workspace_bytes, need)
    st["workspace"] = torch.empty(workspace_bytes, dtype=torch.uint8, device=dev)
    return st


def run(st):
    kind, table, ws, longest = st["kind"], st["block_table"], st["workspace"], st["max_len"]
    for l in st["layers"]:
        desc, packed, cache, q, out = l["desc"], l["packed"], l["cache"], l["q"], l["out"]
        lorc.append_latent(desc, l["x"], packed, st["slot_seq"], st["slot_pos"], table, cache)
        if kind.startswith("prefill"):
            lorc.prefill_attention(desc, q, st["cu_seqlens"], longest, packed, cache, table, out=out, workspace=ws,
                                   plain=kind == "prefill_plain")
        elif kind == "decode_absorbed":
            lorc.decode_attention_absorbed(desc, q, st["ctx_len"], longest, packed, cache, table, out=out, workspace=ws)
        else:
            attend = lorc.decode_attention_plain if kind == "decode_plain" else lorc.decode_attention
            attend(desc, q, st["slot_pos"], st["ctx_len"], longest, packed, cache, table, out=out, workspace=ws)
    return {"out": [l["out"] for l in st["layers"]], "cache": [l["cache"].view(torch.bfloat16) for l in st["layers"]]}


def tolerance(case):
    """Outputs and latents are stored as bf16 (rounding alone: 1.7e-3 in the 2-norm); keys pass through fp16 and softmax
    weights through bf16 or fp16 on the way.  Measured against the same path in fp64 on the same latents, factors and
    queries: outputs 1.7e-3 (prefill) to 2.3e-3 (decode), new latents 1.2e-3 to 2.3e-3."""
    return {"rel": 9e-3, "max": 0.1}
