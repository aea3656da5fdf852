"""lorc_prefill_attention on the GPU against the fp64 oracle, and its consistency with the decode path."""
import numpy as np
import pytest

import lorc_inputs as gen
from lorc_testlib import GpuLayer, Problem, TOL, oracle_prefill, page_gather_indices, rel_err

pytestmark = pytest.mark.gpu

SHAPES = {
    "tiny_d64": dict(d_model=256, n_q_heads=4, n_kv_heads=2, head_dim=64, rank_k=32, rank_v=32,
                     rope_base=10000.0, ctx=[128], seed=10),
    "ragged_mid": dict(d_model=512, n_q_heads=8, n_kv_heads=2, head_dim=128, rank_k=64, rank_v=96,
                       rope_base=10000.0, ctx=[1, 70, 200, 64, 129], seed=11),
    "llama8b_short": dict(d_model=4096, n_q_heads=32, n_kv_heads=8, head_dim=128, rank_k=512, rank_v=512,
                          rope_base=500000.0, ctx=[300, 130], seed=12),
    # groupings that deal the workgroup's waves differently: one head x four query sub-blocks, and a group of three
    # (a pass of two heads, then a pass with one head and idle waves)
    "mha_ragged": dict(d_model=512, n_q_heads=4, n_kv_heads=4, head_dim=128, rank_k=96, rank_v=64,
                       rope_base=10000.0, ctx=[1, 33, 200, 290, 128], seed=14),
    "g3_d64": dict(d_model=256, n_q_heads=6, n_kv_heads=2, head_dim=64, rank_k=64, rank_v=32,
                   rope_base=10000.0, ctx=[97, 260], seed=15),
    "g8_rank768": dict(d_model=1024, n_q_heads=64, n_kv_heads=8, head_dim=128, rank_k=768, rank_v=640,
                       rope_base=500000.0, ctx=[150, 67], seed=13),
}


def make_queries(pb, seed):
    return [gen.queries(N, pb.n_q_heads, pb.head_dim, seed=seed + s) for s, N in enumerate(pb.ctx)]


@pytest.mark.parametrize("name", list(SHAPES))
def test_prefill_matches_oracle(name):
    pb = Problem(**SHAPES[name]).build()
    layer = GpuLayer(pb)
    layer.append_all()
    Q = make_queries(pb, 7000)
    got = layer.prefill(Q)
    ref = oracle_prefill(pb, Q)
    scale = max(np.max(np.abs(r)) for r in ref)
    worst = 0.0
    for g, r in zip(got, ref):
        assert g.shape == r.shape and np.all(np.isfinite(g))
        worst = max(worst, float(np.max(np.abs(g - r))) / scale)
    print(f"{name}: rel err {worst:.3e}")
    assert worst <= TOL


def test_last_prefill_row_equals_decode():
    """Row N-1 of the causal prefill is the decode step with ctx_len = N (same query)."""
    pb = Problem(**SHAPES["ragged_mid"]).build()
    layer = GpuLayer(pb)
    layer.append_all()
    Q = make_queries(pb, 7100)
    pb.q = np.stack([q[-1] for q in Q])
    pre = layer.prefill(Q)
    dec = layer.decode()
    last = np.stack([o[-1] for o in pre])
    assert rel_err(last, dec) <= 1e-2


# The rebuild launch picks its columns per workgroup (256 or 128) and its block order from the number of workgroups and of
# position tiles: each combination, with prompts that leave half of a two-page tile empty and column groups past the last
# head.
REBUILD = {
    "cols256_by_tile": dict(n_q_heads=8, n_kv_heads=8, head_dim=128, rank_k=64, rank_v=96, ctx=[1 + 7 * i % 70 for i in range(70)]),
    "cols256_by_column": dict(n_q_heads=10, n_kv_heads=10, head_dim=128, rank_k=96, rank_v=32, ctx=[1 + 11 * i % 67 for i in range(52)]),
    "cols128_by_column_d64": dict(n_q_heads=17, n_kv_heads=17, head_dim=64, rank_k=32, rank_v=64, ctx=[190, 64, 65, 129]),
    "cols128_by_tile_d64": dict(n_q_heads=5, n_kv_heads=5, head_dim=64, rank_k=64, rank_v=32, ctx=[63, 257]),
}


@pytest.mark.parametrize("name", list(REBUILD))
def test_rebuild_dispatch(name):
    shape = REBUILD[name]
    n = shape["n_kv_heads"] * shape["head_dim"]
    pb = Problem(d_model=(n + 63) // 64 * 64, rope_base=10000.0, seed=19, **shape).build()
    layer = GpuLayer(pb)
    layer.append_all()
    Q = make_queries(pb, 7200)
    ref = oracle_prefill(pb, Q)
    scale = max(np.max(np.abs(r)) for r in ref)
    worst = max(float(np.max(np.abs(g - r))) / scale for g, r in zip(layer.prefill(Q), ref))
    print(f"{name}: rel err {worst:.3e}")
    assert worst <= TOL


@pytest.mark.parametrize("head_dim", [64, 128])
def test_rotated_keys_are_rounded_once(head_dim):
    """With an identity as key factor the rebuilt keys are the latents themselves, and the scratch (1 KiB operand blocks of
    64 lanes x 8 fp16, see lorc_prefill.hip) holds them rotated and rounded to fp16.  An error e of the rotated key moves it to
    a neighbouring fp16 value with probability e / ulp, so the share of keys that are not the nearest fp16 value measures the
    rotation's error below the rounding: composed in fp32 from a base and an offset rotation, each within an ulp or two,
    6.4e-4 (errors of about 1e-6 of the larger coordinate, ulp 2^-11 to 2^-10); with one fp32 angle of up to 31 radians past
    the base in the hardware sine and cosine, 8.5e-4 (head_dim 64) and 7.9e-4 (128)."""
    import torch
    import paper_2410_03111_amd as L
    n, N, h_kv = 2 * head_dim, 8192, 2
    dev = torch.device("cuda:0")
    desc = L.layer_desc(256, 2, h_kv, head_dim, n, n, 10000.0)
    g = torch.Generator().manual_seed(5)
    eye = torch.eye(n, dtype=torch.bfloat16, device=dev)
    A = torch.randn(256, n, generator=g).mul_(0.1).to(dev, torch.bfloat16)
    x = torch.randn(N, 256, generator=g).to(dev, torch.bfloat16)
    i32 = lambda a: torch.as_tensor(a, dtype=torch.int32, device=dev)
    pages = (N + 63) // 64
    table = i32(np.random.default_rng(3).permutation(pages)).view(1, pages)
    cache = torch.zeros(pages * L.page_bytes(desc), dtype=torch.uint8, device=dev)
    packed = L.pack_factors(desc, A, A, eye, eye)
    L.append_latent(desc, x, packed, i32(np.zeros(N)), i32(np.arange(N)), table, cache)
    workspace = torch.zeros(L.prefill_workspace_bytes(desc, 1, N), dtype=torch.uint8, device=dev)
    q = torch.zeros(N, 2, head_dim, dtype=torch.bfloat16, device=dev)
    L.prefill_attention(desc, q, i32([0, N]), N, packed, cache, table, workspace=workspace)
    torch.cuda.synchronize()
    # latents as stored, then the keys in fp64
    idx = page_gather_indices(n, n)
    pool = cache.cpu().numpy().view(np.uint16).reshape(pages, -1)
    lat = np.concatenate([pool[p][idx] for p in table.cpu().numpy()[0]])[:N, :n]
    key = gen.bf16_to_f32(lat).astype(np.float64).reshape(N, h_kv, head_dim)
    half = head_dim // 2
    angle = np.arange(N)[:, None] * 10000.0 ** (-2.0 * np.arange(half) / head_dim)
    c, s = np.cos(angle)[:, None], np.sin(angle)[:, None]
    lo, hi = key[..., :half], key[..., half:]
    exact = np.concatenate([lo * c - hi * s, hi * c + lo * s], axis=-1).astype(np.float16)
    # scratch: [page][KV head][position block][16 coordinates][lane][element], behind a table of 64 doubles (512 bytes)
    raw = workspace.cpu().numpy()[512:512 + pages * 64 * n * 2].view(np.float16).reshape(pages, h_kv, 2, head_dim // 16, 2, 32, 8)
    e = np.arange(8)
    got = np.empty((pages * 64, h_kv, head_dim), np.float16)
    for u in range(head_dim // 16):
        for hf in range(2):
            coord = 16 * u + 8 * (e >> 2) + 4 * hf + (e & 3)
            got[:, :, coord] = raw[:, :, :, u, hf].transpose(0, 2, 3, 1, 4).reshape(pages * 64, h_kv, 8)
    got = got[:N]
    assert np.max(np.abs(got.astype(np.float64) - exact.astype(np.float64))) <= 2.0 ** -9 * np.max(np.abs(key))
    differ = float(np.mean(got != exact))
    print(f"head_dim {head_dim}: {differ:.2e} of the keys are not the nearest fp16 value")
    assert differ <= 7.1e-4


@pytest.mark.parametrize("n_q_heads,head_dim,plain", [(2, 64, False), (2, 128, False), (8, 128, False), (2, 128, True)])
@pytest.mark.parametrize("max_seqlen", [64, 150])
def test_sequences_longer_than_max_seqlen_stay_inside_their_scratch(n_q_heads, head_dim, plain, max_seqlen):
    """cu_seqlens lives on the device, max_seqlen on the host; where the first says more than the second (one and three pages:
    odd, so that half of the last two-page tile is no page of the sequence), the rows inside the pages of max_seqlen are right,
    the others untouched, and so is what follows the workspace."""
    import torch
    n = 2 * head_dim
    pb = Problem(d_model=256, n_q_heads=n_q_heads, n_kv_heads=2, head_dim=head_dim, rank_k=n if plain else 64,
                 rank_v=n if plain else 32, rope_base=10000.0, ctx=[330, 290], seed=31).build()
    layer = GpuLayer(pb, plain=plain)
    layer.append_all()
    L, dev = layer.L, layer.dev
    Q = make_queries(pb, 7300)
    full = layer.prefill(Q)
    pages = (max_seqlen + 63) // 64
    need = L.prefill_workspace_bytes(layer.desc, 2, max_seqlen)
    canary = 4 * 64 * n * 2 + 256
    buf = torch.full((need + canary,), 0x5A, dtype=torch.uint8, device=dev)
    q = torch.from_numpy(np.concatenate(Q, axis=0)).to(dev).to(torch.bfloat16).contiguous()
    out = torch.full_like(q, 77.0)
    cu = torch.tensor([0, 330, 620], dtype=torch.int32, device=dev)
    table = layer.block_table[:, :pages].contiguous()
    L.prefill_attention(layer.desc, q, cu, max_seqlen, layer.packed, layer.cache, table, out=out, workspace=buf[:need], plain=plain)
    torch.cuda.synchronize()
    assert bool((buf[need:] == 0x5A).all())
    o = out.float().cpu().numpy()
    for s, ref in enumerate(full):
        rows = o[330 * s:330 * s + pb.ctx[s]]
        assert rel_err(rows[:64 * pages], ref[:64 * pages]) <= 1e-2
        assert np.all(rows[64 * pages:] == 77.0)
