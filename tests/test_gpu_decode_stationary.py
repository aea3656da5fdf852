"""Parity of the decode path on the shapes that take the split kernel with the key factor held in registers
(head_dim 128, an even number of KV heads, G <= 8, 384 < rank_k <= 512, rank_v <= 512): query-group sizes 1 .. 8, ranks
that are not a multiple of 128 (padded k-steps), ragged and empty contexts, many tiles per split, many splits, pages
that are not cached, shifted and long positions.  Model widths are small so that the fp64 oracle stays cheap."""
import numpy as np
import pytest

import lorc_inputs as gen
from lorc_testlib import GpuLayer, LatentLayer, Problem, TOL, oracle_decode, rel_err
from oracle import lorc_oracle as orc

pytestmark = pytest.mark.gpu

SHAPES = {
    "g4_rank512": dict(n_q_heads=16, n_kv_heads=4, rank_k=512, rank_v=512, ctx=[700, 64, 1, 129]),
    "g8_rank448_416": dict(n_q_heads=32, n_kv_heads=4, rank_k=448, rank_v=416, ctx=[300, 1000]),
    "g1_rank416_v32": dict(n_q_heads=4, n_kv_heads=4, rank_k=416, rank_v=32, ctx=[200, 65]),
    "g2_rank480_empty_and_long": dict(n_q_heads=8, n_kv_heads=4, rank_k=480, rank_v=512, ctx=[0, 2500, 63]),
    "six_kv_heads_rank416": dict(n_q_heads=12, n_kv_heads=6, rank_k=416, rank_v=96, ctx=[1300]),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_stationary_shapes_match_oracle(name):
    shape = dict(SHAPES[name])
    n = shape["n_kv_heads"] * 128
    pb = Problem(d_model=max(512, n), head_dim=128, rope_base=500000.0, seed=61 + len(name), **shape).build()
    layer = GpuLayer(pb)
    layer.append_all()
    got = layer.decode()
    ref = oracle_decode(pb)
    assert np.all(np.isfinite(got))
    for s, N in enumerate(pb.ctx):
        if N == 0:
            assert np.all(got[s] == 0.0)
    live = [s for s, N in enumerate(pb.ctx) if N > 0]
    err = rel_err(got[live], ref[live])
    print(f"{name}: rel err {err:.3e}")
    assert err <= TOL


def test_stationary_unmapped_page_and_shifted_query_positions():
    import torch
    pb = Problem(d_model=512, n_q_heads=16, n_kv_heads=4, head_dim=128, rank_k=512, rank_v=448, rope_base=500000.0,
                 ctx=[330, 200], seed=71).build()
    layer = GpuLayer(pb)
    bt = layer.block_table_np.copy()
    bt[0, 1] = -1                      # positions 64 .. 127 of sequence 0
    bt[0, 4] = layer.n_pages + 9       # positions 256 .. 319
    bt[1, 0] = -7                      # the first tile of sequence 1
    layer.block_table_np = bt
    layer.block_table = torch.from_numpy(bt).to(layer.dev)
    layer.append_all()
    q_pos = [1000, 199]
    got = layer.decode(q_pos=q_pos)
    X = [x.copy() for x in pb.X]
    X[0][64:128] = 0.0
    X[0][256:320] = 0.0
    X[1][0:64] = 0.0
    ref = oracle_decode(Problem(**{**pb.__dict__, "X": X}), q_pos=q_pos)
    assert np.all(np.isfinite(got))
    err = rel_err(got, ref)
    print(f"unmapped pages, shifted query: rel err {err:.3e}")
    assert err <= TOL


def test_stationary_wide_batch_walks_many_tiles_per_workgroup():
    """A batch wide enough that the plan gives every workgroup a long walk (few context splits), ragged lengths."""
    ctx = [1500 - 37 * (s % 9) for s in range(48)]
    pb = Problem(d_model=512, n_q_heads=16, n_kv_heads=4, head_dim=128, rank_k=512, rank_v=512, rope_base=500000.0,
                 ctx=ctx, seed=74).build()
    layer = GpuLayer(pb)
    layer.append_all()
    got = layer.decode()
    sample = [0, 7, 23, 47]
    ref = oracle_decode(pb, seqs=sample)
    err = rel_err(got[sample], ref)
    print(f"wide batch: rel err {err:.3e}")
    assert np.all(np.isfinite(got)) and err <= TOL


def test_stationary_long_positions():
    """20000 positions of one sequence (many context splits of several tiles), angles up to 3e4 rad at base 500000."""
    pb = Problem(d_model=512, n_q_heads=16, n_kv_heads=4, head_dim=128, rank_k=448, rank_v=448, rope_base=500000.0,
                 ctx=[20000, 777], seed=72).build()
    layer = GpuLayer(pb)
    layer.append_all()
    q_pos = [33000, 776]
    got = layer.decode(q_pos=q_pos)
    ref = oracle_decode(pb, q_pos=q_pos)
    err = [rel_err(got[s], ref[s]) for s in range(2)]
    print(f"long walk: rel err {err[0]:.3e}, {err[1]:.3e}")
    assert max(err) <= TOL


def test_stationary_latent_output_matches_full_output():
    """The latent-space entry point shares the split kernel: o_lat B_v must reproduce the full output."""
    import torch
    pb = Problem(d_model=512, n_q_heads=16, n_kv_heads=4, head_dim=128, rank_k=512, rank_v=512, rope_base=10000.0,
                 ctx=[400, 100], seed=73).build()
    layer = GpuLayer(pb)
    layer.append_all()
    L, dev = layer.L, layer.dev
    q = torch.from_numpy(pb.q).to(dev).to(torch.bfloat16).contiguous()
    qp = torch.tensor([n - 1 for n in pb.ctx], dtype=torch.int32, device=dev)
    cl = torch.tensor(pb.ctx, dtype=torch.int32, device=dev)
    o_lat = L.decode_attention_latent(layer.desc, q, qp, cl, max(pb.ctx), layer.packed, layer.cache, layer.block_table)
    torch.cuda.synchronize()
    o_lat = o_lat.float().cpu().numpy().astype(np.float64)
    B_v = layer.dB_v.float().cpu().numpy().astype(np.float64)
    G, d = pb.n_q_heads // pb.n_kv_heads, pb.head_dim
    got = np.stack([np.stack([o_lat[s, h] @ B_v[:, (h // G) * d:(h // G + 1) * d] for h in range(pb.n_q_heads)])
                    for s in range(len(pb.ctx))])
    assert rel_err(got, oracle_decode(pb)) <= TOL


def _latents(shape, seed):
    """A LatentLayer of random latents (falling spectrum), bf16."""
    h_q, h_kv, r_k, r_v, ctx = shape
    rng = np.random.default_rng(seed)
    bf = lambda a: gen.bf16_round(a.astype(np.float32))
    fall = lambda r: (1.0 + np.arange(r)) ** -0.7
    C_k, C_v = ([bf(rng.standard_normal((n, r)) * fall(r) * 4.0) for n in ctx] for r in (r_k, r_v))
    B_k, B_v = (bf(rng.standard_normal((r, h_kv * 128)) / np.sqrt(r)) for r in (r_k, r_v))
    return C_k, C_v, B_k, B_v, bf(rng.standard_normal((len(ctx), h_q, 128)))


def _decode_in_one_split(layer, q, q_pos):
    """With room for one split per sequence only: one workgroup walks all the tiles of a sequence."""
    import torch
    h_q, r_v = layer.h_q, layer.B_v.shape[0]
    b, longest = len(layer.ctx), max(layer.ctx)
    need = b * h_q * (8 + 2 * r_v) + 512
    assert layer.L.decode_kernel_info(layer.desc, b, longest, need)[1] == 1
    ws = torch.empty(need, dtype=torch.uint8, device=layer.dev)
    args = layer.tensors(q, q_pos)
    return layer.L.decode_attention(layer.desc, *args, longest, layer.packed, layer.cache, layer.block_table,
                                    workspace=ws).float().cpu().numpy().astype(np.float64)


WIDE_SHAPES = [(24, 6, 544, 544), (18, 6, 768, 768), (6, 6, 704, 768), (12, 6, 640, 32), (48, 6, 640, 672), (30, 6, 576, 544), (16, 4, 512, 416)]


@pytest.mark.parametrize("h_q,h_kv,r_k,r_v", WIDE_SHAPES)
def test_stationary_pages_not_cached_and_query_positions(h_q, h_kv, r_k, r_v):
    """Pages that are not cached at the start, inside and at the end of a walk (zero latents: score 0, value 0), queries behind and beyond
    the context; NaN wherever nothing is cached.  In splits of one page and in one walk."""
    import torch
    ctx = [330, 200, 100]
    C_k, C_v, B_k, B_v, q = _latents((h_q, h_kv, r_k, r_v, ctx), seed=r_k + h_q)
    layer = LatentLayer(h_q, h_kv, 128, C_k, C_v, B_k, B_v, rope_base=10000.0)
    table = layer.block_table.cpu().numpy().copy()
    for s, page, value in ((0, 1, -1), (0, 2, layer.n_pages + 9), (0, 4, -3), (1, 0, -7), (2, 1, -1)):
        table[s, page] = value
        layer.C_k[s], layer.C_v[s] = layer.C_k[s].copy(), layer.C_v[s].copy()
        layer.C_k[s][64 * page:64 * page + 64] = 0.0
        layer.C_v[s][64 * page:64 * page + 64] = 0.0
    layer.block_table = torch.from_numpy(table).to(layer.dev)
    q_pos = [1000, 199, 20]
    ref = layer.oracle(q, q_pos)
    for got in (layer.decode(q, q_pos), _decode_in_one_split(layer, q, q_pos)):
        assert np.all(np.isfinite(got))
        assert rel_err(got, ref) <= TOL


@pytest.mark.parametrize("h_q,h_kv,r_k,r_v", WIDE_SHAPES + [(32, 4, 160, 160)])
def test_stationary_tiles_far_below_and_above_earlier_ones(h_q, h_kv, r_k, r_v):
    """Scores that are the same within 32 positions and jump by up to 90 (log2) between them, in one walk: the reference falls behind the
    largest by no more than 2^24 and rises again.  Whole numbers in fp16: exact scores; what is left is the rounding of the outputs and of
    the partials (bf16, fp16)."""
    n = 13 * 32 + 9
    levels = np.array([0, -40, -80, -23, -26, 2, 10, -60, 10, 11, -12, -90, 8, -20], float)
    rng = np.random.default_rng(11)
    C_k, B_k = np.zeros((n, r_k)), np.zeros((r_k, h_kv * 128))
    C_k[:, 0] = np.repeat(levels, 32)[:n]
    B_k[0, 63::128] = 1.0                       # the slowest rotation: none at this base
    C_v, B_v = gen.bf16_round(rng.standard_normal((n, r_v)).astype(np.float32)), np.zeros((r_v, h_kv * 128))
    B_v[np.arange(h_kv * 128) % r_v, np.arange(h_kv * 128)] = 1.0
    layer = LatentLayer(h_q, h_kv, 128, [C_k], [C_v], B_k, B_v, rope_base=1e12, softmax_scale=float(np.log(2.0)))
    q = np.zeros((1, h_q, 128))
    q[:, :, 63] = 1.0
    ref = layer.oracle(q)
    for got in (_decode_in_one_split(layer, q, None), layer.decode(q)):
        assert float(np.max(np.abs(got - ref)) / np.max(np.abs(ref))) <= 2 ** -8


@pytest.mark.parametrize("h_q,h_kv,r_k,r_v,ctx", [(24, 6, 544, 544, [400, 100]), (18, 6, 768, 768, [300, 0, 65]), (48, 6, 640, 672, [150]),
                                                  (16, 8, 96, 1024, [150, 400]), (8, 8, 96, 640, [200]), (40, 8, 96, 992, [90, 300])])
def test_latent_output_of_wide_values_matches_the_oracle(h_q, h_kv, r_k, r_v, ctx):
    """The merge that stops before the up-projection, value ranks 544 to 1024: o_lat B_v reproduces the outputs."""
    C_k, C_v, B_k, B_v, q = _latents((h_q, h_kv, r_k, r_v, ctx), seed=r_v)
    layer = LatentLayer(h_q, h_kv, 128, C_k, C_v, B_k, B_v, rope_base=10000.0)
    o_lat = layer.decode(q, latent=True)
    G = h_q // h_kv
    live = [s for s, n in enumerate(ctx) if n > 0]
    assert all(np.all(o_lat[s] == 0.0) for s, n in enumerate(ctx) if n == 0)
    got = np.stack([[o_lat[s, h] @ B_v[:, h // G * 128:h // G * 128 + 128].astype(np.float64) for h in range(h_q)] for s in live])
    ref = []
    for s in live:
        K, V = layer.keys_values(s)
        ref.append(orc.attention_decode(q[s].astype(np.float64), ctx[s] - 1, K, V, np.arange(ctx[s]), layer.base))
    assert rel_err(got, np.stack(ref)) <= TOL


@pytest.mark.parametrize("h_q,r_full,r_k,r_v", [(24, 576, 544, 544), (18, 672, 608, 96), (18, 768, 704, 704), (48, 576, 544, 544), (48, 672, 640, 608)])
def test_nothing_of_an_earlier_launch_is_left_in_lds(h_q, r_full, r_k, r_v):
    """NaN latents first, on every compute unit and in all of the K and V tiles; then a smaller rank, whose padding, first tile and missing
    page must not see them."""
    import torch
    h_kv, ctx = 6, [330, 100, 64]
    C_k, C_v, B_k, B_v, q = _latents((h_q, h_kv, r_k, r_v, ctx), seed=r_k)
    layer = LatentLayer(h_q, h_kv, 128, C_k, C_v, B_k, B_v, rope_base=10000.0)
    table = layer.block_table.cpu().numpy().copy()
    table[0, 0] = table[0, 3] = -1
    for page in (0, 3):
        layer.C_k[0][64 * page:64 * page + 64] = 0.0
        layer.C_v[0][64 * page:64 * page + 64] = 0.0
    layer.block_table = torch.from_numpy(table).to(layer.dev)
    one = np.zeros((64, r_full))
    nan = LatentLayer(h_q, h_kv, 128, [one], [one], np.ones((r_full, h_kv * 128)), np.ones((r_full, h_kv * 128)))
    nan.cache.view(torch.bfloat16).fill_(float("nan"))
    b, n = 256, 640
    i32 = lambda *shape: torch.zeros(*shape, dtype=torch.int32, device=layer.dev)
    args = (nan.desc, torch.ones(b, h_q, 128, dtype=torch.bfloat16, device=layer.dev), i32(b), i32(b) + n, n, nan.packed, nan.cache, i32(b, n // 64))
    form = lambda info: info[0]
    assert form(layer.L.decode_kernel_info(nan.desc, b, n)) == form(layer.L.decode_kernel_info(layer.desc, 3, 330))
    ref = layer.oracle(q)
    for _ in range(3):
        assert bool(torch.isnan(layer.L.decode_attention(*args).float()).all())
        got = layer.decode(q)
        assert np.all(np.isfinite(got))
        assert rel_err(got, ref) <= TOL
