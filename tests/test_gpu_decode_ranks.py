"""The split kernels with the key factor in registers at the ranks their k-step paddings serve (up to 512: 16, 20, 24, 28, 32 steps of 16
and 64-position tiles; above: 18, 21, 24 steps of 32 and 32-position tiles), head counts per workgroup on both sides of eight, value
ranks that leave latent blocks empty, contexts around tile edges; and the fixed-array entry point where only a plan of fewer splits
fits."""
import ctypes

import numpy as np
import pytest

import lorc_inputs as gen
from lorc_testlib import GpuLayer, LatentLayer, Problem, TOL, oracle_decode, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r_k,r_v,h_q,h_kv,ctx", [
    (160, 160, 8, 2, [1, 63, 64, 65, 200]),      # rank below the smallest padding
    (256, 32, 16, 2, [700, 129]),                # rank equal to it; sixteen heads per workgroup, one block of values
    (288, 512, 16, 4, [31, 32, 33, 640]),        # 20 k-steps, two of them empty
    (320, 96, 4, 4, [2000, 0]),                  # groups of one head, an empty context
    (352, 352, 12, 4, [333, 1]),                 # 24 k-steps, three heads per group, odd number of value blocks per wave
    (384, 384, 32, 4, [127, 128, 1000]),
    (448, 480, 20, 4, [65, 500]),                # 28 k-steps, ten heads per workgroup
    (64, 64, 64, 8, [300, 70]),                  # small rank, more than 32 query heads
    # ranks above 512, 32-position tiles: 18, 21 and 24 k-steps of 32, some of them empty
    (544, 544, 24, 6, [1, 31, 32, 33, 63, 64, 65, 200]),
    (576, 576, 32, 8, [700, 129]),
    (608, 32, 6, 6, [333, 0]),
    (672, 640, 12, 6, [31, 96, 640]),
    (704, 768, 18, 6, [97, 1]),
    (768, 768, 32, 8, [127, 128, 1000]),
    (576, 544, 36, 6, [33, 1, 500]),             # groups of six
    (640, 672, 64, 8, [700, 64, 0]),
    (160, 576, 24, 6, [75, 300]),                 # value rank above 512 alone
])
def test_ranks_match_oracle(r_k, r_v, h_q, h_kv, ctx):
    pb = Problem(d_model=max(512, h_kv * 128), n_q_heads=h_q, n_kv_heads=h_kv, head_dim=128, rank_k=r_k, rank_v=r_v,
                 rope_base=10000.0, ctx=ctx, seed=r_k + h_q).build()
    layer = GpuLayer(pb)
    name = layer.L.decode_plan_info(layer.desc, len(ctx), max(ctx))[0]
    assert name == ("decode_stationary_kernel" if 384 < r_k <= 512 else "decode_split_kernel")
    heads = 2 * h_q // h_kv
    if max(r_k, r_v) <= 512:
        form = f"{name}<{max(16, -(-r_k // 64) * 4)}, {1 if heads <= 8 else 2}>"
    else:
        nk = next(k for k in (18, 21, 24) if 32 * k >= max(r_k, r_v))
        form = f"decode_split_kernel<{nk}, {({18: 0, 21: 1, 24: 3} if heads <= 8 else {18: 0, 21: 3})[nk]}, {'true' if heads <= 8 else 'false'}>"
    assert layer.L.decode_kernel_info(layer.desc, len(ctx), max(ctx))[0] == form
    layer.append_all()
    got, ref = layer.decode(), oracle_decode(pb)
    assert np.all(np.isfinite(got))
    for s, n in enumerate(ctx):
        if n == 0:
            assert np.all(got[s] == 0.0)
    live = [s for s, n in enumerate(ctx) if n > 0]
    assert rel_err(got[live], ref[live]) <= TOL


def test_fixed_array_takes_a_plan_of_fewer_splits_where_the_best_one_does_not_fit():
    """484 sequences in a launch sized for 25911 positions: the partials of the best plan exceed the array, those of a plan
    of fewer splits fit.  Same cached latents, so the two differ by the rounding of the partials (fp16) and of the outputs (bf16)."""
    import torch
    b, max_ctx = 484, 25911
    pb = Problem(d_model=1024, n_q_heads=32, n_kv_heads=8, head_dim=128, rank_k=384, rank_v=384, rope_base=10000.0, ctx=[150], seed=5).build()
    layer = GpuLayer(pb)
    layer.append_all()
    L, dev = layer.L, layer.dev
    assert L.decode_workspace_bytes(layer.desc, b, max_ctx) > L.STATIC_WORKSPACE_BYTES
    table = torch.full((b, (max_ctx + 63) // 64), -1, dtype=torch.int32, device=dev)
    table[:, :layer.block_table.shape[1]] = layer.block_table
    q = torch.from_numpy(pb.q).to(dev).to(torch.bfloat16).expand(b, -1, -1).contiguous()
    ctx = torch.randint(1, 151, (b,), generator=torch.Generator().manual_seed(3)).to(torch.int32).to(dev)
    ref = L.decode_attention(layer.desc, q, ctx - 1, ctx, max_ctx, layer.packed, layer.cache, table)
    out = torch.full_like(q, float("nan"))
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    q_pos = ctx - 1
    rc = L._lib.lorc_decode_attention_static(ctypes.byref(layer.desc), ptr(q), ptr(q_pos), ptr(ctx), b, max_ctx, ptr(layer.packed),
                                             ptr(layer.cache), ptr(table), table.shape[1], layer.n_pages, ptr(out), None)
    assert rc == L.OK, L.strerror(rc)
    torch.cuda.synchronize()
    got, ref = out.float(), ref.float()
    assert bool(torch.isfinite(got).all())
    assert float((got - ref).norm() / ref.norm()) <= 2 ** -8   # bf16 outputs (2^-9 each) and fp16 partials (2^-11)


@pytest.mark.parametrize("rank,h_q,b,largest_b,n", [
    (256, 32, 4, 6, 700),     # factor in registers; one workspace for six sequences is smaller than what four take by themselves
    (256, 64, 4, 6, 700),
    (608, 32, 4, 6, 700),
    (608, 64, 4, 6, 700),
    (768, 64, 8, 12, 700),    # three launches
    (1024, 64, 10, 15, 550),
    (512, 32, 6, 11, 350),
    (512, 64, 6, 11, 350),
    (128, 32, 20, 38, 1700),  # streaming kernel
    (1024, 32, 17, 32, 1000),
])
def test_workspace_sized_for_the_largest_batch_serves_smaller_ones(rank, h_q, b, largest_b, n):
    """The call takes the splits that fit, leaves what follows the workspace alone, and differs from a call with a workspace of its own
    size by the rounding of the outputs and of the softmax weights (bf16, relative to the tile's or the split's maximum: 1.7e-3 each in the 2-norm)
    and of the partials (fp16), in both: under 2^-8 together."""
    import torch
    pb = Problem(d_model=1024, n_q_heads=h_q, n_kv_heads=8, head_dim=128, rank_k=rank, rank_v=rank, rope_base=10000.0, ctx=[n], seed=7).build()
    layer = GpuLayer(pb)
    layer.append_all()
    L, dev = layer.L, layer.dev
    need = L.decode_workspace_bytes(layer.desc, largest_b, n)
    assert need < L.decode_workspace_bytes(layer.desc, b, n)
    q = torch.randn(b, h_q, 128, generator=torch.Generator().manual_seed(1)).to(dev).to(torch.bfloat16)
    ctx = torch.tensor([n - 61 * s for s in range(b)], dtype=torch.int32, device=dev)
    table = layer.block_table.expand(b, -1).contiguous()
    args = (layer.desc, q, ctx - 1, ctx, n, layer.packed, layer.cache, table)
    ref = L.decode_attention(*args).float()
    buf = torch.full((need + 4096,), 0x5A, dtype=torch.uint8, device=dev)
    got = L.decode_attention(*args, workspace=buf[:need]).float()
    assert bool(torch.isfinite(got).all()) and bool((buf[need:] == 0x5A).all())
    assert float((got - ref).norm() / ref.norm()) <= 2 ** -8


@pytest.mark.parametrize("h_q,h_kv,r_k,r_v,b,n,symbol", [
    # layers of one or two heads per group on either side of the lines to the three launches and to the streaming kernel
    (40, 40, 64, 64, 12, 130, "decode_split_kernel<16, 1>"), (40, 40, 64, 64, 70, 130, "wide_scores_kernel"),
    (40, 40, 544, 544, 4, 130, "decode_split_kernel<18, 0, true>"), (40, 40, 544, 544, 64, 100, "wide_scores_kernel"),
    (36, 18, 672, 640, 16, 130, "decode_split_kernel<21, 1, true>"), (36, 18, 672, 640, 128, 100, "wide_scores_kernel"),
    (32, 32, 256, 256, 200, 300, "decode_split_kernel<128, 2, 1, 4, 4, 2>"),
    # value ranks above 512, groups on either side of the merge's lines (128, 512): one, two, three, four and eight heads
    (6, 6, 704, 768, 21, 100, None), (6, 6, 704, 768, 22, 100, None), (6, 6, 704, 768, 86, 70, None),
    (12, 6, 544, 576, 85, 70, None), (12, 6, 544, 576, 86, 70, None),
    (18, 6, 96, 608, 22, 100, None), (24, 6, 768, 768, 2, 300, None), (24, 6, 768, 768, 3, 300, None), (24, 6, 768, 768, 100, 70, None),
    (48, 6, 96, 736, 2, 200, None), (48, 6, 640, 672, 8, 100, None), (36, 6, 96, 704, 9, 100, None), (48, 6, 640, 672, 22, 100, None), (20, 20, 96, 1280, 12, 100, None), (20, 20, 96, 1280, 13, 100, None),
])
def test_dispatch_lines_match_oracle(h_q, h_kv, r_k, r_v, b, n, symbol):
    """Three sequences, repeated to the batch: each against the oracle on its latents, and every repetition bit for bit the same."""
    import torch
    rng = np.random.default_rng(b + r_k)
    bf = lambda a: gen.bf16_round(a.astype(np.float32))
    ctx = [n, 1, max(1, n - 37)]
    fall = lambda r: 4.0 * (1.0 + np.arange(r)) ** -0.7
    C_k, C_v = ([bf(rng.standard_normal((m, r)) * fall(r)) for m in ctx] for r in (r_k, r_v))
    B_k, B_v = (bf(rng.standard_normal((r, h_kv * 128)) / np.sqrt(r)) for r in (r_k, r_v))
    q = bf(rng.standard_normal((3, h_q, 128)))
    layer = LatentLayer(h_q, h_kv, 128, C_k, C_v, B_k, B_v, rope_base=10000.0)
    L = layer.L
    info = L.decode_kernel_info(layer.desc, b, n)
    assert symbol is None or info[0] == symbol
    rep = torch.arange(b, device=layer.dev) % 3
    tq, q_pos, cl = layer.tensors(q)
    got = L.decode_attention(layer.desc, tq[rep].contiguous(), q_pos[rep], cl[rep], n, layer.packed, layer.cache, layer.block_table[rep].contiguous())
    for s in range(min(3, b)):
        same = got[s::3].view(torch.int16)
        assert bool((same == same[:1]).all())
    live = min(3, b)
    assert rel_err(got[:live].float().cpu().numpy().astype(np.float64), layer.oracle(q)[:live]) <= TOL
