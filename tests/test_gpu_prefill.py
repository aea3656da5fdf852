"""lorc_prefill_attention on the GPU against the fp64 oracle, and its consistency with the decode path."""
import numpy as np
import pytest

import lorc_inputs as gen
from lorc_testlib import GpuLayer, Problem, TOL, oracle_prefill, rel_err

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
