"""Causal prefill where a row's scores outgrow the maximum of its first tile: the reference of the exponentials then has to
move, once, several times, in the diagonal tile or before it, and for some of a wave's rows only; and where the first tile holds
the largest scores, so that later weights vanish next to it."""
import numpy as np
import pytest

from lorc_testlib import GpuLayer, LatentLayer, Problem, TOL
import lorc_inputs as gen
from oracle import lorc_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h_q,h_kv,head_dim", [(8, 2, 128), (4, 4, 64)])
@pytest.mark.parametrize("scales", [(0.25, 4.0), (0.25, 1.0, 4.0, 4.0, 8.0), (8.0, 0.5, 0.5), (1.0, 0.0625, 8.0)])
def test_reference_moves_with_the_scores(h_q, h_kv, head_dim, scales):
    """Hidden states of the g-th 64 positions are scaled by scales[g] (powers of two: exact in bf16); keys and values follow.
    The oracle's attention takes the latents that the layer cached and its bf16 factors: what is left is the rounding of rotated keys
    and queries to fp16 (2^-11 each), which moves a score s by at most |s| 2^-10 (scores to 8 x 4 sigma = 46 in log2 units: 4.5 % of a
    weight at the very most, and independent from key to key, so a fraction of that in a weighted mean)."""
    n = 64 * (len(scales) - 1) + 41
    pb = Problem(d_model=512, n_q_heads=h_q, n_kv_heads=h_kv, head_dim=head_dim, rank_k=96, rank_v=64, rope_base=10000.0,
                 ctx=[n, 64], seed=31).build()
    pb.X = [x * np.repeat(np.asarray(scales, x.dtype), 64)[:len(x), None] for x in pb.X]
    layer = GpuLayer(pb)
    layer.append_all()
    Q = [gen.queries(N, h_q, head_dim, seed=7300 + s) for s, N in enumerate(pb.ctx)]
    got = layer.prefill(Q)
    B_k, B_v = (b.float().cpu().numpy().astype(np.float64) for b in (layer.dB_k, layer.dB_v))
    for s, N in enumerate(pb.ctx):
        latents = (layer.read_latents(s, N).astype(np.uint32) << 16).view(np.float32).astype(np.float64)
        c_k, c_v = latents[:, :pb.rank_k], latents[:, pb.rank_k:]
        ref = orc.attention_prefill(Q[s].astype(np.float64), orc.split_heads(c_k @ B_k, h_kv, head_dim),
                                    orc.split_heads(c_v @ B_v, h_kv, head_dim), pb.rope_base)
        assert np.all(np.isfinite(got[s]))
        assert float(np.max(np.abs(got[s] - ref))) <= TOL * float(np.max(np.abs(ref)))


@pytest.mark.parametrize("h_q,h_kv,head_dim", [(4, 2, 128), (2, 2, 64)])
def test_a_long_tail_of_small_weights_counts_in_the_sum(h_q, h_kv, head_dim):
    """One key of score 0 first (the row's maximum), 4096 keys of score -15 (log2) behind it: each weighs 2^-15 of the first, below
    fp16's normal range, all of them an eighth of it.  Value column 0 is the first key's share of the row, column 1 the tail's.
    Tolerance: query and key in fp16 move the score by 15 x 2^-11 at most, a weight by 0.5 %; fp16 holds 2^-15 in steps of 2^-24
    (2^-10 at most); the outputs are bf16 (2^-9)."""
    n, r = 4097, 32
    C_k, C_v = np.zeros((n, r)), np.zeros((n, r))
    C_k[1:, 0] = -15.0
    C_v[0, 0] = C_v[1:, 1] = 1.0
    B_k, B_v = np.zeros((r, h_kv * head_dim)), np.zeros((r, h_kv * head_dim))
    for g in range(h_kv):
        B_k[0, g * head_dim + head_dim // 2 - 1] = 1.0      # the slowest rotation: none at this base
        B_v[0, g * head_dim] = B_v[1, g * head_dim + 1] = 1.0
    layer = LatentLayer(h_q, h_kv, head_dim, [C_k], [C_v], B_k, B_v, rope_base=1e12, softmax_scale=float(np.log(2.0)))
    q = np.zeros((n, h_q, head_dim))
    q[:, :, head_dim // 2 - 1] = 1.0
    got = layer.prefill(q)
    rows = [1, 63, 64, 100, 1000, 4096]
    K, V = layer.keys_values(0)
    for i in rows:
        ref = orc.attention_decode(q[i], i, K[:i + 1], V[:i + 1], np.arange(i + 1), layer.base, layer.scale)
        for c in (0, 1):
            assert np.all(np.abs(got[i, :, c] / ref[:, c] - 1.0) <= 0.005 + 2 ** -10 + 2 ** -9), (i, c)


@pytest.mark.parametrize("h_q,h_kv,head_dim", [(16, 8, 128), (8, 8, 64)])
def test_the_largest_weight_of_a_row_is_exact(h_q, h_kv, head_dim):
    """Twenty keys of score 0 in the first tile, then one key of score s (log2) with the only value: its share of the row is 2^s / (20 + 2^s),
    and the weight itself, the row's largest, is 1 and takes no rounding.  s is the one whose 2^s a 16-bit weight holds worst
    (4.3e-4 off).  The mean over 128 (64) x 8 values leaves the rounding of the outputs out: 2^-9 / sqrt(3 x 512) = 5e-5 of it."""
    n, r = 96, 32
    s = max((k / 128.0 for k in range(1, 128)), key=lambda x: abs(float(np.float16(2.0 ** x)) / 2.0 ** x - 1.0))
    assert abs(float(np.float16(2.0 ** s)) / 2.0 ** s - 1.0) > 4e-4
    C_k, C_v = np.full((n, r), 0.0), np.zeros((n, r))
    C_k[:, 0] = -64.0
    C_k[:20, 0] = 0.0
    C_k[66, 0], C_v[66, 0] = s, 1.0
    B_k, B_v = np.zeros((r, h_kv * head_dim)), np.zeros((r, h_kv * head_dim))
    B_k[0, head_dim // 2 - 1::head_dim] = 1.0
    B_v[0] = gen.bf16_round(np.random.default_rng(5).uniform(1.0, 2.0, h_kv * head_dim).astype(np.float32))
    layer = LatentLayer(h_q, h_kv, head_dim, [C_k], [C_v], B_k, B_v, rope_base=1e12, softmax_scale=float(np.log(2.0)))
    q = np.zeros((n, h_q, head_dim))
    q[:, :, head_dim // 2 - 1] = 1.0
    got = layer.prefill(q)
    values = B_v[0].reshape(h_kv, head_dim)[np.arange(h_q) // (h_q // h_kv)]
    for i in (66, 95):
        assert abs(float(np.mean(got[i] / values)) * (20.0 + 2.0 ** s) / 2.0 ** s - 1.0) <= 2e-4
