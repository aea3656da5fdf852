"""Causal prefill where a row's scores outgrow the maximum of its first tile: the reference of the exponentials then has to
move, once, several times, in the diagonal tile or before it, and for some of a wave's rows only; and where the first tile holds
the largest scores, so that later weights vanish next to it."""
import numpy as np
import pytest

from lorc_testlib import GpuLayer, Problem, TOL
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
