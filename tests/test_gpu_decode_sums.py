"""What the decode kernels keep in 32 bits: the softmax sums, and o_lat between the splits' partials and the value up-projection."""
import numpy as np
import pytest

import lorc_inputs as gen
from lorc_testlib import LatentLayer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h_q,h_kv,head_dim,r_k,r_v", [
    (4, 2, 64, 32, 64), (16, 4, 128, 96, 128),                              # streaming kernel
    (16, 4, 128, 160, 160), (32, 4, 128, 384, 256), (16, 4, 128, 448, 512),  # stationary, up to 8 and 16 heads per workgroup
    (64, 8, 128, 64, 96),
    (24, 6, 128, 544, 544), (18, 6, 128, 768, 768), (36, 6, 128, 640, 672),  # ranks 544 to 768
    (40, 8, 128, 96, 1024),                                                 # three launches
])
def test_row_sums_take_the_weights_unrounded(h_q, h_kv, head_dim, r_k, r_v):
    """Every 32nd key has score 0, the others a score whose weight bf16 rounds by 0.36 %.  Values at the former only: the sum of the
    weights decides the outputs, and the mean over at least 32 of them leaves their rounding out (bf16 2^-9, partials 2^-11, uniform:
    1.2e-3 / sqrt(32) = 2e-4; the bound is about five times that, a third of what rounded weights in the sum would do)."""
    s = min((-k / 256.0 for k in range(1, 256)), key=lambda x: float(gen.bf16_round(np.float32([2.0 ** x]))[0]) / 2.0 ** x)
    assert float(gen.bf16_round(np.float32([2.0 ** s]))[0]) / 2.0 ** s - 1.0 < -3.3e-3
    n, width = 200, h_kv * head_dim
    rng = np.random.default_rng(3)
    C_k, C_v = np.zeros((n, r_k)), np.zeros((n, r_v))
    C_k[:, 0] = s
    C_k[::32, 0] = 0.0
    C_v[::32] = gen.bf16_round(rng.uniform(1.0, 2.0, r_v).astype(np.float32))
    B_k, B_v = np.zeros((r_k, width)), np.zeros((r_v, width))
    B_k[0, head_dim // 2 - 1::head_dim] = 1.0      # the slowest rotation: none at this base
    B_v[np.arange(width) % r_v, np.arange(width)] = 1.0
    layer = LatentLayer(h_q, h_kv, head_dim, [C_k], [C_v], B_k, B_v, rope_base=1e12, softmax_scale=float(np.log(2.0)))
    q = np.zeros((1, h_q, head_dim))
    q[:, :, head_dim // 2 - 1] = 1.0
    ratio = layer.decode(q) / layer.oracle(q)
    print(f"mean deviation {np.mean(ratio) - 1.0:.2e}")
    assert abs(float(np.mean(ratio)) - 1.0) <= 1e-3
