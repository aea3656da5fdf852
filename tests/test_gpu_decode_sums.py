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


@pytest.mark.parametrize("h_q,h_kv,head_dim,r_v,b", [
    (32, 8, 128, 1024, 1), (32, 8, 128, 768, 9), (32, 8, 128, 544, 17),   # 8, 72 and 136 groups of four heads
    (24, 8, 128, 768, 2), (40, 8, 128, 1024, 3), (40, 8, 128, 576, 17),   # odd groups
    (64, 8, 128, 1024, 2), (64, 8, 128, 1024, 6), (64, 8, 128, 1024, 20),  # groups of eight
    (16, 16, 128, 768, 2), (16, 16, 128, 768, 16), (16, 16, 128, 768, 33), (32, 16, 64, 1024, 1), (16, 16, 64, 640, 9),
    (40, 40, 128, 1280, 1), (40, 40, 128, 2048, 6),                       # one head per group, ranks above 1024
])
def test_merged_latents_keep_32_bits(h_q, h_kv, head_dim, r_v, b):
    """Queries of zeros: all weights are equal.  The quarters of the context hold the values 1, 2^-9, 2^-17 and 0 in the lower half of the
    latents, 1, 2^-9, 0 and 0 in the upper one; splits lie within a quarter, so that their partials (fp16) and every sum of fp32 are
    exact.  Each output is the difference of two merged latents, 2^-17 / 4, which is lost where they are held in 16 bits."""
    import paper_2410_03111_amd as L
    width, r_k = h_kv * head_dim, 96
    for n in (256, 512, 1024, 2048, 4096):
        ns = L.decode_plan_info(L.layer_desc(64, h_q, h_kv, head_dim, r_k, r_v, 1e12), b, n)[1]
        if ns in (4, 8, 16, 32, 64):
            break
    assert ns in (4, 8, 16, 32, 64)
    C_v = np.zeros((n, r_v))
    C_v[: n // 4] = 1.0
    C_v[n // 4: n // 2] = 2.0 ** -9
    C_v[n // 2: 3 * n // 4, : r_v // 2] = 2.0 ** -17
    B_v = np.zeros((r_v, width))
    B_v[np.arange(width) % (r_v // 2), np.arange(width)] = 1.0
    B_v[r_v // 2 + np.arange(width) % (r_v // 2), np.arange(width)] = -1.0
    empty = b - 1
    layer = LatentLayer(h_q, h_kv, head_dim, [np.zeros((0, r_k))] * empty + [np.zeros((n, r_k))], [np.zeros((0, r_v))] * empty + [C_v],
                        np.zeros((r_k, width)), B_v, rope_base=1e12)
    got = layer.decode(np.zeros((b, h_q, head_dim)))
    assert np.all(got[:empty] == 0.0)
    assert np.all(got[empty] == 2.0 ** -19)
