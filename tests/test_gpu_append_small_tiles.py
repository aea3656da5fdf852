"""The append's 32 x 32 tiles (four waves share the k-steps of a k-tile, their sums meet in LDS): token counts around the lines
to the one-pass kernel and to 64 x 64 tiles, rows and tokens that do not fill a tile, model dimensions that do not fill its ring
of eight k-tiles; and the 64 x 64 tiles just beyond."""
import pytest

import paper_2410_03111_amd as L
from test_gpu_append import _append_and_compare_pool

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("geom,ctx,kernel", [
    ((1024, 2, 64, 64, 32), [32], "append_skinny_kernel"),
    ((1024, 2, 64, 64, 32), [33], "append_kernel<32>"),
    ((1088, 4, 64, 96, 224), [1, 40, 22], "append_kernel<32>"),  # 63 tokens, 17 k-tiles
    ((1024, 8, 128, 512, 512), [64], "append_kernel<32>"),       # 64 workgroups
    ((64, 2, 64, 32, 64), [70, 3], "append_kernel<32>"),         # a single k-tile
    ((576, 8, 128, 512, 512), [200, 56], "append_kernel<32>"),   # 256 workgroups: the last size of these tiles
    ((576, 8, 128, 512, 512), [200, 57], "append_kernel<64>"),
    # 64 x 64 tiles whose rows (96, 1120) and tokens (26, 8, 57) do not fill the last one; 1, 2, 3, 10 and 13 k-tiles
    ((128, 2, 64, 64, 32), [2700, 1, 64, 77], "append_kernel<64>"),
    ((64, 2, 64, 64, 32), [2660, 1, 27], "append_kernel<32>"),
    ((64, 2, 64, 64, 32), [2711, 1, 40], "append_kernel<64>"),
    ((192, 2, 64, 64, 32), [2711, 1, 40], "append_kernel<64>"),
    ((640, 9, 128, 544, 576), [160, 1, 88], "append_kernel<64>"),
    ((832, 9, 128, 544, 576), [200, 57], "append_kernel<64>"),
])
def test_small_tiles_are_bit_exact_with_integer_data(geom, ctx, kernel):
    D, h_kv, d, r_k, r_v = geom
    assert L.append_kernel_info(L.layer_desc(D, 2 * h_kv, h_kv, d, r_k, r_v, 10000.0), sum(ctx)) == kernel
    _append_and_compare_pool(geom, ctx, density=0.2)
