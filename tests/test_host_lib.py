"""CPU-only tests of the C-ABI library: it loads, exports every declared symbol, and its host entry points
(lorc_factorize, lorc_rank_schedule, index helpers, argument validation) agree with the oracle and numpy."""
import ctypes
import os
import re

import numpy as np
import pytest

import lorc_inputs as gen
from oracle import lorc_oracle as orc
from lorc_testlib import k_index, v_index

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
L = pytest.importorskip("paper_2410_03111_amd", reason="liblorc.so not built: python paper_2410_03111_amd/build.py")


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "lorc.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(lorc_[a-z_]+)\s*\(", header))
    assert declared == set(L.EXPORTS)
    lib = ctypes.CDLL(L.LIB_PATH)
    for name in declared:
        assert hasattr(lib, name), name


def test_strerror_texts():
    assert L.strerror(0) == "ok"
    for code in (-1, -2, -3, -4, -5):
        assert L.strerror(code) and "unknown" not in L.strerror(code)
    assert "unknown" in L.strerror(-99)


@pytest.mark.parametrize("rows,cols,rank", [(96, 48, 16), (256, 128, 32), (200, 128, 128), (512, 256, 100)])
def test_factorize_matches_lapack(rows, cols, rank):
    W, sigma = gen.power_law_weight(rows, cols, seed=rows + cols)
    A, B, s, eps = L.factorize(W, rank)
    Wt, s_ref = orc.low_rank_weight(W, rank)
    assert np.max(np.abs(A @ B - Wt)) < 1e-11
    assert np.max(np.abs(s - s_ref)) < 1e-11
    assert abs(eps - orc.rel_frobenius_error(W, Wt)) < 1e-11
    assert np.allclose(B @ B.T, np.eye(rank), atol=1e-11)           # read-side factor: orthonormal rows
    assert np.allclose(np.linalg.norm(A, axis=0), s_ref[:rank], atol=1e-11)
    # documented sign convention: the largest-magnitude entry of every row of B is positive
    assert np.all(B[np.arange(rank), np.argmax(np.abs(B), axis=1)] > 0)


def test_factorize_generic_matrix_and_determinism():
    rng = np.random.default_rng(0)
    W = rng.standard_normal((130, 64)) * np.logspace(0, -6, 64)[None, :]
    A, B, s, eps = L.factorize(W, 20)
    A2, B2, s2, _ = L.factorize(W, 20)
    assert np.array_equal(A, A2) and np.array_equal(B, B2)
    Wt, s_ref = orc.low_rank_weight(W, 20)
    assert np.max(np.abs(A @ B - Wt)) < 1e-10
    assert np.max(np.abs(s - s_ref) / s_ref[0]) < 1e-12


def test_factorize_rejects_bad_arguments():
    W = np.zeros((8, 16))
    with pytest.raises(L.LorcError) as e:
        L.factorize(W, 4)               # rows < cols
    assert e.value.code == L.EINVAL
    W = np.eye(16)[:, :8].copy()
    for bad in (0, 9):
        with pytest.raises(L.LorcError):
            L.factorize(W, bad)
    W[0, 0] = np.nan
    with pytest.raises(L.LorcError):
        L.factorize(W, 4)


def test_rank_schedule_matches_oracle():
    rng = np.random.default_rng(4)
    Lyr, n = 12, 64
    sk = np.sort(rng.random((Lyr, n)) + 0.05, axis=1)[:, ::-1].copy()
    sv = np.sort(rng.random((Lyr, n)) + 0.05, axis=1)[:, ::-1].copy()
    got = L.rank_schedule(sk, sv, d_max=64, d_min=24, align=8)
    kk = [orc.condition_number(s) for s in sk]
    kv = [orc.condition_number(s) for s in sv]
    lc = orc.cumulative_log_condition(kk, kv)
    ref = orc.round_dims(orc.compression_dims(lc, 64, 24), 8, 24, 64)
    assert list(got) == list(ref)
    assert got[0] == 64 and got[-1] == 24 and all(a >= b for a, b in zip(got, got[1:]))
    # threshold on the log cumulative condition number: sensitive (shallow) layers stay uncompressed
    thr = float(lc[3] + lc[4]) / 2
    got_t = L.rank_schedule(sk, sv, d_max=48, d_min=24, align=8, log_threshold=thr)
    assert list(got_t[:4]) == [n] * 4 and all(r <= 48 for r in got_t[4:])


def test_error_bound_matches_oracle():
    rng = np.random.default_rng(6)
    Lyr, n = 7, 40
    sg = np.sort(rng.random((Lyr, n)) * 3 + 0.01, axis=1)[:, ::-1].copy()
    ranks = np.array([5, 40, 0, 17, 39, 1, 20], np.int32)        # includes full rank (term 0) and rank 0
    for lip in (1.0, 0.5, 2.0):
        bound, terms = L.error_bound(sg, ranks, lipschitz=lip)
        ref_b, ref_t = orc.network_error_bound(list(sg), ranks, lipschitz=lip)
        np.testing.assert_allclose(terms, ref_t, rtol=1e-13, atol=0)
        assert abs(bound - ref_b) <= 1e-12 * abs(ref_b)
    assert terms[1] == 0.0
    one, t1 = L.error_bound(sg[:1], ranks[:1])
    assert one == sg[0, 5] == t1[0]                                # one layer: Theorem 1's constant
    with pytest.raises(L.LorcError):
        L.error_bound(sg, np.array([5, 41, 0, 17, 39, 1, 20], np.int32))


def test_page_layout_helpers_match_documented_formulas():
    desc = L.layer_desc(4096, 32, 8, 128, 512, 384, 500000.0)
    assert L.page_bytes(desc) == 64 * (512 + 384) * 2
    seen = set()
    for slot in range(64):
        for j in range(0, 512, 37):
            i = L.cache_index_k(desc, slot, j)
            assert i == k_index(512, slot, j)
            seen.add(i)
        for j in range(0, 384, 29):
            i = L.cache_index_v(desc, slot, j)
            assert i == v_index(512, slot, j)
            seen.add(i)
    assert max(seen) < 64 * (512 + 384)
    assert L.cache_index_k(desc, 64, 0) == -1 and L.cache_index_v(desc, 0, 384) == -1


def test_page_layout_is_a_bijection():
    r_k, r_v = 96, 64
    slot = np.arange(64)[:, None]
    idx = np.concatenate([k_index(r_k, slot, np.arange(r_k)[None, :]), v_index(r_k, slot, np.arange(r_v)[None, :])], axis=1)
    assert sorted(idx.reshape(-1)) == list(range(64 * (r_k + r_v)))


def test_unsupported_geometry_is_reported():
    assert L.page_bytes(L.layer_desc(4096, 32, 8, 96, 512, 512, 1e4)) == 0          # head_dim 96
    assert L.page_bytes(L.layer_desc(4096, 32, 8, 128, 500, 512, 1e4)) == 0         # rank not a multiple of 32
    assert L.page_bytes(L.layer_desc(4096, 32, 8, 128, 512, 512, 1e4, page_size=16)) == 0
    assert L.packed_bytes(L.layer_desc(4096, 30, 8, 128, 512, 512, 1e4)) == 0       # h_q not a multiple of h_kv
    assert L.decode_workspace_bytes(L.layer_desc(4096, 32, 8, 128, 512, 512, 5e5), 16, 4096) > 0


def test_workspace_helpers_accept_an_empty_context():
    """max_ctx = 0 (every context empty) is legal: the split plan must still have one split, not divide by zero."""
    for desc in (L.layer_desc(4096, 32, 8, 128, 512, 512, 5e5), L.layer_desc(256, 4, 2, 64, 32, 32, 1e4),
                 L.layer_desc(8192, 64, 8, 128, 512, 512, 5e5)):
        for b in (1, 16):
            w0 = L.decode_workspace_bytes(desc, b, 0)
            assert 0 < w0 <= L.decode_workspace_bytes(desc, b, 64)
            a0 = L.decode_absorbed_workspace_bytes(desc, b, 0)
            assert 0 < a0 <= L.decode_absorbed_workspace_bytes(desc, b, 64)
    assert L.decode_workspace_bytes(L.layer_desc(4096, 32, 8, 128, 512, 512, 5e5), 16, -1) == 0


@pytest.mark.parametrize("n_q_heads,n_kv_heads", [(32, 8), (8, 8), (64, 16), (40, 40), (64, 64)])
def test_uncompressed_workspace_grows_with_context_and_batch(n_q_heads, n_kv_heads):
    """KV heads a multiple of eight (the one-pass kernel): a workspace sized for the longest context and the largest batch
    serves every smaller call, and it never exceeds scores and partials of the three-launch path (256 bytes per head and
    position tile, 264 per head and split)."""
    n = 128 * n_kv_heads
    desc = L.layer_desc(1024, n_q_heads, n_kv_heads, 128, n, n, 1e4)
    previous = None
    for b in (1, 2, 3, 5, 8, 16, 33, 64, 100, 256, 1000):
        sizes = [L.decode_plain_workspace_bytes(desc, b, 64 * t) for t in list(range(0, 700)) + list(range(700, 9000, 37))]
        assert all(x <= y for x, y in zip(sizes, sizes[1:]))
        assert previous is None or all(x <= y for x, y in zip(previous, sizes))
        for t in (1, 2, 7, 64, 300, 699):
            splits = max(1, min((t + 3) // 4, 512, -(-2048 // (b * n_kv_heads))))
            splits = -(-t // -(-t // splits))
            assert sizes[t] <= b * n_q_heads * (256 * t + 264 * splits) + 768
        previous = sizes


@pytest.mark.parametrize("h_q,h_kv,head_dim,rank,absorbed", [
    (32, 8, 128, 128, False), (32, 8, 64, 256, False), (15, 5, 128, 512, False), (32, 2, 128, 256, False),    # streaming kernel
    (32, 8, 128, 1024, False), (32, 8, 128, 256, False), (32, 8, 128, 512, False), (64, 8, 128, 512, False), (40, 40, 128, 416, False),
    (32, 8, 128, 768, False), (64, 8, 128, 640, False), (64, 8, 128, 768, False), (40, 40, 128, 2048, False), (40, 40, 128, 640, False),
    (64, 64, 128, 64, False), (64, 64, 128, 544, False), (64, 32, 128, 672, False), (32, 32, 128, 256, False),
    (32, 8, 128, 512, True), (64, 8, 128, 512, True), (40, 40, 128, 2048, True)])
def test_a_workspace_sized_for_the_largest_call_serves_them_all(h_q, h_kv, head_dim, rank, absorbed):
    """A plan of few splits exists for every call with no more sequences and no longer contexts, and it covers the context; a workspace
    that holds less than one split per sequence is refused."""
    desc = L.layer_desc(4096, h_q, h_kv, head_dim, rank, rank, 1e4)
    size = L.decode_absorbed_workspace_bytes if absorbed else L.decode_workspace_bytes
    rng = np.random.default_rng(7)
    fewer = 0
    for B, N in [(1, 700), (6, 700), (12, 700), (32, 2000), (16, 4096), (5, 6720), (9, 7488), (64, 300), (3, 40000)] + \
            [(int(rng.integers(2, 80)), int(rng.integers(64, 9000))) for _ in range(30)]:
        need = size(desc, B, N)
        calls = [(b, n) for b in {1, B // 2, B - 1, B} for n in {0, 1, N // 3, N - 64, N - 1, N} if b >= 1 and n >= 0]
        for b, n in calls + [(int(rng.integers(1, B + 1)), int(rng.integers(0, N + 1))) for _ in range(30)]:
            info = L.decode_kernel_info(desc, b, n, need, absorbed)
            assert info is not None, (B, N, b, n)
            assert info[1] * info[2] * 128 >= n and (info[1] - 1) * info[2] * 64 <= n
            fewer += size(desc, b, n) > need
        assert L.decode_kernel_info(desc, B, N, B * h_q * (8 + 2 * rank) - 1, absorbed) is None
    assert fewer > 0   # (some of the calls would have taken more splits)


@pytest.mark.parametrize("h_q,h_kv,rank", [(40, 40, 256), (40, 40, 512), (24, 24, 512), (48, 12, 640), (40, 10, 256), (32, 8, 512)])
def test_stationary_splits_fill_the_xcds(h_q, h_kv, rank):
    """The head pairs of a (sequence, split) share one of eight XCDs of 32 CUs: no other split count gives fewer rounds of an XCD's
    workgroups x (tiles of a split + 2)."""
    desc = L.layer_desc(4096, h_q, h_kv, 128, rank, rank, 1e4)
    for b, n in ((1, 1000), (2, 1000), (4, 4000), (3, 2000), (12, 1000), (16, 4096), (33, 700)):
        tiles = -(-n // 64)
        cost = lambda tps: -(-(-(-b * -(-tiles // tps) // 8) * (h_kv // 2)) // 32) * (tps + 2)
        _, ns, tps = L.decode_kernel_info(desc, b, n)
        assert ns == -(-tiles // tps)
        assert cost(tps) <= min(cost(t) for t in range(1, tiles + 1) if -(-tiles // t) <= 64) * 1.002


@pytest.mark.parametrize("h_q,h_kv,rank,b,n,symbol", [
    (64, 64, 544, 16, 1000, "decode_split_kernel<18, 0, true>"), (64, 64, 544, 32, 1000, "wide_scores_kernel"),
    (64, 64, 544, 64, 100, "wide_scores_kernel"), (64, 64, 544, 16, 4000, "decode_split_kernel<18, 0, true>"),
    (40, 40, 672, 12, 1000, "decode_split_kernel<21, 1, true>"), (40, 40, 672, 16, 1000, "wide_scores_kernel"),
    (64, 32, 672, 32, 1000, "decode_split_kernel<21, 1, true>"), (64, 32, 672, 128, 100, "wide_scores_kernel"),
    (40, 20, 544, 16, 1000, "decode_split_kernel<18, 0, true>"), (40, 20, 544, 32, 1000, "wide_scores_kernel"),
    (40, 20, 544, 200, 300, "decode_split_kernel<18, 0, true>"), (40, 20, 384, 32, 1000, "decode_split_kernel<24, 1>"),
    (40, 40, 64, 1, 1000, "decode_split_kernel<16, 1>"), (40, 40, 64, 32, 1000, "wide_scores_kernel"),
    (40, 40, 128, 32, 1000, "decode_split_kernel<16, 1>"), (40, 40, 384, 64, 100, "decode_split_kernel<24, 1>"),
    (48, 16, 544, 200, 300, "decode_split_kernel<18, 0, true>"), (32, 32, 256, 64, 100, "decode_split_kernel<16, 1>"),
    (32, 32, 256, 200, 300, "decode_split_kernel<128, 2, 1, 4, 4, 2>"), (32, 32, 544, 200, 300, "decode_split_kernel<18, 0, true>"),
    (32, 8, 256, 200, 300, "decode_split_kernel<16, 1>"), (64, 8, 544, 64, 100, "decode_split_kernel<18, 0, false>")])
def test_decode_takes_the_kernel_measured_fastest(h_q, h_kv, rank, b, n, symbol):
    """Sizes on either side of the lines between the stationary kernels and the ones that they replace for most shapes (256 CUs)."""
    assert L.decode_kernel_info(L.layer_desc(4096, h_q, h_kv, 128, rank, rank, 1e4), b, n)[0] == symbol


@pytest.mark.parametrize("h_q,h_kv,rank", [(64, 8, 768), (64, 8, 1024), (40, 40, 1280), (40, 40, 2048)])
def test_value_splits_of_fewer_than_four_tiles_have_a_compute_unit_each(h_q, h_kv, rank):
    """Three launches: one workgroup per (sequence, split, 512 value columns)."""
    desc = L.layer_desc(4096, h_q, h_kv, 128, rank, rank, 1e4)
    for b in range(1, 70):
        for n in (64, 300, 500, 1000, 1500, 2000, 4096):
            _, ns, tps = L.decode_kernel_info(desc, b, n)
            assert ns <= -(-n // 256) or b * ns * -(-rank // 512) <= 256   # (no more than splits of four tiles, or a CU for each)


def test_decode_plan_info_names_the_kernel_and_covers_the_context():
    """Host-only: the reported plan names the kernel the launch will use and its splits cover every tile."""
    for desc, b, ctx in ((L.layer_desc(4096, 32, 8, 128, 512, 512, 5e5), 16, 4096),
                         (L.layer_desc(4096, 32, 8, 128, 768, 768, 5e5), 32, 8192),
                         (L.layer_desc(4096, 32, 8, 128, 384, 384, 5e5), 32, 8192),
                         (L.layer_desc(8192, 64, 8, 128, 512, 512, 5e5), 64, 32768),
                         (L.layer_desc(256, 4, 2, 64, 32, 32, 1e4), 1, 0)):
        name, ns, tps = L.decode_plan_info(desc, b, ctx)
        assert name in ("decode_split_kernel", "decode_stationary_kernel", "wide_scores_kernel")
        assert ns >= 1 and tps >= 1 and ns * tps >= (ctx + 63) // 64
        if desc.n_q_heads <= 32 and (desc.rank_k > 512 or desc.rank_k <= 384 or desc.head_dim != 128):
            assert name == "decode_split_kernel"
    # 64 query heads off the stationary kernel's ranks: three launches
    assert L.decode_plan_info(L.layer_desc(8192, 64, 8, 128, 768, 768, 5e5), 32, 8192)[0] == "wide_scores_kernel"
    assert L.decode_plan_info(L.layer_desc(8192, 64, 8, 128, 512, 512, 5e5), 32, 8192)[0] == "decode_stationary_kernel"
    with pytest.raises(L.LorcError):
        L.decode_plan_info(L.layer_desc(4096, 32, 8, 96, 512, 512, 1e4), 1, 64)


@pytest.mark.parametrize("h_q,h_kv,head_dim,r_k,r_v,symbol", [
    (32, 8, 128, 128, 128, "decode_split_kernel<128, 2, 1, 4, 4, 2>"), (4, 2, 64, 32, 32, "decode_split_kernel<64, 2, 1, 4, 4, 2>"),
    (32, 8, 128, 160, 512, "decode_split_kernel<16, 1>"), (64, 8, 128, 32, 32, "decode_split_kernel<16, 2>"),
    (32, 8, 128, 384, 384, "decode_split_kernel<24, 1>"), (32, 8, 128, 416, 416, "decode_stationary_kernel<28, 1>"),
    (64, 8, 128, 512, 512, "decode_stationary_kernel<32, 2>"), (15, 5, 128, 512, 512, "decode_split_kernel<128, 2, 1, 4, 4, 2>"),
    (32, 8, 128, 544, 544, "decode_split_kernel<18, 0, true>"), (32, 8, 128, 160, 672, "decode_split_kernel<21, 1, true>"),
    (32, 8, 128, 768, 768, "decode_split_kernel<24, 3, true>"), (64, 8, 128, 672, 672, "decode_split_kernel<21, 3, false>"),
    (64, 8, 128, 704, 704, "wide_scores_kernel"), (32, 8, 128, 800, 800, "decode_split_kernel<128, 2, 1, 8, 4, 1>"),
    (40, 40, 128, 2048, 2048, "wide_scores_kernel")])
def test_decode_kernel_info_tells_the_families_apart(h_q, h_kv, head_dim, r_k, r_v, symbol):
    """Streaming kernel (six template arguments), factor in registers to rank 512 (two) and to 768 (three), three launches."""
    desc = L.layer_desc(4096, h_q, h_kv, head_dim, r_k, r_v, 1e4)
    name, ns, tps = L.decode_kernel_info(desc, 4, 2000)
    assert name == symbol
    assert (name.split("<")[0], ns, tps) == L.decode_plan_info(desc, 4, 2000)
    assert L.decode_kernel_info(desc, 4, 2000, workspace_bytes=16) is None


@pytest.mark.parametrize("D,r_k,r_v,T,kernel", [
    (256, 32, 32, 64, "append_skinny_kernel"), (4096, 512, 512, 65, "append_kernel"),
    (2048, 2048, 2048, 48, "append_skinny_kernel"), (2048, 2048, 2048, 56, "append_kernel"),   # 16 and
    (2048, 1280, 1280, 36, "append_skinny_kernel"), (2048, 1280, 1280, 40, "append_kernel"),   # 10 rows per CU
    (3072, 2048, 2048, 33, "append_kernel"), (5120, 2048, 2048, 33, "append_kernel"), (4096, 512, 512, 33, "append_kernel"),
    (4096, 512, 512, 1024, "append_kernel"),                # one 64 x 64 tile per CU
    (4096, 576, 576, 1000, "append_kernel"),                # a few more, token tiles a multiple of eight
    (4096, 576, 576, 900, "append_tile_kernel<2, 5, 4>"),   # ... or not
    (4096, 768, 768, 1000, "append_tile_kernel<2, 5, 4>"), (5120, 2048, 2048, 300, "append_tile_kernel<2, 5, 4>"),
    (4096, 576, 576, 6002, "append_tile_kernel<2, 2, 4>"), (4096, 576, 576, 12320, "append_tile_kernel<2, 2, 4>"),
    (5120, 5120, 5120, 777, "append_tile_kernel<4, 3, 2>"), (5120, 5120, 5120, 1500, "append_tile_kernel<4, 3, 2>"),
    (4096, 512, 512, 12000, "append_gemm_kernel"), (4096, 576, 576, 12288, "append_gemm_kernel"),
    (5120, 2048, 2048, 10000, "append_gemm_kernel"),
    (4096, 768, 768, 18000, "append_gemm_kernel"), (4096, 512, 512, 32768, "append_gemm_kernel"),
    (64, 512, 512, 32768, "append_tile_kernel<4, 3, 2>")])  # (the 256 x 256 tiles' ring wants two k-tiles)
def test_append_takes_the_kernel_measured_fastest(D, r_k, r_v, T, kernel):
    """The kernel that measurement found fastest at sizes on either side of the rule's lines (256 CUs)."""
    n = (max(r_k, r_v) + 127) // 128 * 128
    assert L.append_plan_info(L.layer_desc(D, n // 128, n // 128, 128, r_k, r_v, 1e4), T) == kernel


def test_device_functions_without_torch_raise_import_error(monkeypatch):
    monkeypatch.setattr(L, "torch", L._NoTorch())
    desc = L.layer_desc(4096, 32, 8, 128, 512, 512, 1e4)
    with pytest.raises(ImportError):
        L.append_latent(desc, None, None, None, None, None, None)
    with pytest.raises(ImportError):
        L.pack_factors(desc, None, None, None, None)


def test_append_plan_info_refuses_what_append_refuses():
    with pytest.raises(L.LorcError):
        L.append_plan_info(L.layer_desc(4096, 32, 8, 96, 512, 512, 1e4), 1)
    with pytest.raises(L.LorcError):
        L.append_plan_info(L.layer_desc(4096, 32, 8, 128, 512, 512, 1e4), 0)


def test_bench_refuses_more_than_one_gpu():
    """The build is single-GPU: asking bench.py for more exits with a message before anything touches a device."""
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=300)
    assert r.returncode != 0
    assert "single-GPU" in (r.stdout + r.stderr)
    assert not any(line.startswith("{") for line in r.stdout.splitlines())
