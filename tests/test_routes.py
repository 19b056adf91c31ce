"""Which kernel a call takes, by the library's own rules (no GPU needed): the calls that a rule must leave to the
general kernel because it serves them faster."""
import ctypes
import sys

import pytest
import torch

from paper_2603_10026_amd import binding as B

TILED = (1, 2, 3, 4)   # rf_diag_attention_route: one or two query tiles of 128 or 256 rows per workgroup
KEY_GROUPS, FEW_ROWS = 5, 6


def attention_route(Bt, Hq, Hkv, Lq, Lk, d, causal, dtype=torch.bfloat16):
    q = torch.empty((Bt, Hq, Lq, d), dtype=dtype, device="meta")
    k = torch.empty((Bt, Hkv, Lk, d), dtype=dtype, device="meta")
    return B.rf_diag_attention_route(q, k, k, causal)


@pytest.mark.parametrize("Bt,Hq,Hkv,Lq,Lk,d,causal", [
    # many queries before a short context: a workgroup's own cost is all there is (us tiled / taken before:
    # 12.8 / 38.6, 6.7 / 17.9, 47.3 / 127, 125 / 257, 21.3 / 29.6)
    (27, 16, 4, 607, 31, 64, True), (20, 8, 8, 614, 80, 64, True), (53, 16, 16, 767, 4, 128, True),
    (24, 32, 8, 1770, 3, 128, True), (45, 2, 2, 1376, 18, 128, True),
    # up to 64 rows a head, but more heads than compute units (74 / 101)
    (64, 32, 32, 50, 300, 128, False),
    # the benchmark's prefills, a batch of heads beyond one round, no key at all
    (4, 32, 32, 2048, 2048, 128, False), (4, 32, 32, 2048, 2048, 128, True), (2, 32, 8, 1000, 3001, 128, True),
    (1, 40, 40, 900, 900, 128, False), (1, 4, 4, 300, 0, 128, False),
])
def test_attention_calls_that_stay_with_the_tiled_kernel(Bt, Hq, Hkv, Lq, Lk, d, causal):
    assert attention_route(Bt, Hq, Hkv, Lq, Lk, d, causal) in TILED


@pytest.mark.parametrize("Bt,Hq,Hkv,Lq,Lk,d,causal,route", [
    # (us tiled / taken: 54.5 / 32.1, 12.7 / 8.6, 39.9 / 17.7, 145.5 / 23.3, 16.1 / 9.2)
    (1, 16, 16, 512, 2048, 128, False, KEY_GROUPS), (1, 32, 32, 512, 512, 64, False, KEY_GROUPS),
    # a handful of keys (6.7 / 5.0, 6.7 / 5.2)
    (28, 8, 8, 25, 2, 128, False, FEW_ROWS), (1, 32, 8, 202, 6, 128, True, FEW_ROWS),
    (1, 1, 1, 1371, 2708, 64, True, FEW_ROWS), (6, 256, 32, 1, 1389, 128, True, FEW_ROWS), (6, 16, 2, 1, 565, 128, False, FEW_ROWS),
])
def test_attention_calls_that_leave_the_tiled_kernel(Bt, Hq, Hkv, Lq, Lk, d, causal, route):
    assert attention_route(Bt, Hq, Hkv, Lq, Lk, d, causal) == route


def test_attention_with_a_workspace():
    from test_gpu_attention_split import SPLIT_ATTENTION, _chunks
    for case in SPLIT_ATTENTION:
        assert 2 <= _chunks(case) <= 32, case
    # (us one launch / split: 14.9 / 16.0, 28.5 / 29.3, 5.5 / 7.9, 22.7 / 50.7, 9.1 / 12.9); the benchmark's prefills; no keys
    for case in [(3, 8, 8, 109, 1115, 128, True), (2, 8, 8, 1097, 2467, 64, True), (3, 2, 1, 8, 276, 64, False),
                 (4, 32, 16, 200, 639, 128, False), (1, 32, 8, 76, 490, 128, False), (4, 32, 32, 2048, 2048, 128, False),
                 (4, 32, 32, 2048, 2048, 128, True), (2, 32, 8, 1000, 3001, 128, True), (1, 4, 4, 3, 0, 128, False),
                 (1, 4, 3, 3, 8192, 128, False), (1, 4, 4, 3, 8192, 96, False), (0, 4, 4, 3, 8192, 128, False)]:
        assert _chunks(case) == 0, case
    assert _chunks((1, 4, 4, 3, 8192, 128, False), torch.float32) == 0
    # the states stay below 128 MB
    for case in [(8, 64, 8, 3000, 8192, 64, True), (1, 1, 1, 100000, 8192, 64, False), (64, 64, 64, 64, 100000, 128, False)]:
        q = torch.empty((case[0], case[1], case[3], case[5]), dtype=torch.bfloat16, device="meta")
        k = torch.empty((case[0], case[2], case[4], case[5]), dtype=torch.bfloat16, device="meta")
        dq, dk = B.tensor_desc(q), B.tensor_desc(k)
        r = ctypes.byref
        assert B.load_library().rf_cascade_attention_workspace_bytes(r(dq), r(dk), r(dk), int(case[6])) <= 128 << 20


F32_FEW_ROWS, F32_TWO_TILES, F32_WAVES16, F32_WAVES8, F32_WAVES4 = 11, 12, 13, 14, 15


@pytest.mark.parametrize("Bt,Hq,Hkv,Lq,Lk,d,causal,routes", [
    # (us with one tile of 16 rows / two: 22.2 / 29.7, 11.4 / 13.8)
    (1, 8, 8, 1017, 516, 128, True, (F32_WAVES8, F32_WAVES4)), (2, 4, 1, 944, 409, 64, True, (F32_WAVES8,)),
    # (148 / 111, 61.9 / 50.3)
    (1, 512, 512, 128, 512, 64, False, (F32_TWO_TILES,)), (1, 64, 64, 128, 1000, 128, False, (F32_TWO_TILES,)),
    (1, 1, 1, 128, 512, 64, False, (F32_FEW_ROWS,)), (2, 8, 8, 200, 520, 128, True, (F32_WAVES8,)), (2, 8, 8, 100, 200, 64, False, (F32_WAVES16,)),
])
def test_fp32_attention_routes(Bt, Hq, Hkv, Lq, Lk, d, causal, routes):
    assert attention_route(Bt, Hq, Hkv, Lq, Lk, d, causal, torch.float32) in routes


def test_attention_grids_of_2_to_32_threads_are_left_to_larger_tiles():
    assert attention_route(1 << 19, 16, 16, 17, 16, 64, False) in TILED       # 2^24 tiles of 16 rows, 2^23 of 128
    assert attention_route(1 << 18, 16, 16, 17, 16, 64, False) != 0


def test_attention_refusals_have_no_route():
    assert attention_route(1, 3, 2, 4, 4, 128, False) == 0
    assert attention_route(1, 2, 2, 4, 4, 96, False) == 0


STREAMING, SHORT_CHUNKS = 1, 2   # rf_diag_splitk_route


@pytest.mark.parametrize("Bt,Hq,Hkv,Lq,Lk,S,route", [
    # few workgroups with long chunks (us streaming / short chunks: 21.9 / 32.7, 10.1 / 13.8, 8.6 / 11.5, 41 / 53)
    (11, 4, 1, 1, 2493, 1, STREAMING), (2, 2, 2, 1, 1726, 2, STREAMING), (9, 4, 1, 1, 2543, 4, STREAMING), (1, 32, 4, 1, 8978, 2, STREAMING),
    (16, 32, 8, 1, 32768, 64, STREAMING),          # K and V beyond the line of 128 MB
    # short chunks, and several row tiles per KV head (25.5 / 21.2, 328 / 106)
    (4, 32, 8, 1, 3001, 32, SHORT_CHUNKS), (1, 4, 1, 1, 100, 64, SHORT_CHUNKS), (38, 8, 1, 4, 2700, 4, SHORT_CHUNKS),
    (2, 64, 8, 128, 2048, 8, SHORT_CHUNKS),
    # two row tiles: 2^24 workgroups of 256 threads would pass a grid's 32 bits, half of them do not
    (1, 1, 1, 17, 64, 1 << 23, STREAMING), (1, 1, 1, 17, 64, (1 << 23) - 1, SHORT_CHUNKS),
])
def test_splitk_routes(Bt, Hq, Hkv, Lq, Lk, S, route):
    q = torch.empty((Bt, Hq, Lq, 128), dtype=torch.bfloat16, device="meta")
    k = torch.empty((Bt, Hkv, Lk, 128), dtype=torch.bfloat16, device="meta")
    assert B.rf_diag_splitk_route(q, k, k, S) == route


@pytest.mark.parametrize("M,K,N,large", [
    # many tokens, few channels, a short axis (us large / small tiles: 7.7 / 13.8, 7.7 / 11.0, 10.2 / 13.5, 6.5 / 8.4)
    (1672, 256, 40, True), (1416, 256, 64, True), (34, 512, 8584, True), (1007, 128, 40, True), (1604, 256, 24, True),
    (4096, 8192, 3584, True), (100, 8192, 8192, True),
    # (35.2 / 6.7, 40.5 / 13.6, 47 / 33.6, 77 / 46)
    (1, 4096, 4096, False), (64, 4096, 4096, False), (256, 4096, 4096, False), (64, 8192, 8192, False), (1, 128, 8, False),
])
def test_fp8_tiles(M, K, N, large):
    assert (B.rf_diag_fp8_quant_gemm_tile(M, K, N)[0] == 128) == large


# ---- what the GPU tests cover, held against the rules: a changed rule must not leave a kernel without a test ----
sys.path.insert(0, __file__.rsplit("/", 1)[0])


def test_every_fp8_tile_has_a_gpu_test():
    from test_gpu_fp8_rows import FP8_TILES
    for tile, _, shape in FP8_TILES:
        assert B.rf_diag_fp8_quant_gemm_tile(*shape) == tile, shape
    held = {2: [(m, n) for m in (16, 32, 64) for n in (16, 32, 64)], 4: [(m, n) for m in (16, 32) for n in (16, 32, 64)],
            8: [(16, n) for n in (16, 32, 64)]}
    assert {(t, h) for t, h, _ in FP8_TILES} == {(t, h) for h, ts in held.items() for t in ts}
    # and the rule takes no other tile, over a grid of sizes
    for M in (1, 7, 16, 33, 100, 260, 545, 1000, 2000, 4096):
        for K in (128, 640, 2048, 2176, 4096, 4224, 8192):
            for N in (8, 136, 520, 1032, 4104, 8200):
                t = B.rf_diag_fp8_quant_gemm_tile(M, K, N)
                assert t[0] == 128 or t in held[2 if K <= 2048 else 4 if K <= 4096 else 8], (M, K, N, t)


def test_every_fp8_two_pass_tile_has_a_gpu_test():
    from test_gpu_fp8_two_pass import TWO_PASS_TILES
    tiles = {(256, 256), (128, 128), (64, 128), (64, 64), (32, 64), (32, 32)}
    assert {t for t, _ in TWO_PASS_TILES} == tiles
    for tile, shape in TWO_PASS_TILES:
        assert B.rf_diag_fp8_quant_gemm_ws_tile(*shape) == tile, shape
    for M in (1, 16, 33, 100, 260, 545, 1000, 2000, 4096, 70000):
        for K in (128, 640, 2048, 4096, 8192):
            for N in (8, 136, 520, 1032, 4104, 8200):
                assert B.rf_diag_fp8_quant_gemm_ws_tile(M, K, N) in tiles | {(0, 0)}, (M, K, N)


def test_every_large_fp8_tile_has_a_gpu_test_in_one_launch():
    """The binding takes two launches for most of what the 128-token tiles serve: cases that the C entry point runs."""
    from test_gpu_fp8_two_pass import LARGE_TILES
    assert {t for t, _ in LARGE_TILES} == {(128, 256), (128, 512)}
    for tile, shape in LARGE_TILES:
        assert B.rf_diag_fp8_quant_gemm_tile(*shape) == tile and shape[1] >= 4096, shape


@pytest.mark.parametrize("M,K,N,two", [
    # few tokens or a short axis stay in one launch (us one launch / two: 6.5 / 7.2, 4.3 / 6.3, 4.7 / 6.0, 13.5 / 11.5 and 3.5 more alone)
    (1, 4096, 4096, False), (1, 1920, 1432, False), (9, 640, 1288, False), (1672, 256, 40, False), (64, 4096, 4096, False),
    # (176 / 130, 48 / 26, 43 / 17, 46 / 19, 22 / 13)
    (4096, 8192, 3584, True), (1348, 3456, 2336, True), (141, 3456, 7200, True), (64, 8192, 8192, True),
    (18, 5248, 5712, True),
    # nothing that rf_fp8_quant_gemm refuses, no axis beyond 32-bit offsets
    (300, 100, 1000, False), (300, 1152, 1001, False), (0, 1152, 1000, False), (300, -128, 1000, False), (300, 1 << 23, 1024, False),
])
def test_fp8_workspace(M, K, N, two):
    nbytes = B.load_library().rf_fp8_quant_gemm_workspace_bytes(M, K, N)
    assert (nbytes > 0) == two and nbytes <= (128 << 20) + (64 << 10)
    assert (B.rf_diag_fp8_quant_gemm_ws_tile(M, K, N) != (0, 0)) == two


def test_moe_workspace_of_a_large_batch_serves_smaller_ones():
    """The size is 4 E bytes for each token and slice, a slice for every round of 256 workgroups of 64 tokens: 16384 rows
    of scores and less than S more, whatever the kernels make of it."""
    size = B.moe_routing_workspace_bytes
    for hd in (64, 1024, 1152, 2176, 4096, 8192):
        for E in (32, 64, 128):
            for S in [*range(1, 20000, 37), 5440, 6000, 8000, 1 << 20, (1 << 31) - 1]:
                slices = 1 if hd <= 1024 else min(-(-256 // -(-S // 64)), 64, hd // 128)
                assert size(S, hd, E) == slices * S * E * 4, (S, hd, E)
    # a program that asks once, for 8000 tokens
    assert all(size(S, 4096, 128) <= size(8000, 4096, 128) for S in range(1, 8001))
    # and what the entry point without a workspace takes of the largest hidden size: every other one is too large for it
    assert [S for S in range(2048, 16385, 512) if size(S, 8192, 128) <= B.MOE_ROUTING_NOALLOC_MAX_BYTES] == [2048, 4096, 8192, 16384]


def test_every_rmsnorm_tile_has_a_gpu_test():
    from test_gpu_rmsnorm_rows import RMSNORM_TILES
    for tile, shape in RMSNORM_TILES:
        assert B.rf_diag_rmsnorm_gemm_tile(*shape) == tile, shape
    tiles = {(16, 32), (16, 64), (32, 32), (32, 64), (32, 128), (64, 64), (64, 128)}
    assert {t for t, _ in RMSNORM_TILES} == tiles
    for M in (1, 16, 33, 100, 270, 600, 1000, 2000, 4096):
        for K in (64, 512, 1088, 4096, 8192):
            for N in (8, 72, 520, 1032, 4104, 8200):
                assert B.rf_diag_rmsnorm_gemm_tile(M, K, N) in tiles | {(128, 512)}, (M, K, N)


def test_every_kernel_of_the_small_rmsnorm_tiles_has_a_gpu_test():
    from test_gpu_rmsnorm_rows import RMSNORM_SMALL_TILES
    tile, straight = B.rf_diag_rmsnorm_gemm_tile, B.rf_diag_rmsnorm_gemm_straight
    for want, shape in RMSNORM_SMALL_TILES:
        assert straight(*shape, shape[2] + 24) == want, shape
    both = {((16, 32), True), ((16, 32), False), ((16, 64), True), ((16, 64), False), ((32, 32), True), ((32, 32), False),
            ((32, 64), False)}
    assert {(tile(*s), want) for want, s in RMSNORM_SMALL_TILES} == both
    for M in (1, 5, 16, 17, 33, 100, 400):
        for K in (64, 256, 512, 2048, 4096, 8192):
            for N in (8, 136, 520, 1032, 4104, 8200):
                if tile(M, K, N) in {t for t, _ in both}:
                    assert (tile(M, K, N), straight(M, K, N)) in both, (M, K, N)


@pytest.mark.parametrize("M,K,N,straight", [
    # one row tile against many columns, a handful of rows (us straight / LDS: 6.9 / 7.4, 5.0 / 5.3, 7.55 / 7.9, 5.65 / 6.1, 6.1 / 6.35)
    (3, 2304, 872, True), (2, 768, 4792, True), (19, 1408, 4784, True), (1, 448, 8776, True), (3, 704, 7608, True),
    # several row tiles, rows of w on the same memory channels (15.3 / 13.6, 14.7 / 12.6, 9.0 / 8.4, 5.8 / 4.1)
    (48, 4096, 4096, False), (16, 4096, 4096, False), (37, 2880, 616, False), (4, 5952, 512, False),
])
def test_small_rmsnorm_products_take_the_kernel_that_serves_them_faster(M, K, N, straight):
    assert B.rf_diag_rmsnorm_gemm_straight(M, K, N) == straight


def test_every_rmsnorm_two_pass_tile_has_a_gpu_test():
    from test_gpu_rmsnorm_two_pass import NORM_TILES
    tiles = {(256, 256), (128, 256), (128, 128), (64, 128), (64, 64)}
    assert {t for t, _ in NORM_TILES} == tiles
    for tile, shape in NORM_TILES:
        assert B.rf_diag_rmsnorm_gemm_ws_tile(*shape) == tile, shape
    for M in (1, 48, 100, 600, 1000, 2000, 4096, 30000):
        for K in (64, 512, 1088, 4096, 8192):
            for N in (8, 520, 1032, 4104, 8200):
                assert B.rf_diag_rmsnorm_gemm_ws_tile(M, K, N) in tiles | {(0, 0)}, (M, K, N)


@pytest.mark.parametrize("M,K,N,two", [
    # (us one launch / two: 12.1 / 18, 5.7 / 8.9, 26.9 / 24.9 and 3.5 more alone, 126.9 / 123.7)
    (48, 4096, 4096, False), (300, 1024, 1024, False), (323, 3200, 4208, False), (4096, 4096, 4096, False), (1, 64, 8, False),
    # (90.7 / 69.3, 62.2 / 41.4, 34.0 / 21.9, 30.3 / 20.0)
    (2048, 4096, 4096, True), (1024, 4096, 4096, True), (600, 2048, 4096, True), (2727, 1152, 1360, True),
    # nothing that rf_rmsnorm_gemm refuses, no axis beyond 32-bit offsets
    (1024, 4000, 4096, False), (1024, 4096, 4097, False), (0, 4096, 4096, False), (1024, -64, 4096, False), (1024, 1 << 22, 4096, False),
])
def test_rmsnorm_workspace(M, K, N, two):
    nbytes = B.load_library().rf_rmsnorm_gemm_workspace_bytes(M, K, N)
    assert (nbytes > 0) == two and nbytes <= (128 << 20) + (64 << 10)
    assert (B.rf_diag_rmsnorm_gemm_ws_tile(M, K, N) != (0, 0)) == two


def test_every_attention_kernel_has_gpu_tests_in_each_head_dimension():
    from test_gpu_few_query_tiles import FEW_ATTENTION
    from test_gpu_parity import ATTN_CASES
    from test_gpu_tiled_attention import TILED_ATTENTION
    for case in TILED_ATTENTION:
        assert attention_route(*case[2:], torch.bfloat16 if case[1] == "bf16" else torch.float32) == case[0], case
    seen = {}
    for case in [*FEW_ATTENTION, *ATTN_CASES, *(c[1:] for c in TILED_ATTENTION)]:
        r = attention_route(*case[1:], torch.bfloat16 if case[0] == "bf16" else torch.float32)
        seen.setdefault((r, case[6]), []).append(case)
    for d in (64, 128):
        for r in (1, 2, 3, 4, KEY_GROUPS, FEW_ROWS, F32_FEW_ROWS, F32_TWO_TILES, F32_WAVES8):
            assert len(seen.get((r, d), [])) >= (1 if r in (3, 12) else 2), (r, d, seen.get((r, d)))
    assert seen[F32_WAVES16, 64] and seen[F32_WAVES4, 128]


def test_types_of_one_name_stay_in_one_source():
    """Every source is a translation unit of namespace rf: a type that two of them define has to be in an unnamed
    namespace (one definition rule)."""
    import glob
    import os
    import re
    where = {}
    for path in sorted(glob.glob(os.path.join(os.path.dirname(B.__file__), "csrc", "*.hip"))):
        unnamed = False
        for line in open(path):
            unnamed = line.startswith("namespace {") or (unnamed and not line.startswith("}  // namespace"))
            m = re.match(r"(?:struct|class|enum class)\s+(\w+)\s*[{:]", line)
            if m and not unnamed:
                where.setdefault(m.group(1), []).append(os.path.basename(path))
    assert where and all(len(files) == 1 for files in where.values()), where
