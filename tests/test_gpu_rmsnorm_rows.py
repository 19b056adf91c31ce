"""RMSNorm + linear at few rows: the tiles of rmsnorm_gemm_rows.hip against the fp64 oracle at the
edges of its row tiles (16, 32, 64), of its column tiles (32, 64, 128, groups of 64 columns over 8
XCDs), at contraction axes that leave some of the 4 wavefronts without a step, and on both sides of
the rule that hands over to the large tiles."""
import sys

import pytest
import torch

from oracle import rf_oracle as O
from paper_2603_10026_amd import inputs as I

sys.path.insert(0, __file__.rsplit("/", 1)[0])
from test_gpu_parity import DEV, check, rf, say  # noqa: E402,F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N", [
    (1, 64, 8), (1, 64, 520), (2, 128, 32), (15, 192, 40), (16, 256, 64), (17, 320, 72), (31, 448, 1032), (33, 576, 4096),
    (47, 64 * 9, 8 * 67), (64, 512, 2048), (65, 512, 2056), (100, 1088, 4096), (128, 256, 8200), (129, 640, 4104),
    (256, 192, 1000), (257, 192, 1000),
    # tiles of 32 and 64 rows x 128 columns, ragged in both directions; then the large tiles
    (100, 512, 8200), (256, 576, 4104), (500, 320, 4096), (1000, 1024, 1000), (2047, 192, 1032), (1500, 128, 4104),
    (3000, 256, 2056),
])
def test_rmsnorm_gemm_few_rows(rf, M, K, N):  # noqa: F811
    say(f"rmsnorm_gemm few rows M{M} K{K} N{N}")
    x, g, w = I.rmsnorm_gemm_inputs(I.SEED_BASE + 50 + M, M, K, N)
    tx, tg, tw = (I.to_torch(a, "bf16", DEV) for a in (x, g, w))
    y = torch.full((M, N + 16), float("nan"), dtype=torch.bfloat16, device=DEV)
    rf.rf_rmsnorm_gemm(tx, tg, tw, eps=1e-6, y=y[:, 8:N + 8])
    torch.cuda.synchronize()
    check(y[:, 8:N + 8], O.rmsnorm_gemm(x, g, w, 1e-6), "bf16", "rmsnorm_gemm few rows")
    assert bool(torch.isnan(y[:, :8]).all()) and bool(torch.isnan(y[:, N + 8:]).all())


# (rows, columns) of the output tile and products that take it: every instance (test_routes.py holds the list
# against the rule)
RMSNORM_TILES = [
    ((16, 32), (16, 256, 64)), ((16, 64), (5, 192, 8200)), ((16, 64), (13, 1088, 8200)), ((32, 32), (270, 192, 40)),
    ((32, 64), (601, 128, 72)), ((32, 128), (41, 320, 8200)), ((64, 64), (1999, 192, 72)), ((64, 64), (2000, 64, 8)),
    ((64, 128), (100, 512, 8200)),
]


@pytest.mark.parametrize("tile,shape", RMSNORM_TILES)
def test_rmsnorm_gemm_every_tile(rf, tile, shape):  # noqa: F811
    assert rf.rf_diag_rmsnorm_gemm_tile(*shape) == tile
    test_rmsnorm_gemm_few_rows(rf, *shape)


def test_rmsnorm_gemm_rows_do_not_depend_on_their_batch(rf):  # noqa: F811
    """A row of a small batch, which the small tiles serve, and the same row in a batch of 4096 rows,
    which the 128 x 512 tiles serve, meet the same bf16 roundings (x g, then y): they differ by the
    order of fp32 sums alone.  Sums of 512 products in two orders lie a few 2^-24 sqrt(512) of their
    terms apart, 2e-6 of y's scale; a bf16 value has 2^-8 to its neighbour, so that moves the rounding
    of about one value in a thousand, by one step.  (Rounding w g instead moved half of them.)"""
    M, K, N = 4096, 512, 4096
    say(f"rmsnorm_gemm: rows of a batch of {M} against the same rows in small batches")
    x, g, w = I.rmsnorm_gemm_inputs_device(I.SEED_BASE + 51, M, K, N, device=DEV)
    whole = rf.rf_rmsnorm_gemm(x, g, w)
    for rows in (1, 16, 33, 48, 100, 300):
        part = rf.rf_rmsnorm_gemm(x[7:7 + rows], g, w).double()
        torch.cuda.synchronize()
        want = whole[7:7 + rows].double()
        moved = float((part != want).double().mean())
        print(f"        {rows} rows: {moved:.2e} of the values moved", flush=True)
        assert moved <= 5e-3, rows
        assert float((part - want).norm() / want.norm()) <= 2e-4, rows
        assert bool(((part - want).abs() <= 2.0 ** -7 * want.abs() + 1e-4 * want.abs().max()).all())


# (tiles of up to 32 rows x 64 columns; w in rows of N + 24) operands straight into registers or through LDS, and products
# that go there: every instance (test_routes.py holds the list against the rule)
STRAIGHT, LDS = True, False
RMSNORM_SMALL_TILES = [
    # pieces of 64 k that leave wavefronts without one, the next 4096 values of g after 64 pieces, a handful of rows
    # against much of w, columns that end in a tile's middle
    (STRAIGHT, (6, 64, 8)), (LDS, (6, 512, 40)), (LDS, (7, 576, 136)), (LDS, (20, 4096, 520)), (LDS, (20, 4160, 264)), (LDS, (37, 8192, 264)),
    (LDS, (40, 8256, 72)), (LDS, (130, 12352, 136)), (STRAIGHT, (5, 4352, 2056)), (LDS, (6, 4352, 2056)), (LDS, (300, 1472, 544)),
    (LDS, (64, 768, 2952)),
    # both sides of the rule: short axes
    (STRAIGHT, (9, 256, 4280)), (STRAIGHT, (153, 256, 744)), (LDS, (153, 320, 744)), (LDS, (153, 512, 744)), (LDS, (153, 576, 744)),
    (STRAIGHT, (5, 192, 8200)), (STRAIGHT, (20, 256, 5192)), (STRAIGHT, (33, 256, 4104)),
    # one row tile before many columns, several row tiles
    (STRAIGHT, (9, 320, 4104)), (LDS, (9, 320, 4080)), (STRAIGHT, (9, 320, 4280)), (STRAIGHT, (13, 1024, 8200)), (STRAIGHT, (13, 1088, 8200)),
    (LDS, (34, 1344, 4192)), (STRAIGHT, (20, 1088, 5192)), (STRAIGHT, (20, 1088, 5208)), (STRAIGHT, (32, 1088, 5192)), (LDS, (33, 1088, 5192)),
    # up to five rows: fewer columns the longer the axis
    (STRAIGHT, (5, 1024, 1288)), (LDS, (5, 1024, 1272)), (LDS, (6, 1024, 1288)), (STRAIGHT, (5, 2112, 648)), (LDS, (5, 2112, 632)),
    (STRAIGHT, (5, 4160, 520)), (LDS, (5, 4160, 504)), (STRAIGHT, (2, 2112, 1736)), (STRAIGHT, (3, 2112, 1736)), (STRAIGHT, (3, 896, 2952)),
    (STRAIGHT, (3, 960, 2952)),
    # rows of w 256 bytes apart or a multiple
    (LDS, (9, 320, 4072)), (LDS, (5, 4352, 2024)),
]


@pytest.mark.parametrize("straight,shape", RMSNORM_SMALL_TILES)
def test_rmsnorm_gemm_few_rows_strided(rf, straight, shape):  # noqa: F811
    M, K, N = shape
    tile = rf.rf_diag_rmsnorm_gemm_tile(M, K, N)
    assert tile in ((16, 32), (16, 64), (32, 32), (32, 64))
    assert rf.rf_diag_rmsnorm_gemm_straight(M, K, N, N + 24) == straight
    say(f"rmsnorm_gemm few rows, strided, tile {tile}: M{M} K{K} N{N}")
    x, g, w = I.rmsnorm_gemm_inputs(I.SEED_BASE + 52 + M, M, K, N)
    bx = torch.full((M, K + 72), float("nan"), dtype=torch.bfloat16, device=DEV)
    bw = torch.full((K, N + 24), float("nan"), dtype=torch.bfloat16, device=DEV)
    bx[:, 8:K + 8], bw[:, 8:N + 8] = I.to_torch(x, "bf16", DEV), I.to_torch(w, "bf16", DEV)
    y = torch.full((M + 1, N + 16), float("nan"), dtype=torch.bfloat16, device=DEV)
    rf.rf_rmsnorm_gemm(bx[:, 8:K + 8], I.to_torch(g, "bf16", DEV), bw[:, 8:N + 8], eps=1e-6, y=y[:M, 8:N + 8])
    torch.cuda.synchronize()
    check(y[:M, 8:N + 8], O.rmsnorm_gemm(x, g, w, 1e-6), "bf16", "rmsnorm_gemm few rows, strided")
    assert bool(torch.isnan(y[:, :8]).all()) and bool(torch.isnan(y[:, N + 8:]).all()) and bool(torch.isnan(y[M]).all())
