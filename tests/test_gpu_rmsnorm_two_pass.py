"""RMSNorm + linear with a workspace: the norm and every tile of the product of rmsnorm_gemm_two_pass.hip against the
definition, at the edges of their tiles and stages, and the workspace itself."""
import ctypes
import sys

import pytest
import torch

from paper_2603_10026_amd import binding as B
from paper_2603_10026_amd import inputs as I

sys.path.insert(0, __file__.rsplit("/", 1)[0])
from test_gpu_parity import DEV, rf, say  # noqa: E402,F401

pytestmark = pytest.mark.gpu

# (rows, columns) of the tile and products that take it: ragged in both directions, axes of every form of the norm's
# rows (a wavefront or four a row, 512 to 8192 values held, longer ones)
NORM_TILES = [
    ((256, 256), (3058, 512, 5176)), ((256, 256), (1201, 384, 12968)),
    ((128, 256), (1067, 1408, 5208)), ((128, 256), (1739, 1280, 3024)), ((128, 128), (3437, 1728, 1016)), ((128, 128), (367, 2176, 8136)),
    ((64, 128), (1164, 960, 1488)), ((64, 128), (543, 4032, 3440)), ((64, 64), (2651, 1792, 352)), ((64, 64), (3103, 8128, 168)),
    ((64, 64), (857, 6016, 1032)), ((64, 64), (577, 9024, 1032)),
]


def _inputs(shape, seed):
    return I.rmsnorm_gemm_inputs_device(seed, *shape, device=DEV)


def _close(y, x, g, w, eps):
    """y against the definition in fp64 with x g rounded to bf16, as the entry point promises: what is left is half a
    bf16 step and fp32 sums of K products, 2^-24 K of their magnitudes at the very most (2^-24 sqrt(K) is usual)."""
    xg = (x.float() * g.float()).to(torch.bfloat16).double()
    h = (x.double().square().mean(1, keepdim=True) + eps).rsqrt()
    want, mass = xg @ w.double() * h, xg.abs() @ w.double().abs() * h
    assert bool(((y.double() - want).abs() <= 2.0 ** -8 * want.abs() + 2.0 ** -24 * x.shape[1] * mass).all())


def _abi(x, g, w, y, ws=None, nbytes=0):
    d = [B.tensor_desc(t) for t in (x, g, w, y)]
    r, lib = [ctypes.byref(t) for t in d], B.load_library()
    if ws is None:
        return lib.rf_rmsnorm_gemm(*r, ctypes.c_float(1e-6), B._stream(None))
    return lib.rf_rmsnorm_gemm_ws(*r, ctypes.c_float(1e-6), ctypes.c_void_p(ws.data_ptr()), nbytes, B._stream(None))


@pytest.mark.parametrize("tile,shape", NORM_TILES)
def test_rmsnorm_two_pass_every_tile(rf, tile, shape):  # noqa: F811
    M, K, N = shape
    assert rf.rf_diag_rmsnorm_gemm_ws_tile(M, K, N) == tile
    say(f"rmsnorm_gemm two passes, tile {tile}: M{M} K{K} N{N}")
    x, g, w = _inputs(shape, I.SEED_BASE + 53)
    x[M // 2] = 0.0
    bx = torch.full((M, K + 72), float("nan"), dtype=torch.bfloat16, device=DEV)
    bw = torch.full((K, N + 24), float("nan"), dtype=torch.bfloat16, device=DEV)
    bx[:, 8:K + 8], bw[:, 8:N + 8] = x, w
    y = torch.full((M + 1, N + 16), float("nan"), dtype=torch.bfloat16, device=DEV)
    rf.rf_rmsnorm_gemm(bx[:, 8:K + 8], g, bw[:, 8:N + 8], eps=1e-6, y=y[:M, 8:N + 8])
    torch.cuda.synchronize()
    _close(y[:M, 8:N + 8], x, g, w, 1e-6)
    assert bool((y[M // 2, 8:N + 8] == 0).all())
    assert bool(torch.isnan(y[:, :8]).all()) and bool(torch.isnan(y[:, N + 8:]).all()) and bool(torch.isnan(y[M]).all())


def test_rmsnorm_two_pass_against_one_launch(rf):  # noqa: F811
    """Both meet the same roundings and differ by the order of fp32 sums: one value in a thousand moves, by a bf16
    step.  The C entry points: sizes and alignment are checked, nothing is read before it is written; another stream
    and a graph whose workspace is handed out between replays give the same bits."""
    shape = M, K, N = 1164, 960, 1488
    x, g, w = _inputs(shape, I.SEED_BASE + 54)
    one, two, c = (torch.empty((M, N), dtype=torch.bfloat16, device=DEV) for _ in range(3))
    need = B.load_library().rf_rmsnorm_gemm_workspace_bytes(M, K, N)
    assert need > 0
    ws = torch.full((need + 16,), 0xff, dtype=torch.uint8, device=DEV)
    assert _abi(x, g, w, two, ws, need - 1) == B.RF_ERR_WORKSPACE and _abi(x, g, w, two, ws[8:], need) == B.RF_ERR_WORKSPACE
    assert _abi(x, g, w, two, ws, need) == B.RF_OK and _abi(x, g, w, one) == B.RF_OK
    torch.cuda.synchronize()
    moved = one != two
    assert 0 < float(moved.double().mean()) <= 5e-3
    assert bool(((one.double() - two.double()).abs() <= 2.0 ** -7 * one.double().abs() + 1e-4 * float(one.double().abs().max())).all())
    assert torch.equal(rf.rf_rmsnorm_gemm(x, g, w, eps=1e-6), two)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    rf.rf_rmsnorm_gemm(x, g, w, eps=1e-6, y=c, stream=side)
    torch.cuda.synchronize()
    assert torch.equal(c, two)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rf.rf_rmsnorm_gemm(x, g, w, eps=1e-6, y=c)
    for _ in range(3):
        c.zero_()
        junk = [torch.full((need,), 0xff, dtype=torch.uint8, device=DEV) for _ in range(3)]
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(c, two)
        del junk


@pytest.mark.parametrize("shape", [(1201, 384, 12968), (1164, 960, 1488), (2651, 1792, 352), (857, 6016, 1032), (577, 9024, 1032)])
def test_rmsnorm_two_pass_infinities_and_nan(rf, shape):  # noqa: F811
    """A row with an infinity or a NaN gives NaN, as its scale is 0 or none; the others give what they gave without it."""
    M, K, N = shape
    assert rf.rf_diag_rmsnorm_gemm_ws_tile(M, K, N) != (0, 0)
    say(f"rmsnorm_gemm two passes, infinities and NaN: M{M} K{K} N{N}")
    x, g, w = _inputs(shape, I.SEED_BASE + 56)
    clean = rf.rf_rmsnorm_gemm(x, g, w)
    bad = [0, 7, M // 2, M - 1]
    x[0, 5], x[7, K - 1], x[M // 2, K // 2], x[M - 1, 0] = float("inf"), float("nan"), float("-inf"), float("nan")
    y = rf.rf_rmsnorm_gemm(x, g, w)
    torch.cuda.synchronize()
    assert bool(torch.isnan(y[bad]).all())
    keep = [i for i in range(M) if i not in bad]
    assert torch.equal(y[keep], clean[keep])


def test_rmsnorm_rows_beyond_the_workspace_go_in_turns(rf):  # noqa: F811
    M, K, N = 20001, 4096, 520
    nbytes = B.load_library().rf_rmsnorm_gemm_workspace_bytes(M, K, N)
    assert 0 < nbytes <= (128 << 20) + (64 << 10) < 2 * M * K
    say(f"rmsnorm_gemm in turns: M{M} K{K} N{N}")
    x, g, w = _inputs((M, K, N), I.SEED_BASE + 55)
    y = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV)
    rf.rf_rmsnorm_gemm(x, g, w, eps=1e-6, y=y)
    torch.cuda.synchronize()
    _close(y, x, g, w, 1e-6)
