"""FP8 quant + GEMM with a workspace: the quantisation and every tile of the contraction of
fp8_quant_gemm_two_pass.hip against the two-pass definition, at the edges of their tiles, of the
pieces that their stages and wavefronts take along k, and of the workspace."""
import ctypes
import sys

import numpy as np
import pytest
import torch

from paper_2603_10026_amd import binding as B
from paper_2603_10026_amd import inputs as I

sys.path.insert(0, __file__.rsplit("/", 1)[0])
import fp8_checks as F  # noqa: E402
from test_gpu_fp8_rows import FP8_TILES  # noqa: E402
from test_gpu_parity import DEV, _fp8_tensor, rf, say  # noqa: E402,F401

pytestmark = pytest.mark.gpu

# (tokens, channels) of the tile and products that take it: ragged in both directions, axes that leave stages,
# wavefronts and vectors of the quantisation without work
TWO_PASS_TILES = [
    ((256, 256), (2521, 256, 6496)), ((256, 256), (2755, 3072, 3800)),
    ((128, 256), (3923, 1152, 4736)), ((128, 256), (978, 3840, 7032)), ((128, 128), (1348, 3456, 2344)), ((128, 128), (641, 8320, 4104)),
    ((64, 128), (141, 3456, 7208)), ((64, 128), (1333, 640, 976)), ((64, 64), (119, 640, 5936)), ((64, 64), (545, 5760, 1736)),
    ((32, 64), (39, 5632, 4552)), ((32, 64), (300, 1152, 1000)), ((32, 32), (36, 7680, 2008)), ((32, 32), (33, 4224, 3080)),
]


def _abi(a, w, c, ws=None, ws_bytes=0):
    """The C entry points themselves."""
    d = [B.tensor_desc(t) for t in (a, w, c)]
    lib, r = B.load_library(), ctypes.byref
    if ws is None:
        return lib.rf_fp8_quant_gemm(r(d[0]), r(d[1]), r(d[2]), B._stream(None))
    return lib.rf_fp8_quant_gemm_ws(r(d[0]), r(d[1]), r(d[2]), ctypes.c_void_p(ws.data_ptr()), ws_bytes, B._stream(None))


def _close(c, ta, tw):
    """c against the definition in fp64, from codes that torch rounds.  Every token is quantised with its whole
    maximum, so what is left is half a bf16 step and the matrix instruction's own sums: it aligns the products of
    an instruction to the largest before it adds them, up to 2^-16 of the products' magnitudes; four times that."""
    m = ta.abs().amax(1, keepdim=True)
    # (448.0 / m would be 448 times a reciprocal: not the IEEE quotient)
    codes = torch.where(m > 0, ta * (torch.full_like(m, 448.0) / m), torch.zeros_like(ta)).to(torch.float8_e4m3fn).double()
    want = codes @ tw.double().T * (m.double() / 448.0)
    mass = codes.abs() @ tw.double().abs().T * (m.double() / 448.0)
    assert bool(((c.double() - want).abs() <= 2.0 ** -8 * want.abs() + 2.0 ** -14 * mass).all())


@pytest.mark.parametrize("tile,shape", TWO_PASS_TILES)
def test_fp8_two_pass_every_tile(rf, tile, shape):  # noqa: F811
    M, K, N = shape
    assert rf.rf_diag_fp8_quant_gemm_ws_tile(M, K, N) == tile
    say(f"fp8_quant_gemm two passes, tile {tile}: M{M} K{K} N{N}")
    a, w, w_bits = I.fp8_quant_gemm_inputs(I.SEED_BASE + 70, M, K, N)
    a[M // 2] = 0.0
    big = torch.full((M + 1, K + 64), float("nan"), dtype=torch.bfloat16, device=DEV)
    big[:M, 8:K + 8] = I.to_torch(a, "bf16", DEV)
    wide = torch.full((N, K + 128), 1.0, device=DEV).to(torch.float8_e4m3fn)
    wide.view(torch.uint8)[:, 16:K + 16] = _fp8_tensor(w_bits).view(torch.uint8)
    c = torch.full((M + 1, N + 16), float("nan"), dtype=torch.bfloat16, device=DEV)
    rf.rf_fp8_quant_gemm(big[:M, 8:K + 8], wide[:, 16:K + 16], c=c[:M, 8:N + 8])
    torch.cuda.synchronize()
    _close(c[:M, 8:N + 8], torch.from_numpy(a).to(DEV), torch.from_numpy(np.asarray(w, dtype=np.float32)).to(DEV))
    assert bool((c[M // 2, 8:N + 8] == 0).all())
    assert bool(torch.isnan(c[:, :8]).all()) and bool(torch.isnan(c[:, N + 8:]).all()) and bool(torch.isnan(c[M]).all())


@pytest.mark.parametrize("M,K,N", [(300, 1152, 1000), (256, 4096, 1032)])
def test_fp8_two_pass_against_the_oracle(rf, M, K, N):  # noqa: F811
    say(f"fp8_quant_gemm two passes, oracle: M{M} K{K} N{N}")
    assert rf.rf_diag_fp8_quant_gemm_ws_tile(M, K, N) != (0, 0)
    a, w, w_bits = I.fp8_quant_gemm_inputs(I.SEED_BASE + 71, M, K, N)
    c = rf.rf_fp8_quant_gemm(I.to_torch(a, "bf16", DEV), _fp8_tensor(w_bits))
    torch.cuda.synchronize()
    F.check(I.to_numpy(c), a, w, "fp8_quant_gemm two passes", first_max_rows=list(range(M)))


def test_fp8_two_pass_infinities_and_nan(rf):  # noqa: F811
    """A token with an infinity or a NaN gives NaN, the others what they gave without it."""
    M, K, N = 300, 1152, 1000
    a, w, w_bits = I.fp8_quant_gemm_inputs(I.SEED_BASE + 72, M, K, N)
    ta, tw = I.to_torch(a, "bf16", DEV), _fp8_tensor(w_bits)
    clean = rf.rf_fp8_quant_gemm(ta, tw)
    ta[7, 5], ta[40, K - 1], ta[299, 600] = float("inf"), float("nan"), float("-inf")
    c = rf.rf_fp8_quant_gemm(ta, tw)
    torch.cuda.synchronize()
    bad = [7, 40, 299]
    assert bool(torch.isnan(c[bad]).all())
    keep = [i for i in range(M) if i not in bad]
    assert torch.equal(c[keep], clean[keep])


def test_fp8_tokens_beyond_the_workspace_go_in_turns(rf):  # noqa: F811
    M, K, N = 33000, 4224, 520
    nbytes = B.load_library().rf_fp8_quant_gemm_workspace_bytes(M, K, N)
    assert 0 < nbytes <= (128 << 20) + (64 << 10) < M * K
    say(f"fp8_quant_gemm in turns: M{M} K{K} N{N}")
    a, w = I.fp8_quant_gemm_inputs_device(I.SEED_BASE + 73, M, K, N, DEV)
    c = rf.rf_fp8_quant_gemm(a, w)
    rows = torch.tensor([0, 1, 255, 256, 31487, 31488, 31743, 31744, 31745, 32000, 32999], device=DEV)
    torch.cuda.synchronize()
    _close(c[rows], a[rows].float(), w.float())
    assert bool(torch.isfinite(c).all())


def test_fp8_workspace_is_checked(rf):  # noqa: F811
    M, K, N = 300, 1152, 1000
    a, w = I.fp8_quant_gemm_inputs_device(I.SEED_BASE + 74, M, K, N, DEV)
    c = torch.empty((M, N), dtype=torch.bfloat16, device=DEV)
    need = B.load_library().rf_fp8_quant_gemm_workspace_bytes(M, K, N)
    ws = torch.zeros(need + 16, dtype=torch.uint8, device=DEV)
    assert _abi(a, w, c, ws, need - 1) == B.RF_ERR_WORKSPACE
    assert _abi(a, w, c, ws[8:], need) == B.RF_ERR_WORKSPACE
    ws.fill_(0xff)                                       # NaN codes: nothing may be read before it is written
    assert _abi(a, w, c, ws[:need], need) == B.RF_OK
    torch.cuda.synchronize()
    assert torch.equal(c, rf.rf_fp8_quant_gemm(a, w))


@pytest.mark.parametrize("tile,held,shape", [t for t in FP8_TILES if B.rf_diag_fp8_quant_gemm_ws_tile(*t[2]) != (0, 0)])
def test_fp8_without_a_workspace(rf, tile, held, shape):  # noqa: F811
    """The single-launch tiles at the sizes that the binding serves with a workspace: the C entry point has none."""
    M, K, N = shape
    say(f"fp8_quant_gemm single launch, tile {tile}: M{M} K{K} N{N}")
    _, w, w_bits = I.fp8_quant_gemm_inputs(I.SEED_BASE + 75, 1, K, N)
    rng = np.random.Generator(np.random.PCG64(75 + M))
    e = rng.integers(-7, 1, size=(M, K))
    e[::3] = np.sort(e[::3], axis=1)
    a = (np.exp2(e) * rng.choice([-1.0, 1.0], size=(M, K))).astype(np.float32)
    c = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV)
    assert _abi(I.to_torch(a, "bf16", DEV), _fp8_tensor(w_bits), c) == B.RF_OK
    torch.cuda.synchronize()
    ta, tw = torch.from_numpy(a).to(DEV).double(), torch.from_numpy(np.asarray(w, dtype=np.float32)).to(DEV).double()
    want, mass = ta @ tw.T, ta.abs() @ tw.abs().T
    assert bool(((c.double() - want).abs() <= 2.0 ** -8 * want.abs() + 2.0 ** -14 * mass).all())


def test_fp8_two_pass_in_a_graph_and_on_streams(rf):  # noqa: F811
    """Replays give the eager result while memory of the workspace's size is handed out, filled and given back
    between them; a call on another stream than the current one does too."""
    M, K, N = 600, 2048, 1032
    assert rf.rf_diag_fp8_quant_gemm_ws_tile(M, K, N) != (0, 0)
    a, w = I.fp8_quant_gemm_inputs_device(I.SEED_BASE + 76, M, K, N, DEV)
    eager = rf.rf_fp8_quant_gemm(a, w)
    c = torch.empty_like(eager)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    rf.rf_fp8_quant_gemm(a, w, c=c, stream=side)
    torch.cuda.synchronize()
    assert torch.equal(c, eager)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rf.rf_fp8_quant_gemm(a, w, c=c)
        rf.rf_fp8_quant_gemm(a, w, c=c)
    nbytes = B.load_library().rf_fp8_quant_gemm_workspace_bytes(M, K, N)
    for _ in range(4):
        c.zero_()
        junk = [torch.full((nbytes,), 0xff, dtype=torch.uint8, device=DEV) for _ in range(3)]
        torch.cuda.synchronize()
        graph.replay()
        junk[0].fill_(0x7f)
        torch.cuda.synchronize()
        assert torch.equal(c, eager)
        del junk
        assert torch.equal(rf.rf_fp8_quant_gemm(a, w), eager)


def test_fp8_in_a_capture_that_torch_does_not_know_of(rf):  # noqa: F811
    """No workspace there (its replays would outlive the memory): the single launch, whatever is replayed when."""
    M, K, N = 600, 2048, 1032
    a, w = I.fp8_quant_gemm_inputs_device(I.SEED_BASE + 77, M, K, N, DEV)
    want, c = (torch.empty((M, N), dtype=torch.bfloat16, device=DEV) for _ in range(2))
    assert _abi(a, w, want) == B.RF_OK
    hip = ctypes.CDLL("libamdhip64.so")
    V = ctypes.c_void_p
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph, execg = V(), V()
    with torch.cuda.stream(side):
        s = V(side.cuda_stream)
        assert hip.hipStreamBeginCapture(s, 0) == 0      # global mode
        rf.rf_fp8_quant_gemm(a, w, c=c)
        assert hip.hipStreamEndCapture(s, ctypes.byref(graph)) == 0
    assert hip.hipGraphInstantiate(ctypes.byref(execg), graph, None, None, ctypes.c_size_t(0)) == 0
    for _ in range(3):
        c.zero_()
        torch.cuda.synchronize()
        assert hip.hipGraphLaunch(execg, s) == 0
        torch.cuda.synchronize()
        assert torch.equal(c, want)
    assert hip.hipGraphExecDestroy(execg) == 0 and hip.hipGraphDestroy(graph) == 0
