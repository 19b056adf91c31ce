"""FP8 quant + GEMM with a workspace: the quantisation and every tile of the contraction of
fp8_quant_gemm_two_pass.hip against the incremental definition and against the single launch, at the
edges of their tiles, of the pieces that their stages and wavefronts take along k, and of the workspace."""
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
    ((256, 256), (2755, 3072, 3800)), ((256, 256), (1408, 6272, 6168)), ((256, 256), (3059, 1536, 5200)),
    ((128, 128), (3923, 1152, 4736)), ((128, 128), (978, 3840, 7032)), ((128, 128), (3247, 512, 4728)),
    ((64, 128), (1348, 3456, 2344)), ((64, 128), (641, 8320, 4104)), ((64, 128), (2102, 512, 7736)),
    ((64, 64), (141, 3456, 7208)), ((64, 64), (119, 640, 5936)), ((64, 64), (545, 5760, 1736)),
    ((32, 64), (39, 5632, 4552)), ((32, 64), (74, 768, 5208)), ((32, 64), (647, 8832, 504)),
    ((32, 32), (33, 4224, 3080)), ((32, 32), (3153, 640, 16)), ((32, 32), (8, 4224, 8)), ((32, 32), (36, 12800, 2008)),
]
# tokens x channels of the single launch's large tiles, over axes that its rings go round many times
LARGE_TILES = [((128, 256), (900, 8320, 5000)), ((128, 256), (131, 4224, 7208)), ((128, 512), (1100, 4224, 7400)), ((128, 512), (1999, 8320, 4104))]


def _abi(a, w, c, ws=None, ws_bytes=0):
    """The C entry points themselves."""
    d = [B.tensor_desc(t) for t in (a, w, c)]
    lib, r = B.load_library(), ctypes.byref
    if ws is None:
        return lib.rf_fp8_quant_gemm(r(d[0]), r(d[1]), r(d[2]), B._stream(None))
    return lib.rf_fp8_quant_gemm_ws(r(d[0]), r(d[1]), r(d[2]), ctypes.c_void_p(ws.data_ptr()), ws_bytes, B._stream(None))


def _dequantised(ta):
    """The elements as quantised with the maximum of their row up to the end of their tile of 128 k, in fp64."""
    M, K = ta.shape
    t = ta.view(M, K // 128, 128)
    m = t.abs().amax(2, keepdim=True).cummax(1).values
    # (448.0 / m would be 448 times a reciprocal: not the IEEE quotient)
    codes = torch.where(m > 0, t * (torch.full_like(m, 448.0) / m), torch.zeros_like(t)).to(torch.float8_e4m3fn).double()
    return (codes * (m.double() / 448.0)).view(M, K)


def _close(c, ta, tw):
    """c against the definition in fp64, from codes that torch rounds.  What is left is half a bf16 step, the
    reciprocals of the rescaling (2^-22 each) and the matrix instruction's own sums: it aligns the products of
    an instruction to the largest before it adds them, up to 2^-16 of the products' magnitudes; four times that."""
    hat = _dequantised(ta)
    want, mass = hat @ tw.double().T, hat.abs() @ tw.double().abs().T
    assert bool(((c.double() - want).abs() <= 2.0 ** -8 * want.abs() + 2.0 ** -14 * mass).all())


def _rising(M, K, seed):
    """Tokens whose maximum moves in almost every tile (a third of them), somewhere, or never; none a power of two."""
    rng = np.random.Generator(np.random.PCG64(seed))
    a = rng.standard_normal((M, K)).astype(np.float32)
    a[::3] *= np.exp2(np.linspace(-6, 3, K)).astype(np.float32)
    a[1::3, :128] *= 8.0
    return I.bf16_round(a)


@pytest.mark.parametrize("tile,shape", TWO_PASS_TILES)
def test_fp8_two_pass_every_tile(rf, tile, shape):  # noqa: F811
    M, K, N = shape
    assert rf.rf_diag_fp8_quant_gemm_ws_tile(M, K, N) == tile
    say(f"fp8_quant_gemm two passes, tile {tile}: M{M} K{K} N{N}")
    _, w, w_bits = I.fp8_quant_gemm_inputs(I.SEED_BASE + 70, 1, K, N)
    a = _rising(M, K, 70 + M)
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


@pytest.mark.parametrize("tile,shape", TWO_PASS_TILES)
def test_fp8_result_does_not_depend_on_a_workspace(rf, tile, shape):  # noqa: F811
    """The binding, which has memory here, and the C entry point without any: the same codes, so the same result up
    to the order of fp32 sums; to the bit where both add a tile of 128 k after the other."""
    M, K, N = shape
    say(f"fp8_quant_gemm with and without a workspace: M{M} K{K} N{N}")
    _, w, w_bits = I.fp8_quant_gemm_inputs(I.SEED_BASE + 78, 1, K, N)
    ta, tw = I.to_torch(_rising(M, K, 78 + M), "bf16", DEV), _fp8_tensor(w_bits)
    one = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device=DEV)
    assert _abi(ta, tw, one) == B.RF_OK
    two = rf.rf_fp8_quant_gemm(ta, tw)
    torch.cuda.synchronize()
    if rf.rf_diag_fp8_quant_gemm_tile(M, K, N)[0] == 128 and tile[0] >= 64:
        assert torch.equal(one, two)
    else:
        # sums that lie on either side of a rounding boundary leave as neighbours: a bf16 step, 2^-7 of the value at
        # most, beside what the sums themselves differ by
        mass = _dequantised(ta.float()).abs() @ tw.double().abs().T
        assert bool(((one.double() - two.double()).abs() <= 2.0 ** -7 * one.double().abs() + 2.0 ** -14 * mass).all())


@pytest.mark.parametrize("M,K,N", [(256, 2944, 1032), (171, 4224, 520), (600, 2048, 1032)])
def test_fp8_two_pass_against_the_oracle(rf, M, K, N):  # noqa: F811
    say(f"fp8_quant_gemm two passes, oracle: M{M} K{K} N{N}")
    assert rf.rf_diag_fp8_quant_gemm_ws_tile(M, K, N) != (0, 0)
    a, w, w_bits = I.fp8_quant_gemm_inputs(I.SEED_BASE + 71, M, K, N)
    first = list(range(0, M, 3))                         # these tokens have their maximum in the first element
    a[first, 0] = I.bf16_round(1.5 * np.max(np.abs(a[first]), axis=1))
    c = rf.rf_fp8_quant_gemm(I.to_torch(a, "bf16", DEV), _fp8_tensor(w_bits))
    torch.cuda.synchronize()
    F.check(I.to_numpy(c), a, w, "fp8_quant_gemm two passes", first_max_rows=first)


@pytest.mark.parametrize("tile,shape", LARGE_TILES)
def test_fp8_large_tiles_without_a_workspace(rf, tile, shape):  # noqa: F811
    """The 128-token tiles of the single launch, which the binding takes only where it has no memory: long axes, late
    maxima, strided operands."""
    M, K, N = shape
    assert rf.rf_diag_fp8_quant_gemm_tile(M, K, N) == tile
    say(f"fp8_quant_gemm single launch, tile {tile}: M{M} K{K} N{N}")
    _, w, w_bits = I.fp8_quant_gemm_inputs(I.SEED_BASE + 79, 1, K, N)
    a = _rising(M, K, 79 + M)
    a[M // 2] = 0.0
    rng = np.random.Generator(np.random.PCG64(80))       # powers of two in rising runs: a @ w^T itself
    a[5::7] = (np.exp2(np.sort(rng.integers(-7, 1, size=(len(a[5::7]), K)), axis=1)) *
               rng.choice([-1.0, 1.0], size=(len(a[5::7]), K))).astype(np.float32)
    big = torch.full((M + 1, K + 64), float("nan"), dtype=torch.bfloat16, device=DEV)
    big[:M, 8:K + 8] = I.to_torch(a, "bf16", DEV)
    wide = torch.full((N, K + 128), 1.0, device=DEV).to(torch.float8_e4m3fn)
    wide.view(torch.uint8)[:, 16:K + 16] = _fp8_tensor(w_bits).view(torch.uint8)
    c = torch.full((M + 1, N + 16), float("nan"), dtype=torch.bfloat16, device=DEV)
    assert _abi(big[:M, 8:K + 8], wide[:, 16:K + 16], c[:M, 8:N + 8]) == B.RF_OK
    torch.cuda.synchronize()
    _close(c[:M, 8:N + 8], torch.from_numpy(a).to(DEV), torch.from_numpy(np.asarray(w, dtype=np.float32)).to(DEV))
    ta, tw = torch.from_numpy(a[5::7]).to(DEV).double(), torch.from_numpy(np.asarray(w, dtype=np.float32)).to(DEV).double()
    want, mass = ta @ tw.T, ta.abs() @ tw.abs().T
    assert bool(((c[5:M:7, 8:N + 8].double() - want).abs() <= 2.0 ** -8 * want.abs() + 2.0 ** -14 * mass).all())
    assert bool(torch.isnan(c[:, :8]).all()) and bool(torch.isnan(c[:, N + 8:]).all()) and bool(torch.isnan(c[M]).all())


@pytest.mark.parametrize("M,K,N", [(600, 2048, 1032), (171, 4224, 520)])
def test_fp8_two_pass_infinities_and_nan(rf, M, K, N):  # noqa: F811
    """A token with an infinity or a NaN gives NaN, the others what they gave without it."""
    assert rf.rf_diag_fp8_quant_gemm_ws_tile(M, K, N) != (0, 0)
    a, w, w_bits = I.fp8_quant_gemm_inputs(I.SEED_BASE + 72, M, K, N)
    ta, tw = I.to_torch(a, "bf16", DEV), _fp8_tensor(w_bits)
    clean = rf.rf_fp8_quant_gemm(ta, tw)
    ta[7, 5], ta[40, K - 1], ta[M - 1, 600] = float("inf"), float("nan"), float("-inf")
    c = rf.rf_fp8_quant_gemm(ta, tw)
    torch.cuda.synchronize()
    bad = [7, 40, M - 1]
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
    M, K, N = 600, 2048, 1032
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
