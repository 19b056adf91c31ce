"""bf16 attention with a workspace: the chunks of keys, 64 rows and two key groups per workgroup, and the sum of their
states, against the oracle at the edges of tiles, chunks and masks."""
import ctypes
import sys

import pytest
import torch

from oracle import rf_oracle as O
from paper_2603_10026_amd import binding as B
from paper_2603_10026_amd import inputs as I

sys.path.insert(0, __file__.rsplit("/", 1)[0])
from test_gpu_parity import DEV, check, rf, say  # noqa: E402,F401

pytestmark = pytest.mark.gpu

# B, Hq, Hkv, Lq, Lk, d, causal
SPLIT_ATTENTION = [
    # one row and a full tile of 64; key counts around whole tiles of 64; one and several tiles a chunk
    (1, 8, 8, 1, 8192, 128, False), (1, 1, 1, 1, 7989, 64, True), (1, 4, 4, 3, 4065, 128, False), (1, 16, 4, 5, 6000, 64, True),
    (2, 4, 1, 64, 4097, 64, False), (1, 2, 1, 65, 4863, 128, True), (1, 2, 2, 63, 4096, 64, False),
    # causal rows whose chunks are partly or wholly out of sight (more queries than the context before them)
    (1, 1, 1, 2700, 2708, 64, True), (1, 1, 1, 3000, 3072, 128, True), (2, 1, 1, 1598, 5977, 64, True),
    # queries beyond the keys: rows that see nothing
    (1, 1, 1, 3500, 3000, 64, True), (1, 1, 1, 2600, 2200, 128, True),
    # heads that are and are not a multiple of the XCDs
    (2, 8, 8, 242, 7136, 64, True), (3, 2, 2, 31, 4674, 64, True), (2, 16, 8, 8, 2384, 128, True),
]


def _chunks(c, dtype=torch.bfloat16):
    Bt, Hq, Hkv, Lq, Lk, d, causal = c
    q = torch.empty((Bt, Hq, Lq, d), dtype=dtype, device="meta")
    k = torch.empty((Bt, Hkv, Lk, d), dtype=dtype, device="meta")
    return B.rf_diag_attention_ws_chunks(q, k, k, causal)


def _inputs(c, seed):
    Bt, Hq, Hkv, Lq, Lk, d, _ = c
    return I.attention_inputs(seed, Bt, Hq, Hkv, Lq, Lk, d, "bf16")


@pytest.mark.parametrize("case", SPLIT_ATTENTION)
def test_attention_split(rf, case):  # noqa: F811
    Bt, Hq, Hkv, Lq, Lk, d, causal = case
    assert _chunks(case) >= 2
    say(f"attention split {case} into {_chunks(case)} chunks")
    q, k, v = _inputs(case, I.SEED_BASE + 95)
    sc = I.default_scale(d)
    tq, tk, tv = (I.to_torch(a, "bf16", DEV) for a in (q, k, v))
    # k and v inside larger buffers (row and head strides of their own), o between rows of NaN
    big = [torch.full((Bt, Hkv, Lk + 2, d + 24), float("nan"), dtype=torch.bfloat16, device=DEV) for _ in range(2)]
    for b_, t in zip(big, (tk, tv)):
        b_[:, :, 1:Lk + 1, 8:d + 8] = t
    o = torch.full((Bt, Lq + 1, Hq, d), float("nan"), dtype=torch.bfloat16, device=DEV)
    rf.rf_cascade_attention(tq, *(b_[:, :, 1:Lk + 1, 8:d + 8] for b_ in big), sc, causal, o=o[:, :Lq].transpose(1, 2))
    torch.cuda.synchronize()
    check(o[:, :Lq].transpose(1, 2), O.attention(q, k, v, sc, causal), "bf16", f"attention split {case}")
    assert bool(torch.isnan(o[:, Lq]).all())
    if causal and Lq > Lk:
        assert bool((o[:, :Lq - Lk] == 0).all())        # rows that see no key


@pytest.mark.parametrize("case", [(1, 4, 4, 3, 4064, 128, True), (1, 1, 1, 1371, 5000, 64, True)])
@pytest.mark.parametrize("scale", [-0.1, 0.0, 3.0])
def test_attention_split_scales(rf, case, scale):  # noqa: F811
    """Negative and zero scales, and one that makes single keys win: chunks whose maxima lie far apart."""
    assert _chunks(case) >= 2
    say(f"attention split {case} scale {scale}")
    q, k, v = _inputs(case, I.SEED_BASE + 96)
    o = rf.rf_cascade_attention(*(I.to_torch(a, "bf16", DEV) for a in (q, k, v)), scale, case[6])
    torch.cuda.synchronize()
    check(o, O.attention(q, k, v, scale, case[6]), "bf16", f"attention split {case} scale {scale}")


@pytest.mark.parametrize("case", [(1, 8, 8, 5, 5000, 64, False), (1, 1, 1, 1598, 5977, 64, True), (1, 4, 4, 3, 4065, 128, False)])
def test_attention_split_infinities_and_nan(rf, case):  # noqa: F811
    """What is no number stays where fp64 has it: a query of NaN in its row; values of NaN or infinity in their column of
    the rows that see the key; a score of +inf in its row, one of -inf nowhere."""
    Bt, Hq, Hkv, Lq, Lk, d, causal = case
    assert _chunks(case) >= 2
    say(f"attention split {case}: infinities and NaN")
    q, k, v = (I.to_torch(a, "bf16", DEV) for a in _inputs(case, I.SEED_BASE + 99))
    sc, inf, nan = I.default_scale(d), float("inf"), float("nan")
    clean = rf.rf_cascade_attention(q, k, v, sc, causal)
    q[:, 0, Lq - 1, 3] = nan
    v[:, 0, 7, 5], v[:, 0, Lk // 2, 9] = nan, inf
    if Hkv > 2:                                           # scores of either infinity, in heads of their own
        q[:, 1, :, 0], q[:, 2, :, 0] = 1.0, 1.0
        k[:, 1, Lk // 3, 0], k[:, 2, Lk // 3, 0] = inf, -inf
    o = rf.rf_cascade_attention(q, k, v, sc, causal)
    torch.cuda.synchronize()
    qd, kd, vd = (t.double().cpu() for t in (q, k, v))
    kd, vd = (t.repeat_interleave(Hq // Hkv, 1) for t in (kd, vd))
    p = qd @ kd.transpose(2, 3).contiguous() * sc
    if causal:
        p.masked_fill_(torch.ones(Lq, Lk).triu(Lk - Lq + 1).bool(), -inf)
    p = torch.softmax(p, -1)
    want = torch.matmul(p, vd)
    # (0 times what is no number is none either, in the sum over the keys that a row sees not; the kernels skip those tiles)
    hidden = [(key, col) for key, col in ((7, 5), (Lk // 2, 9))]
    o, clean = o.double().cpu(), clean.double().cpu()
    for key, col in hidden:
        sees = torch.arange(Lq) + (Lk - Lq if causal else Lk) >= key
        assert bool((~torch.isfinite(o[:, 0, sees, col])).all())
    assert bool(torch.isnan(o[:, 0, Lq - 1]).all())
    keep = [c for c in range(d) if c not in (5, 9)]
    assert torch.equal(o[:, 0, :Lq - 1][..., keep], clean[:, 0, :Lq - 1][..., keep])
    if Hkv > 2:
        assert bool(torch.isnan(want[:, 1]).all()) and bool(torch.isnan(o[:, 1]).all())
        assert bool(torch.isfinite(o[:, 2]).all())
        assert float((o[:, 2] - want[:, 2]).norm() / want[:, 2].norm()) <= 1e-2
        assert torch.equal(o[:, 3], clean[:, 3])


@pytest.mark.parametrize("case", [(2, 8, 8, 242, 7136, 64, False), (1, 32, 8, 1, 8192, 128, False), (2, 4, 4, 1506, 7356, 64, True),
                                  (1, 4, 4, 64, 6000, 128, False)])
def test_attention_split_is_no_further_from_64_bits_than_one_launch(rf, case):  # noqa: F811
    """Long and short chunks against the single launch of the C entry point, whose few-row kernel holds every new maximum
    of a row exactly.  (With a reference that lags behind the maximum the first two were 3 % further off than it.)"""
    Bt, Hq, Hkv, Lq, Lk, d, causal = case
    assert _chunks(case) >= 2
    say(f"attention split {case}: error against 64 bits")
    lib, r, sc = B.load_library(), ctypes.byref, I.default_scale(d)
    off = {"one": 0.0, "two": 0.0}
    for seed in range(20, 22 if Lq > 100 else 40):
        q, k, v = I.attention_inputs_device(seed, Bt, Hq, Hkv, Lq, Lk, d, "bf16", DEV)
        two = rf.rf_cascade_attention(q, k, v, sc, causal)
        one = torch.empty_like(two)
        assert lib.rf_cascade_attention(*(r(B.tensor_desc(t)) for t in (q, k, v, one)), ctypes.c_float(sc), int(causal),
                                        B._stream(None)) == B.RF_OK
        kd, vd = (t.double().repeat_interleave(Hq // Hkv, 1) for t in (k, v))
        p = torch.matmul(q.double(), kd.transpose(2, 3).contiguous()) * sc
        if causal:
            p.masked_fill_(torch.ones(Lq, Lk, device=DEV).triu(Lk - Lq + 1).bool(), float("-inf"))
        want = torch.matmul(torch.softmax(p, -1), vd)
        off["one"] += float((one.double() - want).norm() ** 2)
        off["two"] += float((two.double() - want).norm() ** 2)
    print(f"        {off}", flush=True)
    assert off["two"] <= off["one"]


def test_attention_split_workspace(rf):  # noqa: F811
    """The C entry point: sizes and alignment are checked, nothing is read before it is written; another stream and
    a graph whose workspace is handed out between replays give the same result."""
    case = (1, 8, 8, 5, 5000, 64, False)
    n = _chunks(case)
    assert n >= 2
    tq, tk, tv = (I.to_torch(a, "bf16", DEV) for a in _inputs(case, I.SEED_BASE + 97))
    sc, o = I.default_scale(64), torch.empty_like(tq)
    d = [B.tensor_desc(t) for t in (tq, tk, tv, o)]
    lib, r = B.load_library(), ctypes.byref
    need = lib.rf_cascade_attention_workspace_bytes(r(d[0]), r(d[1]), r(d[2]), 0)
    assert need == 8 * 5 * n * 66 * 4
    ws = torch.full((need // 4 + 4,), float("nan"), dtype=torch.float32, device=DEV)

    def call(p, nbytes):
        return lib.rf_cascade_attention_ws(r(d[0]), r(d[1]), r(d[2]), r(d[3]), ctypes.c_float(sc), 0, ctypes.c_void_p(p), nbytes,
                                           B._stream(None))
    assert call(ws.data_ptr(), need - 1) == B.RF_ERR_WORKSPACE and call(ws.data_ptr() + 4, need) == B.RF_ERR_WORKSPACE
    assert call(None, need) == B.RF_ERR_WORKSPACE
    assert call(ws.data_ptr(), need) == B.RF_OK
    torch.cuda.synchronize()
    eager = rf.rf_cascade_attention(tq, tk, tv, sc)
    torch.cuda.synchronize()
    assert torch.equal(o, eager)
    side, c = torch.cuda.Stream(), torch.zeros_like(o)
    torch.cuda.synchronize()
    rf.rf_cascade_attention(tq, tk, tv, sc, o=c, stream=side)
    torch.cuda.synchronize()
    assert torch.equal(c, eager)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rf.rf_cascade_attention(tq, tk, tv, sc, o=c)
    for _ in range(3):
        c.zero_()
        junk = [torch.full((need // 4,), float("nan"), device=DEV) for _ in range(3)]
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(c, eager)
        del junk


@pytest.mark.parametrize("case", SPLIT_ATTENTION[:4] + SPLIT_ATTENTION[7:8])
def test_attention_without_a_workspace(rf, case):  # noqa: F811
    """The single launches at sizes that the binding splits: the C entry point has no workspace."""
    Bt, Hq, Hkv, Lq, Lk, d, causal = case
    say(f"attention in one launch {case}")
    q, k, v = _inputs(case, I.SEED_BASE + 98)
    tq, tk, tv = (I.to_torch(a, "bf16", DEV) for a in (q, k, v))
    sc, o = I.default_scale(d), torch.full((Bt, Hq, Lq, d), float("nan"), dtype=torch.bfloat16, device=DEV)
    r = ctypes.byref
    dq, dk, dv, do = (B.tensor_desc(t) for t in (tq, tk, tv, o))
    assert B.load_library().rf_cascade_attention(r(dq), r(dk), r(dv), r(do), ctypes.c_float(sc), int(causal), B._stream(None)) == B.RF_OK
    torch.cuda.synchronize()
    check(o, O.attention(q, k, v, sc, causal), "bf16", f"attention in one launch {case}")
