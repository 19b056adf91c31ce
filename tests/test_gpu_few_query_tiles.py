"""Attention with few query tiles against the fp64 oracle: the tiles of attention_fewrows.hip and
attention_f32_few.hip and the two key groups of attention_bf16.hip at their edges and on both sides of the rules that choose them."""
import sys

import numpy as np
import pytest
import torch

from oracle import rf_oracle as O
from paper_2603_10026_amd import inputs as I

sys.path.insert(0, __file__.rsplit("/", 1)[0])
from test_gpu_parity import DEV, check, rf, say  # noqa: E402,F401

pytestmark = pytest.mark.gpu


FEW_ATTENTION = [
    # dtype, B, Hq, Hkv, Lq, Lk, d, causal
    ("bf16", 1, 4, 1, 4, 1, 128, False), ("bf16", 2, 6, 2, 5, 31, 64, True), ("bf16", 1, 2, 2, 16, 32, 128, True),
    ("bf16", 1, 8, 2, 17, 129, 64, False), ("bf16", 3, 4, 4, 1, 257, 128, False), ("bf16", 1, 1, 1, 700, 1030, 64, True),
    ("bf16", 1, 3, 1, 33, 20, 128, True),      # Lk < Lq: early rows see no key, tiles span heads
    ("bf16", 8, 8, 8, 40, 100, 64, True),
    # 64 rows per workgroup, the keys over two groups of wavefronts: odd numbers of key tiles, tiles that
    # one group alone sees under the mask, ragged rows and keys
    ("bf16", 2, 32, 8, 197, 318, 64, False), ("bf16", 4, 8, 2, 300, 314, 64, False), ("bf16", 1, 48, 48, 250, 450, 128, False),
    ("bf16", 1, 48, 48, 250, 300, 128, False), ("bf16", 1, 48, 48, 250, 330, 128, True), ("bf16", 1, 64, 64, 200, 260, 64, True),
    ("bf16", 1, 32, 8, 700, 700, 128, True),
    # the tiled kernel from here on: many query tiles
    ("bf16", 8, 32, 32, 200, 130, 64, False), ("bf16", 8, 32, 8, 130, 193, 128, True), ("bf16", 8, 32, 32, 300, 330, 64, True),
    ("f32", 1, 1, 1, 1, 129, 64, False), ("f32", 2, 6, 2, 3, 130, 128, True), ("f32", 1, 4, 1, 5, 511, 64, True),
    ("f32", 1, 2, 2, 7, 513, 128, False), ("f32", 1, 1, 1, 200, 150, 64, True), ("f32", 1, 4, 4, 64, 1100, 64, False),
    # tiles of 16 rows, and of two of them, from here on
    ("f32", 2, 16, 4, 40, 140, 64, True), ("f32", 4, 16, 16, 33, 200, 128, True), ("f32", 4, 32, 32, 50, 140, 64, False),
    ("f32", 8, 32, 32, 65, 100, 64, True), ("f32", 4, 32, 8, 161, 140, 128, True),
]


@pytest.mark.parametrize("dtype,B,Hq,Hkv,Lq,Lk,d,causal", FEW_ATTENTION)
def test_attention_few_query_tiles(rf, dtype, B, Hq, Hkv, Lq, Lk, d, causal):  # noqa: F811
    say(f"attention few tiles {dtype} B{B} Hq{Hq} Hkv{Hkv} Lq{Lq} Lk{Lk} d{d} causal={causal}")
    q, k, v = I.attention_inputs(I.SEED_BASE + 70, B, Hq, Hkv, Lq, Lk, d, dtype)
    scale = -I.default_scale(d) if Lq % 2 else I.default_scale(d)
    if Lk == 31:
        scale = 0.0
    # [B, L, H, d] memory order inside buffers whose other values are NaN: a read past a head's rows
    # that reached the result would show
    def place(a):
        bb, h, ln, dd = a.shape
        t = torch.full((bb, ln + 3, h, dd), float("nan"), dtype=I.to_torch(a, dtype, DEV).dtype, device=DEV)
        t[:, :ln] = I.to_torch(a, dtype, DEV).permute(0, 2, 1, 3)
        return t[:, :ln].permute(0, 2, 1, 3)
    o = place(np.zeros_like(q))
    rf.rf_cascade_attention(place(q), place(k), place(v), scale, causal, o=o)
    torch.cuda.synchronize()
    check(o, O.attention(q, k, v, scale, causal), dtype, "attention few tiles")


def test_splitk_streaming_kernel_agrees_with_the_small_one(rf):  # noqa: F811
    """More than 128 MB of K and V take the streaming kernel; the same call batch by batch takes the
    other.  Their states differ by fp32 rounding and by the bf16 rounding of the probabilities."""
    B, Hq, Hkv, Lq, Lk, S = 4, 24, 8, 7, 16513, 37
    say(f"splitk streaming kernel against the small one B{B} Lk{Lk} S{S}")
    q, k, v = I.attention_inputs_device(I.SEED_BASE + 71, B, Hq, Hkv, Lq, Lk, 128, "bf16", DEV)
    scale = I.default_scale(128)
    whole = rf.alloc_partial_states(q, S)
    rf.rf_cascade_attention_splitk(q, k, v, S, *whole, scale, True)
    for b in range(B):
        part = rf.alloc_partial_states(q[b:b + 1], S)
        rf.rf_cascade_attention_splitk(q[b:b + 1], k[b:b + 1], v[b:b + 1], S, *part, scale, True)
        torch.cuda.synchronize()
        # fp32 scores of 128 products of N(0,1) values: 1e-5; l and acc to the same, acc also 2^-9 per weight
        assert float((whole[0][b] - part[0][0]).abs().max()) <= 1e-4
        assert float(((whole[1][b] - part[1][0]) / part[1][0]).abs().max()) <= 1e-3
        d = (whole[2][b] - part[2][0]).double()
        assert float(d.norm() / part[2][0].double().norm()) <= 2.0 ** -9


@pytest.mark.parametrize("B,Hq,Hkv,Lq,Lk,d,few", [(8, 32, 8, 1, 5, 128, True), (16, 64, 8, 1, 6, 64, True), (16, 16, 2, 2, 40, 128, True),
                                                  (4, 32, 32, 200, 5, 128, False)])
def test_attention_probability_rounding_cancels(rf, B, Hq, Hkv, Lq, Lk, d, few):  # noqa: F811
    """O = acc / l with both sums over the bf16-rounded probabilities: where V has a mean far from zero, here
    values in [1.75, 2), the rounding cancels, and what is left is that of the output, 1/sqrt(12) = 0.289 of
    bf16's spacing there (2^-7) in the mean square.  With l over the unrounded probabilities a row is off by
    another 2^-9 / sqrt(3 Lk) of its value or so, 0.13 of the spacing for five keys: 0.32 in all."""
    route = rf.rf_diag_attention_route(*(torch.empty((B, h, n, d), dtype=torch.bfloat16, device="meta")
                                         for h, n in ((Hq, Lq), (Hkv, Lk), (Hkv, Lk))))
    assert (route == 6) == few, route
    say(f"attention rounding of P: B{B} Hq{Hq} Hkv{Hkv} Lq{Lq} Lk{Lk} d{d}")
    q, k, v = I.attention_inputs(I.SEED_BASE + 75, B, Hq, Hkv, Lq, Lk, d, "bf16")
    rng = np.random.Generator(np.random.PCG64(75))
    v = (1.75 + 2.0 ** -7 * rng.integers(0, 32, size=v.shape)).astype(np.float32)
    o = rf.rf_cascade_attention(*(I.to_torch(a, "bf16", DEV) for a in (q, k, v)), I.default_scale(d))
    torch.cuda.synchronize()
    err = (I.to_numpy(o) - O.attention(q, k, v, I.default_scale(d), False)) * 2.0 ** 7
    rms = float(np.sqrt(np.mean(err ** 2)))
    print(f"        error {rms:.4f} of the spacing", flush=True)
    assert rms <= 0.293
