"""The tiled attention kernels against the fp64 oracle, in calls with heads enough that they are not left to the
kernels for idle chips (small sizes alone no longer reach them): tails of query and key tiles, fewer keys than a
tile or than queries, large logits, negative and zero scale.  Every case names the kernel it is meant for, by
the number that rf_diag_attention_route gives (checked here and, without a GPU, in test_routes.py)."""
import sys

import numpy as np
import pytest
import torch

from oracle import rf_oracle as O
from paper_2603_10026_amd import inputs as I

sys.path.insert(0, __file__.rsplit("/", 1)[0])
from test_gpu_parity import DEV, check, rf, say  # noqa: E402,F401

pytestmark = pytest.mark.gpu

TILED_ATTENTION = [
    # route, dtype, B, Hq, Hkv, Lq, Lk, d, causal
    # 128 query rows per workgroup: a one-row tail tile, Lk = 64 k + 1, Lk < 64, Lk < Lq, one key, a ragged only tile
    (1, "bf16", 8, 32, 32, 129, 129, 128, True), (1, "bf16", 8, 32, 8, 128, 65, 128, False), (1, "bf16", 8, 32, 32, 200, 90, 128, True),
    (1, "bf16", 8, 32, 32, 40, 20, 128, False), (1, "bf16", 4, 40, 40, 130, 193, 128, True),
    (1, "bf16", 8, 32, 32, 129, 40, 64, True), (1, "bf16", 8, 32, 8, 100, 65, 64, False), (1, "bf16", 8, 32, 32, 129, 129, 64, True),
    (1, "bf16", 8, 32, 32, 100, 1, 64, False),
    # 256 query rows
    (2, "bf16", 8, 32, 32, 257, 65, 128, False), (2, "bf16", 4, 40, 40, 300, 20, 128, False), (2, "bf16", 8, 32, 32, 257, 33, 64, False),
    # two tiles of 128 query rows: keys for the last tile's last rows only
    (4, "bf16", 1, 128, 128, 769, 40, 64, True),
    # keys over two groups of wavefronts, Lk < Lq: tiles that see no key, or that one group alone sees
    (5, "bf16", 1, 32, 32, 512, 400, 64, True), (5, "bf16", 1, 32, 32, 512, 400, 128, True),
    # fp32, d = 128: two tiles of 16 rows per workgroup, one over 8 wavefronts, one over 4
    (12, "f32", 1, 64, 64, 128, 520, 128, False), (12, "f32", 2, 64, 8, 33, 129, 64, False),
    (14, "f32", 2, 8, 8, 200, 520, 128, True), (14, "f32", 1, 16, 16, 100, 600, 128, False),
    (15, "f32", 4, 16, 16, 130, 515, 128, True), (13, "f32", 2, 16, 16, 100, 200, 64, True),
    # fp32, d = 64 over 8 wavefronts: whole groups of key tiles, a ragged one behind them and alone
    (14, "f32", 4, 32, 32, 32, 512, 64, False), (14, "f32", 4, 32, 32, 20, 1100, 64, True), (14, "f32", 4, 32, 32, 17, 515, 64, False),
]


@pytest.mark.parametrize("route,dtype,B,Hq,Hkv,Lq,Lk,d,causal", TILED_ATTENTION)
def test_tiled_attention(rf, route, dtype, B, Hq, Hkv, Lq, Lk, d, causal):  # noqa: F811
    say(f"tiled attention {dtype} B{B} Hq{Hq} Hkv{Hkv} Lq{Lq} Lk{Lk} d{d} causal={causal}")
    q, k, v = I.attention_inputs(I.SEED_BASE + 76, B, Hq, Hkv, Lq, Lk, d, dtype)
    tq, tk, tv = (I.to_torch(a, dtype, DEV) for a in (q, k, v))
    assert rf.rf_diag_attention_route(tq, tk, tv, causal) == route
    o = rf.rf_cascade_attention(tq, tk, tv, I.default_scale(d), causal, o=torch.full_like(tq, float("nan")))
    torch.cuda.synchronize()
    check(o, O.attention(q, k, v, I.default_scale(d), causal), dtype, "tiled attention")


@pytest.mark.parametrize("route,B,H,Lq,Lk,d,causal", [
    (1, 8, 32, 100, 193, 128, False), (1, 8, 32, 129, 129, 64, True), (2, 8, 32, 257, 130, 128, False), (2, 8, 32, 257, 130, 64, False),
    (3, 1, 176, 700, 700, 128, True), (5, 2, 32, 200, 333, 64, False), (5, 1, 48, 250, 450, 128, False), (6, 1, 2, 160, 160, 128, False),
])
def test_attention_large_logits_negative_and_zero_scale(rf, route, B, H, Lq, Lk, d, causal):  # noqa: F811
    """Logits of +-100 and more, in the first and in late key tiles: the reference point moves by leaps, the two
    key groups merge states with references far apart.  The same with the order of the scores reversed, and with
    all scores equal."""
    say(f"attention large logits B{B} H{H} Lq{Lq} Lk{Lk} d{d} causal={causal}")
    q, k, v = I.attention_inputs(I.SEED_BASE + 77, B, H, H, Lq, Lk, d, "bf16")
    q[:, :, 3::7] = I.bf16_round(q[:, :, 3::7] * 30.0)
    k[:, ::2, Lk - 5] = I.bf16_round(q[:, ::2, Lq - 1] * 4.0)
    k[:, 1::2, 2] = I.bf16_round(q[:, 1::2, Lq - 1] * 4.0)
    tq, tk, tv = (I.to_torch(a, "bf16", DEV) for a in (q, k, v))
    assert rf.rf_diag_attention_route(tq, tk, tv, causal) == route
    for scale in (I.default_scale(d), -I.default_scale(d), 0.0):
        o = rf.rf_cascade_attention(tq, tk, tv, scale, causal)
        torch.cuda.synchronize()
        check(o, O.attention(q, k, v, scale, causal), "bf16", f"attention large logits, scale {scale:.3f}")
