"""MoE routing at the edges of its token tiles (16, 32, 64), of the single-segment rule (1024 k) and
of the slices, and with infinite scores."""
import sys

import pytest
import torch

from paper_2603_10026_amd import inputs as I

sys.path.insert(0, __file__.rsplit("/", 1)[0])
from test_gpu_parity import DEV, check_routing, rf, say  # noqa: E402,F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,hd,E,topk", [
    (15, 128, 128, 16), (16, 896, 64, 8), (17, 1024, 32, 3), (1, 1152, 128, 8), (16, 2176, 32, 4), (33, 1152, 64, 16),
    (65, 4096, 128, 8), (31, 8192, 128, 2), (1000, 1280, 128, 8),
])
def test_moe_routing_edges(rf, S, hd, E, topk):  # noqa: F811
    say(f"moe_routing edges S{S} hd{hd} E{E} top{topk}")
    x, w = I.moe_routing_inputs(I.SEED_BASE + 80 + S, S, hd, E)
    prob, idx = rf.rf_moe_routing(I.to_torch(x, "bf16", DEV), I.to_torch(w, "bf16", DEV), topk)
    torch.cuda.synchronize()
    check_routing(prob, idx, x, w, topk, "moe_routing edges")


@pytest.mark.parametrize("S,hd,E,topk", [
    # 64 tokens per workgroup on a short axis: more than one round of 16 tokens each, ragged last tiles
    (12001, 256, 128, 1), (12050, 128, 64, 2), (16400, 256, 32, 1), (40003, 384, 128, 16),
    # 16 lanes per token in the cascade, and the call just below
    (3584, 1152, 32, 16), (3585, 1152, 32, 16), (4099, 1280, 64, 8), (6001, 1152, 128, 6),
])
def test_moe_routing_many_tokens(rf, S, hd, E, topk):  # noqa: F811
    say(f"moe_routing many tokens S{S} hd{hd} E{E} top{topk}")
    x, w = I.moe_routing_inputs(I.SEED_BASE + 85 + S, S, hd, E)
    tx, tw = I.to_torch(x, "bf16", DEV), I.to_torch(w, "bf16", DEV)
    prob, idx = rf.rf_moe_routing(tx, tw, topk)
    torch.cuda.synchronize()
    rows = list(range(0, S, 37)) + list(range(S - 40, S))
    check_routing(prob[rows], idx[rows], x[rows], w, topk, "moe_routing many tokens")
    # every token against the same call on a few tokens at a time (other kernels, other orders of the sums):
    # the same decisions but where two scores lie within their error
    part = [rf.rf_moe_routing(tx[i:i + 2000], tw, topk) for i in range(0, S, 2000)]
    same = (torch.cat([p[1] for p in part]) == idx).double().mean()
    assert float(same) >= 0.999
    assert float((torch.cat([p[0] for p in part]) - prob).abs().max()) <= 1e-5


def test_moe_routing_a_grid_of_more_than_2_to_32_threads(rf):  # noqa: F811
    """One token repeated 140 million times (a row pitch of 0): 8.75 million workgroups of 512 threads would
    wrap the grid's 32 bits and leave most tokens without a result."""
    S, hd, E, topk = 140_000_000, 128, 32, 16
    say(f"moe_routing S{S}")
    x = torch.randn((1, hd), dtype=torch.float32, generator=torch.Generator().manual_seed(5)).to(DEV, torch.bfloat16).expand(S, hd)
    w = torch.randn((hd, E), dtype=torch.float32, generator=torch.Generator().manual_seed(6)).to(DEV, torch.bfloat16)
    prob = torch.full((S, topk), -1.0, dtype=torch.float32, device=DEV)
    idx = torch.full((S, topk), -1, dtype=torch.int32, device=DEV)
    rf.rf_moe_routing(x, w, topk, prob=prob, idx=idx)
    torch.cuda.synchronize()
    p, i = torch.topk(torch.softmax(x[0].double() @ w.double(), 0), topk)
    assert torch.equal(idx[S - 1].long(), i) and float((prob[S - 1].double() - p).abs().max()) <= 1e-5
    for lo in range(0, S, 10_000_000):
        assert bool((idx[lo:lo + 10_000_000] == idx[S - 1]).all()) and bool((prob[lo:lo + 10_000_000] == prob[S - 1]).all())


def test_moe_routing_infinite_scores(rf):  # noqa: F811
    """An expert whose score is -inf has probability 0 and is never chosen ahead of a finite one."""
    say("moe_routing: -inf scores")
    for hd in (128, 1152):
        x = torch.ones((3, hd), dtype=torch.bfloat16, device=DEV)
        w = torch.zeros((hd, 64), dtype=torch.bfloat16, device=DEV)
        w[0] = torch.arange(64, device=DEV, dtype=torch.bfloat16) / 16
        w[0, 5::2] = float("-inf")
        prob, idx = rf.rf_moe_routing(x, w, 8)
        torch.cuda.synchronize()
        s = w[0].double()
        p, i = torch.topk(torch.softmax(s, 0), 8)
        assert torch.equal(idx[1].long(), i)
        assert float(((prob[1].double() - p) / p).abs().max()) <= 1e-5


@pytest.mark.parametrize("S,hd,E,topk", [
    # token tiles of 32, 64, 128 (128, 64, 32 experts); slices of 1 to 7 tiles of 128 k, uneven ones, more slices than a
    # batch of the cascade (16), one slice of a long axis
    (31, 1152, 128, 8), (33, 8192, 128, 16), (63, 1280, 64, 1), (65, 4224, 64, 8), (127, 2176, 32, 4), (129, 8064, 32, 8),
    (1999, 3712, 128, 6), (2940, 3456, 64, 6), (3257, 1408, 32, 8), (4000, 5504, 128, 2), (8193, 1152, 128, 3), (8200, 2048, 64, 5),
])
def test_moe_routing_slices(rf, S, hd, E, topk):  # noqa: F811
    say(f"moe_routing slices S{S} hd{hd} E{E} top{topk}")
    x, w = I.moe_routing_inputs(I.SEED_BASE + 90 + S, S, hd, E)
    big = torch.full((S, hd + 64), float("nan"), dtype=torch.bfloat16, device=DEV)
    big[:, 8:hd + 8] = I.to_torch(x, "bf16", DEV)
    ws = torch.full((rf.moe_routing_workspace_bytes(S, hd, E) // 4,), float("nan"), dtype=torch.float32, device=DEV)
    prob, idx = rf.rf_moe_routing(big[:, 8:hd + 8], I.to_torch(w, "bf16", DEV), topk, workspace=ws)
    torch.cuda.synchronize()
    rows = sorted(set(range(0, S, 29)) | set(range(max(0, S - 40), S)))
    check_routing(prob[rows], idx[rows], x[rows], w, topk, "moe_routing slices")


@pytest.mark.parametrize("hd", [128, 1152])
@pytest.mark.parametrize("E", [32, 64, 128])
def test_moe_routing_equal_scores_in_every_place(rf, hd, E):  # noqa: F811
    """Scores that are exact sums: equal ones around every place of the TopK, zeros of either sign, negative scores
    only, and NaN, which is nobody's score and everybody's probability."""
    say(f"moe_routing equal scores hd{hd} E{E}")
    gen = torch.Generator().manual_seed(hd + E)
    S = 40
    x = torch.zeros((S, hd), dtype=torch.float32)
    x[:, 0], x[:, 1] = 1.0, 1.0
    w = torch.zeros((hd, E), dtype=torch.float32)
    w[0] = torch.randint(-6, 3, (E,), generator=gen).float() / 4          # many equal scores
    x[20:, 2] = 1.0
    w[2] = torch.randperm(E, generator=gen).float() / 8 - 32.0             # rows from 20 on: mostly distinct, all negative
    for topk in (1, 7, 8, 16):
        prob, idx = rf.rf_moe_routing(x.to(DEV, torch.bfloat16), w.to(DEV, torch.bfloat16), topk)
        torch.cuda.synchronize()
        s = x.double() @ w.double()
        order = torch.argsort(s, dim=1, descending=True, stable=True)[:, :topk]   # equal scores: lowest index first
        assert torch.equal(idx.cpu().long(), order)
        want = torch.gather(torch.softmax(s, 1), 1, order)
        assert float(((prob.cpu().double() - want) / want).abs().max()) <= 1e-5
    z = torch.zeros((hd, E), dtype=torch.float32)
    z[0, ::2] = -0.0                                                       # scores of -0 and 0 are equal
    prob, idx = rf.rf_moe_routing(x.to(DEV, torch.bfloat16), z.to(DEV, torch.bfloat16), 8)
    torch.cuda.synchronize()
    assert bool((idx.cpu() == torch.arange(8, dtype=torch.int32)).all())
    w[0, 3] = float("nan")
    prob, idx = rf.rf_moe_routing(x.to(DEV, torch.bfloat16), w.to(DEV, torch.bfloat16), 8)
    torch.cuda.synchronize()
    s[:, 3] = -1e30
    order = torch.argsort(s, dim=1, descending=True, stable=True)[:, :8]
    assert torch.equal(idx.cpu().long(), order) and bool(torch.isnan(prob).all())


@pytest.mark.parametrize("S,hd,E,topk,error", [
    (2048, 4096, 128, 8, 2.03e-7), (5620, 3200, 128, 8, 2.01e-7), (6000, 8192, 128, 4, 2.68e-7), (2048, 8192, 64, 8, 1.95e-7),
    (4096, 4096, 32, 4, 1.58e-7),
])
def test_moe_routing_error_against_64_bits(rf, S, hd, E, topk, error):  # noqa: F811
    """The probabilities' distance from fp64, as four wavefronts with a quarter of a tile's steps each left it, and a
    seventh more: short slices and long ones that are added up on the way.  (One chain of sums over a slice is 1.3, with
    long slices up to 6 times as far off.)"""
    say(f"moe_routing error S{S} hd{hd} E{E} top{topk}")
    off = []
    for seed in (3, 4, 5):
        x, w = I.moe_routing_inputs_device(seed, S, hd, E, device=DEV)
        prob, idx = rf.rf_moe_routing(x, w, topk)
        torch.cuda.synchronize()
        want = torch.softmax(x.double() @ w.double(), 1).gather(1, idx.long())
        off.append(float((prob.double() - want).norm() / want.norm()))
    print(f"        {off}", flush=True)
    assert sum(off) / 3 <= 1.15 * error


@pytest.mark.parametrize("S,hd,E,error", [(4000, 1920, 128, 1.83e-7), (5000, 2304, 128, 1.82e-7), (5000, 1152, 128, 1.71e-7),
                                          (8000, 1920, 64, 1.61e-7)])
def test_moe_routing_error_of_a_few_slices(rf, S, hd, E, error):  # noqa: F811
    """One to three slices of the axis leave little to add up after them: no further from fp64 than four wavefronts and
    as many slices as the workspace holds were (the bound).  (4 sums for slices of 5 to 8 tiles and none added up before 16:
    1.97, 2.05, 1.77 and 1.76e-7.)"""
    say(f"moe_routing error S{S} hd{hd} E{E}, few slices")
    off = []
    for seed in (3, 4, 5):
        x, w = I.moe_routing_inputs_device(seed, S, hd, E, device=DEV)
        prob, idx = rf.rf_moe_routing(x, w, 8)
        torch.cuda.synchronize()
        want = torch.softmax(x.double() @ w.double(), 1).gather(1, idx.long())
        off.append(float((prob.double() - want).norm() / want.norm()))
    print(f"        {off}", flush=True)
    assert sum(off) / 3 <= error


@pytest.mark.parametrize("hd", [1152, 3072, 4096, 8192])
@pytest.mark.parametrize("S", [1, 31, 32, 33, 64, 65, 97, 128, 129, 225])
def test_moe_routing_wavefronts_without_tokens(rf, S, hd):  # noqa: F811
    """32 experts: a workgroup's four wavefronts take 32 tokens each, and those past the end take none; slices of one
    and of several tiles.  Scores against fp64 (sums of hd products, 2^-24 each and a few), guard rows untouched."""
    say(f"moe_routing 32 experts, S{S} hd{hd}")
    x, w = I.moe_routing_inputs_device(11 + S, S, hd, 32, device=DEV)
    ws = torch.full((rf.moe_routing_workspace_bytes(S, hd, 32) // 4 + 64,), float("nan"), device=DEV)
    prob = torch.full((S + 1, 8), float("nan"), device=DEV)
    idx = torch.full((S + 1, 8), -7, dtype=torch.int32, device=DEV)
    rf.rf_moe_routing(x, w, 8, prob=prob[:S], idx=idx[:S], workspace=ws[:-64].view(torch.uint8))
    torch.cuda.synchronize()
    want = torch.softmax(x.double() @ w.double(), 1)
    top = want.topk(8, 1).values
    assert float((prob[:S].double() - top).abs().max()) <= 4e-6 * float(top.max())
    assert float((want.gather(1, idx[:S].long()) - top).abs().max()) <= 4e-6 * float(top.max())
    assert bool(torch.isnan(prob[S]).all()) and bool((idx[S] == -7).all()) and bool(torch.isnan(ws[-64:]).all())
