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
