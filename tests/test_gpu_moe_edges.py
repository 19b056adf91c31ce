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
