"""The library under HIP graph capture: every entry point only launches kernels on
the stream it is given (no memset, no synchronisation; where the binding hands a call a
workspace, torch's allocator has it from the graph's pool), so a
sequence of calls can be captured once and replayed.  Each replay is checked
bit for bit against the eager result, with eager work and synchronisations
between the replays, and the eager result is checked against the oracle.
"""
import sys

import numpy as np
import pytest
import torch

from oracle import rf_oracle as O
from paper_2603_10026_amd import inputs as I

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def rf():
    from paper_2603_10026_amd import binding
    binding.load_library()
    return binding


def say(msg):
    print(f"[case] {msg}", flush=True)
    sys.stdout.flush()


def test_captured_sequence_replays_bit_exact(rf):
    say("graph capture of softmax, prefill, split-K + merge, RMSNorm+GEMM, variance, routing, FP8 GEMM")
    seed = I.SEED_BASE + 40
    xs = I.to_torch(I.softmax_inputs(seed, 70, 2048, 2.0, "bf16"), "bf16", DEV)
    q, k, v = (I.to_torch(a, "bf16", DEV) for a in I.attention_inputs(seed + 1, 1, 4, 2, 300, 300, 128, "bf16"))
    qd, kd, vd = (I.to_torch(a, "bf16", DEV) for a in I.attention_inputs(seed + 2, 2, 8, 2, 1, 1500, 128, "bf16"))
    xg, gg, wg = (I.to_torch(a, "bf16", DEV) for a in I.rmsnorm_gemm_inputs(seed + 3, 200, 256, 520))
    xv = I.to_torch(I.variance_inputs(seed + 4, 33, 5000, "f32", 1.0, 2.0), "f32", DEV)
    xm, wm = I.moe_routing_inputs_device(seed + 5, 256, 512, 64, 1.5, "bf16", DEV)
    af, wf = I.fp8_quant_gemm_inputs_device(seed + 6, 200, 256, 520, DEV)
    scale = I.default_scale(128)
    S = 6

    out = dict(
        sm=torch.empty_like(xs), o=torch.empty_like(q), od=torch.empty_like(qd),
        y=torch.empty((200, 520), dtype=torch.bfloat16, device=DEV),
        mean=torch.empty(33, dtype=torch.float32, device=DEV), var=torch.empty(33, dtype=torch.float32, device=DEV),
        prob=torch.empty((256, 4), dtype=torch.float32, device=DEV), idx=torch.empty((256, 4), dtype=torch.int32, device=DEV),
        c=torch.empty((200, 520), dtype=torch.bfloat16, device=DEV))
    pm, pl, pacc = rf.alloc_partial_states(qd, S)
    ws = torch.empty(max(rf.moe_routing_workspace_bytes(256, 512, 64), 16), dtype=torch.uint8, device=DEV)

    def sequence():
        rf.rf_safe_softmax(xs, out["sm"])
        rf.rf_cascade_attention(q, k, v, scale, causal=True, o=out["o"])
        rf.rf_cascade_attention_splitk(qd, kd, vd, S, pm, pl, pacc, scale)
        rf.rf_merge_states(pm, pl, pacc, out["od"])
        rf.rf_rmsnorm_gemm(xg, gg, wg, eps=1e-6, y=out["y"])
        rf.rf_variance(xv, out["mean"], out["var"])
        rf.rf_moe_routing(xm, wm, 4, prob=out["prob"], idx=out["idx"], workspace=ws)
        rf.rf_fp8_quant_gemm(af, wf, c=out["c"])

    sequence()
    torch.cuda.synchronize()
    eager = {n: t.clone() for n, t in out.items()}

    # the eager results themselves are right
    ref = O.attention(I.to_numpy(q), I.to_numpy(k), I.to_numpy(v), scale, True)
    err = float(np.max(np.abs(I.to_numpy(eager["o"]) - ref)))
    assert err <= 2e-2 * float(np.max(np.abs(ref)))
    m_ref, v_ref = O.variance(I.to_numpy(xv))
    assert float(np.max(np.abs(I.to_numpy(eager["var"]) - v_ref))) <= 1e-5 * float(np.max(np.abs(v_ref)))

    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        sequence()                      # warm-up on the capture stream
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        sequence()

    for rep in range(4):
        for t in out.values():
            t.zero_()                   # eager work between the replays
        pacc.fill_(float("nan"))        # stale partial states must not leak into a replay
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for n, t in out.items():
            assert torch.equal(t.view(torch.uint8), eager[n].view(torch.uint8)), f"replay {rep}: {n} differs from eager"
        # eager launches of the same entry points still work after a replay
        sequence()
        torch.cuda.synchronize()
        for n, t in out.items():
            assert torch.equal(t.view(torch.uint8), eager[n].view(torch.uint8)), f"eager after replay {rep}: {n} differs"
