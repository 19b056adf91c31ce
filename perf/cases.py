"""The work that users of this package have it do, as timed cases.

Every case is one pass through the public binding (``paper_2603_10026_amd.binding``) with the
outputs and workspaces a program keeps between calls already allocated.  ``listed()`` holds the
sizes of the repository's benchmark and of its tables of shapes, and beside them the ordinary
and ragged ones a serving or training program meets: a token batch that is no multiple of a
tile, a context that grows by one key per step, a vocabulary of odd length.  ``draw`` spreads
over the ranges these stand for.
"""
import math

import torch

from paper_2603_10026_amd import binding as rf
from paper_2603_10026_amd import inputs

DEV = "cuda:0"
SIZE = {"bf16": 2, "f32": 4}
TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    return [
        # Attention scores or logits of a large batch, one row per (token, head): the benchmark's
        # memory-bound workload.
        dict(name="softmax_bf16_32768x4096", kind="softmax", dtype="bf16", rows=32768, n=4096),
        # Token sampling: fp32 logits of a batch over a vocabulary of odd length, so that only
        # one row in four starts on a 16-byte boundary.
        dict(name="softmax_f32_256x50001", kind="softmax", dtype="f32", rows=256, n=50001),
        # Prefill of four prompts without a mask: the benchmark's headline workload.
        dict(name="attention_bf16_prefill_b4h32l2048d128", kind="attention", dtype="bf16",
             B=4, Hq=32, Hkv=32, Lq=2048, Lk=2048, d=128, causal=False),
        # A prompt of 3001 tokens prefilled in chunks: the last 1000 queries against the whole
        # context, grouped heads, causal.
        dict(name="attention_bf16_causal_b2h32kv8q1000k3001d128", kind="attention", dtype="bf16",
             B=2, Hq=32, Hkv=8, Lq=1000, Lk=3001, d=128, causal=True),
        # The smallest call of the benchmark: one fp32 head, latency and launch cost.
        dict(name="attention_f32_q128k512d64", kind="attention", dtype="f32",
             B=1, Hq=1, Hkv=1, Lq=128, Lk=512, d=64, causal=False),
        # Long-context decode with grouped heads, split over the keys and merged: the benchmark's
        # largest workload in bytes.
        dict(name="decode_b16h32kv8k32768s64", kind="decode",
             B=16, Hq=32, Hkv=8, Lq=1, Lk=32768, d=128, S=64, causal=False),
        # The same step of a small batch at an ordinary context length.
        dict(name="decode_b4h32kv8k3001s32", kind="decode",
             B=4, Hq=32, Hkv=8, Lq=1, Lk=3001, d=128, S=32, causal=False),
        # Normalisation and projection of a prefill: the benchmark's matrix workload.
        dict(name="rmsnorm_gemm_m4096k4096n4096", kind="rmsnorm_gemm", M=4096, K=4096, N=4096),
        # The same projection for the tokens of one decode step of 48 requests.
        dict(name="rmsnorm_gemm_m48k4096n4096", kind="rmsnorm_gemm", M=48, K=4096, N=4096),
        # Per-token FP8 quantisation and projection, the table's longest contraction.
        dict(name="fp8_quant_gemm_m4096k8192n3584", kind="fp8_quant_gemm", M=4096, K=8192, N=3584),
        # Routing of a prefill's tokens over 128 experts, eight of them each.
        dict(name="moe_routing_s2048hd4096e128top8", kind="moe_routing", S=2048, hd=4096, E=128, topk=8),
        # Row statistics of a small matrix, a middle row of the variance table.
        dict(name="variance_f32_128x8192", kind="variance", dtype="f32", rows=128, n=8192),
    ]


def _log(rng, lo, hi):
    """Whole number between lo and hi, even over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _num_splits(B, Hkv, Lk):
    """Splits a program picks: about a thousand (batch, head, chunk) units, chunks of 64 keys or more."""
    return max(1, min(64, -(-1024 // (B * Hkv)), -(-Lk // 64)))


def _draw_attention(rng, dtype):
    fp32 = dtype == "f32"
    hkv = rng.choice([1, 2, 4, 8, 16])
    causal = rng.random() < 0.5
    lq = _log(rng, 1, 1024 if fp32 else 4096)
    # a mask goes with a context that holds the queries
    lk = _log(rng, max(lq, 16) if causal else 16, 2048 if fp32 else 8192)
    return dict(kind="attention", dtype=dtype, B=_log(rng, 1, 8), Hq=hkv * rng.choice([1, 1, 2, 4]), Hkv=hkv,
                Lq=lq, Lk=lk, d=rng.choice([64, 128]), causal=causal)


def _draw_decode(rng):
    b, hkv, lk = _log(rng, 1, 32), rng.choice([1, 2, 4, 8]), _log(rng, 64, 32768)
    lq = rng.choice([1, 1, 1, 1, 2, 4])  # a few draft tokens now and then
    return dict(kind="decode", B=b, Hq=hkv * rng.choice([1, 4, 4, 8]), Hkv=hkv, Lq=lq, Lk=lk, d=128,
                S=_num_splits(b, hkv, lk), causal=lq > 1)


def _draw_one(rng):
    kind = rng.choice(["softmax", "variance", "attention_bf16", "attention_f32", "decode", "rmsnorm_gemm",
                       "fp8_quant_gemm", "moe_routing"])
    if kind in ("softmax", "variance"):
        return dict(kind=kind, dtype=rng.choice(["bf16", "f32"]), rows=_log(rng, 16, 32768), n=_log(rng, 64, 65536))
    if kind == "attention_bf16":
        return _draw_attention(rng, "bf16")
    if kind == "attention_f32":
        return _draw_attention(rng, "f32")
    if kind == "decode":
        return _draw_decode(rng)
    if kind == "rmsnorm_gemm":
        return dict(kind=kind, M=_log(rng, 1, 4096), K=64 * _log(rng, 8, 128), N=8 * _log(rng, 64, 1024))
    if kind == "fp8_quant_gemm":
        return dict(kind=kind, M=_log(rng, 1, 4096), K=128 * _log(rng, 4, 64), N=8 * _log(rng, 64, 1024))
    return dict(kind=kind, S=_log(rng, 1, 4096), hd=128 * _log(rng, 4, 64), E=rng.choice([32, 64, 128]),
                topk=rng.choice([1, 2, 4, 6, 8]))


def draw(rng):
    """One more case of the listed ranges.  The bounds keep it below the largest listed one."""
    while True:
        case = _draw_one(rng)
        w = work(case)
        flops = 8e9 if case.get("dtype") == "f32" else 1.4e11
        if 2e4 <= w["bytes"] <= 2.7e8 and w["flops"] <= flops:
            return case


def _attention_pairs(case):
    """(query, key) pairs of one head."""
    lq, lk = case["Lq"], case["Lk"]
    if not case["causal"]:
        return lq * lk
    return sum(max(0, min(lk, i + 1 + lk - lq)) for i in range(lq))


def work(case):
    k = case["kind"]
    if k == "softmax":
        # maximum, subtraction and exponential, sum, division
        return {"bytes": 2 * SIZE[case["dtype"]] * case["rows"] * case["n"], "flops": 5 * case["rows"] * case["n"]}
    if k == "variance":
        return {"bytes": SIZE[case["dtype"]] * case["rows"] * case["n"] + 8 * case["rows"],
                "flops": 4 * case["rows"] * case["n"]}
    if k in ("attention", "decode"):
        es = SIZE[case.get("dtype", "bf16")]
        q = case["B"] * case["Hq"] * case["Lq"] * case["d"]
        kv = case["B"] * case["Hkv"] * case["Lk"] * case["d"]
        return {"bytes": es * (2 * q + 2 * kv),
                "flops": 4 * case["B"] * case["Hq"] * case["d"] * _attention_pairs(case)}
    if k == "rmsnorm_gemm":
        m, kk, n = case["M"], case["K"], case["N"]
        return {"bytes": 2 * (m * kk + kk + kk * n + m * n), "flops": 2 * m * kk * n}
    if k == "fp8_quant_gemm":
        m, kk, n = case["M"], case["K"], case["N"]
        return {"bytes": 2 * m * kk + kk * n + 2 * m * n, "flops": 2 * m * kk * n}
    s, hd, e = case["S"], case["hd"], case["E"]
    return {"bytes": 2 * (s * hd + hd * e) + 8 * s * case["topk"], "flops": 2 * s * hd * e}


def prepare(case, seed):
    k = case["kind"]
    st = dict(kind=k)
    if k == "softmax":
        x = inputs.softmax_inputs_device(seed, case["rows"], case["n"], 2.0, case["dtype"], DEV)
        st.update(x=x, y=torch.empty_like(x))
    elif k == "variance":
        x = inputs.variance_inputs_device(seed, case["rows"], case["n"], case["dtype"], device=DEV)
        st.update(x=x, mean=torch.empty(case["rows"], dtype=torch.float32, device=DEV),
                  var=torch.empty(case["rows"], dtype=torch.float32, device=DEV))
    elif k in ("attention", "decode"):
        q, kk, v = inputs.attention_inputs_device(seed, case["B"], case["Hq"], case["Hkv"], case["Lq"], case["Lk"],
                                                  case["d"], case.get("dtype", "bf16"), DEV)
        st.update(q=q, k=kk, v=v, o=torch.empty_like(q), scale=inputs.default_scale(case["d"]),
                  causal=case["causal"])
        if k == "decode":
            st.update(S=case["S"], parts=rf.alloc_partial_states(q, case["S"]))
    elif k == "rmsnorm_gemm":
        x, g, w = inputs.rmsnorm_gemm_inputs_device(seed, case["M"], case["K"], case["N"], device=DEV)
        st.update(x=x, g=g, w=w, y=torch.empty((case["M"], case["N"]), dtype=torch.bfloat16, device=DEV))
    elif k == "fp8_quant_gemm":
        a, w = inputs.fp8_quant_gemm_inputs_device(seed, case["M"], case["K"], case["N"], DEV)
        st.update(a=a, w=w, c=torch.empty((case["M"], case["N"]), dtype=torch.bfloat16, device=DEV))
    else:
        S, topk = case["S"], case["topk"]
        x, w = inputs.moe_routing_inputs_device(seed, S, case["hd"], case["E"], device=DEV)
        ws = max(16, rf.moe_routing_workspace_bytes(S, case["hd"], case["E"]))
        st.update(x=x, w=w, topk=topk, prob=torch.empty((S, topk), dtype=torch.float32, device=DEV),
                  idx=torch.empty((S, topk), dtype=torch.int32, device=DEV),
                  workspace=torch.empty(ws, dtype=torch.uint8, device=DEV))
    return st


def run(st):
    k = st["kind"]
    if k == "softmax":
        return rf.rf_safe_softmax(st["x"], st["y"])
    if k == "variance":
        return rf.rf_variance(st["x"], st["mean"], st["var"])
    if k == "attention":
        return rf.rf_cascade_attention(st["q"], st["k"], st["v"], st["scale"], st["causal"], o=st["o"])
    if k == "decode":
        pm, pl, pacc = st["parts"]
        rf.rf_cascade_attention_splitk(st["q"], st["k"], st["v"], st["S"], pm, pl, pacc, st["scale"], st["causal"])
        return rf.rf_merge_states(pm, pl, pacc, st["o"])
    if k == "rmsnorm_gemm":
        return rf.rf_rmsnorm_gemm(st["x"], st["g"], st["w"], eps=1e-6, y=st["y"])
    if k == "fp8_quant_gemm":
        return rf.rf_fp8_quant_gemm(st["a"], st["w"], c=st["c"])
    return rf.rf_moe_routing(st["x"], st["w"], st["topk"], prob=st["prob"], idx=st["idx"], workspace=st["workspace"])


def tolerance(case):
    """Distance of another correct implementation: about four times what lies between the path
    and the same arithmetic in 64 bits, measured over the listed and some dozens of drawn cases."""
    k = case["kind"]
    if k == "fp8_quant_gemm":
        # Rounding to FP8 under one prefix maximum or under another: two roundings of the same
        # values lie sqrt(2) times one rounding's error (2.6 %) apart, whatever the path.
        return {"rel": 5e-2}
    if k == "moe_routing":
        # fp32 sums of up to 8192 products (2.8e-7 seen); experts whose scores tie within that may swap
        return {"rel": 2e-6, "differ": 1e-3}
    if k == "variance":
        return {"rel": 1e-6}  # 7e-8 seen, both storage types; longer rows sum more
    if case.get("dtype") == "f32":
        return {"rel": 2e-6}  # 2.6e-7 seen; the longest key axes sum more
    return {"rel": 1e-2}  # bf16 outputs and probabilities: 2.4e-3 seen
