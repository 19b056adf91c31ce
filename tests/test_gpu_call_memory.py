"""The memory that the binding hands to calls which take a workspace (bf16 attention cut over the keys, RMSNorm + linear
and FP8 quant + GEMM in two launches): beside a capture on another thread, in a capture that torch does not know of, and
on the stream handle that means another stream to every thread."""
import ctypes
import sys
import threading

import pytest
import torch

from paper_2603_10026_amd import binding as B
from paper_2603_10026_amd import inputs as I

sys.path.insert(0, __file__.rsplit("/", 1)[0])
from test_gpu_parity import DEV, rf, say  # noqa: E402,F401

pytestmark = pytest.mark.gpu

# every one asks for more than torch's 1 MB pool of small blocks holds
ATTENTION = (2, 8, 8, 242, 7136, 64)
RMSNORM = (1164, 960, 1488)
FP8 = (600, 2048, 1032)
OPS = ["attention", "rmsnorm", "fp8"]


class Op:
    """One operation: `call` through the binding, `one` the C entry point without a workspace, which takes `need` bytes."""

    def __init__(self, name):
        lib, r, f = B.load_library(), ctypes.byref, ctypes.c_float
        if name == "attention":
            b, hq, hkv, lq, lk, d = ATTENTION
            t = I.attention_inputs_device(I.SEED_BASE + 110, b, hq, hkv, lq, lk, d, "bf16", DEV)
            sc, self.out = I.default_scale(d), torch.empty_like(t[0])
            self.desc = [B.tensor_desc(x) for x in (*t, self.out)]
            self.need = lib.rf_cascade_attention_workspace_bytes(*(r(x) for x in self.desc[:3]), 0)
            self.call = lambda s=None: B.rf_cascade_attention(*t, sc, False, o=self.out, stream=s)
            self.one = lambda: lib.rf_cascade_attention(*(r(x) for x in self.desc), f(sc), 0, B._stream(None))
        elif name == "rmsnorm":
            t = I.rmsnorm_gemm_inputs_device(I.SEED_BASE + 111, *RMSNORM, device=DEV)
            self.out = torch.empty((RMSNORM[0], RMSNORM[2]), dtype=torch.bfloat16, device=DEV)
            self.desc = [B.tensor_desc(x) for x in (*t, self.out)]
            self.need = lib.rf_rmsnorm_gemm_workspace_bytes(*RMSNORM)
            self.call = lambda s=None: B.rf_rmsnorm_gemm(*t, eps=1e-6, y=self.out, stream=s)
            self.one = lambda: lib.rf_rmsnorm_gemm(*(r(x) for x in self.desc), f(1e-6), B._stream(None))
        else:
            t = I.fp8_quant_gemm_inputs_device(I.SEED_BASE + 112, *FP8, DEV)
            self.out = torch.empty((FP8[0], FP8[2]), dtype=torch.bfloat16, device=DEV)
            self.desc = [B.tensor_desc(x) for x in (*t, self.out)]
            self.need = lib.rf_fp8_quant_gemm_workspace_bytes(*FP8)
            self.call = lambda s=None: B.rf_fp8_quant_gemm(*t, c=self.out, stream=s)
            self.one = lambda: lib.rf_fp8_quant_gemm(*(r(x) for x in self.desc), B._stream(None))
        assert self.need > 1 << 20

    def result(self, fn):
        self.out.zero_()
        torch.cuda.synchronize()
        status = fn()
        assert not isinstance(status, int) or status == B.RF_OK
        torch.cuda.synchronize()
        return self.out.clone()


@pytest.mark.parametrize("name", OPS)
def test_a_call_beside_a_capture_on_another_thread(rf, name):  # noqa: F811
    """The call needs memory that torch has to ask the driver for, while this thread captures in global mode: it gets it,
    and the capture goes on."""
    say(f"{name} beside a capture")
    op = Op(name)
    want = op.result(op.call)
    xs = I.to_torch(I.softmax_inputs(I.SEED_BASE + 113, 70, 2048, 2.0, "bf16"), "bf16", DEV)
    soft, ys = rf.rf_safe_softmax(xs), torch.empty_like(xs)
    side, graph, failed = torch.cuda.Stream(), torch.cuda.CUDAGraph(), []
    op.out.zero_()
    torch.cuda.synchronize()

    def other():
        try:
            op.call(side)
        except Exception as e:  # noqa: BLE001
            failed.append(e)
    with torch.cuda.graph(graph):                        # (gives torch's cached memory back first)
        rf.rf_safe_softmax(xs, ys)
        before = torch.cuda.memory_stats()["segment.all.allocated"]
        t = threading.Thread(target=other)
        t.start()
        t.join()
        after = torch.cuda.memory_stats()["segment.all.allocated"]
    torch.cuda.synchronize()
    assert not failed and after > before                 # memory from the driver, not what was there
    assert torch.equal(op.out, want)
    for _ in range(3):
        ys.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(ys, soft)
        assert torch.equal(op.result(op.call), want)


@pytest.mark.parametrize("name", OPS)
def test_a_capture_that_torch_does_not_know_of(rf, name):  # noqa: F811
    """No workspace there (its replays would outlive the memory): the single launch, whatever is replayed when."""
    say(f"{name} in a capture of HIP's own")
    op = Op(name)
    want = op.result(op.one)
    hip, V = ctypes.CDLL("libamdhip64.so"), ctypes.c_void_p
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    graph, execg = V(), V()
    with torch.cuda.stream(side):
        s = V(side.cuda_stream)
        assert hip.hipStreamBeginCapture(s, 0) == 0      # global mode
        op.call()
        assert hip.hipStreamEndCapture(s, ctypes.byref(graph)) == 0
    assert hip.hipGraphInstantiate(ctypes.byref(execg), graph, None, None, ctypes.c_size_t(0)) == 0
    for _ in range(3):
        op.out.zero_()
        torch.cuda.synchronize()
        assert hip.hipGraphLaunch(execg, s) == 0
        torch.cuda.synchronize()
        assert torch.equal(op.out, want)
        junk = torch.full((op.need,), 0xff, dtype=torch.uint8, device=DEV)
        del junk
    assert hip.hipGraphExecDestroy(execg) == 0 and hip.hipGraphDestroy(graph) == 0


@pytest.mark.parametrize("name", OPS)
def test_the_stream_handle_that_is_another_stream_on_every_thread(rf, name):  # noqa: F811
    """hipStreamPerThread (handle 2): memory given back for one thread's stream must not go to another's, so there is
    none."""
    say(f"{name} on hipStreamPerThread")
    op = Op(name)
    want = op.result(op.one)
    op.out.zero_()
    torch.cuda.synchronize()
    taken = torch.cuda.memory_stats()["allocation.all.allocated"]
    op.call(2)
    torch.cuda.synchronize()
    assert torch.cuda.memory_stats()["allocation.all.allocated"] == taken
    assert torch.equal(op.out, want)
