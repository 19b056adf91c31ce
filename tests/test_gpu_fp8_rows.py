"""FP8 quant + GEMM of a few tokens: the tiles of fp8_quant_gemm_rows.hip against the two-pass
definition at the edges of their tiles, of the runs their wavefronts hold, and of the rule that
chooses them."""
import sys

import numpy as np
import pytest
import torch

from paper_2603_10026_amd import inputs as I

sys.path.insert(0, __file__.rsplit("/", 1)[0])
import fp8_checks as F  # noqa: E402
from test_gpu_parity import DEV, _fp8_tensor, rf, say  # noqa: E402,F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N", [
    # (at least 256 channels: the checks compare root mean squares over a token's n channels, which
    # scatter by 1 / sqrt(2 n) of themselves; 8 channels left the 1.25 bound by chance, 1.26)
    # runs of 2, 4 and 8 tiles of 128 k per wavefront and their remainders; wavefronts without a tile
    (1, 128, 512), (16, 896, 520), (17, 1024, 1032), (31, 2048, 264), (33, 2176, 2056), (64, 3968, 264), (65, 4096, 1000),
    (5, 4224, 264), (48, 8064, 520), (128, 1024, 4104), (200, 2048, 2048), (3, 8192, 264),
    # tiles of 64 tokens x 64 channels; the row counts around the line to the large kernel
    (128, 2048, 8192), (1, 8320, 264), (1000, 256, 1000), (1024, 512, 640),
])
def test_fp8_quant_gemm_few_rows(rf, M, K, N):  # noqa: F811
    say(f"fp8_quant_gemm few rows M{M} K{K} N{N}")
    a, w, w_bits = I.fp8_quant_gemm_inputs(I.SEED_BASE + 60 + M, M, K, N)
    first = list(range(0, M, 3))               # these tokens have their maximum in the first element
    a[first, 0] = I.bf16_round(1.5 * np.max(np.abs(a[first]), axis=1))
    if M > 4:
        a[4] = 0.0
    big = torch.full((M + 1, K + 64), float("nan"), dtype=torch.bfloat16, device=DEV)
    big[:M, 8:K + 8] = I.to_torch(a, "bf16", DEV)
    c = torch.full((M, N + 16), float("nan"), dtype=torch.bfloat16, device=DEV)
    rf.rf_fp8_quant_gemm(big[:M, 8:K + 8], _fp8_tensor(w_bits), c=c[:, 8:N + 8])
    torch.cuda.synchronize()
    F.check(I.to_numpy(c[:, 8:N + 8]), a, w, "fp8_quant_gemm few rows", first_max_rows=first)
    assert bool(torch.isnan(c[:, :8]).all()) and bool(torch.isnan(c[:, N + 8:]).all())


@pytest.mark.parametrize("M,K,N", [(4, 1024, 256), (40, 2048, 520), (16, 4096, 264), (3, 8192, 264), (2000, 1024, 512)])
def test_fp8_quant_gemm_only_the_result_has_to_be_in_range(rf, M, K, N):  # noqa: F811
    """Sums over parts of the contraction axis that leave fp32 while the whole does not: 2^114 times 256 over
    half of the axis, the same less over the other half.  Every product is exact in FP8, so the result is."""
    say(f"fp8_quant_gemm range M{M} K{K} N{N}")
    a = np.full((M, K), 2.0 ** 114, dtype=np.float32)
    a[:, K // 2:] = -(2.0 ** 114)
    a[:, K - 16:] = 0.0
    a[M // 2] *= 0.25
    w = torch.full((N, K), 256.0, device=DEV).to(torch.float8_e4m3fn)
    c = rf.rf_fp8_quant_gemm(I.to_torch(a, "bf16", DEV), w)
    torch.cuda.synchronize()
    want = torch.full((M, N), 2.0 ** 126, dtype=torch.float64)
    want[M // 2] *= 0.25
    assert torch.equal(c.double().cpu(), want)
