"""Softmax and variance over rows that start at any element and hold any number of elements, against the fp64
oracle: row lengths around every boundary of the dispatch (one vector, lanes per row, vectors per
lane, wavefronts per row, the registers of a workgroup), at every alignment an element type allows,
x and y aligned differently, in place, with the bytes around every output row left as they were."""
import sys

import numpy as np
import pytest
import torch

from oracle import rf_oracle as O
from paper_2603_10026_amd import inputs as I

sys.path.insert(0, __file__.rsplit("/", 1)[0])
from test_gpu_parity import DEV, check, rf, say  # noqa: E402,F401

pytestmark = pytest.mark.gpu

SOFTMAX_N = {
    "bf16": [1, 7, 8, 9, 31, 33, 63, 65, 129, 255, 257, 511, 513, 1025, 1537, 2049, 3071, 3073, 4095, 4097, 6145, 8191,
             8193, 12289, 24577, 32769, 49153, 65535, 65537],
    "f32": [1, 3, 4, 5, 15, 17, 31, 33, 65, 127, 129, 255, 257, 513, 769, 1025, 1537, 2049, 3073, 4095, 4097, 6145, 8193,
            12289, 24577, 32769, 49153, 65535, 65537],
}


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_softmax_ragged_rows(rf, dtype):  # noqa: F811
    for i, n in enumerate(SOFTMAX_N[dtype]):
        rows = 37 if n < 3000 else 3
        xo, yo = i % 8, (3 * i + 1) % 8           # first element of x and of y: every alignment
        say(f"softmax ragged {dtype} rows={rows} n={n} x+{xo} y+{yo}")
        x = I.softmax_inputs(I.SEED_BASE + 60 + i, rows, n, 2.0, dtype)
        t = I.to_torch(x, dtype, DEV)
        xb = torch.full((rows, n + 9), 50.0, dtype=t.dtype, device=DEV)   # large neighbours: reading one would show
        yb = torch.full((rows, n + 11), -7.0, dtype=t.dtype, device=DEV)
        xb[:, xo:xo + n] = t
        rf.rf_safe_softmax(xb[:, xo:xo + n], yb[:, yo:yo + n])
        torch.cuda.synchronize()
        ref = O.safe_softmax(x)
        check(yb[:, yo:yo + n], ref, dtype, "softmax ragged")
        assert bool((yb[:, :yo] == -7.0).all()) and bool((yb[:, yo + n:] == -7.0).all())
        rf.rf_safe_softmax(xb[:, xo:xo + n], xb[:, xo:xo + n])            # in place
        torch.cuda.synchronize()
        check(xb[:, xo:xo + n], ref, dtype, "softmax ragged in place")
        assert bool((xb[:, :xo] == 50.0).all()) and bool((xb[:, xo + n:] == 50.0).all())


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_variance_ragged_rows(rf, dtype):  # noqa: F811
    for i, n in enumerate(SOFTMAX_N[dtype] + [2047, 4090, 100003]):
        for rows in ((37, 1030) if n < 5000 else (3,)):   # 1024 rows: where 8 vectors per lane are taken
            xo = i % 8
            say(f"variance ragged {dtype} rows={rows} n={n} x+{xo}")
            x = I.variance_inputs(I.SEED_BASE + 70 + i, rows, n, dtype)
            t = I.to_torch(x, dtype, DEV)
            xb = torch.full((rows, n + 9), 1.0e4, dtype=t.dtype, device=DEV)   # large neighbours: reading one would show
            xb[:, xo:xo + n] = t
            mean, var = rf.rf_variance(xb[:, xo:xo + n])
            torch.cuda.synchronize()
            m_ref, v_ref = O.variance(x)
            check(mean, m_ref, "f32", "variance ragged mean")
            if n == 1:
                assert float(var.abs().max()) == 0.0
            else:
                check(var, v_ref, "f32", "variance ragged var")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_variance_mean_of_large_values(rf, dtype):  # noqa: F811
    """A mean is in range wherever its row is, also where the sum of the row, or of one vector of it, is
    not: values of 1e36 and of 2e38, in rows of less than a vector up to the longest that stay in
    registers and beyond, aligned or not."""
    for n in (3, 5, 33, 64, 250, 1000, 1537, 2047, 2048, 20000, 20001):
        for rows in (3, 1030) if n < 5000 else (3,):
            for big in (1e36, 2e38):
                say(f"variance of large values {dtype} rows={rows} n={n} {big}")
                rng = np.random.Generator(np.random.PCG64(n))
                x = I.bf16_round((rng.uniform(0.5, 1.5, (rows, n)) * big).astype(np.float32))
                x[1] = -x[1]
                if big < 1e38:
                    x[2, ::2] *= -0.5
                mean, var = rf.rf_variance(I.to_torch(x, dtype, DEV))
                torch.cuda.synchronize()
                want = x.astype(np.float64).mean(axis=1)
                assert np.all(np.abs(I.to_numpy(mean) - want) <= 1e-5 * big), (n, big)


@pytest.mark.parametrize("mask", ["inf", "lowest"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_softmax_masked_rows(rf, dtype, mask):  # noqa: F811
    """Masked logits, by -inf or by the type's lowest value: a prefix (every lane's first vectors), a
    suffix, scattered ones and whole vectors, in every kernel (several rows per wavefront, one, a
    workgroup, two sweeps), aligned or not.  A row of nothing but the lowest value is uniform, one of
    nothing but -inf is NaN, as by the definition."""
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    mv = float("-inf") if mask == "inf" else torch.finfo(td).min
    for n in (5, 24, 100, 1000, 4096, 4099, 16384, 50001, 65537, 70000, 128256):
        for off in (0, 1):
            say(f"softmax masked by {mask} {dtype} n={n} offset {off}")
            x = torch.from_numpy(I.softmax_inputs(I.SEED_BASE + 90 + n, 6, n, 2.0, dtype)).to(td)
            x[0, : n // 2] = mv
            x[1, n // 2:] = mv
            x[2, ::3] = mv
            x[3, 1:] = mv
            x[4, : n - n // 40 - 1] = mv
            x[5] = mv
            xb = torch.full((6, n + 8), 50.0, dtype=td, device=DEV)
            xb[:, off:off + n] = x.to(DEV)
            y = rf.rf_safe_softmax(xb[:, off:off + n], torch.empty((6, n + 8), dtype=td, device=DEV)[:, off:off + n])
            torch.cuda.synchronize()
            ref = O.safe_softmax(x[:5].double().numpy())
            for r in range(5):                     # row by row: their scales differ
                check(y[r:r + 1], ref[r:r + 1], dtype, f"softmax masked, row {r}")
            if mask == "inf":
                assert bool(torch.isnan(y[5]).all())
            else:
                assert float((y[5].double() * n - 1).abs().max()) <= 1e-2


@pytest.mark.parametrize("dtype,n", [("bf16", 1), ("bf16", 2), ("bf16", 5), ("bf16", 7), ("f32", 1), ("f32", 2), ("f32", 3)])
def test_rows_of_less_than_one_vector(rf, dtype, n):  # noqa: F811
    """A lane per row: row counts around a wavefront and a workgroup, pitched and packed, what lies between the
    rows left as it was."""
    for rows in (1, 63, 64, 255, 257, 1000):
        for gap in (0, 3):
            say(f"tiny rows {dtype} rows={rows} n={n} gap={gap}")
            x = I.softmax_inputs(I.SEED_BASE + 95, rows, n, 2.0, dtype)
            t = I.to_torch(x, dtype, DEV)
            xb = torch.full((rows, n + gap), 50.0, dtype=t.dtype, device=DEV)
            xb[:, :n] = t
            yb = torch.full((rows, n + gap), -7.0, dtype=t.dtype, device=DEV)
            rf.rf_safe_softmax(xb[:, :n], yb[:, :n])
            mean, var = rf.rf_variance(xb[:, :n])
            torch.cuda.synchronize()
            check(yb[:, :n], O.safe_softmax(x), dtype, "softmax tiny rows")
            assert bool((yb[:, n:] == -7.0).all())
            m_ref, v_ref = O.variance(x)
            check(mean, m_ref, "f32", "variance tiny rows, mean")
            if n > 1:
                check(var, v_ref, "f32", "variance tiny rows, var")
            else:
                assert float(var.abs().max()) == 0.0
