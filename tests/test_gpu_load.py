"""The load-time kernels at the edges of their tiles and vectors: the
transpose of W_down (8 x 8 fp16 or 16 x 16 INT8 squares per lane, columns of
any number) byte for byte, and the per-row INT8 quantization (16-byte vectors
held in registers up to 16384 values, single values at the row's end) bit for
bit against the same float32 arithmetic in NumPy, ties, infinities and NaN
included.
"""

import numpy as np
import pytest
import torch

import paper_2411_12692_amd as si

pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.mark.parametrize("k", [1, 7, 8, 17, 127, 256, 515, 1003, 1024])
@pytest.mark.parametrize("d", [128, 640])
def test_transpose_edges(k, d):
    rng = np.random.default_rng(k + d)
    w = rng.integers(0, 1 << 16, (d, k), dtype=np.uint16)  # every bit pattern, NaN among them
    got = si.transpose_down(torch.from_numpy(w.view(np.int16)).to(DEV)).cpu().numpy().view(np.uint16)
    assert np.array_equal(got, w.T)
    q = rng.integers(-128, 128, (d, k), dtype=np.int8)
    assert np.array_equal(si.transpose_down_i8(torch.from_numpy(q).to(DEV)).cpu().numpy(), q.T)


def quantize_ref(w):
    """scale = max |w| / 127 and rint(w / scale) in float32, NaN left out of
    the maximum and clamped like the smallest value."""
    f = w.astype(np.float32)
    with np.errstate(all="ignore"):
        s = (np.fmax.reduce(np.abs(f), axis=1, initial=np.float32(0)) / np.float32(127)).astype(np.float32)
        t = np.rint((f / s[:, None]).astype(np.float32))
    q = np.fmin(np.fmax(t, np.float32(-127)), np.float32(127)).astype(np.int8)
    return np.where(s[:, None] > 0, q, np.int8(0)), s


@pytest.mark.parametrize("n", [1, 7, 8, 9, 2047, 4096, 4097, 4105, 12288, 12296, 16384, 16391, 20003])
def test_quantize_lengths(n):
    rng = np.random.default_rng(n)
    w = np.empty((9, n), np.float16)
    w[:3] = rng.standard_normal((3, n)) * 0.02
    w[3] = rng.integers(-254, 255, n) * 0.5  # halves of the scale 1 (the maximum set below): ties
    w[3, n // 2] = 127.0
    w[4] = rng.integers(-2540, 2541, n) * 2.0 ** -10
    w[5] = rng.integers(-60, 60, n) * 2.0 ** -24  # subnormals
    w[6] = 0
    w[7] = rng.standard_normal(n)
    w[7, n - 1] = np.inf
    w[8] = rng.standard_normal(n)
    w[8, 0] = np.nan
    q, s = si.quantize_rows_i8(torch.from_numpy(w.view(np.int16)).to(DEV))
    qr, sr = quantize_ref(w)
    assert np.array_equal(s.cpu().numpy().view(np.uint32), sr.view(np.uint32))
    assert np.array_equal(q.cpu().numpy(), qr)


def test_quantize_every_quotient_near_a_half():
    """Every fp16 value from 1/8 up to the row's maximum, over every seventh
    fp16 maximum from 1 to 2 (a binade has every fraction of the quotients):
    the product with the inverse must never decide a tie differently from the
    division."""
    maxima = np.arange(1024, 2048, 7).astype(np.uint16) | np.uint16(0x3800)
    vals = np.arange(0x3000, 0x4000, dtype=np.uint16)
    rows = np.broadcast_to(vals, (maxima.size, vals.size)).copy().view(np.float16)
    top = maxima.view(np.float16)
    rows = np.minimum(rows, top[:, None])
    rows[:, 0] = top
    q, s = si.quantize_rows_i8(torch.from_numpy(rows.view(np.int16)).to(DEV))
    qr, sr = quantize_ref(rows)
    assert np.array_equal(s.cpu().numpy().view(np.uint32), sr.view(np.uint32))
    assert np.array_equal(q.cpu().numpy(), qr)
