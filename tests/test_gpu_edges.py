"""Kernels at the sizes where their tiling and their dispatch can go wrong:
edges of tiles and chunks, remainders, the smallest and largest of a range,
and both sides of every rule that picks a kernel.  Against the fp64 oracle,
with the gates of gpu_util (reading of the stated bars)."""

import numpy as np
import pytest

import workloads as W
from oracle import acache_oracle as O
from tests.gpu_util import assert_close, down, up, up_i32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def A():
    from paper_2608_26140_amd import acache
    return acache


# ----------------------------------------------------------------------------- argmax and confidence

@pytest.mark.parametrize("dtype,n", [
    ("bf16", 1), ("bf16", 8), ("bf16", 2048), ("bf16", 2056), ("bf16", 16376), ("bf16", 16384), ("bf16", 16387),
    ("bf16", 32768 + 8), ("bf16", 4 * 8192 + 5), ("f32", 4), ("f32", 1023), ("f32", 8192), ("f32", 4 * 4096 + 3),
])
def test_argmax_positions(A, dtype, n):
    """The largest value at the first and last element, at chunk, wave and
    unrolled-round edges and in the tail; the same value twice (the lowest
    index wins); +inf twice; -inf and NaN rows.  Confidences to fp32 rounding:
    a sum of n terms in a tree of at most n / 1024 + 30 additions, each within
    2^-24, and exponentials within 4 ulp."""
    import torch
    rng = np.random.default_rng(n)
    spots = sorted({min(n - 1, p) for p in (0, 7, 8, 511, 2047, 2048, 8191, 8192, 16383, n // 2, n - 9, n - 1) if p >= 0})
    rows = len(spots) + 5
    vals = np.clip(rng.standard_normal((rows, n)) * 3, -20, 11).astype(np.float32)
    for i, p in enumerate(spots):
        vals[i, p] = 12.0
        if p + 1 < n:
            vals[i, min(n - 1, p + 1 + 3 * i)] = 12.0  # a tie further on
    vals[-1, :] = np.nan
    vals[-2, :] = -np.inf
    vals[-3, :] = np.nan
    vals[-3, n // 2:] = -np.inf
    vals[-4, [n // 3, n - 1]] = np.inf
    vals[-5, ::2] = np.nan
    bits = W.bf16_bits_from_f32(vals) if dtype == "bf16" else vals
    conf = torch.full((rows,), -1.0, dtype=torch.float32, device="cuda")
    out = A.acache_argmax_commit(up(bits, dtype), conf=conf)
    x = O.from_bits(bits, dtype)
    np.testing.assert_array_equal(out.cpu().numpy(), O.greedy_commit(x))
    np.testing.assert_allclose(conf.cpu().numpy(), O.confidence(x), rtol=2.0 ** -24 * (n / 1024 + 40) + 1e-6, atol=1e-30)
