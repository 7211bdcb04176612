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


# ----------------------------------------------------------------------------- fp32 path

@pytest.mark.parametrize("M,N,K,acc", [
    (1, 1, 1, 0), (16, 16, 16, 1), (17, 33, 20, 1), (15, 47, 18, 0), (90, 256, 688, 1), (3, 600, 1029, 0),
    (1024, 1024, 132, 0),   # 256 tiles of 64 x 64: the last size of the small-product kernel
    (1025, 1024, 132, 1),   # the first of the other
])
def test_linear_f32_edges(A, M, N, K, acc):
    """Both fp32 products on either side of their rule, with and without
    16-byte loads (K % 4), rows and columns that do not fill a tile."""
    a = W.draw_tensor((M, K), "f32", seed=M)
    w = W.draw_tensor((N, K), "f32", std=0.05, seed=N + K)
    c0 = W.draw_tensor((M, N), "f32", seed=5)
    dims = A.make_dims(256, 4, 4, 64, 688, "f32")
    c = up(c0, "f32").clone()
    A.acache_linear(dims, up(a, "f32"), up(w, "f32"), out=c, accumulate=bool(acc))
    ref = O.from_bits(a, "f32") @ O.from_bits(w, "f32").T + (c0.astype(np.float64) if acc else 0.0)
    assert_close(down(c), ref, "f32", f"linear {M}x{N}x{K}")


@pytest.mark.parametrize("H,Hkv,dh", [(4, 4, 64), (4, 2, 32), (2, 1, 128), (2, 2, 2), (3, 1, 30), (2, 2, 20), (4, 1, 112)])
def test_attention_and_scores_f32_edges(A, H, Hkv, dh):
    """Row tiles of 16 and key tiles of 16 over 8 waves: one key, one row,
    fewer keys than waves' tiles, remainders, requests without rows, absent
    slots (logit 0, value 0); head sizes with and without 16-byte loads."""
    import torch
    rows, keys = [1, 16, 0, 17, 33], [1, 15, 9, 128, 301]
    n_slots = sum(keys) + 5
    q = W.draw_tensor((sum(rows), H * dh), "f32", seed=1)
    kp = W.draw_tensor((n_slots, Hkv * dh), "f32", seed=2)
    vp = W.draw_tensor((n_slots, Hkv * dh), "f32", seed=3)
    slots = W.draw_permutation(n_slots, seed=4)[:sum(keys)].copy()
    slots[[20, 40, sum(keys) - 1]] = [-1, n_slots, n_slots + 7]
    cu_rows = np.concatenate([[0], np.cumsum(rows)]).astype(int).tolist()
    cu_keys = np.concatenate([[0], np.cumsum(keys)]).astype(int).tolist()
    dims = A.make_dims(256, H, Hkv, dh, 128, "f32")
    # pools laid out for 16-byte rows: a row stride that is a multiple of 4
    ld = -(-Hkv * dh // 4) * 4
    pools = []
    for p in (kp, vp):
        t = torch.full((n_slots, ld), float("nan"), device="cuda")
        t[:, :Hkv * dh] = up(p, "f32")
        pools.append(t)
    lse = torch.empty((sum(rows), H), dtype=torch.float32, device="cuda")
    out = A.acache_attention(dims, cu_rows, cu_keys, up(q, "f32"), up_i32(slots), *pools, lse=lse)
    f = lambda a: O.from_bits(a, "f32")  # noqa: E731
    kz = np.concatenate([f(kp).reshape(-1, Hkv, dh), np.zeros((1, Hkv, dh))])
    vz = np.concatenate([f(vp).reshape(-1, Hkv, dh), np.zeros((1, Hkv, dh))])
    sl = np.where((slots < 0) | (slots >= n_slots), n_slots, slots)
    o_ref, lse_ref = O.attention_via_slots(f(q).reshape(-1, H, dh), kz, vz, sl, cu_rows, cu_keys)
    assert_close(down(out), o_ref.reshape(sum(rows), H * dh), "f32", "attention out")
    assert_close(down(lse), lse_ref, "f32", "attention lse")
    # scores of 29 + 0 + 5 masked queries against 37 affix keys
    q_rows = W.draw_permutation(sum(rows), seed=5)[:34]
    cu_q, aff = [0, 29, 29, 34], slots[60:97]
    scores = torch.zeros((3, len(aff)), dtype=torch.float32, device="cuda")
    qa = up(q, "f32")
    if H * dh % 4 == 0:
        A.acache_score(dims, qa, up_i32(q_rows), cu_q, pools[0], up_i32(aff), scores)
        ref = O.scores_via_slots(f(q).reshape(-1, H, dh), q_rows, cu_q, kz[:-1], aff, "affix", None)
        assert_close(down(scores), ref, "f32", "scores")
