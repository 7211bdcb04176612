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


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n", [64, 1000, 20000])
def test_argmax_any_bits(A, dtype, n):
    """Rows of any bits: NaNs of every kind (quiet, signalling, negative),
    infinities and denormals.  Confidences within the bound of
    test_argmax_positions."""
    import torch
    rng = np.random.default_rng(n)
    exp0, snan, ninf = (0x7F, 0x7F81, 0xFF80) if dtype == "bf16" else (0x7FFFFF, 0x7F800001, 0xFF800000)
    word = 16 if dtype == "bf16" else 32
    sign = 1 << (word - 1)
    bits = rng.integers(0, 1 << word, size=(24, n), dtype=np.uint64)
    bits[:8] = rng.integers(1, exp0 + 1, size=(8, n)) | np.where(rng.random((8, n)) < 0.5, sign, 0)  # denormals
    bits[8:16] = np.where(rng.random((8, n)) < 0.5, snan, bits[:8])
    bits[16:20] = np.where(rng.random((4, n)) < 0.9, sign | snan, ninf)  # nothing above -inf
    bits[20:24, ::3] = snan
    dev = torch.from_numpy(bits.astype(np.uint16).view(np.int16)).view(torch.bfloat16).cuda() if dtype == "bf16" \
        else torch.from_numpy(bits.astype(np.uint32).view(np.int32)).cuda().view(torch.float32)
    wide = bits.astype(np.uint32) << (32 - word)
    with np.errstate(invalid="ignore"):
        x = np.where((wide & 0x7FFFFFFF) > 0x7F800000, np.nan, wide.view(np.float32).astype(np.float64))
        want, want_conf = O.greedy_commit(x), O.confidence(x)
    conf = torch.full((24,), -1.0, dtype=torch.float32, device="cuda")
    out = A.acache_argmax_commit(dev, conf=conf)
    np.testing.assert_array_equal(out.cpu().numpy(), want)
    np.testing.assert_allclose(conf.cpu().numpy(), want_conf, rtol=2.0 ** -24 * (n / 1024 + 40) + 1e-6, atol=1e-30)


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


@pytest.mark.parametrize("keys,lost", [
    (65, [64]),                                     # alone in its tile of 16
    (64, range(16, 32)),                            # all of one wave's keys
    (300, [*range(0, 48), *range(128, 144), 299]),  # some waves' first tile, others' second
])
def test_attention_f32_infinite_logits(A, keys, lost):
    """Keys with a logit of -inf weigh nothing, whichever wave reads them, and
    the affix-normalised scores leave them out."""
    import torch
    H, dh, rows = 2, 32, 20
    q = np.abs(W.draw_tensor((rows, H * dh), "f32", seed=1))
    kp = W.draw_tensor((keys, H * dh), "f32", seed=2)
    vp = W.draw_tensor((keys, H * dh), "f32", seed=3)
    kp[list(lost), ::dh] = -np.inf
    dims = A.make_dims(256, H, H, dh, 128, "f32")
    slots, lse = up_i32(np.arange(keys)), torch.empty((rows, H), dtype=torch.float32, device="cuda")
    out = A.acache_attention(dims, [0, rows], [0, keys], up(q, "f32"), slots, up(kp, "f32"), up(vp, "f32"), lse=lse)
    keep = np.setdiff1d(np.arange(keys), list(lost))
    heads = lambda t: O.from_bits(t, "f32").reshape(-1, H, dh)  # noqa: E731
    o_ref, lse_ref = O.attention_via_slots(heads(q), heads(kp), heads(vp), keep, [0, rows], [0, len(keep)])
    assert_close(down(out), o_ref.reshape(rows, H * dh), "f32", "attention out")
    assert_close(down(lse), lse_ref, "f32", "attention lse")
    scores = torch.zeros((1, keys), dtype=torch.float32, device="cuda")
    A.acache_score(dims, up(q, "f32"), up_i32(np.arange(rows)), [0, rows], up(kp, "f32"), slots, scores)
    ref = np.zeros((1, keys))
    ref[0, keep] = O.scores_via_slots(heads(q), np.arange(rows), [0, rows], heads(kp), keep, "affix", None)[0]
    assert_close(down(scores), ref, "f32", "scores")


# ----------------------------------------------------------------------------- bf16 products of few rows

@pytest.mark.parametrize("M", [1, 16, 31, 33, 64, 65, 96, 97, 128, 129, 192, 193, 256, 257])
@pytest.mark.parametrize("N,K,acc", [
    (256, 64, 0),       # one K step
    (768, 192, 1),      # fewer K steps than the ring holds
    (4608, 512, 0),     # narrow: split along K where a workspace is given
    (8448, 320, 1),     # wider than the split path takes, a last workgroup that is part full
    (12288, 2048, 0),   # staggered K starts
    (33280, 128, 1),    # more tiles than CUs: workgroups take several
])
def test_linear_few_rows(A, M, N, K, acc):
    """Both sides of every row bucket and of the last row count of the kernel
    for few rows; with and without a workspace (K splits)."""
    import torch
    a = W.draw_tensor((M, K), "bf16", seed=M)
    w = W.draw_tensor((N, K), "bf16", std=0.05, seed=N + K)
    c0 = W.draw_tensor((M, N), "bf16", seed=7)
    dims = A.make_dims(4096, 32, 32, 128, 256, "bf16")
    ws = A.workspace(dims, M, 1, 0)
    da, dw = up(a, "bf16"), up(w, "bf16")
    # the oracle's product, in fp64 on the device: the same bits as inputs
    ref = da.double() @ dw.double().t() + (up(c0, "bf16").double() if acc else 0.0)
    got = []
    for work in (None, ws):
        c = up(c0, "bf16").clone()
        A.acache_linear(dims, da, dw, out=c, accumulate=bool(acc), ws=work)
        assert_close(down(c), ref.cpu().numpy(), "bf16", f"linear {M}x{N}x{K} ws {work is not None}")
        again = up(c0, "bf16").clone()
        A.acache_linear(dims, da, dw, out=again, accumulate=bool(acc), ws=work)
        assert torch.equal(c, again)  # sums in a fixed order
        got.append(c)


@pytest.mark.parametrize("B,blk", [(1, 16), (1, 32), (2, 32), (3, 32), (4, 33), (5, 32), (8, 32), (7, 37), (2, 193), (3, 239)])
@pytest.mark.parametrize("H,Hkv,F,d", [(4, 4, 1024, 512), (6, 2, 896, 768), (32, 32, 12160, 256), (20, 4, 9472, 512)])
def test_layer_few_rows(A, B, blk, H, Hkv, F, d):
    """acache_layer_recompute at row counts on both sides of the few-row
    kernel's buckets (16 .. 259 rows): the rotary, K/V store, SwiGLU and
    split-K epilogues, against the oracle's block in fp64; some rows have no
    valid write slot (nothing stored)."""
    import torch
    rng = np.random.default_rng(B * blk + H)
    dh, M, S = 128, B * blk, blk + 40
    shapes = dict(w_qkv=((H + 2 * Hkv) * dh, d), w_o=(d, H * dh), w_gate_up=(2 * F, d), w_down=(d, F))
    bits = {n: W.draw_tensor(s, "bf16", std=0.04, seed=i) for i, (n, s) in enumerate(shapes.items())}
    bits["attn_norm"] = bits["mlp_norm"] = W.draw_tensor((d,), "bf16", seed=9)
    x0 = W.draw_tensor((M, d), "bf16", seed=10)
    n_slots = B * S + 3
    kp, vp = (W.draw_tensor((n_slots, Hkv * dh), "bf16", seed=11 + i) for i in range(2))
    read = rng.permutation(n_slots)[:B * S].reshape(B, S)
    write = read[:, 40:].copy()
    pos = rng.integers(0, 9000, size=(B, blk))
    bad = write.reshape(-1).copy()
    bad[M // 2] = n_slots + 5  # dropped; its key keeps the pool's row
    dims = A.make_dims(d, H, Hkv, dh, F, "bf16")
    dev = {n: up(b, "bf16") for n, b in bits.items()}
    x, gk, gv = up(x0, "bf16").clone(), up(kp, "bf16").clone(), up(vp, "bf16").clone()
    ws = A.workspace(dims, M, B, 0)
    A.acache_layer_recompute(dims, dev, [b * blk for b in range(B + 1)], [b * S for b in range(B + 1)], x,
                             up_i32(pos.reshape(-1)), up_i32(bad), up_i32(read.reshape(-1)), gk, gv, ws)
    # the same block in fp64 with plain torch operations
    D = lambda t: t.double()  # noqa: E731
    norm = lambda t, g: t / torch.sqrt((t * t).mean(1, keepdim=True) + 1e-5) * D(g)  # noqa: E731
    xr = D(up(x0, "bf16"))
    y = norm(xr, dev["attn_norm"])
    qkv = (y @ D(dev["w_qkv"]).t()).view(M, H + 2 * Hkv, dh)
    th = 10000.0 ** (-2.0 * torch.arange(64, device="cuda", dtype=torch.float64) / dh)
    an = torch.from_numpy(pos.reshape(-1)).cuda().double()[:, None, None] * th
    rot = torch.cat([qkv[..., :64] * an.cos() - qkv[..., 64:] * an.sin(),
                     qkv[..., 64:] * an.cos() + qkv[..., :64] * an.sin()], 2)
    K, V = D(up(kp, "bf16")), D(up(vp, "bf16"))
    ok = torch.from_numpy(bad < n_slots).cuda()
    wsl = torch.from_numpy(bad).cuda().long()[ok]
    K[wsl] = rot[:, H:H + Hkv].reshape(M, -1)[ok]
    V[wsl] = qkv[:, H + Hkv:].reshape(M, -1)[ok]
    assert_close(down(gk), K.cpu().numpy(), "bf16", "K pool")
    assert_close(down(gv), V.cpu().numpy(), "bf16", "V pool")
    o = torch.zeros(M, H * dh, dtype=torch.float64, device="cuda")
    for b in range(B):
        sl = torch.from_numpy(read[b]).cuda().long()
        for h in range(H):
            g = slice(h // (H // Hkv) * dh, (h // (H // Hkv) + 1) * dh)
            lg = rot[b * blk:(b + 1) * blk, h] @ K[sl][:, g].t() / np.sqrt(dh)
            o[b * blk:(b + 1) * blk, h * dh:(h + 1) * dh] = torch.softmax(lg, 1) @ V[sl][:, g]
    xr = xr + o @ D(dev["w_o"]).t()
    gu = norm(xr, dev["mlp_norm"]) @ D(dev["w_gate_up"]).t()
    xr = xr + (torch.nn.functional.silu(gu[:, :F]) * gu[:, F:]) @ D(dev["w_down"]).t()
    assert_close(down(x), xr.cpu().numpy(), "bf16", "layer rows")


# ----------------------------------------------------------------------------- decode-step attention

@pytest.mark.parametrize("H,Hkv,B,blk,L,k,priv", [
    (4, 4, 1, 32, 1024, 205, 77),     # one request, both kinds split along their keys
    (4, 4, 3, 20, 200, 40, 30),       # 32 queries of a wavefront across requests: per-lane masks
    (8, 2, 4, 32, 640, 100, 65),      # grouped heads as further rows of a tile
    (6, 1, 2, 17, 129, 129, 40),      # every affix key an anchor: private keys alone
    (4, 2, 2, 32, 130, 0, 32),        # no anchors
    (32, 32, 8, 32, 2048, 410, 300),  # the 256-query kernel on the shared affix
    (32, 32, 9, 32, 1031, 700, 33),   # the same, a part-full query tile and key tile, whole tiles masked
    (32, 8, 16, 64, 4096, 819, 64),   # the same with grouped heads, several requests' rows a tile
])
def test_decode_attention(A, H, Hkv, B, blk, L, k, priv):
    """acache_layer_decode against the block in fp64: the shared affix minus
    each request's anchors plus its private slots, some of them out of range
    (zero key, zero value)."""
    import torch
    rng = np.random.default_rng(L + H)
    dh, d, F, M = 128, 256, 256, B * blk
    shapes = dict(w_qkv=((H + 2 * Hkv) * dh, d), w_o=(d, H * dh), w_gate_up=(2 * F, d), w_down=(d, F))
    bits = {n: W.draw_tensor(s, "bf16", std=0.08, seed=i) for i, (n, s) in enumerate(shapes.items())}
    bits["attn_norm"] = bits["mlp_norm"] = W.draw_tensor((d,), "bf16", seed=9)
    x0 = W.draw_tensor((M, d), "bf16", seed=10)
    n_slots = L + B * priv + 3
    kp, vp = (W.draw_tensor((n_slots, Hkv * dh), "bf16", seed=11 + i) for i in range(2))
    perm = rng.permutation(n_slots)
    affix, private = perm[:L].copy(), perm[L:L + B * priv].reshape(B, priv).copy()
    anchors = np.stack([np.sort(rng.permutation(L)[:k]) for _ in range(B)]).astype(np.int32)
    if k >= 700:  # two whole key tiles of request 0 are anchors
        rest = rng.permutation(np.concatenate([np.arange(64, 128), np.arange(256, L)]))[:k - 128]
        anchors[0] = np.sort(np.concatenate([np.arange(0, 64), np.arange(128, 192), rest]))
    write = private[:, priv - blk:].copy() if priv >= blk else private[:, :0]
    if priv < blk:
        write = np.full((B, blk), -1)  # rows whose K/V go nowhere
    affix[L // 2], private[0, 0] = n_slots + 9, -5
    pos = rng.integers(0, 9000, size=M)
    dims = A.make_dims(d, H, Hkv, dh, F, "bf16")
    dev = {n: up(b, "bf16") for n, b in bits.items()}
    x, gk, gv = up(x0, "bf16").clone(), up(kp, "bf16").clone(), up(vp, "bf16").clone()
    ws = A.workspace(dims, M, B, L)
    run = lambda xx: A.acache_layer_decode(  # noqa: E731
        dims, dev, B, blk, xx, up_i32(pos), up_i32(write.reshape(-1)), up_i32(affix),
        up_i32(anchors) if k else None, k, up_i32(private.reshape(-1)), priv, gk, gv, ws)
    run(x)
    again = up(x0, "bf16").clone()
    run(again)
    assert torch.equal(x, again)  # partials merged in a fixed order
    D = lambda t: t.double()  # noqa: E731
    norm = lambda t, g: t / torch.sqrt((t * t).mean(1, keepdim=True) + 1e-5) * D(g)  # noqa: E731
    xr = D(up(x0, "bf16"))
    q = (norm(xr, dev["attn_norm"]) @ D(dev["w_qkv"]).t()[:, :H * dh]).view(M, H, dh)
    th = 10000.0 ** (-2.0 * torch.arange(64, device="cuda", dtype=torch.float64) / dh)
    an = torch.from_numpy(pos).cuda().double()[:, None, None] * th
    q = torch.cat([q[..., :64] * an.cos() - q[..., 64:] * an.sin(), q[..., 64:] * an.cos() + q[..., :64] * an.sin()], 2)
    # the keys as stored (the rows' own K/V, checked by the projection's tests)
    zero = torch.zeros(1, Hkv * dh, dtype=torch.float64, device="cuda")
    K, V = torch.cat([D(gk), zero]), torch.cat([D(gv), zero])
    o = torch.zeros(M, H * dh, dtype=torch.float64, device="cuda")
    for b in range(B):
        keep = np.ones(L, bool)
        keep[anchors[b]] = False
        view = np.concatenate([affix[keep], private[b]])
        sl = torch.from_numpy(np.where((view < 0) | (view >= n_slots), n_slots, view)).cuda().long()
        kb, vb = K[sl], V[sl]
        for h in range(H):
            g = slice(h // (H // Hkv) * dh, (h // (H // Hkv) + 1) * dh)
            lg = q[b * blk:(b + 1) * blk, h] @ kb[:, g].t() / np.sqrt(dh)
            o[b * blk:(b + 1) * blk, h * dh:(h + 1) * dh] = torch.softmax(lg, 1) @ vb[:, g]
    xr = xr + o @ D(dev["w_o"]).t()
    gu = norm(xr, dev["mlp_norm"]) @ D(dev["w_gate_up"]).t()
    xr = xr + (torch.nn.functional.silu(gu[:, :F]) * gu[:, F:]) @ D(dev["w_down"]).t()
    assert_close(down(x), xr.cpu().numpy(), "bf16", "decode rows")


# ----------------------------------------------------------------------------- 192-wide tiles

@pytest.mark.parametrize("M,N,K,acc", [
    (384, 12288, 256, 0),    # 192 x 192 tiles: whole rows and columns
    (717, 12288, 128, 1),    # a part-full last row tile
    (600, 8448, 192, 0),     # N a multiple of neither: the last tile's fragments repeat and are skipped
    (1024, 12288, 64, 1),    # 192 x 256, one K step
    (1000, 24576, 192, 0),
    (2048, 12544, 128, 1),
    (1536, 4096, 256, 0), (4500, 4096, 128, 1),
])
def test_linear_tile_shapes(A, M, N, K, acc):
    a = W.draw_tensor((M, K), "bf16", seed=M)
    w = W.draw_tensor((N, K), "bf16", std=0.05, seed=N + K)
    c0 = W.draw_tensor((M, N), "bf16", seed=7)
    dims = A.make_dims(4096, 32, 32, 128, 256, "bf16")
    da, dw = up(a, "bf16"), up(w, "bf16")
    ref = (da.double() @ dw.double().t() + (up(c0, "bf16").double() if acc else 0.0)).cpu().numpy()
    for work in (None, A.workspace(dims, M, 1, 0)):
        c = up(c0, "bf16").clone()
        A.acache_linear(dims, da, dw, out=c, accumulate=bool(acc), ws=work)
        assert_close(down(c), ref, "bf16", f"linear {M}x{N}x{K} ws {work is not None}")
