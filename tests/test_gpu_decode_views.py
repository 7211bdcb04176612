"""acache_layer_decode over views whose requests share a wavefront (blocks
that are no multiple of 32 rows, with anchors that cover whole 64-key tiles of
the affix for one request and not for its neighbours), and over more rows than
the workspace holds attention partials for."""

import numpy as np
import pytest

import workloads as W
from tests.gpu_util import assert_close, down, up, up_i32

pytestmark = pytest.mark.gpu

DH = 128


def anchors_of(pattern, B, L):
    """[B, k] anchors in whole 64-key tiles; request b covers
    first   tile 0 if b is even, the last whole tile otherwise;
    strips  every second tile, from tile b % 2 on (so whichever tile a key
            split starts at, every second request has no key in it);
    halves  the first half of the affix or the second (whole splits)."""
    n = L // 64
    tiles = []
    for b in range(B):
        if pattern == "first":
            tiles.append([0 if b % 2 == 0 else n - 1])
        elif pattern == "strips":
            tiles.append(list(range(b % 2, n - n % 2, 2)))
        else:
            tiles.append(list(range(b % 2 * (n // 2), (b % 2 + 1) * (n // 2))))
    return np.stack([np.concatenate([np.arange(64 * t, 64 * t + 64) for t in ts]) for ts in tiles]).astype(np.int32)


def check_decode(H, Hkv, B, blk, L, priv, anchors):
    from paper_2608_26140_amd import acache as A
    from tests import block_reference as R
    rng = np.random.default_rng(L + H + blk)
    d, F, M, k = 256, 256, B * blk, anchors.shape[1]
    # standard deviation 0.05: with 0.08 the MLP of single rows amplifies the bf16
    # rounding of the stored intermediates alone (fp64 arithmetic otherwise; 256
    # rows over 1024 + 40 keys, row 50) to 0.0328 of the RMS in one element, and
    # the gate's 8 x RMS error stands at 0.0342 there
    dev = R.weights(d, H, Hkv, F, std=0.05)
    x0 = up(W.draw_tensor((M, d), "bf16", seed=10), "bf16")
    n_slots = L + B * priv
    pools = [up(W.draw_tensor((n_slots, Hkv * DH), "bf16", seed=11 + i), "bf16") for i in range(2)]
    perm = rng.permutation(n_slots)
    affix, private = perm[:L], perm[L:].reshape(B, priv)
    write = private[:, priv - blk:] if priv >= blk else np.full((B, blk), -1)
    pos = rng.integers(0, 9000, size=M)
    dims = A.make_dims(d, H, Hkv, DH, F, "bf16")
    x = x0.clone()
    A.acache_layer_decode(dims, dev, B, blk, x, up_i32(pos), up_i32(write.reshape(-1)), up_i32(affix),
                          up_i32(anchors), k, up_i32(private.reshape(-1)), priv, *pools,
                          A.workspace(dims, M, B, L))
    # the block in fp64 over each request's own list of keys (as stored)
    views = [np.concatenate([np.delete(affix, anchors[b]), private[b]]) for b in range(B)]
    q = R.qkv(dev, x0.double(), pos, H, Hkv)[0]
    ref = R.out_mlp(dev, x0.double(), R.attend(q, *pools, views, blk))
    assert_close(down(x), ref.cpu().numpy(), "bf16", "decode rows")


@pytest.mark.parametrize("pattern", ["first", "strips", "halves"])
@pytest.mark.parametrize("H,Hkv,B,blk,L,priv", [
    (32, 32, 2, 16, 1024, 717),   # one wavefront of two requests
    (28, 4, 4, 8, 4096, 40),      # four requests a wavefront, grouped heads as further rows
    (4, 2, 3, 20, 650, 30),       # requests that begin inside a wavefront, a part-full last key tile
    (4, 4, 8, 16, 1024, 65),
    (4, 4, 5, 40, 640, 64),
    (32, 32, 8, 32, 2048, 64),    # whole wavefronts a request: the 256-query kernel
])
def test_tiles_masked_for_some(pattern, H, Hkv, B, blk, L, priv):
    check_decode(H, Hkv, B, blk, L, priv, anchors_of(pattern, B, L))


@pytest.mark.parametrize("H,Hkv,B,blk", [
    (8, 2, 5, 4201),   # 21,005 rows where 20,164 fit: two groups of requests (2 and 3)
    (8, 2, 3, 11000),  # one request a group
    (8, 4, 2, 20300),  # a request beyond one group: slices of its rows
])
def test_more_rows_than_partials(H, Hkv, B, blk):
    check_decode(H, Hkv, B, blk, 200, 40, anchors_of("first", B, 200))


@pytest.mark.parametrize("H,Hkv,B,blk,L,priv", [
    (32, 32, 16, 16, 1024, 40),    # more workgroups than run at a time, the shared ones longer
    (32, 32, 17, 16, 128, 330),    # the private ones longer
    (32, 32, 17, 16, 330, 330),    # alike
    (28, 4, 40, 30, 200, 700),     # grouped heads, the private ones longer
])
def test_either_kind_first(H, Hkv, B, blk, L, priv):
    check_decode(H, Hkv, B, blk, L, priv, anchors_of("first", B, L))
