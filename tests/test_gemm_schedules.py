"""bf16 products on every schedule the planner has: each shape below is first
held to the schedule it is here for (on the CPU, so that a change of the
planner cannot leave a schedule untested unnoticed), then run against fp64."""

import ctypes

import numpy as np
import pytest

import workloads as W

STORE, ACCUM, PARTIAL, QKV, SWIGLU = range(5)


def schedule(epi, M, N, K, ws=True):
    """((tile's weight rows, activation rows), whole rounds ahead of a stream-K
    region, tiles in that region); tile (0, 0): the kernel for few rows."""
    from paper_2608_26140_amd import acache as A
    out = (ctypes.c_int32 * 4)()
    A.lib.acache_gemm_schedule(epi, M, N, K, int(ws), out)
    return (out[0], out[1]), out[2], out[3]


# M, N, K and the schedule with a workspace
LINEAR = [
    (717, 768, 1024, ((256, 256), 0, 9)),       # stream-K alone
    (700, 2048, 4096, ((256, 256), 0, 24)),
    (6528, 2560, 2048, ((256, 256), 1, 4)),     # a whole round, then stream-K
    (9000, 4096, 12288, ((256, 256), 2, 64)),   # a down projection: two rounds, then stream-K
    (284, 256, 256, ((256, 128), 0, 3)),        # stream-K on the half tile
    (300, 2048, 4096, ((256, 128), 0, 24)),
    (8193, 1024, 4096, ((256, 128), 1, 4)),
    (966, 8192, 64, ((256, 128), 0, 0)),
    (2048, 12544, 64, ((256, 256), 0, 0)),      # 392 tiles of one K step on 256 persistent workgroups
]

# H, Hkv, d, F, M; the schedule of the Q/K/V and of the gate/up projection.
# (H + 2 Hkv) * 128 and 2 F are no multiples of 192.
LAYERS = [
    (4, 2, 256, 640, 385, ((192, 192), 0, 0), ((192, 192), 0, 0)),
    (126, 2, 256, 8576, 385, ((192, 256), 0, 0), ((192, 256), 0, 0)),
    (94, 2, 256, 6400, 900, ((256, 192), 0, 0), ((256, 192), 0, 0)),
    (2, 1, 512, 256, 385, ((256, 256), 0, 4), ((256, 256), 0, 4)),
    (2, 1, 512, 256, 257, ((256, 128), 0, 6), ((256, 128), 0, 6)),
    (126, 2, 512, 8320, 1000, ((256, 256), 1, 4), ((256, 256), 1, 4)),
]


@pytest.mark.parametrize("M,N,K,want", LINEAR)
def test_linear_schedules(M, N, K, want):
    assert schedule(STORE, M, N, K) == want
    assert schedule(ACCUM, M, N, K) == want
    assert schedule(STORE, M, N, K, ws=False)[2] == 0  # no stream-K without space for its pieces


@pytest.mark.parametrize("H,Hkv,d,F,M,qkv,gate_up", LAYERS)
def test_layer_schedules(H, Hkv, d, F, M, qkv, gate_up):
    nq = (H + 2 * Hkv) * 128
    assert nq % 192 and 2 * F % 192
    assert schedule(QKV, M, nq, d) == qkv
    assert schedule(SWIGLU, M, 2 * F, d) == gate_up


def test_few_rows_schedules():
    for epi in range(5):
        assert schedule(epi, 128, 12288, 4096)[0] == (0, 0)
        assert schedule(epi, 257, 12288, 4096)[0] != (0, 0)
    assert schedule(ACCUM, 256, 8192, 4096)[0] == (0, 0)  # narrow, with space for K splits


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,want", LINEAR)
def test_linear(M, N, K, want):
    import torch
    from paper_2608_26140_amd import acache as A
    from tests.gpu_util import assert_close, down, up
    assert schedule(STORE, M, N, K) == want  # on this device too
    a = up(W.draw_tensor((M, K), "bf16", seed=M), "bf16")
    w = up(W.draw_tensor((N, K), "bf16", std=0.05, seed=N + K), "bf16")
    c0 = up(W.draw_tensor((M, N), "bf16", seed=7), "bf16")
    dims = A.make_dims(256, 2, 2, 128, 128, "bf16")
    ws = A.workspace(dims, M, 1, 0)
    ref = a.double() @ w.double().t()
    for acc in (False, True):
        out = [c0.clone() for _ in range(3)]
        for c, space in zip(out, (ws, ws, None)):
            A.acache_linear(dims, a, w, out=c, accumulate=acc, ws=space)
        want_c = (ref + c0.double() if acc else ref).cpu().numpy()
        assert_close(down(out[0]), want_c, "bf16", f"linear {M}x{N}x{K} accumulate {acc}")
        assert torch.equal(out[0], out[1])  # the pieces are added in a fixed order
        # the data-parallel schedule: one bf16 ulp, plus the order of fp32 sums near zero
        sk, dp = down(out[0]), down(out[2])
        assert np.all(np.abs(sk - dp) <= 2.0 ** -7 * np.maximum(np.abs(sk), np.abs(dp)) + 1e-6 * np.abs(want_c).max())


@pytest.mark.gpu
@pytest.mark.parametrize("M", [192, 193, 224, 256])
@pytest.mark.parametrize("N,K", [(256, 1024), (512, 512), (2048, 768), (2304, 768)])
def test_linear_few_rows_accumulate(M, N, K):
    """Both sides of the rows and columns from which on a product added to its
    output goes through K splits sooner."""
    from paper_2608_26140_amd import acache as A
    from tests.gpu_util import assert_close, down, up
    a = up(W.draw_tensor((M, K), "bf16", seed=M), "bf16")
    w = up(W.draw_tensor((N, K), "bf16", std=0.05, seed=N + K), "bf16")
    c = up(W.draw_tensor((M, N), "bf16", seed=7), "bf16")
    dims = A.make_dims(256, 2, 2, 128, 128, "bf16")
    ref = (a.double() @ w.double().t() + c.double()).cpu().numpy()
    A.acache_linear(dims, a, w, out=c, accumulate=True, ws=A.workspace(dims, M, 1, 0))
    assert_close(down(c), ref, "bf16", f"linear {M}x{N}x{K}")


@pytest.mark.gpu
@pytest.mark.parametrize("H,Hkv,d,F,M,qkv,gate_up", LAYERS)
def test_layer(H, Hkv, d, F, M, qkv, gate_up):
    """The rotary, K/V store and SwiGLU epilogues of those tiles; a row without
    a valid write slot stores nothing."""
    from paper_2608_26140_amd import acache as A
    from tests import block_reference as R
    from tests.gpu_util import assert_close, down, up, up_i32
    rng = np.random.default_rng(M + H)
    S, n_slots = M + 40, M + 47
    dev = R.weights(d, H, Hkv, F, std=0.05)
    x0 = up(W.draw_tensor((M, d), "bf16", seed=10), "bf16")
    K, V = (up(W.draw_tensor((n_slots, Hkv * 128), "bf16", seed=11 + i), "bf16") for i in range(2))
    read = rng.permutation(n_slots)[:S]
    write, pos = read[40:].copy(), rng.integers(0, 9000, size=M)
    write[M // 3] = n_slots
    dims = A.make_dims(d, H, Hkv, 128, F, "bf16")
    q, k_new, v_new = R.qkv(dev, x0.double(), pos, H, Hkv)
    k_ref, v_ref = down(K), down(V)
    ok = write < n_slots
    k_ref[write[ok]] = k_new.reshape(M, -1).cpu().numpy()[ok]
    v_ref[write[ok]] = v_new.reshape(M, -1).cpu().numpy()[ok]
    x = x0.clone()
    A.acache_layer_recompute(dims, dev, [0, M], [0, S], x, up_i32(pos), up_i32(write), up_i32(read), K, V,
                             A.workspace(dims, M, 1, 0))
    assert_close(down(K), k_ref, "bf16", "K pool")
    assert_close(down(V), v_ref, "bf16", "V pool")
    ref = R.out_mlp(dev, x0.double(), R.attend(q, K, V, [read], M))
    assert_close(down(x), ref.cpu().numpy(), "bf16", "rows")
