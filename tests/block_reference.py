"""The transformer block in fp64 with plain torch operations, in three parts,
from bf16 tensors on the device: reference of the layer calls' tests."""

import numpy as np
import torch

DH = 128


def norm(t, g, eps=1e-5):
    return t / torch.sqrt((t * t).mean(1, keepdim=True) + eps) * g.double()


def qkv(w, x, pos, H, Hkv, rope_base=10000.0):
    """[M, heads, 128] rotated queries, rotated keys, values of the rows x."""
    p = (norm(x, w["attn_norm"]) @ w["w_qkv"].double().t()).view(len(x), H + 2 * Hkv, DH)
    th = rope_base ** (-2.0 * torch.arange(64, device=x.device, dtype=torch.float64) / DH)
    an = torch.from_numpy(np.asarray(pos)).to(x.device).double()[:, None, None] * th
    rot = torch.cat([p[..., :64] * an.cos() - p[..., 64:] * an.sin(),
                     p[..., 64:] * an.cos() + p[..., :64] * an.sin()], 2)
    return rot[:, :H], rot[:, H:H + Hkv], p[:, H + Hkv:]


def attend(q, K, V, views, rows):
    """Row block b of q (rows each) over the pool slots views[b]; K and V are
    the pools [n_slots, Hkv * 128]."""
    M, H, _ = q.shape
    K, V = (p.double().view(len(p), -1, DH) for p in (K, V))
    rep = H // K.shape[1]
    o = torch.zeros(M, H, DH, dtype=torch.float64, device=q.device)
    for b, view in enumerate(views):
        sl, r = torch.from_numpy(np.asarray(view)).to(q.device), slice(b * rows, (b + 1) * rows)
        for h in range(H):
            o[r, h] = torch.softmax(q[r, h] @ K[sl, h // rep].t() / np.sqrt(DH), 1) @ V[sl, h // rep]
    return o.reshape(M, H * DH)


def out_mlp(w, x, o):
    """The rows after the output projection and the MLP, both with residual."""
    x = x + o @ w["w_o"].double().t()
    gu = norm(x, w["mlp_norm"]) @ w["w_gate_up"].double().t()
    F = gu.shape[1] // 2
    return x + (torch.nn.functional.silu(gu[:, :F]) * gu[:, F:]) @ w["w_down"].double().t()


def weights(d, H, Hkv, F, std=0.08):
    """A layer's bf16 weights on the device."""
    import workloads as W
    from tests.gpu_util import up
    shapes = dict(w_qkv=((H + 2 * Hkv) * DH, d), w_o=(d, H * DH), w_gate_up=(2 * F, d), w_down=(d, F))
    w = {n: up(W.draw_tensor(s, "bf16", std=std, seed=i), "bf16") for i, (n, s) in enumerate(shapes.items())}
    w["attn_norm"] = w["mlp_norm"] = up(W.draw_tensor((d,), "bf16", seed=9), "bf16")
    return w
