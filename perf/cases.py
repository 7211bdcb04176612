"""What a program that serves with this package has it do, as cases for timing and comparing.

Each case goes through the package's own entry points (AffixBatch.refresh and
.probe, decode_step, the head's calls) as a serving loop calls them: token ids
in, rows, scores or logits and the key/value pools out.  Weights, embeddings and
the cached keys and values are drawn on the GPU from the seed with the spread a
stack with N(0, 0.02^2) weights and unit RMSNorm gains gives them (a normalised
row times a projection has a standard deviation of 0.02 sqrt(d)).

Kinds
  refresh  maps, embedding gather and the layer over anchors and own rows (the
           call at every recomputation point)
  probe    the same over the own rows only, with the scores of the affix keys
           (the call that precedes the selection)
  decode   one step of block decoding: queries of the current block only
  head     the end of a step: final norm, vocabulary projection, most likely
           token and confidence of every row, commits over a threshold
  select   the calls between probe and refresh: top-K of the scores, slot maps,
           gather of the rows' embeddings
  call     probe, refresh and the head's logits over a stack of layers
"""

import math

import torch

from paper_2608_26140_amd import acache as A
from paper_2608_26140_amd import driver as D

# The shapes the package's workloads are made of: LLaDA-8B's block (one key/value head
# per query head), Dream-7B's (grouped heads, wider MLP), and the two fp32 layers.
MODELS = {
    "llada": dict(d_model=4096, n_heads=32, n_kv_heads=32, head_dim=128, d_ff=12288, dtype="bf16"),
    "dream": dict(d_model=3584, n_heads=28, n_kv_heads=4, head_dim=128, d_ff=18944, dtype="bf16"),
    "f32": dict(d_model=256, n_heads=4, n_kv_heads=4, head_dim=64, d_ff=688, dtype="f32"),
    "f32-gqa": dict(d_model=128, n_heads=4, n_kv_heads=2, head_dim=32, d_ff=256, dtype="f32"),
}
VOCAB = 126464
EPS, BASE = 1e-5, 10000.0
TAU = 0.9  # commit threshold of block decoding


def _layers(kind, name, model, batch, affix, after, mask, ratio, before=0, layers=1, page=0, norm="affix"):
    """before / affix / after / mask: lengths of a request's spans, in that order; page: slots per
    key/value block (0: one flat range of slots per request)."""
    c = dict(kind=kind, model=model, batch=batch, before=before, affix=affix, after=after, mask=mask,
             anchors=int(math.floor(ratio * affix + 0.5)), layers=layers, page=page, norm=norm)
    return dict(c, name=name) if name else c


def _head(name, model, batch, block):
    c = dict(kind="head", model=model, batch=batch, block=block)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the fp32 layer of the numerics tests: 90 rows of 256, all launches and latency
        _layers("refresh", "refresh-f32-b1", "f32", 1, 128, 32, 32, 0.2),
        # the host-free middle of a step: Eq. 6's selection and the maps for a batch of eight
        _layers("select", "select-llada-b8", "llada", 8, 2048, 128, 256, 0.2),
        # one user decoding: 32 rows, every weight read for them
        _layers("decode", "decode-llada-b1", "llada", 1, 1024, 256, 256, 0.2),
        # a small batch on the grouped-head model, affix between two own spans
        _layers("decode", "decode-dream-b4", "dream", 4, 4096, 256, 256, 0.2, before=512),
        # the serving batch decoding: 1024 rows over a shared affix of 8192 keys
        _layers("decode", "decode-llada-b32", "llada", 32, 8192, 256, 256, 0.2),
        # one user's recomputation point: 717 rows
        _layers("refresh", "refresh-llada-b1", "llada", 1, 1024, 256, 256, 0.2),
        # eight users, 6354 rows
        _layers("refresh", "refresh-llada-b8", "llada", 8, 2048, 128, 256, 0.2),
        # four users on the grouped-head model, 7372 rows
        _layers("refresh", "refresh-dream-b4", "dream", 4, 4096, 256, 256, 0.2, before=512),
        # the serving batch at a recomputation point: 68 800 rows, paged slots
        _layers("refresh", "refresh-llada-b32", "llada", 32, 8192, 256, 256, 0.2, page=256),
        # the one-shot probe of eight users: a layer that also scores its affix keys
        _layers("probe", "probe-llada-b8", "llada", 8, 2048, 128, 256, 0.2),
        # the end of a decode step of eight users: 256 rows against the whole vocabulary
        _head("head-llada-b8", "llada", 8, 32),
        # a whole small call over three layers, no size a multiple of a tile
        _layers("call", "call-llada-b3", "llada", 3, 613, 77, 51, 0.2, layers=3),
    ]


def draw(rng):
    def span(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["refresh", "refresh", "decode", "decode", "probe", "head", "select", "call", "f32"])
    model = rng.choice(["llada", "llada", "dream"])
    batch = span(1, 32)
    if kind == "f32":
        return _layers(rng.choice(["refresh", "probe"]), None, rng.choice(["f32", "f32-gqa"]), rng.randint(1, 2),
                       span(64, 400), span(16, 64), span(8, 48), rng.uniform(0.1, 0.4), before=rng.choice([0, 20]))
    if kind == "head":
        return _head(None, model, batch, rng.choice([16, 32, 32]))
    affix, after, mask = span(512, 8192), span(64, 384), rng.choice([128, 256, span(64, 256)])
    before = rng.choice([0, 0, span(32, 512)])
    ratio = rng.choice([0.1, 0.2, 0.2, 0.4])
    norm = rng.choice(["affix", "affix", "full"]) if kind == "probe" else "affix"
    layers = 1
    if kind == "call":
        batch, affix, layers = min(batch, 4), min(affix, 2048), rng.choice([2, 3])
    page = rng.choice([0, 256]) if kind in ("refresh", "probe") else 0
    most = max(work(c)["flops"] for c in listed())
    while True:
        c = _layers(kind, None, model, batch, affix, after, mask, ratio, before=before, layers=layers, page=page, norm=norm)
        if work(c)["flops"] <= most:
            return c
        batch -= 1


# ---------------------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) + 0x26140)


def _normal(g, shape, std, dtype):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).mul_(std).to(dtype)


def _sizes(c):
    m = MODELS[c["model"]]
    z = dict(m, B=c["batch"], dt=torch.bfloat16 if m["dtype"] == "bf16" else torch.float32, hq=m["n_heads"] * m["head_dim"],
             hkv=m["n_kv_heads"] * m["head_dim"])
    if c["kind"] == "head":
        return z
    z.update(S=c["before"] + c["affix"] + c["after"] + c["mask"], L=c["affix"], ab=c["before"], G=c["mask"], K=c["anchors"])
    z["mb"] = z["S"] - z["G"]
    z["P"] = z["S"] - z["L"]  # own rows of a request
    z["R"] = z["K"] + z["P"]  # rows a refresh recomputes
    bs = c["page"]
    z["base"] = -(-z["L"] // bs) * bs if bs else z["L"]      # first private slot
    up = lambda n: -(-n // bs) * bs  # noqa: E731
    z["slots"] = z["base"] + z["B"] * (up(z["R"]) if bs else z["R"])
    # private slots of a request: a paged batch takes whole pages for the rows it has
    z["stride"] = up(z["P"] if c["kind"] == "probe" else z["R"]) if bs else z["R"]
    z["block"] = min(32, z["G"])
    z["blk"] = (z["G"] // z["block"]) // 2                   # the block that decodes
    return z


def _weights(g, z):
    d, hq, hkv, F, dt = z["d_model"], z["hq"], z["hkv"], z["d_ff"], z["dt"]
    gain = lambda: _normal(g, (d,), 0.1, torch.float32).add_(1.0).to(dt)  # noqa: E731
    return dict(attn_norm=gain(), w_qkv=_normal(g, (hq + 2 * hkv, d), 0.02, dt), w_o=_normal(g, (d, hq), 0.02, dt),
                mlp_norm=gain(), w_gate_up=_normal(g, (2 * F, d), 0.02, dt), w_down=_normal(g, (d, F), 0.02, dt))


def _inputs(c, seed):
    """Everything a case is made of, as plain tensors."""
    z, g = _sizes(c), _gen(seed)
    d, dt, B = z["d_model"], z["dt"], z["B"]
    i = dict(z=z)
    if c["kind"] == "head":
        n = B * c["block"]
        w = _normal(g, (VOCAB, d), 0.02, dt)
        # rows that favour one token, as a trained model's do: of each request half the rows are sure
        # of it (probability over 0.95), half are not (under 0.3); none is near the threshold
        t = torch.randint(0, VOCAB, (n,), generator=g, device="cuda")
        wt, x = w[t].float(), _normal(g, (n, d), 1.0, torch.float32)
        x -= (x * wt).sum(1, keepdim=True) / (wt * wt).sum(1, keepdim=True) * wt
        u = torch.rand(n, generator=g, device="cuda")
        at = torch.arange(n, device="cuda")
        logit = torch.where(at % 2 == 0, 16.0 + 3.0 * u, 8.5 + 2.5 * u) * (1.02 if d > 3600 else 1.03)
        x += (logit / (wt * wt).sum(1)).unsqueeze(1) * wt
        return dict(i, x=x.to(dt), gain=torch.ones(d, device="cuda", dtype=dt), w=w)
    S, L, K = z["S"], z["L"], z["K"]
    i["anchors"] = torch.sort(torch.rand((B, L), generator=g, device="cuda").argsort(1)[:, :K], 1).values.to(torch.int32)
    if z["dtype"] == "f32":
        i["emb"] = _normal(g, (B * S, d), 1.0, dt)
        i["ids"] = None
    else:
        i["emb"] = _normal(g, (VOCAB, d), 0.02, dt)
        ids = torch.randint(0, VOCAB - 1, (B, S), generator=g, device="cuda")
        ids[:, z["ab"]:z["ab"] + L] = ids[:1, z["ab"]:z["ab"] + L]  # the shared affix
        masked = ids[:, z["mb"]:]
        masked[torch.rand(masked.shape, generator=g, device="cuda") < (0.5 if c["kind"] == "decode" else 1.0)] = VOCAB - 1
        i["ids"] = ids.to(torch.int32).contiguous()
    if c["kind"] == "select":
        i["scores"] = torch.rand((B, L), generator=g, device="cuda").pow_(4.0)  # few keys take most of the mass
        return i
    i["layers"] = [_weights(g, z) for _ in range(c["layers"])]
    kv = 0.02 * math.sqrt(d)
    rows = z["base"] if c["kind"] != "decode" else z["slots"]  # a decode step finds its request's rows in the cache too
    i["k"] = [_normal(g, (rows, z["hkv"]), kv, dt) for _ in range(c["layers"])]
    i["v"] = [_normal(g, (rows, z["hkv"]), kv, dt) for _ in range(c["layers"])]
    if c["kind"] == "call":
        i["gain"], i["head"] = torch.ones(d, device="cuda", dtype=dt), _normal(g, (VOCAB, d), 0.02, dt)
    return i


def prepare(case, seed):
    i = _inputs(case, seed)
    z = i["z"]
    dims = A.make_dims(z["d_model"], z["n_heads"], z["n_kv_heads"], z["head_dim"], z["d_ff"], z["dtype"], EPS, BASE)
    i32 = dict(dtype=torch.int32, device="cuda")
    if case["kind"] == "head":
        n = z["B"] * case["block"]
        return dict(case=case, dims=dims, x=i["x"], gain=i["gain"], w=i["w"], block=case["block"],
                    rows=torch.arange(n, **i32), pos=torch.arange(n, **i32), ids=torch.full((n,), VOCAB - 1, **i32),
                    logits=torch.empty((n, VOCAB), dtype=z["dt"], device="cuda"), pick=torch.empty(n, **i32),
                    conf=torch.empty(n, dtype=torch.float32, device="cuda"), flags=torch.zeros(n, **i32),
                    count=torch.empty(z["B"], **i32), ws=A.workspace(dims, n, z["B"], 0))
    layers = i.get("layers") or []
    batch = D.AffixBatch(D.Model(dims, layers), z["S"], z["ab"], z["L"], z["mb"], z["G"], z["B"], i["emb"],
                         None if i["ids"] is None else i["ids"].view(-1), private_stride=z["R"], max_rows=z["R"],
                         block_size=case["page"] or None)
    for n in range(len(layers)):
        batch.k_pools[n][:i["k"][n].shape[0]] = i["k"][n]
        batch.v_pools[n][:i["v"][n].shape[0]] = i["v"][n]
    s = dict(case=case, dims=dims, batch=batch, anchors=i["anchors"] if z["K"] else None, k=z["K"], scores=i.get("scores"))
    if case["kind"] == "decode":
        s["plan"] = D.DecodePlan(batch, z["K"], z["block"], z["G"] // z["block"], full=False)
        s["blk"], s["maps"] = z["blk"], batch.maps(s["anchors"], z["K"])
    if case["kind"] == "call":
        s["gain"], s["head"] = i["gain"], i["head"]
        s["rows"] = D.block_row_index(batch, z["K"], z["mb"], z["block"])
    return s


def run(s):
    kind, b = s["case"]["kind"], s.get("batch")
    if kind == "refresh":
        x, _ = b.refresh(s["anchors"], s["k"])
        return dict(x=x, k=b.k_pools[0], v=b.v_pools[0])
    if kind == "probe":
        norm = A.ACACHE_NORM_FULL if s["case"]["norm"] == "full" else A.ACACHE_NORM_AFFIX
        scores, x, _ = b.probe(norm)
        return dict(scores=scores, x=x, k=b.k_pools[0], v=b.v_pools[0])
    if kind == "decode":
        x = D.decode_step(b, s["plan"], s["blk"], s["maps"], s["anchors"])
        return dict(x=x, k=b.k_pools[0], v=b.v_pools[0])
    if kind == "select":
        anchors = A.acache_topk(s["scores"], s["k"])
        m = b.maps(anchors, s["k"])
        return dict(m, anchors=anchors, x=b.gather_inputs(m))
    if kind == "call":
        scores, _, _ = b.probe(outputs=False)
        x, _ = b.refresh(s["anchors"], s["k"])
        h = A.acache_gather_rows(x, s["rows"])
        y = A.acache_rmsnorm(s["dims"], h, s["gain"])
        logits = A.acache_linear(s["dims"], y, s["head"], ws=b.ws)
        return dict(scores=scores, x=x, logits=logits, k=b.k_pools[-1], v=b.v_pools[-1])
    h = A.acache_gather_rows(s["x"], s["rows"])
    y = A.acache_rmsnorm(s["dims"], h, s["gain"])
    A.acache_linear(s["dims"], y, s["w"], out=s["logits"], ws=s["ws"])
    A.acache_argmax_commit(s["logits"], out=s["pick"], conf=s["conf"])
    s["flags"].zero_()
    A.acache_threshold_commit(s["block"], s["pick"], s["conf"], TAU, s["flags"], s["pos"], s["ids"], s["count"])
    return {n: s[n] for n in ("logits", "pick", "conf", "flags", "ids", "count")}


# ---------------------------------------------------------------------------- what it takes, and what it gives
def work(case):
    z = _sizes(case)
    d, es = z["d_model"], 2 if z["dtype"] == "bf16" else 4
    if case["kind"] == "head":
        n = z["B"] * case["block"]
        return dict(bytes=es * (VOCAB * d + n * d + n * VOCAB) + 24 * n, flops=2.0 * n * VOCAB * d)
    B, S, L, R, G, hq, hkv, F = (z[n] for n in ("B", "S", "L", "R", "G", "hq", "hkv", "d_ff"))
    ids = 4 * B * S
    if case["kind"] == "select":
        return dict(bytes=4 * B * (L + z["K"] + 3 * R + S + G) + ids + 2 * es * B * R * d, flops=0.0)
    per_row = 2.0 * (d * (2 * hq + 2 * hkv) + 3 * d * F)
    weights = es * (d * (2 * hq + 2 * hkv) + 3 * d * F)

    def layer(rows, keys, kv_rows):  # rows through the layer, keys each attends to, cached rows read
        return dict(bytes=weights + es * (2 * rows * d + 2 * (rows + kv_rows) * hkv), flops=rows * (per_row + 4.0 * keys * hq))

    score = dict(bytes=4 * B * L, flops=2.0 * B * G * L * hq)
    if case["kind"] == "decode":
        return layer(B * z["block"], S, L + B * (R - z["block"]))
    refresh = layer(B * R, S, L)
    if case["kind"] == "refresh":
        return dict(refresh, bytes=refresh["bytes"] + ids)
    probe = layer(B * z["P"], S, L)
    if case["kind"] == "probe":
        return dict(bytes=probe["bytes"] + score["bytes"] + ids, flops=probe["flops"] + score["flops"])
    n, rows = case["layers"], B * z["block"]
    last = dict(bytes=es * hq * d, flops=2.0 * B * G * hq * d)  # the probe's last layer: queries and scores only
    return dict(bytes=n * refresh["bytes"] + (n - 1) * probe["bytes"] + last["bytes"] + score["bytes"] + es * VOCAB * (d + rows),
                flops=n * refresh["flops"] + (n - 1) * probe["flops"] + last["flops"] + n * score["flops"] + 2.0 * rows * VOCAB * d)


def tolerance(case):
    # measured against exact(): f32 2e-7; a bf16 layer's rows 0.007, its scores 0.0007, its keys and
    # values 0.002; three layers and the logits 0.013; the head's logits 0.0024.  Two paths that round
    # at the same places but sum in another order lie up to sqrt(2) of that apart.
    if case["kind"] == "select":
        return "exact"
    if MODELS[case["model"]]["dtype"] == "f32":
        return {"rel": 5e-6, "max": 1e-4}
    if case["kind"] == "head":
        return {"rel": 1e-2, "max": 0.1}
    return {"rel": 2.5e-2 if case["kind"] == "call" else 1.2e-2, "max": 0.1}


def _norm64(x, g):
    return x / torch.sqrt((x * x).mean(1, keepdim=True) + EPS) * g.double()


def _rotate64(t, pos, dh):
    """Half-split rotary embedding of rows [n, heads * dh] at positions pos [n]."""
    n = t.shape[0]
    theta = BASE ** (-2.0 * torch.arange(dh // 2, device="cuda", dtype=torch.float64) / dh)
    a = (pos.double()[:, None] * theta)[:, None, :]
    t = t.view(n, -1, dh)
    lo, hi = t[..., :dh // 2], t[..., dh // 2:]
    return torch.cat([lo * torch.cos(a) - hi * torch.sin(a), hi * torch.cos(a) + lo * torch.sin(a)], 2).reshape(n, -1)


def _linear64(x, w, rows=8192):
    w = w.double()
    return torch.cat([x[r:r + rows] @ w.t() for r in range(0, x.shape[0], rows)])


def _layer64(z, w, x, pos, req, write, read, kp, vp, score=None):
    """One block in 64 bits.  x, pos, write: rows; req: rows of each request; read: slots of each
    request's keys; kp, vp: the pools, written at write.  score = (rows of the masked queries per
    request, norm, scores [B, L])."""
    dh, H, Hkv, hq, hkv, F = z["head_dim"], z["n_heads"], z["n_kv_heads"], z["hq"], z["hkv"], z["d_ff"]
    qkv = _linear64(_norm64(x, w["attn_norm"]), w["w_qkv"])
    q = _rotate64(qkv[:, :hq], pos, dh)
    kp[write] = _rotate64(qkv[:, hq:hq + hkv], pos, dh)
    vp[write] = qkv[:, hq + hkv:]
    del qkv
    o = torch.empty_like(q)
    scale = 1.0 / math.sqrt(dh)
    for b in range(z["B"]):
        k, v, kl = kp[read[b]], vp[read[b]], kp[:z["L"]]
        for h in range(H):
            col, kv = slice(h * dh, (h + 1) * dh), slice(h // (H // Hkv) * dh, (h // (H // Hkv) + 1) * dh)
            logit = q[req[b], col] @ k[:, kv].t() * scale
            if score is not None:
                at, norm, scores = score
                s = q[at[b], col] @ kl[:, kv].t() * scale
                full = torch.logsumexp(q[at[b], col] @ k[:, kv].t() * scale, 1, keepdim=True) if norm == "full" else None
                scores[b] += torch.exp(s - (torch.logsumexp(s, 1, keepdim=True) if full is None else full)).sum(0)
            o[req[b], col] = torch.softmax(logit, 1) @ v[:, kv]
    x = x + _linear64(o, w["w_o"])
    del o, q
    y = _norm64(x, w["mlp_norm"])
    out = []
    for r in range(0, x.shape[0], 4096):
        gu = _linear64(y[r:r + 4096], w["w_gate_up"])
        out.append(_linear64(gu[:, :F] * torch.sigmoid(gu[:, :F]) * gu[:, F:], w["w_down"]))
    return x + torch.cat(out)


def exact(case, seed):
    if case["kind"] == "select":
        return None
    i = _inputs(case, seed)
    z = i["z"]
    if case["kind"] == "head":
        logits = _linear64(_norm64(i["x"].double(), i["gain"]), i["w"])
        return dict(logits=logits, pick=None, conf=torch.softmax(logits, 1).max(1).values, flags=None, ids=None, count=None)
    B, S, L, ab = z["B"], z["S"], z["L"], z["ab"]
    x_src = i["emb"][i["ids"].view(-1).long()] if i["ids"] is not None else i["emb"]

    def plan(anchors):
        """Positions a call recomputes per request, ascending, their slots, and every key's slot."""
        pos, write, read = [], [], []
        for b in range(B):
            rec = torch.ones(S, dtype=torch.bool, device="cuda")
            rec[ab:ab + L] = False
            if anchors is not None:
                rec[ab + anchors[b].long()] = True
            p = rec.nonzero().view(-1)
            w = z["base"] + b * z["stride"] + torch.arange(len(p), device="cuda")
            r = torch.arange(S, device="cuda") - ab
            r[p] = w
            pos.append(p), write.append(w), read.append(r)
        return pos, write, read

    def pools(n):
        out = []
        for t in (i["k"][n], i["v"][n]):
            p = torch.zeros((z["slots"], z["hkv"]), dtype=torch.float64, device="cuda")
            p[:t.shape[0]] = t.double()
            out.append(p)
        return out

    def stack(pos, write, read, n_layers, kvs, score=None):
        x = torch.cat([x_src[b * S + p] for b, p in enumerate(pos)]).double()
        at, req = 0, []
        for p in pos:
            req.append(slice(at, at + len(p)))
            at += len(p)
        for n in range(n_layers):
            x = _layer64(z, i["layers"][n], x, torch.cat(pos), req, torch.cat(write), read, *kvs[n], score=score)
        return x

    def masked(pos):
        at, out = 0, []
        for p in pos:
            out.append(at + ((p >= z["mb"]).nonzero().view(-1)))
            at += len(p)
        return out

    kvs = [pools(n) for n in range(case["layers"])]
    sel = plan(i["anchors"] if z["K"] else None)
    if case["kind"] == "refresh":
        x = stack(*sel, 1, kvs)
        return dict(x=x, k=kvs[0][0], v=kvs[0][1])
    if case["kind"] == "decode":
        lo = z["mb"] + z["blk"] * z["block"]
        keep = [(p >= lo) & (p < lo + z["block"]) for p in sel[0]]
        x = stack([p[m] for p, m in zip(sel[0], keep)], [w[m] for w, m in zip(sel[1], keep)], sel[2], 1, kvs)
        return dict(x=x, k=kvs[0][0], v=kvs[0][1])
    scores = torch.zeros((B, L), dtype=torch.float64, device="cuda")
    own = plan(None)
    x = stack(*own, case["layers"], kvs, score=(masked(own[0]), case["norm"], scores))
    if case["kind"] == "probe":
        return dict(scores=scores, x=x, k=kvs[0][0], v=kvs[0][1])
    x = stack(*sel, case["layers"], kvs)
    rows = torch.cat([(sel[0][b] >= z["mb"]).nonzero().view(-1)[:z["block"]] + b * z["R"] for b in range(B)])
    logits = _linear64(_norm64(x[rows], i["gain"]), i["head"])
    return dict(scores=scores, x=x, logits=logits, k=kvs[-1][0], v=kvs[-1][1])
