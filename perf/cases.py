"""The work that a user of this library has it do, as cases that can be timed and checked.

A control step is Alg. 1 on two frames (selection, layer ratio, and the embedding of the
patches that are recomputed), the sparse prefill over the rows that are not reused, and the
greedy decode of the other action tokens.  The cases are those calls, alone and together,
through the public binding: one environment and batches of them, step 0 (full recompute) and
later steps, the three operand modes, and the three decoder shapes of this repository.

Decoder layers all do the same work, so calls on a decoder run on a few of them; one case is
the whole control step at full depth.  Weights are N(0, 1.28 / sqrt(d_model)) (0.02 at the 7B
shape); the output head is the
embedding table rolled by some rows and scaled, so that a token has a clear successor and the
greedy choice does not hang on rounding, as with trained weights."""
import math

import torch

import paper_2502_02175_amd as V

DEV = "cuda:0"

# tiny: the smoke shape; 7b: the Llama-2 layout of a 7B decoder; gqa: grouped queries (12 / 2 heads)
MODELS = {
    "tiny": dict(d=256, hq=4, hkv=4, hd=64, f=688, vocab=256, base=1.0e4),
    "7b": dict(d=4096, hq=32, hkv=32, hd=128, f=11008, vocab=32000, base=1.0e4),
    "gqa": dict(d=1536, hq=12, hkv=2, hd=128, f=8960, vocab=32000, base=1.0e6),
}
EPS = 1e-6
OPERAND = {"bf16": V.OPERAND_BF16, "f16": V.OPERAND_F16, "f16w8": V.OPERAND_F16_W8}
BANK = 4   # distinct layers that are drawn; a deeper decoder repeats them


def listed():
    return [
        # everything before the decoder for one environment: a 224 x 224 frame, 14 x 14 patches
        dict(name="front_1x256", kind="front", batch=1, gh=16, gw=16, patch=14, redraw=0.3, layers=32, d=4096),
        # the same for eight environments with a finer grid
        dict(name="front_8x1024", kind="front", batch=8, gh=32, gw=32, patch=14, redraw=0.3, layers=32, d=4096),
        # the smallest control step: launches and latency
        dict(name="step_tiny", kind="step", model="tiny", layers=2, batch=1, gh=8, gw=8, patch=14, text=16,
             redraw=0.25, new=3, operand="f16", adaptive=True),
        # one 7B stream: 109 of 288 rows recomputed, and step 0, which recomputes all of them
        dict(name="sparse_7b_1x288", kind="prefill", model="7b", layers=4, batch=1, vis=256, text=32,
             reuse=0.7, operand="f16", adaptive=False),
        dict(name="full_7b_1x288", kind="prefill", model="7b", layers=4, batch=1, vis=256, text=32,
             reuse=0.0, operand="f16", adaptive=False),
        # two camera views and a chunk of 56 action rows read off one pass, few tokens reused
        dict(name="sparse_7b_1x601", kind="prefill", model="7b", layers=4, batch=1, vis=512, text=89,
             reuse=0.16, operand="bf16", adaptive=False),
        # eight 7B streams of 1057 tokens, each with its own reuse list
        dict(name="sparse_7b_8x1057", kind="prefill", model="7b", layers=4, batch=8, vis=1024, text=33,
             reuse=0.7, operand="f16", adaptive=False),
        # 32 streams of the grouped-query model, reuse growing over the layers
        dict(name="sparse_gqa_32x304", kind="prefill", model="gqa", layers=4, batch=32, vis=256, text=48,
             reuse=0.85, operand="bf16", adaptive=True),
        # the action tokens after the first: one stream, one stream with 8-bit weights, 32 streams
        dict(name="decode_7b_1", kind="decode", model="7b", layers=4, batch=1, len=288, new=6, operand="f16"),
        dict(name="decode_7b_1_w8", kind="decode", model="7b", layers=4, batch=1, len=288, new=6, operand="f16w8"),
        dict(name="decode_gqa_32", kind="decode", model="gqa", layers=4, batch=32, len=304, new=6, operand="f16"),
        # the whole control step of one 7B environment at full depth
        dict(name="step_7b", kind="step", model="7b", layers=32, batch=1, gh=16, gw=16, patch=14, text=32,
             redraw=0.3, new=6, operand="f16", adaptive=False),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        kind = rng.choice(["front", "step", "prefill", "prefill", "prefill", "decode"])
        model = rng.choice(["7b", "7b", "gqa", "tiny"]) if kind != "step" else rng.choice(["tiny", "gqa"])
        operand = rng.choice(["f16", "f16", "bf16", "f16w8"])
        c = dict(kind=kind, batch=log_int(1, 32))
        if kind == "front":
            c.update(gh=rng.randint(7, 32), gw=rng.randint(7, 32), patch=rng.choice([14, 14, 14, 16, 8, 13]),
                     redraw=round(rng.uniform(0.05, 0.9), 2), layers=rng.choice([2, 28, 32]),
                     d=rng.choice([256, 1536, 4096]))
        else:
            c.update(model=model, operand=operand, layers=rng.randint(2, 4))
        if kind == "step":
            c.update(batch=log_int(1, 8), gh=rng.randint(7, 18), gw=rng.randint(7, 18), patch=14, text=rng.randint(12, 48),
                     redraw=round(rng.uniform(0.05, 0.6), 2), new=rng.randint(1, 6), adaptive=rng.random() < 0.5)
        if kind == "prefill":
            c.update(vis=log_int(49, 1024), text=rng.randint(12, 90),
                     reuse=rng.choice([0.0, round(rng.uniform(0.05, 0.95), 2), round(rng.uniform(0.4, 0.95), 2)]),
                     adaptive=rng.random() < 0.4)
            if c["reuse"] == 0.0:
                c["adaptive"] = False
        if kind == "decode":
            c.update(len=log_int(60, 1100), new=rng.randint(1, 7))
        w, top = work(c), work(listed()[6])
        if w["flops"] <= top["flops"] and w["bytes"] <= 4 * top["bytes"]:
            return c


# ------------------------------------------------------------------------------------------
# inputs, from the seed alone
# ------------------------------------------------------------------------------------------
def _gen(seed, *tags):
    g = torch.Generator(device=DEV)
    s = int(seed) & 0xFFFFFFFF
    for t in tags:
        s = (s * 1000003 + int(t) + 1) & 0x7FFFFFFFFFFFFFFF
    g.manual_seed(s)
    return g


def _normal(g, shape, std=1.0):
    return (torch.randn(shape, generator=g, device=DEV) * std).bfloat16()


def _on_e4m3_grid(w):
    """Weights that 8-bit storage holds without loss (codes times a power of two per row): what
    a user of that mode has trained or calibrated for it."""
    top = w.float().abs().amax(dim=1, keepdim=True)
    s = torch.exp2(torch.ceil(torch.log2(top / 448.0)))
    return ((w.float() / s).to(torch.float8_e4m3fn).float() * s).bfloat16()


def _layer(m, seed, l, w8):
    g = _gen(seed, 1, l % BANK)
    q, kv = m["hq"] * m["hd"], m["hkv"] * m["hd"]
    std = 1.28 / math.sqrt(m["d"])
    w = {"wqkv": _normal(g, (q + 2 * kv, m["d"]), std), "wo": _normal(g, (m["d"], q), std),
         "w_gate_up": _normal(g, (2 * m["f"], m["d"]), std), "w_down": _normal(g, (m["d"], m["f"]), std)}
    if w8:
        w = {k: _on_e4m3_grid(v) for k, v in w.items()}
    for k in ("g_attn", "g_ffn"):
        w[k] = (1.0 + 0.1 * torch.randn(m["d"], generator=g, device=DEV)).bfloat16()
    return w


def _head(m, seed, w8):
    g = _gen(seed, 2)
    table = _normal(g, (m["vocab"], m["d"]))
    head = (table.float() * (1.28 / math.sqrt(m["d"]))).bfloat16().roll(m["vocab"] // 3 + 1, 0).contiguous()
    if w8:
        head = _on_e4m3_grid(head)
    return {"g_final": (1.0 + 0.1 * torch.randn(m["d"], generator=g, device=DEV)).bfloat16(),
            "w_head": head, "embed": table}


def _layers(c, m, seed):
    bank = {l: _layer(m, seed, l, c["operand"] == "f16w8") for l in range(min(BANK, c["layers"]))}
    return lambda l: bank[l % BANK]


def _frames(c, seed):
    """Frame t-1 uniform noise; frame t the same with +-2 of sensor noise and a share of the
    patches re-drawn."""
    g, B, p = _gen(seed, 3), c["batch"], c["patch"]
    H, W = c["gh"] * p, c["gw"] * p
    prev = torch.randint(0, 256, (B, H, W, 3), generator=g, device=DEV, dtype=torch.int16)
    cur = (prev + torch.randint(-2, 3, prev.shape, generator=g, device=DEV, dtype=torch.int16)).clamp(0, 255)
    fresh = torch.randint(0, 256, prev.shape, generator=g, device=DEV, dtype=torch.int16)
    changed = torch.rand((B, c["gh"], c["gw"]), generator=g, device=DEV) < c["redraw"]
    mask = changed.repeat_interleave(p, 1).repeat_interleave(p, 2)[..., None]
    cur = torch.where(mask, fresh, cur)
    return prev.to(torch.uint8), cur.to(torch.uint8), changed.reshape(B, -1)


def _statistics(c, seed, vis):
    """Text-to-vision attention of the step before: sharper with depth, as Sec. 3.4 assumes."""
    g = _gen(seed, 4)
    x = torch.randn((c["layers"], c["batch"], vis), generator=g, device=DEV)
    depth = torch.arange(c["layers"], device=DEV).view(-1, 1, 1) / max(1, c["layers"])
    return (0.8 * torch.softmax(x * (0.3 + 1.5 * depth), dim=2)).contiguous()


def _embeddings(c, m, seed, vis, head, changed):
    """Embeddings of the steps t-1 and t: text rows are rows of the table (the instruction
    stays), visual rows change where the frame does."""
    g, B = _gen(seed, 5), c["batch"]
    ids = torch.randint(0, m["vocab"], (B, c["text"]), generator=g, device=DEV)
    text = head["embed"][ids].float()
    e0 = _normal(g, (B, vis, m["d"])).float()
    e1 = torch.where(changed[..., None], _normal(g, (B, vis, m["d"])).float(), e0)
    return torch.cat([e0, text], 1).contiguous(), torch.cat([e1, text], 1).contiguous()


def _lists(c, seed):
    """Reuse lists: every stream has its own, of its own length; -> order [B, stride], count [B],
    layer_count [B, layers] or None, and the changed (not reused) positions."""
    g, B, vis = _gen(seed, 6), c["batch"], c["vis"]
    share = torch.rand(B, generator=g, device=DEV) * 0.1 + 0.95 if B > 1 else torch.ones(B, device=DEV)
    count = (c["reuse"] * vis * share).round().clamp(0, vis).to(torch.int32)
    stride = max(1, min(vis, int(round(c["reuse"] * vis * 1.05))))
    count = count.clamp(max=stride)
    perm = torch.rand((B, vis), generator=g, device=DEV).argsort(1).to(torch.int32)
    order = perm[:, :stride].contiguous()
    reused = torch.zeros((B, vis), dtype=torch.bool, device=DEV)
    live = torch.arange(stride, device=DEV)[None, :] < count[:, None]
    reused.scatter_(1, order.long(), live)
    per_layer = None
    if c["adaptive"]:  # the first layer reuses nothing, the last all of the list
        ramp = torch.arange(c["layers"], device=DEV).float() / max(1, c["layers"] - 1)
        per_layer = (ramp[None, :] * count[:, None]).to(torch.int32).contiguous()
    return order, count, per_layer, ~reused, stride


# ------------------------------------------------------------------------------------------
# what a program keeps
# ------------------------------------------------------------------------------------------
class _Ctx:
    """A context with its weights and its KV cache."""

    def __init__(self, m, layers, batch, seq, operand):
        self.cfg = V.ModelCfg(layers, m["d"], m["hq"], m["hkv"], m["hd"], m["f"], m["vocab"], EPS, m["base"],
                              batch, -(-seq // 32) * 32, OPERAND[operand])
        self.handle = V.vlac_create(self.cfg)
        self.kv = torch.empty(V.vlac_kv_cache_bytes(self.cfg), dtype=torch.uint8, device=DEV)
        for b in range(batch):
            V.vlac_reset_stream(self.handle, b, self.kv)

    def __del__(self):
        if getattr(self, "handle", None):
            V.vlac_destroy(self.handle)
            self.handle = None


def _decoder(c, m, seed, seq):
    ctx = _Ctx(m, c["layers"], c["batch"], seq, c["operand"])
    get = _layers(c, m, seed)
    for l in range(c["layers"]):
        V.vlac_set_layer_weights(ctx.handle, l, get(l))
    head = _head(m, seed, c["operand"] == "f16w8")
    V.vlac_set_head_weights(ctx.handle, head["g_final"], head["w_head"], head["embed"])
    torch.cuda.synchronize()
    return ctx, head


def _selection_buffers(c, vis):
    B, k = c["batch"], max(1, int(0.7 * vis))
    i32 = dict(dtype=torch.int32, device=DEV)
    return dict(top_k=k, idx=torch.zeros((B, k), **i32), order=torch.zeros((B, k), **i32), count=torch.zeros(B, **i32),
                relevance=torch.zeros((B, vis), device=DEV), alpha=torch.zeros((B, c["layers"]), device=DEV),
                per_layer=torch.zeros((B, c["layers"]), **i32))


def _prefill_buffers(c, m, L, vis):
    B = c["batch"]
    return dict(stats=torch.zeros((c["layers"], B, vis), device=DEV), hidden=torch.zeros((B, L, m["d"]), device=DEV),
                logits=torch.zeros((B, m["vocab"]), device=DEV), token=torch.zeros(B, dtype=torch.int32, device=DEV))


def _decode_buffers(c, m):
    return dict(tokens=torch.zeros((c["batch"], c["new"]), dtype=torch.int32, device=DEV),
                token_logits=torch.zeros((c["batch"], c["new"], m["vocab"]), device=DEV))


def prepare(case, seed):
    c, s = case, {"c": case}
    if c["kind"] == "front":
        vis = c["gh"] * c["gw"]
        s["prev"], s["cur"], _ = _frames(c, seed)
        s["attn"] = _statistics(c, seed, vis)
        s["proj"] = _normal(_gen(seed, 7), (3 * c["patch"] ** 2, c["d"]), math.sqrt(3.0 / (3 * c["patch"] ** 2)))
        # (nothing of the decoder is used but its depth and its width)
        s["ctx"] = _Ctx(dict(d=c["d"], hq=4, hkv=4, hd=64, f=16, vocab=32, base=1e4), c["layers"], c["batch"], 32, "f16")
        s.update(_selection_buffers(c, vis))
        s["embeds"] = torch.zeros((c["batch"], vis + 32, c["d"]), device=DEV)
        return s
    m = MODELS[c["model"]]
    if c["kind"] == "decode":
        s["ctx"], head = _decoder(c, m, seed, c["len"] + c["new"])
        emb = _normal(_gen(seed, 5), (c["batch"], c["len"], m["d"])).float()
        s["first"] = torch.randint(0, m["vocab"], (c["batch"],), generator=_gen(seed, 8), device=DEV).to(torch.int32)
        V.vlac_sparse_prefill(s["ctx"].handle, emb, c["batch"], 0, c["len"], None, None, 1, None, s["ctx"].kv, None, None,
                              None, torch.zeros(c["batch"], dtype=torch.int32, device=DEV))
        s.update(_decode_buffers(c, m))
        torch.cuda.synchronize()
        return s
    if c["kind"] == "step":
        vis = c["gh"] * c["gw"]
        L = vis + c["text"]
        s["ctx"], head = _decoder(c, m, seed, L + c["new"])
        s["prev"], s["cur"], changed = _frames(c, seed)
        s["attn"] = _statistics(c, seed, vis)
        s.update(_selection_buffers(c, vis))
        s.update(_decode_buffers(c, m))
    else:
        vis = c["vis"]
        L = vis + c["text"]
        s["ctx"], head = _decoder(c, m, seed, L)
        s["list"], s["n"], s["by_layer"], changed, s["stride"] = _lists(c, seed)
    e0, s["embeds"] = _embeddings(c, m, seed, vis, head, changed)
    s.update(_prefill_buffers(c, m, L, vis))
    s["vis"] = vis
    # the step before: a full prefill of frame t-1 leaves the cache that this step starts from
    V.vlac_sparse_prefill(s["ctx"].handle, e0, c["batch"], vis, c["text"], None, None, 1, None, s["ctx"].kv, None, None,
                          None, s["token"])
    torch.cuda.synchronize()
    return s


# ------------------------------------------------------------------------------------------
# one pass
# ------------------------------------------------------------------------------------------
def _select(s, tau_task):
    c, ctx = s["c"], s["ctx"].handle
    B, vis = c["batch"], c["gh"] * c["gw"]
    V.vlac_select_static(ctx, s["prev"], s["cur"], B, c["gh"] * c["patch"], c["gw"] * c["patch"], c["patch"], 249, 250,
                         s["top_k"], s["attn"], None, tau_task, s["idx"], s["order"], s["count"], s["relevance"], s["top_k"])
    V.vlac_layer_ratio(ctx, s["attn"], B, vis, 1.5, s["count"], s["alpha"], s["per_layer"])


def run(state):
    s, c = state, state["c"]
    ctx, B = s["ctx"].handle, c["batch"]
    if c["kind"] == "front":
        _select(s, 0.5)
        V.vlac_embed_patches(ctx, s["cur"], B, c["gh"] * c["patch"], c["gw"] * c["patch"], c["patch"], s["proj"],
                             s["order"], s["count"], s["top_k"], None, s["embeds"], s["embeds"].shape[1])
        return {k: s[k] for k in ("idx", "order", "count", "relevance", "alpha", "per_layer", "embeds")}
    if c["kind"] == "decode":
        V.vlac_decode_action(ctx, B, c["len"], c["new"], s["first"], s["ctx"].kv, s["tokens"], s["token_logits"])
        return {"tokens": s["tokens"], "token_logits": s["token_logits"]}
    if c["kind"] == "prefill":
        sparse = c["reuse"] > 0
        V.vlac_sparse_prefill(ctx, s["embeds"], B, s["vis"], c["text"], s["list"] if sparse else None,
                              s["n"] if sparse else None, s["stride"], s["by_layer"], s["ctx"].kv, s["stats"], s["hidden"],
                              s["logits"], s["token"])
        return {k: s[k] for k in ("stats", "hidden", "logits", "token")}
    _select(s, 1.0)
    V.vlac_sparse_prefill(ctx, s["embeds"], B, s["vis"], c["text"], s["order"], s["count"], s["top_k"],
                          s["per_layer"] if c["adaptive"] else None, s["ctx"].kv, s["stats"], s["hidden"], s["logits"],
                          s["token"])
    V.vlac_decode_action(ctx, B, s["vis"] + c["text"], c["new"], s["token"], s["ctx"].kv, s["tokens"], s["token_logits"])
    return {k: s[k] for k in ("count", "order", "alpha", "stats", "hidden", "logits", "token", "tokens", "token_logits")}


# ------------------------------------------------------------------------------------------
# what a pass cannot do without
# ------------------------------------------------------------------------------------------
def _pass_work(m, c, rows, seen, layers, per_weight):
    """One pass of `rows` rows (all streams), each seeing `seen` positions; cache of c["batch"] streams."""
    q, kv = m["hq"] * m["hd"], m["hkv"] * m["hd"]
    weights = (q + 2 * kv) * m["d"] + m["d"] * q + 3 * m["f"] * m["d"]
    by = layers * (weights * per_weight + c["batch"] * seen * 2 * kv * 2) + m["vocab"] * m["d"] * per_weight
    fl = layers * (2.0 * rows * weights + 4.0 * rows * seen * q) + 2.0 * c["batch"] * m["vocab"] * m["d"]
    return by + c["batch"] * m["vocab"] * 4, fl


def work(case):
    c = case
    by = fl = 0.0
    if c["kind"] in ("front", "step"):
        vis = c["gh"] * c["gw"]
        by += c["batch"] * (2 * vis * 3 * c["patch"] ** 2 + c["layers"] * vis * 4)
        if c["kind"] == "front":
            live = c["batch"] * vis * max(c["redraw"], 1 - 0.35)  # at most half of the most similar 70 % is reused
            by += 3 * c["patch"] ** 2 * c["d"] * 2 + live * c["d"] * 4
            fl += 2.0 * live * 3 * c["patch"] ** 2 * c["d"]
            return {"bytes": by, "flops": fl}
    m = MODELS[c["model"]]
    pw = 1 if c["operand"] == "f16w8" else 2
    if c["kind"] == "decode":
        L = c["len"]
    else:
        vis = c["vis"] if c["kind"] == "prefill" else c["gh"] * c["gw"]
        L = vis + c["text"]
        reuse = c["reuse"] if c["kind"] == "prefill" else min(0.7, 1 - c["redraw"])
        rows = c["batch"] * (L - vis * reuse * (0.5 if c["adaptive"] else 1.0))
        b, f = _pass_work(m, c, rows, L, c["layers"], pw)
        by += b + 2 * rows * m["d"] * 4 + c["layers"] * c["batch"] * vis * 4
        fl += f - c["layers"] * 2.0 * rows * L * m["hq"] * m["hd"]  # (causal: about half of the keys)
    for t in range(c.get("new", 0)):
        b, f = _pass_work(m, c, c["batch"], L + t + 1, c["layers"], pw)
        by, fl = by + b, fl + f
    return {"bytes": float(by), "flops": float(fl)}


def tolerance(case):
    c = case
    if c["kind"] == "front":
        # fp32 sums over 3 patch^2 products and over the layers; counts: floor() of an fp32 product
        return {"rel": 1e-5, "max": 1e-4, "differ": 0.001}
    # 16-bit operands, rounded at every layer (fp32 sums): four times the distance from exact()
    # that the roundings alone leave (fp16: 1.0e-3 over 4 layers, 2.5e-3 over 32; bf16: 7e-3 over 4)
    deep = c["layers"] > 8
    if c["operand"] == "bf16":
        return {"rel": 0.03, "max": 0.3, "differ": 0.002}
    return {"rel": 0.01 if deep else 0.004, "max": 0.1 if deep else 0.04, "differ": 0.002}


# ------------------------------------------------------------------------------------------
# the same in 64 bits
# ------------------------------------------------------------------------------------------
def _norm(x, g):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + EPS) * g.double()


def _rope(x, pos, m):
    """x [rows, heads, hd], pos [rows]: rotate-half pairing."""
    h = m["hd"] // 2
    ang = pos.double()[:, None] * torch.pow(torch.tensor(m["base"], dtype=torch.float64, device=DEV),
                                            -torch.arange(h, device=DEV).double() / h)
    cos, sin = ang.cos()[:, None, :], ang.sin()[:, None, :]
    a, b = x[..., :h], x[..., h:]
    return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)


def _exact_layer(m, w, h, pos, stream, K, Vv, vis, text, stats):
    """Rows (stream[i], pos[i]) of the residual stream h [rows, d]; K, Vv [B, T, hkv, hd] are updated in place.
    stats: [B, vis] to fill, or None."""
    q, kv, hd, grp = m["hq"] * m["hd"], m["hkv"] * m["hd"], m["hd"], m["hq"] // m["hkv"]
    y = _norm(h, w["g_attn"]) @ w["wqkv"].double().t()
    Q = _rope(y[:, :q].reshape(-1, m["hq"], hd), pos, m)
    K[stream, pos] = _rope(y[:, q:q + kv].reshape(-1, m["hkv"], hd), pos, m)
    Vv[stream, pos] = y[:, q + kv:].reshape(-1, m["hkv"], hd)
    out = torch.empty((h.shape[0], q), dtype=torch.float64, device=DEV)
    for b in range(K.shape[0]):
        mine = (stream == b).nonzero()[:, 0]
        p = pos[mine]
        T = int(p.max()) + 1
        k = K[b, :T].repeat_interleave(grp, 1).permute(1, 2, 0).contiguous()
        v = Vv[b, :T].repeat_interleave(grp, 1).permute(1, 0, 2).contiguous()
        a = torch.matmul(Q[mine].permute(1, 0, 2).contiguous(), k) / math.sqrt(hd)
        a = a.masked_fill(torch.arange(T, device=DEV)[None, None, :] > p[None, :, None], float("-inf")).softmax(-1)
        out[mine] = torch.matmul(a, v).permute(1, 0, 2).reshape(len(mine), q)
        if stats is not None:
            stats[b] = a[:, p >= vis, :vis].sum((0, 1)) / (m["hq"] * text)
    h = h + out @ w["wo"].double().t()
    y = _norm(h, w["g_ffn"]) @ w["w_gate_up"].double().t()
    gate, up = y[:, :m["f"]], y[:, m["f"]:]
    return h + (gate * torch.sigmoid(gate) * up) @ w["w_down"].double().t()


def _exact_prefill(c, m, get, head, emb, vis, cache, alive):
    """alive [layers][B, L]: the rows that are recomputed.  -> stats, hidden, logits of the last position."""
    B, L, d = emb.shape
    H = emb.double().clone()
    stats = torch.zeros((c["layers"], B, max(vis, 1)), dtype=torch.float64, device=DEV)
    text = L - vis
    for l in range(c["layers"]):
        st, ps = alive[l].nonzero(as_tuple=True)
        H[st, ps] = _exact_layer(m, get(l), H[st, ps], ps, st, cache[l][0], cache[l][1], vis, text,
                                 stats[l] if vis else None)
    hidden = torch.where(alive[-1][..., None], _norm(H, head["g_final"]), torch.zeros((), dtype=torch.float64, device=DEV))
    return stats, hidden, hidden[:, L - 1] @ head["w_head"].double().t()


def _exact_decode(c, m, get, head, first, L, cache):
    B, tok, out = c["batch"], first.long(), []
    stream = torch.arange(B, device=DEV)
    for t in range(c["new"]):
        h = head["embed"][tok].double()
        pos = torch.full((B,), L + t, dtype=torch.long, device=DEV)
        for l in range(c["layers"]):
            h = _exact_layer(m, get(l), h, pos, stream, cache[l][0], cache[l][1], 0, 0, None)
        out.append(_norm(h, head["g_final"]) @ head["w_head"].double().t())
        tok = out[-1].argmax(-1)
    return torch.stack(out, 1)


def _exact_selection(c, seed, tau_task):
    """-> reused lists in reuse order, relevance, alpha."""
    B, p, gh, gw = c["batch"], c["patch"], c["gh"], c["gw"]
    vis = gh * gw
    prev, cur, _ = _frames(c, seed)

    def patches(f):
        return f.double().reshape(B, gh, p, gw, p * 3).permute(0, 1, 3, 2, 4).reshape(B, vis, -1)

    a, b = patches(prev), patches(cur)
    sim = (a * b).sum(-1) ** 2 / ((a * a).sum(-1) * (b * b).sum(-1))
    attn = _statistics(c, seed, vis)
    score = torch.zeros((B, vis), device=DEV)
    for l in range(c["layers"]):
        score = score + attn[l]
    score = score / c["layers"]
    top_k, n_rel = max(1, int(0.7 * vis)), vis - math.floor(tau_task * vis)
    order = []
    for i in range(B):
        ranked = sim[i].sort(descending=True, stable=True)[1]
        ranked = ranked[sim[i][ranked] >= (249 / 250) ** 2][:top_k]
        keep = torch.zeros(vis, dtype=torch.bool, device=DEV)
        keep[ranked] = True
        keep[score[i].sort(descending=True, stable=True)[1][:n_rel]] = False
        mine = keep.nonzero()[:, 0]
        order.append(mine[score[i][mine].sort(stable=True)[1]])
    x = attn.double() / attn.double().sum(-1, keepdim=True)
    ent = -(x * x.log()).sum(-1)
    ratio = torch.zeros_like(ent)
    ratio[1:] = (ent[:-1] - ent[1:]) / ent[:-1]
    alpha = (1.5 * ratio.cumsum(0)).clamp(0, 1).cummax(0)[0].t().contiguous()
    return order, attn.double().mean(0), alpha, cur


def exact(case, seed):
    c = case
    with torch.no_grad():
        if c["kind"] == "front":
            order, rel, alpha, cur = _exact_selection(c, seed, 0.5)
            B, p, vis = c["batch"], c["patch"], c["gh"] * c["gw"]
            proj = _normal(_gen(seed, 7), (3 * p * p, c["d"]), math.sqrt(3.0 / (3 * p * p))).double()
            px = cur.double().reshape(B, c["gh"], p, c["gw"], p * 3).permute(0, 1, 3, 2, 4).reshape(B, vis, -1)
            emb = torch.zeros((B, vis + 32, c["d"]), dtype=torch.float64, device=DEV)
            emb[:, :vis] = (px / 127.5 - 1.0) @ proj
            for b in range(B):
                emb[b, order[b]] = 0
            return {"idx": None, "order": None, "count": None, "relevance": rel, "alpha": alpha, "per_layer": None,
                    "embeds": emb}
        m = MODELS[c["model"]]
        get, head, B = _layers(c, m, seed), _head(m, seed, c["operand"] == "f16w8"), c["batch"]
        w8 = c["operand"] == "f16w8"
        if c["kind"] == "decode":
            vis, L = 0, c["len"]
            e0 = _normal(_gen(seed, 5), (B, L, m["d"])).float()
        else:
            vis = c["vis"] if c["kind"] == "prefill" else c["gh"] * c["gw"]
            L = vis + c["text"]
            if c["kind"] == "prefill":
                order, count, by_layer, changed, _ = _lists(c, seed)
                lists = [order[b, :int(count[b])].long() for b in range(B)]
            else:
                lists, _, alpha, _ = _exact_selection(c, seed, 1.0)
                changed = _frames(c, seed)[2]
                by_layer = None
                if c["adaptive"]:
                    n = torch.tensor([len(x) for x in lists], device=DEV)
                    by_layer = torch.floor(alpha.float() * n[:, None].float()).long()
            e0, e1 = _embeddings(c, m, seed, vis, head, changed)
        T = L + c.get("new", 0)
        cache = [torch.zeros((2, B, T, m["hkv"], m["hd"]), dtype=torch.float64, device=DEV) for _ in range(c["layers"])]
        every = torch.ones((B, L), dtype=torch.bool, device=DEV)
        _exact_prefill(c, m, get, head, e0, vis, cache, [every] * c["layers"])
        if c["kind"] == "decode":
            first = torch.randint(0, m["vocab"], (B,), generator=_gen(seed, 8), device=DEV)
            return {"tokens": None, "token_logits": _exact_decode(c, m, get, head, first, L, cache)}
        alive = []
        for l in range(c["layers"]):
            a = every.clone()
            if c["kind"] == "step" or c["reuse"] > 0:
                for b in range(B):
                    n = len(lists[b]) if by_layer is None else int(by_layer[b, l])
                    a[b, lists[b][:n]] = False
            alive.append(a)
        stats, hidden, logits = _exact_prefill(c, m, get, head, e1, vis, cache, alive)
        out = {"stats": stats, "hidden": hidden, "logits": logits, "token": None}
        if c["kind"] == "step":
            out.update(count=None, order=None, alpha=alpha, tokens=None,
                       token_logits=_exact_decode(c, m, get, head, logits.argmax(-1), L, cache))
        return out
