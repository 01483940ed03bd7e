"""What a user of the framework has it do, as a list of measurable cases.

Every case is one pass through a public entry point of paper_2605_18710_amd.binding: a training
step of one module (forward, loss or given upstream gradient, backward), a whole stage of
colocated modules, or an optimizer step.  Transformer cases hold one layer (two where the first
and the last layer of a stack take different roads), so that a change of rounding stays
inside the layer; the stage runs stacks of several layers.

A case is a dict of plain values.  `kind` says which family it belongs to:

  encoder     pre-norm layer, LayerNorm, GELU, biases, full attention (vision / audio encoders)
  decoder     RMSNorm, SwiGLU, no biases, causal attention; rotary embedding and grouped
              key/value heads as options
  projector   Linear, GELU, Linear between an encoder and a decoder
  patch_stem  image -> patches -> tokens
  text_stem   image tokens followed by embedding rows; its backward forms the embedding gradient
  conv_stem   the two-convolution audio stem
  optimizer   AdamW over the flat parameters of a module
  stage       vision encoder + projector beside a decoder, each on its own share of the CUs
"""
import math

import torch

from paper_2605_18710_amd import binding as mb

CUS = 256


# ------------------------------------------------------------------------------- the cases
def _encoder(batch, seq, hidden, heads, mlp, layers=1, dtype="bf16", **kw):
    return dict(kind="encoder", dtype=dtype, batch=batch, seq=seq, hidden=hidden, heads=heads, mlp=mlp, layers=layers, **kw)


def _decoder(batch, seq, hidden, heads, mlp, layers=1, dtype="bf16", kv_heads=0, rope=0.0, **kw):
    return dict(kind="decoder", dtype=dtype, batch=batch, seq=seq, hidden=hidden, heads=heads, mlp=mlp, layers=layers,
                kv_heads=kv_heads, rope=rope, **kw)


def listed():
    return [
        # the smallest call: the decoder of the fp32 workload, 256 tokens; launches and latency
        _decoder(2, 128, 128, 4, 384, dtype="f32", name="decoder_f32_tiny"),
        # ViT-B/16 layer at 224 px, batch 8: ragged 196 tokens, tiles too few for the chip
        _encoder(8, 196, 768, 12, 3072, layers=2, name="vit_b_layers"),
        # ViT-L/14 layer at 336 px, batch 16: an ordinary encoder size
        _encoder(16, 576, 1024, 16, 4096, name="vit_l_layer"),
        # audio encoder layer: 1500 frames, not a multiple of any tile
        _encoder(8, 1500, 1280, 20, 5120, name="audio_layer"),
        # layer of a small language model (the decoder beside the ViT-B) with the options that
        # language models use: rotary embedding and four query heads per key/value head
        _decoder(8, 1024, 2048, 16, 5632, kv_heads=4, rope=10000.0, name="decoder_small_gqa_rope"),
        # the largest: layer of the 7B-shaped decoder, 8 x 4096 tokens
        _decoder(8, 4096, 4096, 32, 11008, name="decoder_7b_layer"),
        # vision-to-language projector of the ViT-B workload
        dict(kind="projector", dtype="bf16", batch=8, seq=196, in_dim=768, out_dim=2048, name="projector"),
        # patch embedding at 336 px with 14 x 14 patches: 588 values per patch
        dict(kind="patch_stem", dtype="bf16", batch=16, grid=24, patch=14, hidden=1024, name="patch_stem_336"),
        # embedding of text behind a varying number of image tokens, vocabulary 32000
        dict(kind="text_stem", dtype="bf16", batch=8, seq=1024, hidden=2048, vocab=32000, n_img=196, counts=True, name="text_stem"),
        # convolutional audio stem: 3000 frames of 80 mel bins -> 1500 tokens
        dict(kind="conv_stem", dtype="bf16", batch=8, seq=1500, in_dim=80, hidden=1280, name="conv_stem_audio"),
        # AdamW over a 7B-shaped decoder layer, with an fp32 master copy
        dict(kind="optimizer", dtype="bf16", hidden=4096, heads=32, mlp=11008, master=True, name="adamw_7b_layer"),
        # a stage: ViT-B and projector on 64 CUs beside the small language model on 192
        dict(kind="stage", dtype="bf16", batch=8, vit_seq=196, vit_hidden=768, vit_heads=12, vit_layers=3,
             llm_seq=1024, llm_hidden=2048, llm_heads=16, llm_mlp=5632, llm_layers=1, vit_cus=64, name="stage_vit_llm"),
    ]


def _log(rng, lo, hi):
    """Whole number, uniform over the logarithm of [lo, hi]."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    largest = _flops(listed()[5])
    kind = rng.choice(["f32", "encoder", "encoder", "decoder", "decoder", "projector", "patch_stem", "text_stem",
                       "conv_stem", "optimizer", "stage"])
    if kind == "f32":
        d, heads = rng.choice([16, 32, 64]), rng.choice([2, 4, 8])
        h = d * heads
        f = 4 * rng.randint(h // 2, h)
        b, n = rng.randint(1, 4), _log(rng, 8, 256)
        if rng.random() < 0.5:
            return _encoder(b, n, h, heads, f, dtype="f32")
        return _decoder(b, n, h, heads, f, dtype="f32", kv_heads=rng.choice([0, heads // 2]), rope=rng.choice([0.0, 10000.0]))
    if kind == "encoder":
        d = rng.choice([64, 64, 128])
        heads = rng.randint(6, 25) if d == 64 else rng.randint(4, 25)
        h = d * heads
        return _encoder(rng.randint(1, 16), _log(rng, 49, 1500), h, heads, 4 * h)
    if kind == "decoder":
        heads = rng.choice([8, 12, 16, 24, 32, 40])
        h = 128 * heads
        f = 64 * int(h * rng.uniform(2.5, 3.5) / 64)
        c = _decoder(rng.randint(1, 8), _log(rng, 128, 4096), h, heads, f, kv_heads=rng.choice([0, 0, heads // 4, heads // 2]),
                     rope=rng.choice([0.0, 10000.0]))
        while _flops(c) > largest:
            c["batch"] = max(1, c["batch"] // 2)
        return c
    if kind == "projector":
        return dict(kind="projector", dtype="bf16", batch=rng.randint(1, 16), seq=_log(rng, 49, 1500),
                    in_dim=64 * rng.randint(8, 50), out_dim=128 * rng.randint(8, 40))
    if kind == "patch_stem":
        return dict(kind="patch_stem", dtype="bf16", batch=rng.randint(1, 16), grid=rng.randint(7, 32), patch=rng.choice([14, 16]),
                    hidden=64 * rng.randint(6, 50))
    if kind == "text_stem":
        n = _log(rng, 128, 4096)
        return dict(kind="text_stem", dtype="bf16", batch=rng.randint(1, 8), seq=n, hidden=128 * rng.randint(4, 40),
                    vocab=_log(rng, 1000, 64000), n_img=rng.randint(0, n // 2), counts=rng.random() < 0.5)
    if kind == "conv_stem":
        return dict(kind="conv_stem", dtype="bf16", batch=rng.randint(1, 8), seq=_log(rng, 100, 1500), in_dim=rng.choice([80, 128]),
                    hidden=64 * rng.randint(6, 20))
    if kind == "optimizer":
        heads = rng.choice([4, 8, 16, 24, 32])
        h = 128 * heads
        return dict(kind="optimizer", dtype="bf16", hidden=h, heads=heads, mlp=64 * int(h * rng.uniform(2.5, 3.5) / 64),
                    master=rng.random() < 0.5)
    heads = rng.choice([8, 12, 16])
    vit_heads = rng.choice([6, 8, 12])
    return dict(kind="stage", dtype="bf16", batch=rng.randint(1, 8), vit_seq=_log(rng, 49, 256), vit_hidden=64 * vit_heads,
                vit_heads=vit_heads, vit_layers=rng.randint(1, 3), llm_seq=_log(rng, 128, 1024), llm_hidden=128 * heads,
                llm_heads=heads, llm_mlp=64 * int(128 * heads * 2.75 / 64), llm_layers=1, vit_cus=rng.choice([32, 64, 96, 128]))


# ----------------------------------------------------------- module descriptions and sizes
def _desc(c):
    """The module descriptor (binding.Module's cfg) of a case."""
    k = c["kind"]
    if k == "encoder":
        return dict(kind="encoder", batch=c["batch"], seq=c["seq"], hidden=c["hidden"], heads=c["heads"], mlp=c["mlp"],
                    layers=c["layers"], norm="layernorm", act="gelu", causal=0, bias=1, eps=1e-5)
    if k == "decoder":
        return dict(kind="decoder", batch=c["batch"], seq=c["seq"], hidden=c["hidden"], heads=c["heads"], mlp=c["mlp"],
                    layers=c["layers"], norm="rmsnorm", act="swiglu", causal=1, bias=0, eps=1e-5,
                    kv_heads=c["kv_heads"], rope=c["rope"])
    if k == "projector":
        return dict(kind="projector", batch=c["batch"], seq=c["seq"], in_dim=c["in_dim"], out_dim=c["out_dim"])
    if k == "patch_stem":
        return dict(kind="patch_stem", batch=c["batch"], seq=c["grid"] ** 2, hidden=c["hidden"], patch=c["patch"],
                    in_dim=3 * c["patch"] ** 2)
    if k == "text_stem":
        return dict(kind="text_stem", batch=c["batch"], seq=c["seq"], hidden=c["hidden"], vocab=c["vocab"], n_img=c["n_img"])
    if k == "conv_stem":
        return dict(kind="conv_stem", batch=c["batch"], seq=c["seq"], in_dim=c["in_dim"], hidden=c["hidden"])
    if k == "optimizer":        # the descriptor only lays out the parameters; one short sequence keeps the workspace small
        return dict(kind="decoder", batch=1, seq=16, hidden=c["hidden"], heads=c["heads"], mlp=c["mlp"], layers=1,
                    norm="rmsnorm", act="swiglu", causal=1, bias=0, eps=1e-5)
    raise KeyError(k)


def _stage_modules(c):
    """(name, case, has a target) of a stage's modules, in order; the first two share a quota."""
    return [("vit", _encoder(c["batch"], c["vit_seq"], c["vit_hidden"], c["vit_heads"], 4 * c["vit_hidden"], layers=c["vit_layers"]), False),
            ("proj", dict(kind="projector", dtype="bf16", batch=c["batch"], seq=c["vit_seq"], in_dim=c["vit_hidden"], out_dim=c["llm_hidden"]), False),
            ("llm", _decoder(c["batch"], c["llm_seq"], c["llm_hidden"], c["llm_heads"], c["llm_mlp"], layers=c["llm_layers"]), True)]


def _shapes(c):
    """Parameter tensors of a module case: name -> shape."""
    k = c["kind"]
    if k in ("encoder", "decoder", "optimizer"):
        h, f, H = c["hidden"], c["mlp"], c["heads"]
        kv = c.get("kv_heads") or H
        qw = (H + 2 * kv) * (h // H)
        s = {}
        for l in range(c.get("layers", 1)):
            p = "L%d." % l
            if k == "encoder":
                s.update({p + "ln1_g": (h,), p + "ln1_b": (h,), p + "w_qkv": (h, qw), p + "b_qkv": (qw,), p + "w_o": (h, h), p + "b_o": (h,),
                          p + "ln2_g": (h,), p + "ln2_b": (h,), p + "w_1": (h, f), p + "b_1": (f,), p + "w_2": (f, h), p + "b_2": (h,)})
            else:
                s.update({p + "rms1_g": (h,), p + "w_qkv": (h, qw), p + "w_o": (h, h), p + "rms2_g": (h,), p + "w_gu": (h, 2 * f),
                          p + "w_down": (f, h)})
        return s
    if k == "projector":
        a, b = c["in_dim"], c["out_dim"]
        return {"w_1": (a, b), "b_1": (b,), "w_2": (b, b), "b_2": (b,)}
    if k == "patch_stem":
        return {"w_stem": (3 * c["patch"] ** 2, c["hidden"]), "b_stem": (c["hidden"],), "pos": (c["grid"] ** 2, c["hidden"])}
    if k == "text_stem":
        return {"table": (c["vocab"], c["hidden"])}
    if k == "conv_stem":
        a, h = c["in_dim"], c["hidden"]
        return {"w_c1": (3 * a, h), "b_c1": (h,), "w_c2": (3 * h, h), "b_c2": (h,), "pos": (c["seq"], h)}
    raise KeyError(k)


def _in_out(c):
    """Shapes of a module case's input and output."""
    k = c["kind"]
    if k in ("encoder", "decoder"):
        t = c["batch"] * c["seq"]
        return (t, c["hidden"]), (t, c["hidden"])
    if k == "projector":
        t = c["batch"] * c["seq"]
        return (t, c["in_dim"]), (t, c["out_dim"])
    if k == "patch_stem":
        side = c["grid"] * c["patch"]
        return (c["batch"], 3, side, side), (c["batch"] * c["grid"] ** 2, c["hidden"])
    if k == "text_stem":
        return (c["batch"] * c["n_img"], c["hidden"]), (c["batch"] * c["seq"], c["hidden"])
    if k == "conv_stem":
        return (c["batch"], 2 * c["seq"], c["in_dim"]), (c["batch"] * c["seq"], c["hidden"])
    raise KeyError(k)


def _count(shape):
    n = 1
    for v in shape:
        n *= v
    return n


# --------------------------------------------------------------------------------- inputs
def _dtype(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _inputs(c, seed):
    """What the module starts from, from the seed alone: parameters by name (matrices N(0, 0.02),
    gains near 1, biases near 0), the staged input, and the upstream gradient or the target."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    td = _dtype(c)

    def normal(shape, std=1.0, mean=0.0):
        return torch.randn(shape, generator=g, device="cuda").mul_(std).add_(mean).to(td)

    P = {n: normal(s, 0.02, 1.0 if n.endswith("_g") else 0.0) for n, s in _shapes(c).items()}
    if c["kind"] == "optimizer":
        n = sum(_count(s) for s in _shapes(c).values())
        return dict(P=P, grad=normal((n,), 1e-3), m=torch.randn(n, generator=g, device="cuda").mul_(1e-4),
                    v=torch.rand(n, generator=g, device="cuda").mul_(1e-6))
    si, so = _in_out(c)
    inp = dict(P=P)
    if c["kind"] == "patch_stem":          # pixels in [0, 1)
        inp["x"] = torch.rand(si, generator=g, device="cuda").to(td)
    else:
        inp["x"] = normal(si)
    if c["kind"] == "decoder":
        inp["target"] = normal(so)
    else:                                   # an upstream gradient of the size a mean-squared loss would send
        inp["dy"] = normal(so, 2.0 / _count(so))
    if c["kind"] == "text_stem":
        B, N, V = c["batch"], c["seq"], c["vocab"]
        # token ids of running text: frequency falls with rank (log-uniform ranks)
        u = torch.rand((B, N if c["counts"] else N - c["n_img"]), generator=g, device="cuda", dtype=torch.float64)
        inp["ids"] = (torch.exp(u * math.log(V + 1.0)) - 1.0).floor().clamp_(0, V - 1).to(torch.int32)
        if c["counts"]:
            inp["counts"] = torch.randint(0, c["n_img"] + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    return inp


# --------------------------------------------------------------------- prepare, run
_plan = None          # the CU shares whose streams the process holds


def _streams(vit_cus):
    """A program reserves the streams of its plan once, before training."""
    global _plan
    if _plan != vit_cus:
        mb.pool_clear()
        mb.pool_reserve(CUS - vit_cus, 0)
        mb.pool_reserve(vit_cus, CUS - vit_cus)
        _plan = vit_cus


class _Ready:
    """A module with its parameters loaded and its buffers in place."""

    def __init__(self, c, seed):
        inp = _inputs(c, seed)
        self.c = c
        self.module = mb.Module(_desc(c), c["dtype"])
        for n, t in inp["P"].items():
            off, rows, cols = self.module.tensors[n]
            assert rows * cols == t.numel(), n
            self.module.params[off:off + rows * cols].copy_(t.reshape(-1))
        if c["kind"] == "optimizer":
            n = self.module.param_elems
            assert inp["grad"].numel() == n
            self.module.grads[:n].copy_(inp["grad"])
            self.module.init_optimizer(c["master"])
            self.module.opt_state[:n].copy_(inp["m"])
            self.module.opt_state[n:2 * n].copy_(inp["v"])
            return
        self.x, self.dy, self.target = inp["x"], inp.get("dy"), inp.get("target")
        so = _in_out(c)[1]
        self.y = torch.empty(so, dtype=_dtype(c), device="cuda")
        # stems that read raw data have no input gradient to send on
        self.dx = None if c["kind"] in ("patch_stem", "conv_stem") else torch.empty_like(self.x)
        self.loss = torch.zeros(1, device="cuda") if self.target is not None else None
        if c["kind"] == "text_stem":
            self.module.bind_ids(inp["ids"])
            if c["counts"]:
                self.module.bind_image_counts(inp["counts"])

    def __del__(self):
        self.module.destroy()

    def outputs(self, whole=False):
        m = self.module
        out = {"y": self.y}
        if self.dx is not None and self.dx.numel():
            out["dx"] = self.dx
        if self.loss is not None:
            out["loss"] = self.loss
        if whole:
            out["grads"] = m.grads[:m.param_elems]
        else:
            out["grads"] = {n: m.grads[off:off + rows * cols] for n, (off, rows, cols) in m.tensors.items()}
        return out


def prepare(case, seed):
    if case["kind"] == "stage":
        parts = [_Ready(c, seed * 4 + i) for i, (_, c, _t) in enumerate(_stage_modules(case))]
        _streams(case["vit_cus"])
        return dict(case=case, parts=parts)
    return dict(case=case, part=_Ready(case, seed))


def run(state):
    c = state["case"]
    if c["kind"] == "stage":
        parts, v = state["parts"], c["vit_cus"]
        mb.stage_run([p.module for p in parts], [p.x for p in parts], [p.y for p in parts], [v, v, CUS - v], [CUS - v, CUS - v, 0],
                     mb.STRIPED, mb.COLOCATED, dy=[p.dy for p in parts], target=[p.target for p in parts],
                     dx=[p.dx for p in parts], loss=[p.loss for p in parts])
        return {n: p.outputs(whole=True) for p, (n, _, _t) in zip(parts, _stage_modules(c))}
    p = state["part"]
    if c["kind"] == "optimizer":
        p.module.adamw_step(CUS, None, step=10, lr=1e-4, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.1)
        n = p.module.param_elems
        out = {"params": p.module.params[:n], "m": p.module.opt_state[:n], "v": p.module.opt_state[n:2 * n]}
        if c["master"]:
            out["master"] = p.module.opt_state[2 * n:3 * n]
        return out
    p.module.step(CUS, None, p.x, p.y, dy=p.dy, target=p.target, dx=p.dx, loss=p.loss)
    return p.outputs()


# -------------------------------------------------------------------------- work, tolerance
def _flops(c):
    """Model flops of one pass (backward = 2x forward where there is an input gradient)."""
    k = c["kind"]
    if k == "stage":
        return sum(_flops(m) for _, m, _t in _stage_modules(c))
    if k in ("encoder", "decoder"):
        T, N, B, h, f, H = c["batch"] * c["seq"], c["seq"], c["batch"], c["hidden"], c["mlp"], c["heads"]
        kv = c.get("kv_heads") or H
        qw = (H + 2 * kv) * (h // H)
        mats = 2.0 * T * h * (qw + h) + (6.0 if k == "decoder" else 4.0) * T * h * f
        return 3.0 * c["layers"] * (mats + 4.0 * B * N * N * h * (0.5 if k == "decoder" else 1.0))
    if k == "projector":
        return 6.0 * c["batch"] * c["seq"] * (c["in_dim"] + c["out_dim"]) * c["out_dim"]
    if k == "patch_stem":                   # forward and weight gradient
        return 4.0 * c["batch"] * c["grid"] ** 2 * 3 * c["patch"] ** 2 * c["hidden"]
    if k == "conv_stem":                    # first convolution without its input gradient
        T, h = c["batch"] * c["seq"], c["hidden"]
        return 4.0 * 2 * T * 3 * c["in_dim"] * h + 6.0 * T * 3 * h * h
    if k == "optimizer":
        return 12.0 * sum(_count(s) for s in _shapes(c).values())
    return 0.0


def _bytes(c):
    if c["kind"] == "stage":
        return sum(_bytes(m) for _, m, _t in _stage_modules(c))
    n = sum(_count(s) for s in _shapes(c).values())
    e = 2 if c["dtype"] == "bf16" else 4
    if c["kind"] == "optimizer":            # gradient read; parameters, moments and master read and written
        return n * (e + 2 * e + 16 + (8 - e if c["master"] else 0))
    si, so = _in_out(c)
    x, y = _count(si), _count(so)
    dx = 0 if c["kind"] in ("patch_stem", "conv_stem") else x
    if c["kind"] == "text_stem":            # of the table only the rows that occur are read: at most one per position
        return e * (x + y + y + dx + n) + min(n, y) * e
    return e * (x + n + y + y + dx + n)     # input, parameters, output, its gradient or target, input gradient, gradients


def work(case):
    return {"bytes": float(_bytes(case)), "flops": float(_flops(case))}


def tolerance(case):
    """fp32: sums of a few hundred to a few thousand terms in another order.  bf16: products of
    bf16 values with fp32 sums; the tensors between kernels are rounded to bf16, and a gradient at the end of a
    layer has passed a dozen such roundings (measured against 64 bits: 0.2 to 0.8 % of the norm)."""
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 1e-4}
    if case["kind"] == "optimizer":         # fp32 state; only the stored parameters are rounded to bf16
        return {"rel": 2e-3, "max": 2e-2}
    if case["kind"] == "text_stem":         # copies, and sums rounded once
        return {"rel": 4e-3, "max": 2e-2}
    return {"rel": 2e-2, "max": 0.4}


# -------------------------------------------------------------------- the same in 64 bits
def _attention64(qkv, c):
    """Softmax attention, one sample at a time (the score matrices are formed again in backward)."""
    from torch.utils.checkpoint import checkpoint
    B, N, H, h = c["batch"], c["seq"], c["heads"], c["hidden"]
    kv, d, causal = c.get("kv_heads") or H, h // H, c["kind"] == "decoder"
    if c.get("rope"):
        ang = (torch.arange(N, device="cuda", dtype=torch.float64)[:, None]
               * c["rope"] ** (-2.0 * torch.arange(d // 2, device="cuda", dtype=torch.float64) / d)[None, :])
        cos, sin = ang.cos()[:, None, :], ang.sin()[:, None, :]
    mask = torch.ones((N, N), dtype=torch.bool, device="cuda").triu(1) if causal else None

    def one(rows):
        q, k, v = rows.split([H * d, kv * d, kv * d], dim=1)
        q, k, v = q.reshape(N, H, d), k.reshape(N, kv, d), v.reshape(N, kv, d)
        if c.get("rope"):
            def turn(t):
                a, b = t[..., 0::2], t[..., 1::2]
                return torch.stack([a * cos - b * sin, a * sin + b * cos], dim=-1).reshape(t.shape)
            q, k = turn(q), turn(k)
        k, v = k.repeat_interleave(H // kv, dim=1), v.repeat_interleave(H // kv, dim=1)
        q, kt, v = q.transpose(0, 1).contiguous(), k.permute(1, 2, 0).contiguous(), v.transpose(0, 1).contiguous()
        s = torch.matmul(q, kt) / math.sqrt(d)
        if causal:
            s = s.masked_fill(mask, -math.inf)
        return torch.matmul(torch.softmax(s, dim=-1), v).transpose(0, 1).reshape(N, H * d)

    rows = qkv.reshape(B, N, -1)
    return torch.cat([checkpoint(one, rows[b], use_reentrant=False) for b in range(B)])


def _forward64(c, P, x, inp):
    F = torch.nn.functional
    k = c["kind"]
    if k in ("encoder", "decoder"):
        def norm(t, p, w):
            if k == "encoder":
                return F.layer_norm(t, (t.shape[1],), P[p + "ln%d_g" % w], P[p + "ln%d_b" % w], 1e-5)
            return t * torch.rsqrt(t.square().mean(1, keepdim=True) + 1e-5) * P[p + "rms%d_g" % w]
        for l in range(c["layers"]):
            p = "L%d." % l
            qkv = norm(x, p, 1) @ P[p + "w_qkv"]
            o = _attention64(qkv + P[p + "b_qkv"] if k == "encoder" else qkv, c) @ P[p + "w_o"]
            x = x + (o + P[p + "b_o"] if k == "encoder" else o)
            u = norm(x, p, 2)
            if k == "encoder":
                x = x + F.gelu(u @ P[p + "w_1"] + P[p + "b_1"]) @ P[p + "w_2"] + P[p + "b_2"]
            else:
                gate, up = (u @ P[p + "w_gu"]).chunk(2, dim=1)
                x = x + (F.silu(gate) * up) @ P[p + "w_down"]
        return x
    if k == "projector":
        return F.gelu(x @ P["w_1"] + P["b_1"]) @ P["w_2"] + P["b_2"]
    if k == "patch_stem":
        B, g, p = c["batch"], c["grid"], c["patch"]
        tok = x.reshape(B, 3, g, p, g, p).permute(0, 2, 4, 1, 3, 5).reshape(B, g * g, 3 * p * p)
        return (tok @ P["w_stem"] + P["b_stem"] + P["pos"]).reshape(B * g * g, -1)
    if k == "text_stem":
        B, N, h, ni = c["batch"], c["seq"], c["hidden"], c["n_img"]
        ids, img, rows = inp["ids"].long(), x.reshape(B, ni, h), []
        for b in range(B):
            cnt = int(inp["counts"][b]) if c["counts"] else ni
            rows += [img[b, :cnt], P["table"][ids[b, cnt:] if c["counts"] else ids[b]]]
        return torch.cat(rows)
    B, n = c["batch"], c["seq"]             # conv_stem: taps gathered, then a matrix product
    def taps(t, stride):
        t = F.pad(t, (0, 0, 1, 1))
        m = (t.shape[1] - 3) // stride + 1
        return torch.cat([t[:, i:i + stride * (m - 1) + 1:stride] for i in range(3)], dim=2)
    a = F.gelu(taps(x, 1) @ P["w_c1"] + P["b_c1"])
    return (F.gelu(taps(a, 2) @ P["w_c2"] + P["b_c2"]) + P["pos"]).reshape(B * n, -1)


def _exact_module(c, seed, whole=False):
    inp = _inputs(c, seed)
    P = {n: t.double().requires_grad_() for n, t in inp["P"].items()}
    x = inp["x"].double()
    wants_dx = c["kind"] not in ("patch_stem", "conv_stem") and x.numel() > 0
    x.requires_grad_(wants_dx)
    y = _forward64(c, P, x, inp)
    out = {"y": y.detach()}
    if c["kind"] == "decoder":
        loss = (y - inp["target"].double()).square().mean()
        loss.backward()
        out["loss"] = loss.detach().reshape(1)
    else:
        y.backward(inp["dy"].double())
    if wants_dx:
        out["dx"] = x.grad
    grads = {n: (P[n].grad if P[n].grad is not None else torch.zeros_like(P[n])).reshape(-1) for n in P}
    out["grads"] = torch.cat(list(grads.values())) if whole else grads
    return out


def exact(case, seed):
    if case["kind"] == "stage":
        return {n: _exact_module(c, seed * 4 + i, whole=True) for i, (n, c, _t) in enumerate(_stage_modules(case))}
    if case["kind"] != "optimizer":
        return _exact_module(case, seed)
    inp = _inputs(case, seed)
    f = lambda v: torch.tensor(v, dtype=torch.float32).double().item()          # the settings reach the update as fp32
    lr, b1, b2, eps, wd, step = f(1e-4), f(0.9), f(0.95), f(1e-8), f(0.1), 10
    p, g = torch.cat([t.reshape(-1) for t in inp["P"].values()]).double(), inp["grad"].double()
    m = b1 * inp["m"].double() + (1 - b1) * g
    v = b2 * inp["v"].double() + (1 - b2) * g * g
    p = p - lr * ((m / (1 - b1 ** step)) / ((v / (1 - b2 ** step)).sqrt() + eps) + wd * p)
    out = {"params": p, "m": m, "v": v}
    if case["master"]:
        out["master"] = p
    return out
