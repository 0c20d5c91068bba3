"""Performance cases of the checkpointed LoRA step: what a fine-tuning program calls, at the
shapes this repository is configured for (`mebp_inputs.CONFIGS`).

A case is one call of the C ABI on resident device data: a layer's forward or its recompute
and backward, the final block (LM head, cross-entropy and its gradient), or a whole training
step. The optimizer's update is left out: it changes its own inputs, so that a repeated pass
is another computation; it is a stream over the adapters.
"""
import math

import torch

from mebp_inputs import ALL7, CONFIGS, PROJ, QKVO
from paper_2510_03425_amd import _lib as L
from paper_2510_03425_amd.device import make_config, ptr, stream_handle

DEV = "cuda"
F64 = torch.float64

# The options beyond the plain block that the named families have.
ARCH = {
    "qwen2.5-0.5b": dict(qkv_bias=True),
    "qwen2.5-1.5b": dict(qkv_bias=True),
    "gemma3-1b": dict(qk_norm=True, sandwich_norm=True, embed_scale=True),
    "gemma3-4b": dict(qk_norm=True, sandwich_norm=True, embed_scale=True),
}


def _case(kind, model, batch, seq, arch=False, layer=0, rank=None, modules=None):
    c = CONFIGS[model]
    return {"kind": kind, "model": model, "batch": batch, "seq": seq, "arch": arch, "layer": layer,
            "rank": rank or c.lora_rank, "modules": modules or ("all" if c.lora_modules == ALL7 else "qkvo")}


def listed():
    cases = {
        # one short prompt: the smallest layer call, bound by launches and latency
        "forward-0.5b-b1-t128": _case("forward", "qwen2.5-0.5b", 1, 128),
        # the phone-sized fine-tuning step's layer (256 tokens), with the family's q/k/v biases
        "backward-0.5b-bias-b1-t256": _case("backward", "qwen2.5-0.5b", 1, 256, arch=True),
        # a ragged micro-batch: no size is a multiple of a tile
        "backward-0.5b-b3-t333": _case("backward", "qwen2.5-0.5b", 3, 333, rank=16, modules="all"),
        # head norms and sandwich norms, one key/value head of 256, a sliding-window layer
        "forward-1b-norms-b1-t512": _case("forward", "gemma3-1b", 1, 512, arch=True),
        # the same family's shape without the options, one sequence
        "backward-1b-b1-t512": _case("backward", "gemma3-1b", 1, 512),
        # an ordinary batch: 4096 tokens, both directions of the checkpointed loop
        "forward-1.5b-b4-t1024": _case("forward", "qwen2.5-1.5b", 4, 1024),
        "backward-1.5b-b4-t1024": _case("backward", "qwen2.5-1.5b", 4, 1024),
        # the benchmark's workload: 16384 tokens; a sliding-window and a global layer
        "forward-4b-b8-t2048": _case("forward", "gemma3-4b", 8, 2048),
        "backward-4b-b8-t2048": _case("backward", "gemma3-4b", 8, 2048, layer=5),
        # the final block, at the phone-sized step and at the benchmark's workload
        "lm-head-0.5b-b1-t256": _case("lm_head", "qwen2.5-0.5b", 1, 256),
        "lm-head-4b-b8-t2048": _case("lm_head", "gemma3-4b", 8, 2048),
        # a whole phone-sized step: embedding, 24 layers forward, final block, 24 backward
        "step-0.5b-b1-t256": _case("step", "qwen2.5-0.5b", 1, 256),
    }
    return [dict(c, name=n) for n, c in cases.items()]


def draw(rng):
    kind = rng.choice(["forward", "backward", "forward", "backward", "lm_head", "step"])
    model = rng.choice(["qwen2.5-0.5b"] if kind == "step" else ["qwen2.5-0.5b", "gemma3-1b", "qwen2.5-1.5b", "gemma3-4b"])
    tokens = math.exp(rng.uniform(math.log(96), math.log(1024 if kind == "step" else 16384)))
    batch = rng.choice([1, 1, 2, 3, 4, 8])
    seq = min(2048, max(32, int(tokens / batch)))
    layer = rng.choice([0, 5]) if CONFIGS[model].global_every and kind != "step" else 0
    return _case(kind, model, batch, seq, arch=rng.random() < 0.3, layer=layer, rank=rng.choice([8, 16]),
                 modules=rng.choice(["qkvo", "all"]))


# ------------------------------------------------------------------------------- inputs
def _config(case):
    c = CONFIGS[case["model"]].with_(batch=case["batch"], seq=case["seq"], lora_rank=case["rank"],
                                     lora_alpha=2.0 * case["rank"], lora_modules=ALL7 if case["modules"] == "all" else QKVO)
    return c.with_(**ARCH[case["model"]]) if case["arch"] else c


def _compress(gen, rows, cols, group=32):
    """A random weight matrix, compressed offline: codes [rows][cols/2], fp16 scales."""
    ng = -(-cols // group)
    q4 = torch.empty((rows, cols // 2), dtype=torch.uint8, device=DEV)
    sc = torch.empty((rows, ng), dtype=torch.float16, device=DEV)
    step = max(1, (1 << 26) // cols)
    for r in range(0, rows, step):
        n = min(step, rows - r)
        w = torch.zeros((n, ng * group), device=DEV)
        w[:, :cols] = torch.randn((n, cols), generator=gen, device=DEV) * 0.02
        w = w.view(n, ng, group)
        s = (w.abs().amax(-1) / 7).half()
        q = (w / s.float().unsqueeze(-1)).round_().nan_to_num_(0.0).clamp_(-7, 7).to(torch.int16).view(n, -1)[:, :cols] & 15
        q4[r:r + n] = (q[:, 0::2] | (q[:, 1::2] << 4)).to(torch.uint8)
        sc[r:r + n] = s
    return q4, sc


def _inputs(case, seed):
    """Every input of the case's call, on the device, from the seed alone."""
    cfg = _config(case)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)

    def normal(*shape, std=1.0, mean=0.0):
        return torch.randn(shape, generator=gen, device=DEV) * std + mean

    def norm_w(n):
        return normal(n, std=0.1, mean=1.0)

    d, dh, r, N = cfg.hidden, cfg.head_dim, cfg.lora_rank, cfg.n_tokens
    inp = {"cfg": cfg, "layers": []}
    for _ in range({"lm_head": 0, "step": cfg.n_layers}.get(case["kind"], 1)):
        y = {"w": {p: _compress(gen, *cfg.proj_shape(p)) for p in PROJ}, "norm_attn": norm_w(d), "norm_mlp": norm_w(d)}
        if cfg.qkv_bias:
            y["bias"] = {p: normal(cfg.proj_shape(p)[0], std=0.1) for p in "qkv"}
        if cfg.qk_norm:
            y["qk_norm"] = (norm_w(dh), norm_w(dh))
        if cfg.sandwich_norm:
            y["post_norm"] = (norm_w(d), norm_w(d))
        y["A"] = {p: normal(r, cfg.proj_shape(p)[1], std=1.0 / r) for p in cfg.lora_modules}
        y["B"] = {p: normal(cfg.proj_shape(p)[0], r, std=0.02) for p in cfg.lora_modules}
        inp["layers"].append(y)
    if case["kind"] in ("lm_head", "step"):
        inp["emb"] = _compress(gen, cfg.vocab, d)
        # final-norm weights for logits with a standard deviation of about 4 (confident rows
        # beside flat ones, as a trained model has them)
        inp["norm_final"] = norm_w(d) * (4 / (0.02 * math.sqrt(d)))
        inp["ids"] = torch.randint(0, cfg.vocab, (cfg.batch, cfg.seq), generator=gen, device=DEV, dtype=torch.int32)
    if case["kind"] != "step":
        inp["x"] = normal(N, d)
    if case["kind"] == "backward":
        inp["dy"] = normal(N, d, std=1.0 / N)  # a mean loss over the tokens
    return inp


def prepare(case, seed):
    inp = _inputs(case, seed)
    cfg = inp["cfg"]
    ccfg = make_config(cfg)
    n = len(inp["layers"])
    st = {"kind": case["kind"], "layer": case["layer"], "inp": inp, "ccfg": ccfg, "B": cfg.batch, "T": cfg.seq}
    base, lora, grads = (L.MebpLayerBase * n)(), (L.MebpLayerLora * n)(), (L.MebpLayerLoraGrad * n)()
    # the gradients of one projection over all layers are one tensor
    gr = {}
    if case["kind"] in ("backward", "step"):
        for p in cfg.lora_modules:
            o, i = cfg.proj_shape(p)
            gr["dA." + p] = torch.zeros((n, cfg.lora_rank, i), device=DEV)
            gr["dB." + p] = torch.zeros((n, o, cfg.lora_rank), device=DEV)
    for l, y in enumerate(inp["layers"]):
        for i, p in enumerate(PROJ):
            q4, sc = y["w"][p]
            base[l].w[i].q4, base[l].w[i].scale = ptr(q4), ptr(sc)
            if p in y["A"]:
                lora[l].A[i], lora[l].B[i] = ptr(y["A"][p]), ptr(y["B"][p])
            if "dA." + p in gr:
                grads[l].dA[i], grads[l].dB[i] = ptr(gr["dA." + p][l]), ptr(gr["dB." + p][l])
        base[l].norm_attn, base[l].norm_mlp = ptr(y["norm_attn"]), ptr(y["norm_mlp"])
        for i, p in enumerate("qkv"):
            if "bias" in y:
                base[l].bias[i] = ptr(y["bias"][p])
        if "qk_norm" in y:
            base[l].q_norm, base[l].k_norm = (ptr(t) for t in y["qk_norm"])
        if "post_norm" in y:
            base[l].post_attn_norm, base[l].post_mlp_norm = (ptr(t) for t in y["post_norm"])
    st.update(base=base, lora=lora, grads=grads, gr=gr)
    if "emb" in inp:
        st["emb"] = L.MebpQ4(q4=ptr(inp["emb"][0]), scale=ptr(inp["emb"][1]))
        st["loss"] = torch.zeros(1, device=DEV)
    st["out"] = torch.zeros((cfg.n_tokens, cfg.hidden), device=DEV)  # x_out, or the input's gradient
    if case["kind"] == "step":
        st["ckpt"] = torch.empty((n + 1, cfg.n_tokens, cfg.hidden), device=DEV)
    st["ws_bytes"] = L.mebp_workspace_bytes(ccfg, cfg.batch, cfg.seq)
    st["ws"] = torch.empty(st["ws_bytes"], dtype=torch.uint8, device=DEV)
    return st


def run(st):
    inp, kind, out = st["inp"], st["kind"], st["out"]
    tail = (st["B"], st["T"])
    ws = (ptr(st["ws"]), st["ws_bytes"], stream_handle())
    if kind == "forward":
        L.mebp_layer_forward_ckpt(st["ccfg"], st["layer"], st["base"][0], st["lora"][0], ptr(inp["x"]), ptr(out), *tail, *ws)
        return out
    if kind == "backward":
        L.mebp_layer_recompute_backward(st["ccfg"], st["layer"], st["base"][0], st["lora"][0], ptr(inp["x"]), ptr(inp["dy"]),
                                        ptr(out), st["grads"][0], *tail, *ws)
        return dict(st["gr"], dx=out)
    if kind == "lm_head":
        L.mebp_lm_head_ce_backward(st["ccfg"], st["emb"], ptr(inp["norm_final"]), ptr(inp["x"]), ptr(inp["ids"]), *tail,
                                   ptr(st["loss"]), ptr(out), *ws)
        return {"loss": st["loss"], "dx": out}
    L.mebp_train_step(st["ccfg"], st["emb"], st["base"], ptr(inp["norm_final"]), st["lora"], ptr(inp["ids"]), *tail,
                      ptr(st["ckpt"]), ptr(st["loss"]), st["grads"], ptr(out), *ws)
    return dict(st["gr"], loss=st["loss"], dx=out)


# ------------------------------------------------------------------------------- work
def work(case):
    """Matrix products and attention of the method (the backward recomputes its forward from
    the checkpoint, except the down projection, whose output it does not need); compressed
    weights, inputs and outputs once."""
    cfg = _config(case)
    N, d, V, r = cfg.n_tokens, cfg.hidden, cfg.vocab, cfg.lora_rank
    shapes = {p: cfg.proj_shape(p) for p in PROJ}
    P = sum(o * i for o, i in shapes.values())
    P_fwd = P - shapes["down"][0] * shapes["down"][1]
    ab = sum(sum(shapes[p]) for p in cfg.lora_modules)
    wbytes = sum(o * (i / 2 + 2 * -(-i // 32)) for o, i in shapes.values()) + 4.0 * r * ab
    emb_bytes = V * (d / 2 + 2 * -(-d // 32))

    def pairs(layer):
        W = cfg.layer_window(layer)
        return cfg.batch * sum(min(t + 1, W) if W else t + 1 for t in range(cfg.seq))

    def fwd(layer):
        return 2.0 * N * P + 4.0 * cfg.head_dim * cfg.n_heads * pairs(layer) + 2.0 * N * r * ab

    def bwd(layer):
        return 2.0 * N * (P_fwd + P) + 12.0 * cfg.head_dim * cfg.n_heads * pairs(layer) + 8.0 * N * r * ab

    if case["kind"] == "forward":
        return {"bytes": wbytes + 8.0 * N * d, "flops": fwd(case["layer"])}
    if case["kind"] == "backward":
        return {"bytes": wbytes + 12.0 * N * d + 4.0 * r * ab, "flops": bwd(case["layer"])}
    if case["kind"] == "lm_head":
        return {"bytes": emb_bytes + 8.0 * N * d, "flops": 4.0 * N * d * V}
    n = cfg.n_layers
    return {"bytes": n * (wbytes + 4.0 * r * ab + 4.0 * N * d) + emb_bytes,
            "flops": sum(fwd(l) + bwd(l) for l in range(n)) + 4.0 * N * d * V}


def tolerance(case):
    """About four times the distance from the 64-bit result: fp16 operands and activations in
    the forward products, bf16 operands and gradients in the backward ones, 32-bit sums."""
    return {"rel": {"forward": 2.5e-3, "backward": 2.4e-2, "lm_head": 2.2e-3, "step": 4e-2}[case["kind"]]}


# ------------------------------------------------------------------------------- 64 bits
def _dense(q4, sc, group=32):
    rows, half = q4.shape
    q = torch.stack([q4 & 15, q4 >> 4], dim=-1).view(rows, 2 * half).to(torch.int8)
    q = torch.where(q > 7, q - 16, q).to(F64)
    return q * sc.to(F64).repeat_interleave(group, dim=1)[:, :2 * half]


def _rms(x, w, eps):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * w.to(F64)


def _layer64(cfg, layer, y, A, B, x):
    N, T, dh, H, KV = cfg.n_tokens, cfg.seq, cfg.head_dim, cfg.n_heads, cfg.n_kv_heads

    def proj(p, v):
        o = v @ _dense(*y["w"][p]).t()
        if p in A:
            o = o + cfg.lora_scale * (v @ A[p].t()) @ B[p].t()
        return o

    a = _rms(x, y["norm_attn"], cfg.rms_eps)
    q, k, v = (proj(p, a) for p in "qkv")
    if "bias" in y:
        q, k, v = (t + y["bias"][p].to(F64) for t, p in zip((q, k, v), "qkv"))
    q, k, v = q.view(N, H, dh), k.view(N, KV, dh), v.view(N, KV, dh)
    if "qk_norm" in y:
        q, k = _rms(q, y["qk_norm"][0], cfg.rms_eps), _rms(k, y["qk_norm"][1], cfg.rms_eps)
    t = torch.arange(T, device=DEV, dtype=F64)
    ang = t[:, None] * cfg.layer_theta(layer) ** (-torch.arange(0, dh, 2, device=DEV, dtype=F64) / dh)
    cos, sin = (f(ang).repeat(cfg.batch, 1)[:, None] for f in (torch.cos, torch.sin))

    def rope(z):
        z1, z2 = z[..., :dh // 2], z[..., dh // 2:]
        return torch.cat([z1 * cos - z2 * sin, z2 * cos + z1 * sin], -1)

    q, k = rope(q), rope(k)
    gap = torch.arange(T, device=DEV)[:, None] - torch.arange(T, device=DEV)
    hidden = gap < 0
    if cfg.layer_window(layer):
        hidden = hidden | (gap >= cfg.layer_window(layer))
    outs = []
    for b in range(cfg.batch):
        rows = slice(b * T, (b + 1) * T)
        qb = q[rows].transpose(0, 1).contiguous()
        kb, vb = (z[rows].repeat_interleave(H // KV, dim=1).transpose(0, 1).contiguous() for z in (k, v))
        s = (torch.matmul(qb, kb.transpose(1, 2).contiguous()) / math.sqrt(dh)).masked_fill(hidden, -math.inf)
        outs.append(torch.matmul(s.softmax(-1), vb).transpose(0, 1).reshape(T, H * dh))
    t_o = proj("o", torch.cat(outs))
    h = x + (_rms(t_o, y["post_norm"][0], cfg.rms_eps) if "post_norm" in y else t_o)
    c = _rms(h, y["norm_mlp"], cfg.rms_eps)
    g = proj("gate", c)
    act = torch.nn.functional.silu(g) if cfg.act == "silu" else torch.nn.functional.gelu(g, approximate="tanh")
    t_d = proj("down", act * proj("up", c))
    return h + (_rms(t_d, y["post_norm"][1], cfg.rms_eps) if "post_norm" in y else t_d)


def _layer_grads64(cfg, layer, y, x, dy):
    x = x.to(F64).requires_grad_()
    A, B = ({p: t.to(F64).requires_grad_() for p, t in y[k].items()} for k in "AB")
    mods = list(A)
    out = _layer64(cfg, layer, y, A, B, x)
    g = torch.autograd.grad(out, [x] + [A[p] for p in mods] + [B[p] for p in mods], dy.to(F64))
    n = len(mods)
    return g[0], dict(zip(mods, g[1:1 + n])), dict(zip(mods, g[1 + n:]))


def _head64(inp, x):
    cfg = inp["cfg"]
    E = _dense(*inp["emb"])
    ids = inp["ids"].long()
    n = cfg.batch * (cfg.seq - 1)
    loss = torch.zeros((), dtype=F64, device=DEV)
    dx = torch.zeros(x.shape, dtype=F64, device=DEV)
    for b in range(cfg.batch):
        rows = slice(b * cfg.seq, (b + 1) * cfg.seq)
        xb = x[rows].to(F64).requires_grad_()
        hf = _rms(xb, inp["norm_final"], cfg.rms_eps)
        lg = hf.detach()[:-1] @ E.t()
        tgt = ids[b, 1:, None]
        lse = lg.logsumexp(-1, keepdim=True)
        loss += (lse - lg.gather(1, tgt)).sum() / n
        lg = lg.sub_(lse).exp_()
        lg.scatter_add_(1, tgt, torch.full_like(tgt, -1, dtype=F64))
        dhf = torch.zeros_like(hf)
        dhf[:-1] = (lg @ E) / n
        del lg
        dx[rows] = torch.autograd.grad(hf, xb, dhf)[0]
    return loss.view(1), dx


def exact(case, seed):
    inp = _inputs(case, seed)
    cfg, kind, layers = inp["cfg"], case["kind"], inp["layers"]

    def forward(layer, y, x):
        A, B = ({p: t.to(F64) for p, t in y[k].items()} for k in "AB")
        with torch.no_grad():
            return _layer64(cfg, layer, y, A, B, x.to(F64))

    def stacked(parts):
        return {"%s.%s" % (n, p): torch.stack([g[i][p] for g in parts]) for i, n in ((1, "dA"), (2, "dB")) for p in cfg.lora_modules}

    if kind == "forward":
        return forward(case["layer"], layers[0], inp["x"])
    if kind == "backward":
        got = _layer_grads64(cfg, case["layer"], layers[0], inp["x"], inp["dy"])
        return dict(stacked([got]), dx=got[0])
    if kind == "lm_head":
        loss, dx = _head64(inp, inp["x"])
        return {"loss": loss, "dx": dx}
    xs = [_dense(*(t[inp["ids"].long().view(-1)] for t in inp["emb"]))]
    if cfg.embed_scale:
        xs[0] = xs[0] * math.sqrt(cfg.hidden)
    for l, y in enumerate(layers):
        xs.append(forward(l, y, xs[l]))
    loss, g = _head64(inp, xs[-1])
    parts = [None] * len(layers)
    for l in reversed(range(len(layers))):
        parts[l] = _layer_grads64(cfg, l, layers[l], xs[l], g)
        g = parts[l][0]
    return dict(stacked(parts), loss=loss, dx=g)
