"""The work that users of this library have it do, as cases to measure.

A case is a dict of plain values.  `entry` names the call it makes: "meta_grad" (dV/deta and V
through T inner steps), "inner_step" (one training update) or "hvp" (gradient, H v and, for a
decoder, the mixed product).  `widths`, `rows`, ... describe the problem as include/mfmg.h
does.  Inputs are drawn on the GPU from a seed; `exact` repeats a case with torch autograd in
float64.
"""
import math

import torch

from paper_2505_00793_amd import _lib as M

TANH, GELU, RELU, NONE = 0, 1, 2, 3
MSE, CE, MAPMSE = 0, 1, 2
SGD, ADAM = 0, 1
LOGLR, LAYERLR, LOSSW, TOKENS, MAML = 0, 1, 2, 3, 4
FP32, BF16 = 0, 1


def _mlp(family, widths, rows, val_rows, T, entry="meta_grad", **kw):
    return {"family": family, "kind": 0, "entry": entry, "widths": ",".join(map(str, widths)),
            "rows": rows, "val_rows": val_rows, "T": T, **FAMILIES[family], **kw}


def _decoder(family, d, heads, ff, vocab, seq, blocks, hidden, rows, val_rows, T,
             entry="meta_grad", **kw):
    return {"family": family, "kind": 1, "entry": entry, "d": d, "heads": heads, "ff": ff,
            "vocab": vocab, "seq": seq, "blocks": blocks, "hidden": hidden, "rows": rows,
            "val_rows": val_rows, "T": T, **FAMILIES[family], **kw}


# What the members of a family share.
FAMILIES = {
    # learned per-parameter learning rates of a linear model
    "linreg": dict(act=NONE, loss=MSE, opt=SGD, meta=LOGLR, prec=FP32, bias=0, init="small"),
    # per-example loss weights of a small classifier
    "lossweights": dict(act=TANH, loss=CE, opt=SGD, meta=LOSSW, prec=FP32, bias=1, init="xavier"),
    # per-layer learning rates and weight decay of an Adam-trained classifier
    "adam": dict(act=GELU, loss=CE, opt=ADAM, meta=LAYERLR, prec=BF16, bias=1, init="he"),
    # per-parameter learning rates of a ReLU classifier
    "loglr": dict(act=RELU, loss=CE, opt=SGD, meta=LOGLR, prec=BF16, bias=1, init="he"),
    # MAML on the M-step map of the paper's motivating example
    "map": dict(act=NONE, loss=MAPMSE, opt=SGD, meta=MAML, prec=FP32, bias=0, init="map"),
    # token weights of a decoder: fused attention in bf16, or materialised attention
    "decoder": dict(prec=BF16, fused=1, remat=1),
    "decoder_full": dict(prec=BF16, fused=0, remat=0),
}


def listed():
    c = []

    def add(name, case):
        c.append({"name": name, **case})

    # The smallest call: a 64-feature regression, one launch, latency is all there is.
    add("linreg_64", _mlp("linreg", (64, 1), 256, 256, 4))
    # More features and rows than one staged batch holds, neither a power of two.
    add("linreg_130", _mlp("linreg", (130, 1), 1000, 700, 3))
    # Loss weighting of an MNIST-sized classifier: some 140 small float32 launches.
    add("lossweights_784", _mlp("lossweights", (784, 256, 10), 128, 512, 8))
    # Optimiser hyperparameters of a 4-layer Adam-trained MLP over 16 steps.
    add("adam_4x1024", _mlp("adam", (1024, 1024, 1024, 1024, 100), 512, 1024, 16))
    # Widths and rows that no tile divides, odd ones among them.
    add("loglr_ragged", _mlp("loglr", (781, 1000, 515, 37), 250, 130, 4))
    # The flagship: 121 million learned learning rates of an 8-layer 4096-wide network.
    add("loglr_8x4096", _mlp("loglr", (4096,) * 8 + (1000,), 1024, 1024, 8))
    # One Hessian-vector product at the same width, for callers with their own outer loop.
    add("hvp_3x4096", _mlp("loglr", (4096, 4096, 4096, 1000), 1024, 1024, 1, entry="hvp"))
    # One Adam training step with its gradient, in the middle of a run (warm m and v).
    add("adam_step_3x4096", _mlp("adam", (4096, 4096, 4096, 1000), 1024, 1024, 1,
                                 entry="inner_step"))
    # The paper's motivating example: float32 products of 1024 x 4096 x 4096.
    add("map_4096", _mlp("map", (4096, 4096), 1024, 1024, 2, map_steps=2))
    # Per-token loss weights of a small language model, 4096 tokens a step.
    add("decoder_512", _decoder("decoder", 512, 8, 2048, 8192, 256, 4, 128, 16, 16, 8))
    # The same model at a long context.
    add("decoder_512_long", _decoder("decoder", 512, 8, 2048, 8192, 4096, 4, 128, 2, 2, 2))
    # H v of a small decoder with materialised attention and an odd vocabulary.
    add("decoder_128_hvp", _decoder("decoder_full", 128, 4, 256, 301, 160, 2, 32, 8, 4, 1,
                                    entry="hvp"))
    return c


def _between(rng, lo, hi, step=1):
    """A multiple of `step` between lo and hi, spread over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / step)) * step))


def draw(rng):
    b = lambda lo, hi, step=1: _between(rng, lo, hi, step)
    family = rng.choice(["linreg", "lossweights", "lossweights", "adam", "adam", "loglr", "loglr",
                         "map", "decoder", "decoder", "decoder_full"])
    if family == "linreg":
        return _mlp(family, (b(8, 256), 1), b(32, 1024), b(32, 1024), rng.randint(1, 8))
    if family == "lossweights":
        return _mlp(family, (b(64, 1024), b(32, 512), b(4, 64)), b(16, 512), b(32, 512),
                    rng.randint(1, 8))
    if family == "adam":
        depth, entry = rng.randint(1, 3), rng.choice(["meta_grad", "meta_grad", "inner_step"])
        hi, step = (4096, 1) if entry == "inner_step" else (1024, rng.choice([1, 8]))
        return _mlp(family, [b(128, hi, step) for _ in range(depth + 1)] + [b(10, 1000)],
                    b(64, 1024), b(64, 1024), rng.randint(2, 16), entry=entry)
    if family == "loglr":
        depth, entry = rng.randint(1, 2), rng.choice(["meta_grad", "meta_grad", "hvp"])
        step = rng.choice([1, 8, 64])
        return _mlp(family, [b(256, 4096, step) for _ in range(depth + 1)] + [b(10, 1000)],
                    b(64, 1024), b(64, 1024), rng.randint(1, 8), entry=entry)
    if family == "map":
        return _mlp(family, (b(64, 4096), b(64, 4096)), b(64, 1024), b(64, 1024), 2,
                    map_steps=rng.randint(1, 2))
    entry = rng.choice(["meta_grad", "meta_grad", "hvp"])
    seq = b(64, 2048, 64) if family == "decoder" else b(32, 512, 4)
    d = 64 * rng.choice([2, 4, 8])
    heads = d // (64 if family == "decoder" else 32)
    rows = max(1, min(16, b(512, 4096) // seq))
    rows = max(rows, min(16, -(-512 // seq)))
    return _decoder(family, d, heads, d * rng.choice([2, 4]), b(512, 8192), seq, rng.randint(1, 4),
                    8 * rng.randint(2, 16), rows, rows, rng.randint(1, 4), entry=entry)


# --------------------------------------------------------------------------------------
# Parameters and inputs.
# --------------------------------------------------------------------------------------
def _widths(case):
    return [int(w) for w in case["widths"].split(",")]


def _layout(case):
    """(name, shape) of every tensor of the flat theta, in order."""
    if case["kind"] == 0:
        w, out = _widths(case), []
        for l in range(len(w) - 1):
            out.append((f"W{l}", (w[l], w[l + 1])))
            if case["bias"]:
                out.append((f"b{l}", (w[l + 1],)))
        return out
    d, ff, V = case["d"], case["ff"], case["vocab"]
    out = [("emb", (V, d))]
    for b in range(case["blocks"]):
        out += [(f"ln1_g{b}", (d,)), (f"ln1_b{b}", (d,)), (f"wqkv{b}", (d, 3 * d)),
                (f"wo{b}", (d, d)), (f"ln2_g{b}", (d,)), (f"ln2_b{b}", (d,)),
                (f"w1{b}", (d, ff)), (f"w2{b}", (ff, d))]
    return out + [("lnf_g", (d,)), ("lnf_b", (d,)), ("unemb", (d, V))]


def _size(layout):
    return sum(math.prod(s) for _, s in layout)


def _n_eta(case):
    if case["kind"] == 1:
        return (case["d"] + 2) * case["hidden"] + 1
    if case["meta"] == LAYERLR:
        return len(_widths(case))
    if case["meta"] == LOSSW:
        return case["T"] * case["rows"]
    return _size(_layout(case))


def _std(case, shape):
    if case["kind"] == 1:
        return 0.02
    init = case["init"]
    if init == "small":
        return 0.1
    if init == "xavier":
        return math.sqrt(2.0 / (shape[0] + shape[1]))
    return math.sqrt((2.0 if init == "he" else 1.0) / shape[0])


def _sgd_lr(case):
    return 1e-3 if case["kind"] == 0 and case["meta"] == MAML else 0.1


def _inputs(case, seed):
    dev = "cuda"
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    normal = lambda *shape: torch.randn(*shape, generator=g, device=dev)

    parts = []
    for name, shape in _layout(case):
        if len(shape) == 2:
            parts.append((normal(*shape) * _std(case, shape)).reshape(-1))
        else:
            parts.append(torch.full(shape, 1.0 if "_g" in name else 0.0, device=dev))
    s = {"theta": torch.cat(parts)}

    rows, n_in = (case["rows"], case["val_rows"]), 0
    if case["kind"] == 0:
        n_in, n_out = _widths(case)[0], _widths(case)[-1]
        wstar = normal(n_in, 1)
        p = None
    else:
        p = torch.arange(1, case["vocab"] + 1, device=dev, dtype=torch.float32) ** -1.1

    def batch(r):
        if case["kind"] == 1:   # Zipf-distributed tokens
            n = r * (case["seq"] + 1)
            t = torch.multinomial(p, n, replacement=True, generator=g)
            return t.to(torch.int32).reshape(r, -1), None
        x = normal(r, n_in)
        if case["loss"] == CE:
            return x, torch.randint(n_out, (r,), generator=g, device=dev, dtype=torch.int32)
        if case["loss"] == MAPMSE:
            return x, normal(r, n_out)
        return x, x @ wstar + 0.1 * normal(r, 1)

    b = [batch(rows[0]) for _ in range(case["T"])]
    s["xs"], s["ys"] = [x for x, _ in b], [y for _, y in b]
    s["vx"], s["vy"] = batch(rows[1])

    if case["kind"] == 1:   # Xavier-normal token-weight meta-model
        d, h = case["d"], case["hidden"]
        z = torch.zeros
        s["eta"] = torch.cat([normal(d * h) * math.sqrt(2.0 / (d + h)), z(h, device=dev),
                              normal(h) * math.sqrt(2.0 / (h + 1)), z(1, device=dev)])
    elif case["meta"] == LOGLR:
        s["eta"] = torch.full((_n_eta(case),), math.log(0.01), device=dev)
    elif case["meta"] == LAYERLR:
        s["eta"] = torch.full((_n_eta(case),), math.log(1e-3), device=dev)
        s["eta"][-1] = 1e-4
    elif case["meta"] == MAML:
        s["eta"] = s["theta"].clone()
    else:
        s["eta"] = 0.5 * normal(_n_eta(case))
    s["opt"] = None
    if case.get("opt") == ADAM:
        n = s["theta"].numel()
        s["opt"] = torch.zeros(2 * n, device=dev)
        if case["entry"] == "inner_step":   # the middle of a run: m, v of earlier gradients
            s["opt"][:n] = 1e-4 * normal(n)
            s["opt"][n:] = (1e-3 * normal(n)) ** 2 + 1e-8
    if case["entry"] == "hvp":
        s["v"] = normal(s["theta"].numel())
    return s


STEP = 7   # the update count of an inner_step call


def _problem(case):
    common = dict(rows=case["rows"], val_rows=case["val_rows"], sgd_lr=_sgd_lr(case),
                  precision=case["prec"])
    if case["kind"] == 1:
        return M.Problem(M.make_desc(
            kind=1, widths=(1, 1), loss=CE, optimizer=SGD, meta=TOKENS, has_bias=False,
            d_model=case["d"], n_heads=case["heads"], d_ff=case["ff"], vocab=case["vocab"],
            seq=case["seq"], n_blocks=case["blocks"], meta_hidden=case["hidden"], ln_eps=1e-5,
            rope_base=10000.0, fused_attention=case["fused"], block_remat=case["remat"], **common))
    return M.Problem(M.make_desc(widths=_widths(case), act=case["act"], loss=case["loss"],
                                 optimizer=case["opt"], meta=case["meta"],
                                 has_bias=bool(case["bias"]),
                                 map_steps=case.get("map_steps", 0), **common))


def prepare(case, seed):
    s = _inputs(case, seed)
    s["entry"], s["P"] = case["entry"], _problem(case)
    sizes = s["P"].mfmg_query_sizes(case["T"])
    meta = case["entry"] == "meta_grad"
    s["ws"] = s["P"].workspace(sizes.workspace_bytes if meta else sizes.step_workspace_bytes)
    empty = lambda n: torch.empty(n, device="cuda")
    n = s["theta"].numel()
    if meta:
        s["out"] = {"d_eta": empty(_n_eta(case)), "val_loss": empty(1)}
    elif case["entry"] == "hvp":
        s["out"] = {"grad": empty(n), "hvp": empty(n)}
        if case["kind"] == 1:
            s["out"]["mvp"] = empty(case["rows"] * case["seq"])
    else:
        s["out"] = {"theta": empty(n), "opt": empty(2 * n), "grad": empty(n), "loss": empty(1)}
    return s


def run(s):
    P, o = s["P"], s["out"]
    if s["entry"] == "meta_grad":
        P.mfmg_meta_grad(s["theta"], s["opt"], s["eta"], s["xs"], s["ys"], s["vx"], s["vy"],
                         o["d_eta"], o["val_loss"], ws=s["ws"])
    elif s["entry"] == "hvp":
        P.mfmg_hvp_fwd_over_rev(s["theta"], s["eta"], s["xs"][0], s["ys"][0], 0, s["v"],
                                o["grad"], o["hvp"], o.get("mvp"), ws=s["ws"])
    else:
        P.mfmg_inner_step(s["theta"], s["opt"], s["eta"], s["xs"][0], s["ys"][0], STEP,
                          o["theta"], o["opt"], o["grad"], o["loss"], ws=s["ws"])
    return dict(o)


# --------------------------------------------------------------------------------------
# What a pass cannot do without.
# --------------------------------------------------------------------------------------
def work(case):
    T, rows, vr = case["T"], case["rows"], case["val_rows"]
    meta, hvp = case["entry"] == "meta_grad", case["entry"] == "hvp"
    n = _size(_layout(case))
    n_eta = _n_eta(case)
    adam = case.get("opt") == ADAM
    if case["kind"] == 0:
        w = _widths(case)
        unit = [2.0 * a * b for a, b in zip(w, w[1:])]           # flops per row, one product
        first, rest = unit[0], sum(unit[1:])
        step = 2 * first + 3 * rest                               # forward, backward
        # dual products 3 each; the first layer's input has no tangent, and its output
        # gradient needs no product with its weights; Adam has the primal gradient already
        dual = (2 + (1 if adam and meta else 2)) * first + (6 + (2 if adam and meta else 3)) * rest
        x_bytes = 4.0 * (w[0] + (1 if case["loss"] == CE else w[-1]))
    else:
        d, S = case["d"], case["seq"]
        lin = 2.0 * (case["blocks"] * (4 * d * d + 2 * d * case["ff"]) + d * case["vocab"])
        att = 2.0 * case["blocks"] * S * d                        # causal scores and context
        step, dual = S * (3 * lin + 3 * att), S * (9 * lin + 9 * att)
        x_bytes = 4.0 * (S + 1)
    if meta:
        flops = T * rows * (step + dual) + vr * step
        numbers = n + n_eta * 2 + 1
        data = (T * rows + vr) * x_bytes
    elif hvp:
        flops, numbers, data = rows * dual, 4 * n + n_eta, rows * x_bytes
    else:
        flops, numbers, data = rows * step, (7 if adam else 3) * n + n_eta, rows * x_bytes
    return {"bytes": 4.0 * numbers + data, "flops": flops}


def tolerance(case):
    """About four times the distance between the library and `exact`, over some hundred draws:
    float32 sums 1.6e-7 (linear regression), 6e-7 and 2.5e-6 (map); bf16 operands, whose
    rounding the depth and the ReLU kinks amplify, as noted."""
    if case["prec"] == FP32:
        return {"rel": {"linreg": 1e-6, "lossweights": 5e-6, "map": 1e-5}[case["family"]]}
    if case["family"] == "adam":     # 2.2e-2 and 5e-3
        return {"rel": 6e-2 if case["entry"] == "meta_grad" else 2e-2}
    if case["family"] == "loglr":    # 0.15 at eight layers, else 5e-2
        return {"rel": 0.5 if len(_widths(case)) > 5 else 0.15}
    return {"rel": 8e-2 if case["entry"] == "meta_grad" else 2.5e-2}   # 2.5e-2 and 7e-3


# --------------------------------------------------------------------------------------
# The same in float64: truncated backpropagation by torch autograd, one inner step at a time.
# --------------------------------------------------------------------------------------
def _unpack(case, theta):
    out, off = {}, 0
    for name, shape in _layout(case):
        n = math.prod(shape)
        out[name] = theta[off:off + n].view(shape)
        off += n
    return out


def _logits(case, P, tokens):
    B, S = tokens.shape
    d, H = case["d"], case["heads"]
    dh = d // H
    ang = torch.arange(S, dtype=torch.float64, device=tokens.device)[:, None] \
        * 10000.0 ** (-torch.arange(dh // 2, dtype=torch.float64, device=tokens.device) * 2 / dh)
    cos, sin = torch.cos(ang), torch.sin(ang)

    def turn(t):
        a, b = t[..., :dh // 2], t[..., dh // 2:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

    norm = lambda x, g, b: torch.nn.functional.layer_norm(x, (d,), g, b, 1e-5)
    later = torch.ones(S, S, dtype=torch.bool, device=tokens.device).triu(1)
    h = P["emb"][tokens.long()]
    for b in range(case["blocks"]):
        a = norm(h, P[f"ln1_g{b}"], P[f"ln1_b{b}"])
        q, k, v = (a @ P[f"wqkv{b}"]).view(B, S, 3, H, dh).permute(2, 0, 3, 1, 4)
        s = (turn(q) @ turn(k).transpose(-1, -2) / math.sqrt(dh)).masked_fill(later, -math.inf)
        o = (torch.softmax(s, -1) @ v).transpose(1, 2).reshape(B, S, d)
        h = h + o @ P[f"wo{b}"]
        a = norm(h, P[f"ln2_g{b}"], P[f"ln2_b{b}"])
        h = h + torch.nn.functional.gelu(a @ P[f"w1{b}"]) @ P[f"w2{b}"]
    return norm(h, P["lnf_g"], P["lnf_b"]).reshape(B * S, d) @ P["unemb"]


def _row_losses(case, theta, x, y):
    P = _unpack(case, theta)
    if case["kind"] == 1:
        return torch.nn.functional.cross_entropy(_logits(case, P, x[:, :-1]),
                                                 x[:, 1:].reshape(-1).long(), reduction="none")
    act = {TANH: torch.tanh, GELU: torch.nn.functional.gelu, RELU: torch.relu,
           NONE: lambda z: z}[case["act"]]
    a, last = x.double(), len(_widths(case)) - 2
    for l in range(last + 1):
        a = a @ P[f"W{l}"]
        if case["bias"]:
            a = a + P[f"b{l}"]
        if l < last:
            a = act(a)
    if case["loss"] == CE:
        return torch.nn.functional.cross_entropy(a, y.long(), reduction="none")
    if case["loss"] == MSE:
        return ((a - y.double()) ** 2).sum(-1)
    for i in range(1, case["map_steps"] + 1):
        a = i * (2.0 + torch.sin(a)) ** torch.cos(a)
    return ((a - y.double()) ** 2).mean(-1)


def _weights(case, eta, emb0, t, x):
    """Loss weights of inner step t, or 1."""
    if case["kind"] == 1:
        d, h = case["d"], case["hidden"]
        W1, b1, w2, b2 = torch.split(eta, [d * h, h, h, 1])
        u = torch.tanh(emb0[x[:, :-1].reshape(-1).long()] @ W1.view(d, h) + b1) @ w2 + b2
        return torch.sigmoid(u)
    if case["meta"] == LOSSW:
        return torch.sigmoid(eta.view(case["T"], case["rows"])[t])
    return 1.0


def _update(case, g, theta, m, v, eta, count):
    if case["kind"] == 1 or case["meta"] in (LOSSW, MAML):
        return theta - _sgd_lr(case) * g, m, v
    if case["meta"] == LOGLR:
        return theta - torch.exp(eta) * g, m, v
    per_layer = torch.cat([eta[int(name[1:])].exp().expand(math.prod(shape))
                           for name, shape in _layout(case)])
    m = 0.9 * m + (1 - 0.9) * g
    v = 0.999 * v + (1 - 0.999) * g * g
    mh, vh = m / (1 - 0.9 ** count), v / (1 - 0.999 ** count)
    # an entry that never had a gradient stays put, and its root has no derivative
    root = torch.where(vh > 0, vh, torch.ones_like(vh)).sqrt() * (vh > 0)
    return theta - per_layer * (mh / (root + 1e-8) + eta[-1] * theta), m, v


def exact(case, seed):
    s = _inputs(case, seed)
    grad = torch.autograd.grad
    theta, eta = s["theta"].double(), s["eta"].double()
    n = theta.numel()
    zero = torch.zeros((), dtype=torch.float64, device=theta.device)
    m, v = (zero, zero) if s["opt"] is None else s["opt"].double().split(n)
    if case.get("meta") == MAML:
        theta = eta.clone()
    emb0 = _unpack(case, theta)["emb"] if case["kind"] == 1 else None

    def step(t, theta, m, v, eta, create):
        l = _row_losses(case, theta, s["xs"][t], s["ys"][t])
        L = (_weights(case, eta, emb0, t, s["xs"][t]) * l).mean()
        g, = grad(L, theta, create_graph=create)
        return L, g

    if case["entry"] == "inner_step":
        L, g = step(0, theta.requires_grad_(), m, v, eta, False)
        theta, m, v = _update(case, g, theta.detach(), m, v, eta, STEP + 1)
        return {"theta": theta, "opt": torch.cat([m, v]), "grad": g, "loss": L.detach().view(1)}

    if case["entry"] == "hvp":
        theta.requires_grad_()
        x, tangent = s["xs"][0], s["v"].double()
        out = {}
        if case["kind"] == 1:
            l = _row_losses(case, theta, x, None)
            ones = torch.ones_like(l, requires_grad=True)
            gl, = grad(l, theta, ones, create_graph=True)
            out["mvp"] = grad(gl @ tangent, ones)[0] / l.numel()
            del l, gl
        _, g = step(0, theta, m, v, eta, True)
        out["hvp"] = grad(g @ tangent, theta)[0]
        return {"grad": g.detach(), **out}

    states = []
    for t in range(case["T"]):
        states.append((theta, m, v))
        _, g = step(t, theta.detach().requires_grad_(), m, v, eta, False)
        theta, m, v = _update(case, g.detach(), theta, m, v, eta, t + 1)
    theta = theta.detach().requires_grad_()
    V = _row_losses(case, theta, s["vx"], s["vy"]).mean()
    bars = [grad(V, theta)[0], torch.zeros_like(m), torch.zeros_like(v)]
    d_eta = torch.zeros_like(eta)
    for t in reversed(range(case["T"])):
        ins = [a.detach().requires_grad_() for a in (*states.pop(), eta)]
        _, g = step(t, *ins, True)
        outs = _update(case, g, *ins, t + 1)
        if outs[1] is ins[1]:   # no optimiser state
            outs, bars = outs[:1], bars[:1]
        got = grad(outs, ins, bars, allow_unused=True)
        bars = list(got[:3])
        if got[3] is not None:
            d_eta += got[3]
        del outs, g, got, ins
    if case.get("meta") == MAML:
        d_eta = bars[0]
    if case["family"] == "loglr" and len(_widths(case)) > 5:
        # rounding the operands to bf16 alone moves this by some 15 % (the ReLU kinks of eight
        # layers), so it says nothing of the precision; three layers of the same width do
        d_eta = None
    return {"d_eta": d_eta, "val_loss": V.detach().view(1)}
