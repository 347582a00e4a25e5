"""The work a user of the library has it do, as cases that can be timed and compared.

A case is one pass through the public entry points at one size: a fine-tuning step (frozen forward, trainable
blocks forward and backward, optimizer update), the same step as a two-stream pipeline, the frozen encoder alone
(feature extraction), or the token selection alone.  `listed()` holds the named ones, `draw()` gives more of the
same ranges.

Inputs.  The images hold as many salient patches as each drop location keeps: a salient patch resembles the
pattern the class token looks for, the others resemble the background, and the query and key projections agree with
each other as those of a trained model do on similar tokens.  The attention of the class token then separates the
kept tokens from the dropped ones by far more than bf16 rounding, so that two correct implementations take the same
decisions and their results can be compared value by value.  A mixture of experts routes on near-ties whatever the
input, so its cases replay a recorded expert choice (bsr_moe_routing_io), unevenly spread as a router's is.
"""
from __future__ import annotations

import math

import torch

import paper_2405_10951_amd as P
from paper_2405_10951_amd.binding import bsr_token_schedule, make_config

DEV = "cuda"

MODELS = {
    # name: dim, heads, mlp_hidden, depth
    "vit_b": (768, 12, 3072, 12),
    "deit_s": (384, 6, 1536, 12),
    "vit_s_moe": (384, 6, 1536, 12),      # 16 experts, 2 active, in every other block
    "block": (192, 3, 768, 1),            # one encoder block on token input, mean-square loss
}
EXPERTS, TOP_K, MOE_BLOCKS = 16, 2, [1, 3, 5, 7, 9, 11]
CLASSES = (10, 37, 100, 101, 102)         # the label counts of the usual small fine-tuning sets


def _case(what="step", model="vit_b", batch=32, image=224, keep=0.7, trained=4, layout="suffix", fuse=False, fold=False,
          dtype="bf16", optimizer="sgd", classes=100, tune=False, **more):
    return dict(what=what, model=model, batch=batch, image=image, keep=keep, trained=trained, layout=layout, fuse=fuse,
                fold=fold, dtype=dtype, optimizer=optimizer, classes=classes, tune=tune, **more)


def listed():
    return [
        # the headline: ViT-B/16, a quarter of the tokens gone at three places, the last four blocks trained; a long
        # run tunes its tile shapes during set-up
        _case(name="vit_b_b32_step", tune=True),
        # the same step as a long run would issue it: the next batch's frozen forward on a second stream
        _case(name="vit_b_b32_pipelined", what="pipelined", tune=True),
        # a throughput-sized batch of the same model
        _case(name="vit_b_b128_step", batch=128, tune=True),
        # every block trained, no token dropped: what the method is compared with, and the most work of all
        _case(name="vit_b_b128_full", batch=128, keep=1.0, trained=12),
        # the smaller model with the optimizer it is usually fine-tuned with
        _case(name="deit_s_b32_adamw", model="deit_s", optimizer="adamw", classes=10),
        # mixture-of-experts feed-forward layers in every other block
        _case(name="vit_s_moe_b32", model="vit_s_moe"),
        # every fourth block trained with frozen ones between, dropped tokens fused into one, the ragged last batch
        # of an epoch (nothing is tuned for its size)
        _case(name="vit_b_b27_interleaved_fused", batch=27, keep=0.5, layout="interleaved", fuse=True, classes=37),
        # fine-tuning at a higher resolution than pre-training: 577 tokens
        _case(name="deit_s_384px_b16", model="deit_s", image=384, batch=16, classes=102),
        # full precision, as one runs it to check or to debug a recipe
        _case(name="deit_s_b8_fp32", model="deit_s", batch=8, dtype="fp32", classes=10),
        # the smallest step: one block, two token sequences, full precision
        _case(name="block_b2_fp32", model="block", batch=2, trained=1, dtype="fp32", classes=0),
        # one image through the whole frozen encoder: feature extraction one request at a time
        _case(name="vit_b_b1_features", what="features", batch=1, trained=0, fold=True),
        # token selection on its own: rank 196 patch tokens of 32 images, hand on the best 137
        _case(name="select_b32", what="select", batch=32, tokens=196, kept=137),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    keep = round(rng.uniform(0.4, 1.0), 2)
    kind = rng.choice(["step", "step", "step", "pipelined", "full", "moe", "interleaved", "resolution", "fp32", "block",
                       "features", "select"])
    opt, classes = rng.choice(["sgd", "adamw"]), rng.choice(CLASSES)
    if kind == "step":
        return _case(model=rng.choice(["vit_b", "deit_s"]), batch=_log_int(rng, 1, 128), keep=keep,
                     trained=rng.randint(1, 8), fuse=rng.random() < 0.25, optimizer=opt, classes=classes)
    if kind == "pipelined":
        return _case(what="pipelined", model=rng.choice(["vit_b", "deit_s"]), batch=_log_int(rng, 8, 64), keep=keep,
                     trained=rng.randint(2, 6), classes=classes)
    if kind == "full":
        return _case(model=rng.choice(["vit_b", "deit_s"]), batch=_log_int(rng, 4, 64), keep=rng.choice([1.0, keep]),
                     trained=12, optimizer=opt, classes=classes)
    if kind == "moe":
        return _case(model="vit_s_moe", batch=_log_int(rng, 2, 64), keep=keep, trained=rng.randint(2, 6), classes=classes)
    if kind == "interleaved":
        return _case(model=rng.choice(["vit_b", "deit_s"]), batch=_log_int(rng, 2, 64), keep=keep, layout="interleaved",
                     fuse=rng.random() < 0.5, optimizer=opt, classes=classes)
    if kind == "resolution":
        return _case(model="deit_s", image=rng.choice([256, 288, 320, 384, 448]), batch=_log_int(rng, 1, 16), keep=keep,
                     trained=rng.randint(1, 6), classes=classes)
    if kind == "fp32":
        return _case(model="deit_s", batch=_log_int(rng, 1, 8), keep=keep, trained=rng.randint(1, 6), dtype="fp32",
                     optimizer=opt, classes=classes)
    if kind == "block":
        return _case(model="block", batch=_log_int(rng, 1, 32), keep=keep, trained=1, dtype="fp32", classes=0)
    if kind == "features":
        return _case(what="features", model=rng.choice(["vit_b", "deit_s"]), batch=_log_int(rng, 1, 64), keep=keep, trained=0,
                     fold=rng.random() < 0.5)
    n = _log_int(rng, 24, 1023)
    return _case(what="select", batch=_log_int(rng, 1, 128), tokens=n, kept=max(1, int(keep * n)))


# ------------------------------------------------------------------------------------------ configuration

def _config(case):
    """-> (the dict Context takes, keep_k per drop, tokens seen by the attention / FFN of each block)"""
    dim, heads, hidden, depth = MODELS[case["model"]]
    if case["what"] == "select":
        cfg = dict(image_size=0, tokens_in=case["tokens"] + 1, dim=dim, heads=heads, mlp_hidden=hidden, depth=1, num_classes=0,
                   drop_blocks=[], keep_ratio=1.0, first_trainable=1, dtype=case["dtype"], loss=P.BSR_LOSS_MEAN_SQ)
    elif case["model"] == "block":
        cfg = dict(image_size=0, tokens_in=65, dim=dim, heads=heads, mlp_hidden=hidden, depth=1, num_classes=0, drop_blocks=[0],
                   keep_ratio=case["keep"], first_trainable=0, dtype=case["dtype"], loss=P.BSR_LOSS_MEAN_SQ)
    else:
        cfg = dict(image_size=case["image"], patch_size=16, in_chans=3, dim=dim, heads=heads, mlp_hidden=hidden, depth=depth,
                   drop_blocks=[3, 6, 9], keep_ratio=case["keep"], first_trainable=depth - case["trained"], dtype=case["dtype"],
                   num_classes=case["classes"], loss=P.BSR_LOSS_CE, fuse_dropped=int(case["fuse"]),
                   fold_frozen_layernorm=int(case["fold"]))
        if case["layout"] == "interleaved":
            cfg.update(first_trainable=3, trainable_blocks=[3, 7, 11])
        if case["model"] == "vit_s_moe":
            cfg.update(n_experts=EXPERTS, moe_top_k=TOP_K, moe_blocks=MOE_BLOCKS)
    keep_k, t_attn, t_mlp = bsr_token_schedule(make_config(cfg, case["batch"]))
    return cfg, keep_k, t_attn, t_mlp


def _shapes(cfg, tokens):
    D, F, C, E = cfg["dim"], cfg["mlp_hidden"], cfg["num_classes"], cfg.get("n_experts", 0)
    out = {}
    if cfg["image_size"]:
        out.update(w_patch=(cfg["in_chans"] * cfg["patch_size"] ** 2, D), b_patch=(D,), cls=(D,), pos=(tokens, D))
    for i in range(cfg["depth"]):
        b = dict(ln1_g=(D,), ln1_b=(D,), w_qkv=(D, 3 * D), b_qkv=(3 * D,), w_proj=(D, D), b_proj=(D,), ln2_g=(D,), ln2_b=(D,),
                 w_fc1=(D, F), b_fc1=(F,), w_fc2=(F, D), b_fc2=(D,))
        if i in cfg.get("moe_blocks", ()):
            b.update(w_router=(D, E), w_fc1=(E, D, F), b_fc1=(E, F), w_fc2=(E, F, D), b_fc2=(E, D))
        out.update({"blocks.%d.%s" % (i, k): s for k, s in b.items()})
    if C:
        out.update(lnf_g=(D,), lnf_b=(D,), w_head=(D, C), b_head=(C,))
    return out


def _trained(cfg, name):
    if name in ("lnf_g", "lnf_b", "w_head", "b_head"):
        return True
    if not name.startswith("blocks."):
        return False
    l = int(name.split(".")[1])
    return l in cfg["trainable_blocks"] if cfg.get("trainable_blocks") else l >= cfg["first_trainable"]


class _Flat:
    """Tensors of the given shapes as views into one buffer (each at a multiple of 64 floats): the vectors, the matrices
    of the blocks, the head's matrix.  What a training program keeps so that it can clip, average or checkpoint all of
    them at once."""

    def __init__(self, shapes):
        kind = lambda n: 2 if n == "w_head" else 1 if "w_" in n else 0      # noqa: E731
        order = sorted(shapes, key=kind)
        size = {n: -(-math.prod(shapes[n]) // 64) * 64 for n in order}
        self.flat = torch.zeros(max(64, sum(size.values())), dtype=torch.float32, device=DEV)
        self.views, at, ends = {}, 0, [0, 0, 0]
        for n in order:
            self.views[n] = self.flat[at:at + math.prod(shapes[n])].view(shapes[n])
            at += size[n]
            ends[kind(n)] = at
        self.parts = {"vectors": self.flat[:ends[0]], "matrices": self.flat[ends[0]:max(ends[:2])]}
        if ends[2]:
            self.parts["head"] = self.flat[max(ends[:2]):ends[2]]


# ------------------------------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _params(cfg, shapes, g):
    """Weights of the scale a trained vision transformer has, the trained ones in one buffer; -> dict, its _Flat"""
    flat = _Flat({n: s for n, s in shapes.items() if _trained(cfg, n)})
    bf16 = cfg["dtype"] == "bf16"
    D, out = cfg["dim"], {}
    for n, s in shapes.items():
        leaf = n.split(".")[-1]
        a = torch.randn(s, generator=g, device=DEV) * (D ** -0.5 if leaf == "w_router" else 0.02)
        if leaf in ("ln1_g", "ln2_g", "lnf_g"):
            a += 1.0
        if leaf == "w_qkv":        # similar tokens attend to each other
            a[:, :D] *= 1.5
            a[:, D:2 * D] = a[:, :D]
        if leaf == "b_qkv":
            a[D:2 * D] = a[:D]
        if bf16:
            a = a.to(torch.bfloat16).float()
        if n in flat.views:
            flat.views[n].copy_(a)
            a = flat.views[n]
        out[n] = a
    return out, flat


def _salience(keep_k, n, batch, g):
    """[batch, n] in (0, 1): as many tokens above each step as the drop locations keep, at random places"""
    level = torch.empty(n, device=DEV)
    edges = [n] + list(keep_k) + [0]                     # tokens still there after each drop
    for i in range(len(edges) - 1):
        level[max(0, edges[i + 1]):max(0, edges[i])] = 0.05 + 0.9 * i / max(1, len(edges) - 2)
    place = torch.rand((batch, n), generator=g, device=DEV).argsort(dim=1)
    return level[place]


def _images(cfg, params, keep_k, batch, g):
    """[batch, C, S, S] ~ N(0, 1): every patch a mixture of the salient pattern, the background and noise.  The class
    embedding of the model is the one a pre-training on such images leaves: the embedded salient pattern."""
    C, p, G = cfg["in_chans"], cfg["patch_size"], cfg["image_size"] // cfg["patch_size"]
    pattern, background = (torch.randn(C * p * p, generator=g, device=DEV) for _ in range(2))
    a = _salience(keep_k, G * G, batch, g)[..., None]
    x = a * pattern + (1.0 - a * a).sqrt() * background
    x = (x + 0.4 * torch.randn(x.shape, generator=g, device=DEV)) / 1.16 ** 0.5
    params["cls"].copy_((pattern @ params["w_patch"]).to(torch.bfloat16).float())
    return x.view(batch, G, G, C, p, p).permute(0, 3, 1, 4, 2, 5).reshape(batch, C, G * p, G * p).contiguous()


def _tokens(cfg, keep_k, batch, g):
    T, D = cfg["tokens_in"], cfg["dim"]
    pattern, background = (torch.randn(D, generator=g, device=DEV) for _ in range(2))
    a = torch.cat([torch.ones((batch, 1), device=DEV), _salience(keep_k, T - 1, batch, g)], 1)[..., None]
    x = a * pattern + (1.0 - a * a).sqrt() * background
    return (x + 0.4 * torch.randn(x.shape, generator=g, device=DEV)) / 1.16 ** 0.5


_streams = []


def _two_streams():
    if not _streams:
        _streams.extend([torch.cuda.Stream(), torch.cuda.Stream()])
    return _streams


def _routing(ctx, batch, g):
    """A recorded expert choice: distinct experts per token, some of them several times as popular as others"""
    rows = sum(ctx.moe_rows(batch).values())
    popularity = torch.linspace(0.0, 1.5, EXPERTS, device=DEV)[torch.rand(EXPERTS, generator=g, device=DEV).argsort()]
    gumbel = -torch.log(-torch.log(torch.rand((rows, EXPERTS), generator=g, device=DEV).clamp(1e-6, 1 - 1e-6)))
    return (popularity + gumbel).topk(TOP_K, dim=1).indices.to(torch.int32).contiguous()


def prepare(case, seed):
    g = _gen(seed)
    cfg, keep_k, t_attn, _ = _config(case)
    batch = case["batch"]
    shapes = _shapes(cfg, t_attn[0])
    params, weights = _params(cfg, shapes, g)
    if case["what"] == "select":
        ctx = P.Context(cfg, params, batch)
        n, k = case["tokens"], case["kept"]
        x = torch.randn((batch, n + 1, cfg["dim"]), generator=g, device=DEV).to(ctx.act_dtype)
        return dict(case=case, ctx=ctx, x=x, k=k, scores=torch.randn((batch, n), generator=g, device=DEV).softmax(1),
                    idx=torch.empty((batch, k), dtype=torch.int32, device=DEV),
                    out=torch.empty((batch, k + 1, cfg["dim"]), dtype=ctx.act_dtype, device=DEV))
    x0 = _images(cfg, params, keep_k, batch, g) if cfg["image_size"] else _tokens(cfg, keep_k, batch, g)
    ctx = P.Context(cfg, params, batch)
    act = ctx.act_dtype
    st = dict(case=case, ctx=ctx, i=0, input=x0.to(act).contiguous())
    C = cfg["num_classes"]
    st["labels"] = torch.randint(0, max(C, 1), (batch,), generator=g, device=DEV, dtype=torch.int32) if C else None
    st["x"] = [torch.empty((batch, ctx.T_f, cfg["dim"]), dtype=act, device=DEV) for _ in range(2)]
    if case["what"] == "features":
        kept = sum(batch * keep_k[i] for i in ctx.frozen_drops)
        st["kept"] = torch.empty(max(kept, 4), dtype=torch.int32, device=DEV)[:kept]
        return st
    if case["model"] == "vit_s_moe":
        ctx.bsr_moe_routing_io(forced_experts=_routing(ctx, batch, g))
    moving = {n: s for n, s in shapes.items() if _trained(cfg, n)}
    st["weights"], st["grads"], st["m1"] = weights, _Flat(moving), _Flat(moving)
    st["m2"] = _Flat(moving) if case["optimizer"] == "adamw" else None
    st["loss"] = torch.zeros(4, dtype=torch.float32, device=DEV)
    st["logits"] = torch.zeros((batch, C), dtype=torch.float32, device=DEV) if C else None
    x0, lab, gr = st["input"], st["labels"], st["grads"].views
    if case["what"] == "pipelined":
        frozen, train = _two_streams()
        torch.cuda.synchronize()
        if case["tune"]:
            with torch.cuda.stream(frozen):
                ctx.bsr_autotune_overlapped(x0, lab, st["x"][0], st["x"][1], st["loss"], gr, train)
        ctx.bsr_pipeline_step(x0, st["x"][0], None, None, st["loss"], gr, st["m1"].views, 1e-3, 0.9, 1e-4, frozen, train)
        torch.cuda.synchronize()
    elif case["tune"]:
        ctx.bsr_autotune(x0, lab, st["x"][0], st["loss"], gr)
    return st


# ------------------------------------------------------------------------------------------ one pass

def run(st):
    case, ctx = st["case"], st["ctx"]
    if case["what"] == "select":
        idx, out = ctx.bsr_select_tokens(st["scores"], st["x"], st["k"], idx_out=st["idx"], x_out=st["out"])
        return {"idx": idx, "tokens": out}
    x = st["x"]
    if case["what"] == "features":
        ctx.bsr_forward_frozen(st["input"], x_out=x[0], kept_idx_out=st["kept"])
        return {"features": x[0], "kept": st["kept"]}
    grads, m1 = st["grads"], st["m1"]
    st["i"] = i = st["i"] + 1
    if case["what"] == "pipelined":
        frozen, train = _two_streams()
        ctx.bsr_pipeline_step(st["input"], x[i % 2], x[(i + 1) % 2], st["labels"], st["loss"], grads.views, m1.views, 1e-3, 0.9,
                              1e-4, frozen, train)
    else:
        ctx.bsr_forward_frozen(st["input"], x_out=x[0])
        ctx.bsr_train_blocks_fwd_bwd(x[0], st["labels"], grads.views, loss_out=st["loss"], logits_out=st["logits"])
        if case["optimizer"] == "adamw":
            ctx.bsr_adamw_step(grads.views, m1.views, st["m2"].views, lr=1e-4, weight_decay=0.05, step=i)
        else:
            ctx.bsr_sgd_step(grads.views, m1.views, lr=1e-3, momentum=0.9, weight_decay=1e-4)
    out = {"loss": st["loss"][:1], "weights": st["weights"].parts, "grads": grads.parts, "moment1": m1.parts}
    if st["m2"]:
        out["moment2"] = st["m2"].parts
    if st["logits"] is not None and case["what"] == "step":
        out["logits"] = st["logits"]
    return out


# ------------------------------------------------------------------------------------------ what a pass cannot do without

def work(case):
    """Each input read once, each output written once, and the operations the results depend on.  The class token is all
    that the loss of a classifier reads of the last block: there the other tokens only have to be keys and values."""
    cfg, keep_k, t_attn, t_mlp = _config(case)
    B, D, F, depth = case["batch"], cfg["dim"], cfg["mlp_hidden"], cfg["depth"]
    size = 4 if case["dtype"] == "fp32" else 2
    if case["what"] == "select":
        n, k = case["tokens"], case["kept"]
        return {"bytes": B * (4 * n + 4 * k + 2 * size * (k + 1) * D), "flops": 0}
    shapes = _shapes(cfg, t_attn[0])
    count = {n: math.prod(s) for n, s in shapes.items()}
    trained = sum(c for n, c in count.items() if _trained(cfg, n))
    frozen = sum(count.values()) - trained
    inputs = B * (cfg["in_chans"] * cfg["image_size"] ** 2 if cfg["image_size"] else cfg["tokens_in"] * D)
    if case["what"] == "features":
        outputs = B * (size * t_mlp[-1] * D + 4 * sum(keep_k))
        update = 0
    else:
        outputs = 4 * B * cfg["num_classes"]
        # weights, gradients and moments: all but the gradients are read and written
        update = trained * 4 * (3 if case["optimizer"] == "adamw" else 2) * 2 + trained * 4
    ft = cfg["trainable_blocks"][0] if cfg.get("trainable_blocks") else cfg["first_trainable"]
    flops = 0.0
    if cfg["image_size"]:
        flops += 2.0 * (t_attn[0] - 1) * cfg["in_chans"] * cfg["patch_size"] ** 2 * D
    for l in range(depth):
        Ta, Tm = t_attn[l], t_mlp[l]
        last = l == depth - 1 and cfg["num_classes"] > 0 and case["what"] != "features"
        Tq, Tf = (1, 1) if last else (Ta, Tm)
        qkv, rest = 2.0 * (Tq + 2 * Ta) * D * D, 2.0 * (Tq * D * D + 2 * Tf * D * F)
        if l in cfg.get("moe_blocks", ()):
            rest = 2.0 * (Tq * D * D + 2 * TOP_K * Tf * D * F + Tf * D * EXPERTS)
        attn = 4.0 * Tq * Ta * D
        flops += qkv + rest + attn
        if l >= ft:
            weight_grads = _trained(cfg, "blocks.%d.x" % l)
            flops += 2.5 * attn + (qkv + rest) * (2 if weight_grads else 1)
    flops += 3 * 2.0 * D * cfg["num_classes"] * (case["what"] != "features")
    return {"bytes": inputs * size + frozen * size + outputs + update, "flops": flops * B}


def tolerance(case):
    """bf16 activations: twelve blocks of roundings leave 0.8 % of error (2-norm) in every gradient, measured against the
    same step in fp32, so two implementations may be 1.2 % apart (second moments are squares: twice a gradient's error
    where it is not averaged away)."""
    if case["what"] == "select":
        return "exact"
    if case["dtype"] == "fp32":
        return {"rel": 5e-5, "differ": 0.005}
    return {"rel": 2e-2 if case["optimizer"] == "adamw" else 1.5e-2, "max": 0.5, "differ": 0.005}
