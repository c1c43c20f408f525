"""The work that users of this library have it do, as cases that can be timed.

A case is a dict of plain values.  Its "kind" names the entry point that it
goes through, the other values give sizes, precision and options:

  encode      vl.Encoder.encode on a batch of images (image tower)
  text        vl.TextEncoder.encode on a batch of prompts (text tower)
  train       one contrastive training step: Trainer.forward, the loss with
              its gradients, Trainer.backward to every weight gradient
  attention   vl_attention on packed sequences
  attention_backward   vl_attention_backward on packed sequences
  contrastive vl_contrastive_loss on a batch of matched pairs
  score       vl_score of image embeddings against resident texts

Towers run either whole or cut to two blocks of their own widths, which keeps
a layer's shapes and lets outputs be held against 64-bit arithmetic.  Ragged
batches take their sizes from the case's "shapes" number, so a case's work is
the same for every seed.  Weights are N(0, 0.02^2) with LayerNorm gains
around 1, pixels U[0, 1), texts and embeddings unit vectors, as in the
repository's synthetic workloads.
"""
from __future__ import annotations

import math
import random
from types import SimpleNamespace

import torch
import torch.nn.functional as F

from paper_2505_00690_amd import vl

_SD = 1.0 / math.sqrt(12.0)

# name: patch, width, blocks, heads, mlp, projection, base grid, planes
_TOWERS = {
    "s16_rgbd": (16, 384, 12, 6, 1536, 256, 8, 4),    # 128 px RGB-D observations
    "b16": (16, 768, 12, 12, 3072, 512, 14, 3),
    "l14": (14, 1024, 24, 16, 4096, 768, 24, 3),
}
# vocab, context, width, blocks, heads, mlp, projection
_TEXT = (49408, 77, 768, 12, 12, 3072, 768)
_EPS = 1e-5


# ------------------------------------------------------------------- cases
def listed():
    return [
        # One environment's RGB-D frame per policy step, the whole observation
        # encoder replayed as a graph: the smallest call, latency bound.
        dict(name="rgbd_frame", kind="encode", tower="s16_rgbd", blocks=12, precision="bf16",
             images=1, px="128", shapes=0, graphs=True, split=False),
        # The headline batch: ViT-L/14 at 336 px, whole tower, two overlapped
        # parts, exact-shape graph.  The largest case.
        dict(name="l14_336_b32", kind="encode", tower="l14", blocks=24, precision="bf16",
             images=32, px="336", shapes=0, graphs=True, split=True),
        # Mixed-resolution offline encoding: 96 images of 224, 336 and 448 px.
        dict(name="b16_mixed_b96", kind="encode", tower="b16", blocks=2, precision="bf16",
             images=96, px="224,336,448", shapes=3, graphs=False, split=False),
        # One serving batch with FP8 weights: a few requests' images of four
        # resolutions, eager launches.
        dict(name="l14_serve_fp8w_b11", kind="encode", tower="l14", blocks=2, precision="fp8w",
             images=11, px="224,336,384,448", shapes=4, graphs=False, split=False),
        # The MXFP8 variant on the headline shape.
        dict(name="l14_336_mxfp8_b32", kind="encode", tower="l14", blocks=2, precision="mxfp8",
             images=32, px="336", shapes=0, graphs=False, split=True),
        # The FP32 tower, which results are checked against.
        dict(name="b16_224_fp32_b8", kind="encode", tower="b16", blocks=2, precision="fp32",
             images=8, px="224", shapes=0, graphs=False, split=False),
        # Encoding a set of class prompts (short, one in ten at full context).
        dict(name="text_prompts_1000", kind="text", blocks=2, precision="bf16", texts=1000,
             shapes=5),
        # A contrastive training step: forward, loss, every weight gradient.
        dict(name="train_l14_336_b32", kind="train", tower="l14", blocks=2, precision="bf16",
             images=32),
        # Attention alone over ragged sequences, up to the longest accepted.
        dict(name="attention_ragged", kind="attention", dtype="bf16", heads=16, head_dim=64,
             causal=False, seqs=24, longest=2049, shapes=6),
        # Its backward at the image tower's lengths.
        dict(name="attention_backward_577", kind="attention_backward", dtype="bf16", heads=16,
             head_dim=64, seqs=32, longest=577, shapes=0),
        # The loss and embedding gradients of a large contrastive batch.
        dict(name="contrastive_1024", kind="contrastive", n=1024, dim=768, head="softmax"),
        # Zero-shot scores of a batch against the resident class texts.
        dict(name="score_64x1000", kind="score", n=64, texts=1000, dim=512, head="softmax"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    shapes = rng.randrange(7, 1 << 20)
    kind = rng.choice(["rgbd", "l14", "b16", "serve", "mxfp8", "fp32", "text", "train",
                       "attention", "attention_backward", "contrastive", "score"])
    if kind == "rgbd":     # 1 .. 256 environments' frames
        return dict(kind="encode", tower="s16_rgbd", blocks=12, precision="bf16",
                    images=_log(rng, 1, 256), px="128", shapes=shapes,
                    graphs=rng.random() < 0.5, split=False)
    if kind == "l14":
        return dict(kind="encode", tower="l14", blocks=rng.choice([2, 24]), precision="bf16",
                    images=_log(rng, 1, 31), px=rng.choice(["224", "336"]), shapes=shapes,
                    graphs=rng.random() < 0.5, split=rng.random() < 0.5)
    if kind == "b16":
        return dict(kind="encode", tower="b16", blocks=2, precision="bf16",
                    images=_log(rng, 1, 128), px=rng.choice(["224", "224,336,448"]),
                    shapes=shapes, graphs=False, split=rng.random() < 0.5)
    if kind == "serve":
        return dict(kind="encode", tower="l14", blocks=2, precision="fp8w",
                    images=_log(rng, 1, 32), px="224,336,384,448", shapes=shapes,
                    graphs=rng.random() < 0.5, split=False)
    if kind == "mxfp8":
        return dict(kind="encode", tower="l14", blocks=2, precision="mxfp8",
                    images=_log(rng, 1, 48), px=rng.choice(["224", "336"]), shapes=shapes,
                    graphs=False, split=rng.random() < 0.5)
    if kind == "fp32":
        return dict(kind="encode", tower=rng.choice(["s16_rgbd", "b16", "l14"]), blocks=2,
                    precision="fp32", images=_log(rng, 1, 24), px="224", shapes=shapes,
                    graphs=False, split=False)
    # (FP32 runs at a fraction of the BF16 rate: its draws stay smaller.)
    if kind == "text":
        f32 = rng.random() < 0.3
        return dict(kind="text", blocks=2, precision="fp32" if f32 else "bf16",
                    texts=_log(rng, 1, 256 if f32 else 2048), shapes=shapes)
    if kind == "train":
        f32 = rng.random() < 0.25
        return dict(kind="train", tower="b16" if f32 else rng.choice(["b16", "l14"]), blocks=2,
                    precision="fp32" if f32 else "bf16", images=_log(rng, 2, 8 if f32 else 40))
    if kind == "attention":
        f32 = rng.random() < 0.3
        return dict(kind="attention", dtype="fp32" if f32 else "bf16",
                    heads=rng.choice([6, 12, 16]), head_dim=rng.choice([64, 64, 32]),
                    causal=rng.random() < 0.5, seqs=_log(rng, 1, 16 if f32 else 64),
                    longest=_log(rng, 16, 577 if f32 else 2049), shapes=shapes)
    if kind == "attention_backward":
        f32 = rng.random() < 0.3
        return dict(kind="attention_backward", dtype="fp32" if f32 else "bf16",
                    heads=rng.choice([6, 12, 16]), head_dim=rng.choice([64, 64, 32]),
                    seqs=_log(rng, 1, 4 if f32 else 32), longest=_log(rng, 16, 577 if f32 else 1025),
                    shapes=shapes)
    if kind == "contrastive":
        return dict(kind="contrastive", n=_log(rng, 8, 2400), dim=rng.choice([256, 512, 768]),
                    head=rng.choice(["softmax", "sigmoid"]))
    return dict(kind="score", n=_log(rng, 1, 256), texts=4 * _log(rng, 4, 2048),
                dim=rng.choice([256, 512, 768]), head=rng.choice(["softmax", "sigmoid"]))


# ------------------------------------------------------------------- shapes
def _tower(case):
    p, w, _, h, m, pd, g, c = _TOWERS[case["tower"]]
    return SimpleNamespace(patch=p, width=w, layers=case["blocks"], heads=h, mlp=m, proj_dim=pd,
                           base_grid=g, ln_eps=_EPS, chan_mean=(0.5,) * c, chan_std=(_SD,) * c,
                           channels=c, pool="cls")


def _text_tower(case):
    v, ctx, w, _, h, m, pd = _TEXT
    return SimpleNamespace(vocab=v, ctx=ctx, width=w, layers=case["blocks"], heads=h, mlp=m,
                           proj_dim=pd, ln_eps=_EPS)


def _sizes(case):
    if case["kind"] == "train":
        c = _tower(case)
        return [(c.patch * c.base_grid,) * 2] * case["images"]
    px = [int(x) for x in case["px"].split(",")]
    r = random.Random(case["shapes"])
    return [(s, s) for s in (r.choice(px) for _ in range(case["images"]))]


def _prompt_lengths(case):
    r = random.Random(case["shapes"])
    return [77 if r.random() < 0.1 else r.randint(5, 20) for _ in range(case["texts"])]


def _lengths(case):
    """Sequence lengths up to `longest`; shapes 0: all of them that long."""
    r = random.Random(case["shapes"])
    n, m = case["seqs"], case["longest"]
    return [m] + [m if case["shapes"] == 0 else r.randint(1, m) for _ in range(n - 1)]


def _tokens(c, sizes):
    return [1 + (h // c.patch) * (w // c.patch) for h, w in sizes]


def _layout(c, text=False):
    """(name, shape) of every weight in blob order."""
    D, M = c.width, c.mlp
    if text:
        out = [("tok", (c.vocab, D)), ("pos", (c.ctx, D))]
    else:
        out = [("patch_w", (D, c.channels, c.patch, c.patch)), ("patch_b", (D,)), ("cls", (D,)),
               ("pos", (1 + c.base_grid ** 2, D))]
    for i in range(c.layers):
        out += [(f"{i}.{n}", s) for n, s in (
            ("ln1_g", (D,)), ("ln1_b", (D,)), ("qkv_w", (3 * D, D)), ("qkv_b", (3 * D,)),
            ("o_w", (D, D)), ("o_b", (D,)), ("ln2_g", (D,)), ("ln2_b", (D,)),
            ("fc1_w", (M, D)), ("fc1_b", (M,)), ("fc2_w", (D, M)), ("fc2_b", (D,)))]
    return out + [("lnf_g", (D,)), ("lnf_b", (D,)), ("proj", (c.proj_dim, D))]


# ------------------------------------------------------------------- inputs
def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + salt)
    return g


def _weights(c, seed, text=False):
    lay = _layout(c, text)
    blob = torch.empty(sum(math.prod(s) for _, s in lay), device="cuda")
    blob.normal_(0.0, 0.02, generator=_gen(seed, 1))
    o = 0
    for name, s in lay:
        n = math.prod(s)
        if name.endswith("_g"):
            blob[o:o + n] += 1.0
        o += n
    return blob


def _pixels(c, sizes, seed):
    n = c.channels * sum(h * w for h, w in sizes)
    return torch.rand(n, device="cuda", generator=_gen(seed, 2))


def _ids(case, seed):
    """Start-of-text, words, end-of-text, back to back."""
    vocab = _TEXT[0]
    lens = torch.tensor(_prompt_lengths(case), device="cuda")
    ids = torch.randint(0, vocab - 2, (int(lens.sum()),), device="cuda", dtype=torch.int32,
                        generator=_gen(seed, 3))
    end = lens.cumsum(0)
    ids[end - lens] = vocab - 2
    ids[end - 1] = vocab - 1
    return ids


def _unit(n, dim, seed, salt):
    return F.normalize(torch.randn(n, dim, device="cuda", generator=_gen(seed, salt)), dim=1)


def _pairs(n, dim, seed):
    """Texts, and embeddings that lean towards their own text."""
    t = _unit(n, dim, seed, 4)
    return F.normalize(0.12 * t + _unit(n, dim, seed, 5), dim=1), t


def _qkv(case, seed):
    T, D = sum(_lengths(case)), case["heads"] * case["head_dim"]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    return torch.randn(T, 3 * D, device="cuda", generator=_gen(seed, 6)).to(dt)


def _d_out(case, seed):
    T, D = sum(_lengths(case)), case["heads"] * case["head_dim"]
    return torch.randn(T, D, device="cuda", generator=_gen(seed, 7))


def _loss_constants(head):
    return (100.0, 0.0) if head == "softmax" else (10.0, -10.0)


def prepare(case, seed):
    kind, s = case["kind"], SimpleNamespace(case=case)
    if kind == "encode":
        c = _tower(case)
        s.sizes = _sizes(case)
        s.model = vl.Encoder(c, _weights(c, seed), case["precision"], graphs=case["graphs"],
                             split=case["split"])
        if case["graphs"] and case["px"].count(",") == 0:   # fixed shapes: exact graphs
            vl.vl_model_set_option(s.model.handle, vl.VL_OPT_GRAPH_BUCKETS, 0)
        s.pixels = _pixels(c, s.sizes, seed)
        s.out = torch.empty(len(s.sizes), c.proj_dim, device="cuda")
    elif kind == "text":
        c = _text_tower(case)
        s.lengths = _prompt_lengths(case)
        s.model = vl.TextEncoder(c, _weights(c, seed, True), case["precision"])
        s.ids = _ids(case, seed)
        s.out = torch.empty(case["texts"], c.proj_dim, device="cuda")
    elif kind == "train":
        c = _tower(case)
        s.sizes = _sizes(case)
        w = _weights(c, seed)
        s.model = vl.Trainer(c, w, case["precision"], split=True)
        s.pixels = _pixels(c, s.sizes, seed)
        s.texts = _unit(case["images"], c.proj_dim, seed, 4)
        s.out = torch.empty(case["images"], c.proj_dim, device="cuda")
        s.grads = torch.empty(w.numel(), device="cuda")
    elif kind == "attention":
        s.lengths = _lengths(case)
        s.qkv = _qkv(case, seed)
        s.out = s.qkv.new_empty(s.qkv.shape[0], s.qkv.shape[1] // 3)
        s.ws = torch.empty(vl.vl_attention_workspace_bytes(s.lengths), dtype=torch.uint8,
                           device="cuda")
    elif kind == "attention_backward":
        s.lengths = _lengths(case)
        s.qkv = _qkv(case, seed)
        s.out = s.qkv.new_empty(s.qkv.shape[0], s.qkv.shape[1] // 3)
        vl.vl_attention(s.qkv, s.lengths, case["heads"], case["head_dim"], False, s.out)
        s.d_out = _d_out(case, seed)
        s.d_qkv = torch.empty_like(s.qkv)
        s.ws = torch.empty(vl.vl_attention_backward_workspace_bytes(
            s.lengths, case["heads"], case["head_dim"]), dtype=torch.uint8, device="cuda")
    elif kind == "contrastive":
        s.emb, s.texts = _pairs(case["n"], case["dim"], seed)
    else:
        s.emb = _unit(case["n"], case["dim"], seed, 5)
        s.texts = _unit(case["texts"], case["dim"], seed, 4)
        s.scores = torch.empty(case["n"], case["texts"], device="cuda")
        s.top1 = torch.empty(case["n"], dtype=torch.int32, device="cuda")
    return s


def run(s):
    case, kind = s.case, s.case["kind"]
    if kind == "encode":
        return s.model.encode(s.pixels, s.sizes, out=s.out)
    if kind == "text":
        return s.model.encode(s.ids, s.lengths, out=s.out)
    if kind == "train":
        emb = s.model.forward(s.pixels, s.sizes, out=s.out)
        scale, bias = _loss_constants("sigmoid")
        loss, d_emb, d_texts, d_sb = vl.vl_contrastive_loss(emb, s.texts, "sigmoid", scale, bias)
        grads = s.model.backward(s.pixels, s.sizes, d_emb, grads_out=s.grads)
        return {"emb": emb, "loss": loss, "d_texts": d_texts, "d_scale_bias": d_sb,
                "grads": grads}
    if kind == "attention":
        vl.vl_attention(s.qkv, s.lengths, case["heads"], case["head_dim"], case["causal"], s.out,
                        s.ws)
        return s.out
    if kind == "attention_backward":
        vl.vl_attention_backward(s.qkv, s.out, s.d_out, s.lengths, case["heads"],
                                 case["head_dim"], s.d_qkv, s.ws)
        return s.d_qkv
    scale, bias = _loss_constants(case["head"])
    if kind == "contrastive":
        loss, d_emb, d_texts, d_sb = vl.vl_contrastive_loss(s.emb, s.texts, case["head"], scale,
                                                            bias)
        return {"loss": loss, "d_emb": d_emb, "d_texts": d_texts, "d_scale_bias": d_sb}
    vl.vl_score(s.emb, s.texts, case["head"], scale, bias, s.scores, s.top1)
    return {"scores": s.scores, "top1": s.top1}


# --------------------------------------------------------------------- work
def _weight_bytes(c, precision, text=False):
    per = {"fp32": 4, "bf16": 2, "fp8w": 1, "mxfp8": 1 + 1 / 32}[precision]
    n = 0.0
    for name, s in _layout(c, text):
        block = name.split(".")[-1] in ("qkv_w", "o_w", "fc1_w", "fc2_w")
        if name != "tok":
            n += math.prod(s) * (per if block else 4)
    return n


def _block_flops(c, toks, causal=False):
    T, D = sum(toks), c.width
    pairs = sum(n * (n + 1) / 2 if causal else n * n for n in toks)
    return c.layers * (2.0 * T * D * 4 * D + 4.0 * T * D * c.mlp + 4.0 * pairs * D)


def _encode_work(case):
    c, sizes = _tower(case), _sizes(case)
    toks = _tokens(c, sizes)
    f = _block_flops(c, toks) + 2.0 * len(sizes) * c.width * c.proj_dim
    f += 2.0 * sum(n - 1 for n in toks) * c.channels * c.patch ** 2 * c.width
    b = _weight_bytes(c, case["precision"])
    b += 4.0 * c.channels * sum(h * w for h, w in sizes) + 4.0 * len(sizes) * c.proj_dim
    return b, f


def work(case):
    kind = case["kind"]
    if kind == "encode":
        b, f = _encode_work(case)
    elif kind == "text":
        c, lens = _text_tower(case), _prompt_lengths(case)
        f = _block_flops(c, lens, causal=True) + 2.0 * len(lens) * c.width * c.proj_dim
        b = _weight_bytes(c, case["precision"], True) + sum(lens) * (4.0 + 4.0 * c.width)
        b += 4.0 * len(lens) * c.proj_dim
    elif kind == "train":
        c = _tower(case)
        b, f = _encode_work(case)
        n, f = case["images"], 3.0 * f
        f += 6.0 * n * n * c.proj_dim
        b += 4.0 * sum(math.prod(s) for _, s in _layout(c)) + 8.0 * n * c.proj_dim
    elif kind in ("attention", "attention_backward"):
        lens, D = _lengths(case), case["heads"] * case["head_dim"]
        pairs = sum(n * (n + 1) / 2 if case.get("causal") else n * n for n in lens)
        e = 2 if case["dtype"] == "bf16" else 4
        back = kind == "attention_backward"
        f = (10.0 if back else 4.0) * pairs * D
        b = sum(lens) * D * (e * 7 + 4.0 if back else e * 4.0)
    elif kind == "contrastive":
        n, d = case["n"], case["dim"]
        b, f = 16.0 * n * d + 12, 6.0 * n * n * d
    else:
        n, m, d = case["n"], case["texts"], case["dim"]
        b, f = 4.0 * (n * d + m * d + n * m + n), 2.0 * n * m * d
    return {"bytes": float(b), "flops": float(f)}


# ------------------------------------------------------ 64-bit reference values
def _rounded(name, w, precision):
    """A weight as the model holds it, in float64."""
    if precision == "fp32" or name.split(".")[-1] not in ("qkv_w", "o_w", "fc1_w", "fc2_w"):
        return w.double()
    if precision == "bf16":
        return w.bfloat16().double()
    if precision == "fp8w":
        s = w.abs().amax(1, keepdim=True) / 448.0
        return (w / s).to(torch.float8_e4m3fn).double() * s.double()
    b = w.double().reshape(w.shape[0], -1, 32)
    x = torch.floor(torch.log2(b.abs().amax(-1, keepdim=True))) - 8.0
    q = (b / torch.exp2(x)).clamp(-448.0, 448.0).float().to(torch.float8_e4m3fn).double()
    return (q * torch.exp2(x)).reshape(w.shape)


def _split_blob(c, blob, precision, text=False):
    p, o = {}, 0
    for name, s in _layout(c, text):
        n = math.prod(s)
        p[name] = _rounded(name, blob[o:o + n].reshape(s), precision)
        o += n
    return p


def _attend(q, k, v, causal):
    """softmax(q k^T / sqrt(d)) v per head; q, k, v [heads, n, d] float64."""
    s = q @ k.transpose(1, 2).contiguous() / math.sqrt(q.shape[-1])
    if causal:
        n = s.shape[-1]
        s = s.masked_fill(torch.ones(n, n, dtype=torch.bool, device=s.device).triu(1),
                          -math.inf)
    return torch.softmax(s, -1) @ v


def _heads(x, h):
    return x.reshape(x.shape[0], h, -1).transpose(0, 1).contiguous()


def _packed_attention(qkv, lens, heads, causal):
    out = []
    for part in torch.split(qkv, lens):
        q, k, v = (_heads(t, heads) for t in part.chunk(3, 1))
        out.append(_attend(q, k, v, causal).transpose(0, 1).reshape(part.shape[0], -1))
    return torch.cat(out)


def _blocks(x, lens, p, c, causal):
    D = (c.width,)
    for i in range(c.layers):
        w = {n: p[f"{i}.{n}"] for n in ("ln1_g", "ln1_b", "qkv_w", "qkv_b", "o_w", "o_b", "ln2_g",
                                        "ln2_b", "fc1_w", "fc1_b", "fc2_w", "fc2_b")}
        y = F.layer_norm(x, D, w["ln1_g"], w["ln1_b"], c.ln_eps)
        a = _packed_attention(F.linear(y, w["qkv_w"], w["qkv_b"]), lens, c.heads, causal)
        x = x + F.linear(a, w["o_w"], w["o_b"])
        y = F.layer_norm(x, D, w["ln2_g"], w["ln2_b"], c.ln_eps)
        x = x + F.linear(F.gelu(F.linear(y, w["fc1_w"], w["fc1_b"])), w["fc2_w"], w["fc2_b"])
    return x


def _head(x, rows, p, c):
    z = F.layer_norm(x[rows], (c.width,), p["lnf_g"], p["lnf_b"], c.ln_eps)
    return F.normalize(F.linear(z, p["proj"]), dim=1, eps=1e-12)


def _encode64(c, p, pixels, sizes):
    pos, D = p["pos"], c.width
    grid = pos[1:].T.reshape(1, D, c.base_grid, c.base_grid)
    mean = torch.tensor(c.chan_mean, dtype=torch.float64, device="cuda").view(1, -1, 1, 1)
    std = torch.tensor(c.chan_std, dtype=torch.float64, device="cuda").view(1, -1, 1, 1)
    toks, o, P = [], 0, c.patch
    w = p["patch_w"].reshape(D, -1)
    for h, wd in sizes:
        n = c.channels * h * wd
        img = (pixels[o:o + n].double().reshape(1, c.channels, h, wd) - mean) / std
        o += n
        gh, gw = h // P, wd // P
        t = F.linear(F.unfold(img[..., :gh * P, :gw * P], P, stride=P)[0].T, w, p["patch_b"])
        g = grid if (gh, gw) == (c.base_grid,) * 2 else F.interpolate(
            grid, size=(gh, gw), mode="bilinear", align_corners=False)
        toks.append(torch.cat([(p["cls"] + pos[0])[None], t + g[0].reshape(D, -1).T]))
    lens = [len(t) for t in toks]
    x = _blocks(torch.cat(toks), lens, p, c, False)
    start = torch.tensor([0] + lens[:-1], device="cuda").cumsum(0)
    return _head(x, start, p, c)


def _loss64(e, t, head, scale, bias):
    l = scale * e @ t.T.contiguous() + bias
    if head == "softmax":
        i = torch.arange(len(l), device=l.device)
        return 0.5 * (F.cross_entropy(l, i) + F.cross_entropy(l.T, i))
    z = 2.0 * torch.eye(len(l), dtype=l.dtype, device=l.device) - 1.0
    return -F.logsigmoid(z * l).sum() / len(l)


def exact(case, seed):
    kind = case["kind"]
    if kind == "encode":
        c, sizes = _tower(case), _sizes(case)
        p = _split_blob(c, _weights(c, seed), case["precision"])
        with torch.no_grad():
            return _encode64(c, p, _pixels(c, sizes, seed), sizes)
    if kind == "text":
        c, lens = _text_tower(case), _prompt_lengths(case)
        p = _split_blob(c, _weights(c, seed, True), case["precision"], True)
        ids = _ids(case, seed).long()
        place = torch.cat([torch.arange(n) for n in lens]).cuda()
        with torch.no_grad():
            x = _blocks(p["tok"][ids] + p["pos"][place], lens, p, c, True)
            return _head(x, torch.tensor(lens, device="cuda").cumsum(0) - 1, p, c)
    if kind == "train":
        c, sizes = _tower(case), _sizes(case)
        p = _split_blob(c, _weights(c, seed), case["precision"])
        for w in p.values():
            w.requires_grad_()
        emb = _encode64(c, p, _pixels(c, sizes, seed), sizes)
        sb = torch.tensor(_loss_constants("sigmoid"), dtype=torch.float64, device="cuda",
                          requires_grad=True)
        t = _unit(case["images"], c.proj_dim, seed, 4).double().requires_grad_()
        loss = _loss64(emb, t, "sigmoid", sb[0], sb[1])
        loss.backward()
        return {"emb": emb.detach(), "loss": loss.detach()[None], "d_texts": t.grad,
                "d_scale_bias": sb.grad,
                "grads": torch.cat([p[n].grad.reshape(-1) for n, _ in _layout(c)])}
    if kind == "attention":
        with torch.no_grad():
            return _packed_attention(_qkv(case, seed).double(), _lengths(case), case["heads"],
                                     case["causal"])
    if kind == "attention_backward":
        qkv = _qkv(case, seed).double().requires_grad_()
        out = _packed_attention(qkv, _lengths(case), case["heads"], False)
        out.backward(_d_out(case, seed).double())
        return qkv.grad
    scale, bias = _loss_constants(case["head"])
    if kind == "contrastive":
        e, t = (x.double().requires_grad_() for x in _pairs(case["n"], case["dim"], seed))
        sb = torch.tensor((scale, bias), dtype=torch.float64, device="cuda", requires_grad=True)
        loss = _loss64(e, t, case["head"], sb[0], sb[1])
        loss.backward()
        if case["head"] == "softmax":       # the bias cancels: its gradient is 0 by definition
            sb.grad[1] = 0.0
        return {"loss": loss.detach()[None], "d_emb": e.grad, "d_texts": t.grad,
                "d_scale_bias": sb.grad}
    e = _unit(case["n"], case["dim"], seed, 5).double()
    t = _unit(case["texts"], case["dim"], seed, 4).double()
    l = scale * e @ t.T.contiguous() + bias
    s = torch.softmax(l, 1) if case["head"] == "softmax" else torch.sigmoid(l)
    return {"scores": s, "top1": None}
