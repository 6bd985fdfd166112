"""Workloads that a control program runs, through the public entry points.

A program that drives a robot with a gated KV cache makes one of a few calls
per camera frame: the patch selection alone, a control step with token-by-token
decode, a prompt pass that feeds an action chunk, a step of several episodes
at once, or any of them behind the vision encoder.  The listed cases are these
calls at this repository's own shapes (the 7B shape mostly as a slice of a few
layers, so that a case stands for a layer's work and its tolerance is a
layer's); `draw` gives others of the same ranges.

Tokens that are fed back are given (a recorded action sequence is replayed):
two implementations whose logits differ by a rounding would otherwise part at
the first near-tie and could not be compared; the work is the same.  The
tokens themselves are the argmax of the logits that a case returns.
"""
import math
from fractions import Fraction

import numpy as np
import torch

from paper_2608_10824_amd import gvc
from paper_2608_10824_amd.session import Session, desc_from
from synth.configs import VLAConfig

def _case(kind, **kw):
    c = dict(kind=kind, batch=1, layers=2, d=4096, heads=32, ffn=11008, vocab=32000, bins=256, img=224, patch=14,
             views=1, text=20, proprio=0, chunk=0, bidir=False, decode=1, static_pct=50, spread_pct=0, full=False,
             decay=False, signals=False, min_margin=False, vit_layers=0, vit_dim=0, vit_heads=0, vit_ffn=0)
    c.update(kw)
    return c


def listed():
    return [
        # the patch selection by itself, as a program calls it per frame to decide whether to step at all
        _case("select", name="select_1x224", layers=32, static_pct=60, decay=True),
        # the smallest control step: a two-layer decoder of width 256, everything is launches and latency
        _case("step", name="tiny_step", layers=2, d=256, heads=4, ffn=688, vocab=1024, img=112, text=8, decode=7,
              static_pct=70),
        # the headline: one control step of the whole 7B decoder at 50% reuse, 7 tokens decoded one by one
        _case("step", name="step_7b_50", layers=32, decode=7, static_pct=50),
        # 7B layers, prompt pass at 50% reuse (148 of 276 rows) that ends in one token
        _case("step", name="prompt_7b_148", layers=4, static_pct=50),
        # 7B layers, the step after the gate fired (all 276 rows), recording the instruction attention for the
        # task-relevance and entropy selections of the next step
        _case("step", name="prompt_7b_276_signals", layers=4, full=True, signals=True),
        # 7B layers, OFT action chunk: two cameras, 56 action queries decoded in parallel, 60% of 512 patches reused
        _case("step", name="chunk_7b_282", layers=4, views=2, proprio=1, chunk=56, bidir=True, decode=56,
              static_pct=60, min_margin=True),
        # the same query after the gate fired: all 589 rows, causal action rows
        _case("step", name="chunk_7b_589", layers=4, views=2, proprio=1, chunk=56, decode=56, full=True,
              min_margin=True),
        # three robots in one process, each with its own amount of motion, reuse falling with depth
        _case("step", name="batch3_7b_ragged", layers=4, batch=3, decode=7, static_pct=55, spread_pct=35, decay=True),
        # sixteen episodes (evaluation, data collection): the prompt pass at 50% reuse, 2368 rows
        _case("step", name="batch16_7b_prompt", layers=2, batch=16, static_pct=50),
        # sixteen slow scenes: 90% reuse, so the 7-token decode is most of the step
        _case("step", name="batch16_7b_decode", layers=4, batch=16, decode=7, static_pct=90),
        # the ViT-L/14 encoder and projector in front of two 7B layers
        _case("step", name="vit_l14_7b", layers=2, static_pct=50, vit_layers=24, vit_dim=1024, vit_heads=16,
              vit_ffn=4096),
        # a mid-size decoder with head dimension 128 and a ragged FFN, two small cameras, 5-token decode
        _case("step", name="mid_step", layers=6, d=2048, heads=16, ffn=5504, vocab=4096, img=112, views=2, text=9,
              decode=5, static_pct=40),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["select", "step", "step", "step", "step"])
    patch = rng.choice([8, 14, 14, 16])
    side = rng.randint(4, 16)
    views = rng.choice([1, 1, 1, 2])
    dh = rng.choice([64, 128, 128])
    heads = max(2, round(_log(rng, 256, 4096) / dh))
    d = heads * dh
    ffn = 16 * max(4, round(d * rng.uniform(2.0, 3.6) / 16))
    batch = rng.choice([1, 1, 1, 2, 3, 5, 8, 13, 16])
    text = rng.randint(2, 32)
    c = _case(kind, batch=batch, layers=rng.randint(1, 4), d=d, heads=heads, ffn=ffn, vocab=16 * round(_log(rng, 64, 2000)),
              img=side * patch, patch=patch, views=views, text=text, static_pct=rng.randint(0, 95),
              spread_pct=rng.choice([0, 0, 15, 40]), decay=rng.random() < 0.3, full=rng.random() < 0.2,
              decode=rng.randint(1, 8))
    if kind == "select":
        c.update(layers=rng.randint(1, 40), decode=1)
        return c
    if rng.random() < 0.25:    # an action chunk in place of the token-by-token decode
        n = rng.randint(4, 56)
        c.update(chunk=n, decode=n, proprio=rng.randint(0, 2), bidir=rng.random() < 0.5, min_margin=True)
    elif views * side * side + text < 640 and rng.random() < 0.2:
        c["signals"] = True
    if rng.random() < 0.2:
        vh = rng.choice([2, 4, 6, 8, 12, 16])
        c.update(vit_layers=rng.randint(1, 12), vit_dim=64 * vh, vit_heads=vh, vit_ffn=32 * rng.randint(2 * vh, 8 * vh))
    return c


# ------------------------------------------------------------------ sizes

def _patches(c):
    return c["views"] * (c["img"] // c["patch"]) ** 2


def _prompt(c):
    return _patches(c) + c["text"] + c["proprio"] + c["chunk"]


def _statics(c):
    """Static patches of each episode: static_pct of them, spread_pct up and down over the episodes."""
    N, B = _patches(c), c["batch"]
    out = []
    for b in range(B):
        off = 0.0 if B == 1 else c["spread_pct"] * (2.0 * b / (B - 1) - 1.0)
        out.append(int(N * min(98.0, max(0.0, c["static_pct"] + off)) / 100.0))
    return out


def _permille(c):
    """Reuse proportion per layer: everything, or falling from 800 to 200 per mille with depth."""
    L = c["layers"]
    return [800 - (600 * l) // max(1, L - 1) for l in range(L)] if c["decay"] else [1000] * L


def _config(c):
    return VLAConfig(name=c.get("name", "case"), batch=c["batch"], n_layers=c["layers"], d_model=c["d"],
                     n_heads=c["heads"], ffn=c["ffn"], vocab=c["vocab"], n_bins=c["bins"], img=c["img"],
                     patch=c["patch"], n_views=c["views"], n_text=c["text"], n_proprio=c["proprio"],
                     n_action_q=c["chunk"], n_decode=c["decode"], parallel_decode=c["chunk"] > 0,
                     reduce_min=c["min_margin"], reuse_permille=_permille(c), entropy_reuse=c["signals"],
                     task_topk=_patches(c) // 2 if c["signals"] else 0, action_bidir=c["bidir"],
                     vit_layers=c["vit_layers"], vit_dim=c["vit_dim"] or 1024, vit_heads=c["vit_heads"] or 16,
                     vit_ffn=c["vit_ffn"] or 4096)


# ------------------------------------------------------------------ inputs

def _weights(c, seed):
    """bf16 weights, normal with standard deviation 1/sqrt(fan in); the action-bin rows of the head are larger, so
    that the margins spread as a trained policy's do."""
    dev = "cuda"
    g = torch.Generator(device=dev)
    g.manual_seed(seed * 2 + 1)

    def mat(n, k, std=None):
        w = torch.empty(n, k, dtype=torch.bfloat16, device=dev)
        return w.normal_(0.0, std or 1.0 / math.sqrt(k), generator=g)

    def vec(n, mean):
        return torch.empty(n, dtype=torch.float32, device=dev).uniform_(mean - 0.06, mean + 0.06,
                                                                        generator=g).bfloat16()

    d, F, V = c["d"], c["ffn"], c["vocab"]
    pd = c["patch"] ** 2 * 3
    lm = mat(V, d)
    lm[V - c["bins"]:] = mat(c["bins"], d, 6.0 / math.sqrt(d))
    w = {"embed": mat(V, d, 0.5), "patch_proj": mat(d, pd), "lm_head": lm, "final_norm": vec(d, 1.0), "layers": []}
    for _ in range(c["layers"]):
        w["layers"].append({"wq": mat(d, d), "wk": mat(d, d), "wv": mat(d, d), "wo": mat(d, d), "wg": mat(F, d),
                            "wu": mat(F, d), "wd": mat(d, F), "attn_norm": vec(d, 1.0), "ffn_norm": vec(d, 1.0)})
    if c["vit_layers"]:
        D, Fv, S = c["vit_dim"], c["vit_ffn"], (c["img"] // c["patch"]) ** 2
        v = {"patch_w": mat(D, pd), "patch_b": vec(D, 0.0), "pos": mat(S, D, 0.3), "post_g": vec(D, 1.0),
             "post_b": vec(D, 0.0), "proj1": mat(d, D), "proj1_b": vec(d, 0.0), "proj2": mat(d, d),
             "proj2_b": vec(d, 0.0), "layers": []}
        for _ in range(c["vit_layers"]):
            v["layers"].append({"ln1_g": vec(D, 1.0), "ln1_b": vec(D, 0.0), "wq": mat(D, D), "bq": vec(D, 0.0),
                                "wk": mat(D, D), "bk": vec(D, 0.0), "wv": mat(D, D), "bv": vec(D, 0.0),
                                "wo": mat(D, D), "bo": vec(D, 0.0), "ln2_g": vec(D, 1.0), "ln2_b": vec(D, 0.0),
                                "w1": mat(Fv, D), "b1": vec(Fv, 0.0), "w2": mat(D, Fv), "b2": vec(D, 0.0)})
        w["vit"] = v
    return w


def _inputs(c, seed):
    """Two consecutive frames per episode: the static patches differ by the sensor's noise (0 or 1 per value in a
    few per cent of the values, so their cosines are all different), the others by their content."""
    dev = "cuda"
    g = torch.Generator(device=dev)
    g.manual_seed(seed * 2)
    B, V, img, p = c["batch"], c["views"], c["img"], c["patch"]
    side, N = img // p, _patches(c)
    prev = torch.randint(0, 255, (B, V, img, img, 3), generator=g, device=dev, dtype=torch.uint8)
    fresh = torch.randint(0, 255, (B, V, img, img, 3), generator=g, device=dev, dtype=torch.uint8)
    noise = (torch.rand((B, V, img, img, 3), generator=g, device=dev) < 0.04).to(torch.uint8)
    order = torch.rand((B, N), generator=g, device=dev).argsort(dim=1).argsort(dim=1)
    k = torch.tensor(_statics(c), device=dev)
    static = order < k[:, None]
    per_pixel = static.view(B, V, side, 1, side, 1).expand(B, V, side, p, side, p).reshape(B, V, img, img, 1)
    cur = torch.where(per_pixel, prev + noise, fresh)
    ids = torch.randint(0, c["vocab"] - c["bins"], (B, c["text"]), generator=g, device=dev, dtype=torch.int32)
    n_extra = c["proprio"] + c["chunk"]
    extra = torch.randn((B, n_extra, c["d"]), generator=g, device=dev) * 0.5 if n_extra else None
    fed = torch.randint(c["vocab"] - c["bins"], c["vocab"], (B, c["decode"]), generator=g, device=dev,
                        dtype=torch.int32)
    return {"prev": prev.contiguous(), "cur": cur.contiguous(), "ids": ids, "extra": extra, "fed": fed}


TAU = (249, 250)


def _margins_compare(c):
    """A margin is the difference of two probabilities: near a tie its relative error is anything, so one is only
    returned among at least five (and the smallest, which the gate of a chunk takes, never by itself)."""
    return c["batch"] * c["decode"] >= 5


def prepare(case, seed):
    c = case
    x = _inputs(c, seed)
    if c["kind"] == "select":
        cfg = _config(dict(c, chunk=0, proprio=0))
        B, L, N = c["batch"], c["layers"], _patches(c)
        return {"c": c, "x": x, "desc": desc_from(cfg), "q": _permille(c),
                "mask": torch.zeros(B, L, N, dtype=torch.uint8, device="cuda"),
                "n": torch.zeros(B, dtype=torch.int32, device="cuda"),
                "stream": torch.cuda.current_stream().cuda_stream}
    s = Session(_config(c), _weights(c, seed))
    st = {"c": c, "x": x, "s": s, "fed": None if c["chunk"] else x["fed"]}
    # the step before: a full pass over the previous frame fills the cache
    s.step_prefill(x["prev"], x["ids"], x["extra"])
    s.decode_actions(forced_tokens=st["fed"])
    s.margin_gate(force=[0] * c["batch"])
    return st


def run(state):
    c, x = state["c"], state["x"]
    if c["kind"] == "select":
        gvc.select_static_noalloc(state["desc"], x["cur"].data_ptr(), x["prev"].data_ptr(), TAU[0], TAU[1], state["q"],
                                  state["mask"].data_ptr(), state["n"].data_ptr(), state["stream"])
        return {"mask": state["mask"], "n_static": state["n"]}
    s = state["s"]
    out = {}
    mask = None
    if not c["full"] and not c["signals"]:   # (with the signals on, the selection is whole numbers decided on float sums)
        out["mask"], out["n_static"] = s.select_static(x["cur"], x["prev"], TAU)
        mask = out["mask"]
    s.step_prefill(x["cur"], x["ids"], x["extra"], mask)
    _, margins, out["logits"] = s.decode_actions(logits=True, forced_tokens=state["fed"])
    gate, _ = s.margin_gate(force=[0] * c["batch"])
    if _margins_compare(c):
        out["margins"] = margins
        if not c["min_margin"]:
            out["gate"] = np.array(gate)
    if c["decode"] == 1 or c["chunk"]:
        # the hidden states of every token after the last layer, as a program reads them for another head
        out["hidden"] = s.read(gvc.STATE_H, c["layers"])
    if c["signals"]:
        out["attention"] = s.read(gvc.STATE_TV)
        out["entropy"] = s.read(gvc.STATE_ENTROPY)
    return out


# ------------------------------------------------------------------ work

def _rows(c):
    """Rows recomputed per layer, summed over the episodes."""
    P, B = _prompt(c), c["batch"]
    if c["full"] or c["signals"]:
        return [B * P] * c["layers"]
    return [sum(P - q * k // 1000 for k in _statics(c)) for q in _permille(c)]


def work(case):
    c = case
    B, N, P, d, F, V, L = c["batch"], _patches(c), _prompt(c), c["d"], c["ffn"], c["vocab"], c["layers"]
    frame = B * c["views"] * c["img"] ** 2 * 3
    if c["kind"] == "select":
        return {"bytes": 2 * frame + B * L * N + 4 * B, "flops": 6 * frame}
    layer = 4 * d * d + 3 * d * F
    rows = _rows(c)
    head_rows = B * (c["chunk"] or 1)
    pd = c["patch"] ** 2 * 3
    # prompt pass: the weights once, each recomputed row's hidden state in and out and its keys and values, the
    # keys and values of the others, the logits
    by = 2 * (L * layer + V * d) + 2 * frame + sum(8 * r * d + 4 * r * d + 4 * (B * P - r) * d for r in rows) \
        + 4 * head_rows * V
    fl = sum(2 * r * layer + 4 * r * (P / 2) * d for r in rows) + 2 * head_rows * V * d
    if c["vit_layers"]:
        D, Fv, S = c["vit_dim"], c["vit_ffn"], N // c["views"]
        wv = c["vit_layers"] * (4 * D * D + 2 * D * Fv) + pd * D + D * d
        by += 2 * (wv + d * d)
        fl += 2 * B * N * wv + 4 * c["vit_layers"] * B * N * S * D + 2 * rows[0] * d * d
    else:
        by += 2 * pd * d
        fl += 2 * rows[0] * pd * d
    if not c["chunk"]:
        # each decode pass: the weights and the head once, every episode's keys and values, the logits
        for j in range(1, c["decode"]):
            by += 2 * (L * layer + V * d) + 4 * L * B * (P + j) * d + 4 * B * V
            fl += 2 * B * (L * layer + V * d) + 4 * L * B * (P + j) * d
    return {"bytes": by, "flops": fl}


def tolerance(case):
    if case["kind"] == "select":
        return "exact"
    # bf16 operands and caches: a rounding that falls the other way is 2^-9 of a value and travels through the
    # layers that follow.  With every projection's sum over k cut in other places, hidden states measured 0.002
    # apart, attention 0.002, logits 0.003 to 0.004 (0.07 of their root mean square at most) and margins, which are
    # differences of probabilities, up to 0.017.
    return {"rel": 0.03 if _margins_compare(case) else 0.012, "max": 0.3}


# ------------------------------------------------------------------ the same in 64 bits

def _patch_rows(c, frame):
    """[B][N][p*p*3] values of a frame's patches, view-major, raster, each in H, W, C order."""
    B, V, img, p = c["batch"], c["views"], c["img"], c["patch"]
    s = img // p
    return frame.view(B, V, s, p, s, p, 3).permute(0, 1, 2, 4, 3, 5, 6).reshape(B, V * s * s, p * p * 3)


def _exact_masks(c, x):
    """mask [B][L][N] and the static counts, in whole numbers."""
    u, v = _patch_rows(c, x["cur"]).long().cpu(), _patch_rows(c, x["prev"]).long().cpu()
    dot, uu, vv = (u * v).sum(-1).tolist(), (u * u).sum(-1).tolist(), (v * v).sum(-1).tolist()
    B, N, L = c["batch"], _patches(c), c["layers"]
    mask, counts = torch.zeros(B, L, N, dtype=torch.uint8), []
    for b in range(B):
        cos2 = [Fraction(a * a, q * r) if q and r else Fraction(int(not q and not r))
                for a, q, r in zip(dot[b], uu[b], vv[b])]
        ranked = sorted((n for n in range(N) if cos2[n] > Fraction(TAU[0] ** 2, TAU[1] ** 2)),
                        key=lambda n: (-cos2[n], n))
        counts.append(len(ranked))
        for l, q in enumerate(_permille(c)):
            mask[b, l, ranked[: q * len(ranked) // 1000]] = 1
    return mask, torch.tensor(counts, dtype=torch.int32)


def _gelu(x):
    return 0.5 * x * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (x + 0.044715 * x ** 3)))


def _softmax_attend(q, k, v, last):
    """q [H][M][e], k and v [H][K][e]; row m sees keys 0..last[m]."""
    sc = q @ k.transpose(1, 2).contiguous() / math.sqrt(q.shape[-1])
    sc.masked_fill_(torch.arange(k.shape[1], device=q.device)[None, :] > last[:, None], -math.inf)
    p = torch.softmax(sc, dim=-1)
    return p @ v, p


def _exact_vision(c, w, frame):
    """[B][N][d] embeddings of the visual tokens."""
    f = _patch_rows(c, frame).double() / 255.0
    if not c["vit_layers"]:
        return f @ w["patch_proj"].double().t()
    vw = w["vit"]
    B, N, D, H = c["batch"], _patches(c), c["vit_dim"], c["vit_heads"]
    S, e = N // c["views"], D // H
    eps = _config(c).vit_eps

    def ln(h, g, b):
        m = h.mean(-1, keepdim=True)
        return (h - m) / torch.sqrt(((h - m) ** 2).mean(-1, keepdim=True) + eps) * g.double() + b.double()

    def lin(h, a, b):
        return h @ a.double().t() + b.double()

    h = lin(f.reshape(B * c["views"], S, -1), vw["patch_w"], vw["patch_b"]) + vw["pos"].double()
    last = torch.full((S,), S - 1, device=h.device)
    for lw in vw["layers"]:
        y = ln(h, lw["ln1_g"], lw["ln1_b"])
        q, k, v = (lin(y, lw["w" + i], lw["b" + i]) for i in "qkv")
        split = lambda t: t.view(S, H, e).transpose(0, 1).contiguous()  # noqa: E731
        o = torch.stack([_softmax_attend(split(q[i]), split(k[i]), split(v[i]), last)[0].transpose(0, 1).reshape(S, D)
                         for i in range(h.shape[0])])
        h = h + lin(o, lw["wo"], lw["bo"])
        h = h + lin(_gelu(lin(ln(h, lw["ln2_g"], lw["ln2_b"]), lw["w1"], lw["b1"])), lw["w2"], lw["b2"])
    h = ln(h, vw["post_g"], vw["post_b"])
    return lin(_gelu(lin(h, vw["proj1"], vw["proj1_b"])), vw["proj2"], vw["proj2_b"]).reshape(B, N, -1)


def exact(case, seed):
    """One step after a full pass over the previous frame.  The fed-back tokens are rows after the prompt, so the
    decode is the rest of one causal pass."""
    c = case
    x = _inputs(c, seed)
    if c["kind"] == "select":
        mask, n = _exact_masks(c, x)
        return {"mask": mask, "n_static": n}
    w = _weights(c, seed)
    cfg = _config(c)
    B, N, P, L, d, H = c["batch"], _patches(c), _prompt(c), c["layers"], c["d"], c["heads"]
    e = d // H
    D = 0 if c["chunk"] else c["decode"] - 1
    T = P + D
    dev = "cuda"
    out = {}
    reused = torch.zeros(B, L, T, dtype=torch.bool, device=dev)
    if not c["full"] and not c["signals"]:
        out["mask"], out["n_static"] = _exact_masks(c, x)
        reused[:, :, 1:N + 1] = out["mask"].to(dev).bool()
    emb = w["embed"].double()

    def embed(frame):
        h = torch.empty(B, T, d, dtype=torch.float64, device=dev)
        h[:, 1:N + 1] = _exact_vision(c, w, frame)
        t = emb[x["ids"].long()]
        h[:, 0], h[:, N + 1:N + c["text"]] = t[:, 0], t[:, 1:]
        if x["extra"] is not None:
            h[:, N + c["text"]:P] = x["extra"].double()
        if D:
            h[:, P:] = emb[x["fed"][:, :D].long()]
        return h

    def rms(h, g):
        return h / torch.sqrt((h * h).mean(-1, keepdim=True) + cfg.rms_eps) * g.double()

    pos = torch.arange(T, device=dev)
    ang = pos[:, None].double() * cfg.rope_theta ** (-torch.arange(0, e, 2, device=dev).double() / e)
    cos, sin = ang.cos(), ang.sin()

    def rope(t, rows):   # [M][H][e]
        a, b = t[..., : e // 2], t[..., e // 2:]
        cs, sn = cos[rows][:, None], sin[rows][:, None]
        return torch.cat([a * cs - b * sn, b * cs + a * sn], dim=-1)

    last = pos.clone()
    if c["bidir"]:
        last[P - c["chunk"]:P] = P - 1
    before, now = embed(x["prev"]), embed(x["cur"])
    if not c["full"] and not c["signals"]:
        now = torch.where(reused[:, 0, :, None], before, now)
    if c["signals"]:
        out["attention"] = torch.zeros(B, L, H, N, dtype=torch.float64, device=dev)
        out["entropy"] = torch.zeros(B, L, H, dtype=torch.float64, device=dev)
    for l, lw in enumerate(w["layers"]):
        W = {k: t.double() for k, t in lw.items()}
        nb, nn = torch.empty_like(before), torch.empty_like(now)
        for b in range(B):
            kept = None
            for h, o, fresh in ((before[b], nb[b], None), (now[b], nn[b], ~reused[b, l])):
                rows = pos if fresh is None else pos[fresh]
                hr = h[rows]
                y = rms(hr, W["attn_norm"])
                q, k, v = (y @ W[i].t() for i in ("wq", "wk", "wv"))
                q, k, v = rope(q.view(-1, H, e), rows), rope(k.view(-1, H, e), rows), v.view(-1, H, e)
                if fresh is None:
                    kept = (k, v)
                else:
                    k, v = kept[0].index_copy(0, rows, k), kept[1].index_copy(0, rows, v)
                a, pr = _softmax_attend(q.transpose(0, 1).contiguous(), k.transpose(0, 1).contiguous(),
                                        v.transpose(0, 1).contiguous(), last[rows])
                if c["signals"] and fresh is not None:
                    instr = pr[:, N + 1:N + c["text"]]
                    out["attention"][b, l] = instr[:, :, 1:N + 1].sum(1)
                    ent = -(torch.where(instr > 0, instr * instr.clamp_min(1e-300).log(), instr)).sum(-1)
                    out["entropy"][b, l] = (ent / torch.arange(N + 2, N + c["text"] + 1, device=dev).double().log()).sum(-1)
                r = hr + a.transpose(0, 1).reshape(-1, d) @ W["wo"].t()
                y = rms(r, W["ffn_norm"])
                g = y @ W["wg"].t()
                z = r + (g * torch.sigmoid(g) * (y @ W["wu"].t())) @ W["wd"].t()
                if fresh is None:
                    o[:] = z
                else:
                    o[:] = nb[b]
                    o[rows] = z
        before, now = nb, nn
    heads = now[:, P - c["chunk"]:P] if c["chunk"] else now[:, P - 1:P + D]
    lg = rms(heads, w["final_norm"]) @ w["lm_head"].double().t()
    top = torch.softmax(lg, dim=-1)[..., c["vocab"] - c["bins"]:].topk(2, dim=-1).values
    out["logits"] = lg
    if _margins_compare(c):
        out["margins"] = top[..., 0] - top[..., 1]
        if not c["min_margin"]:
            out["gate"] = out["margins"].mean(-1)
    if c["decode"] == 1 or c["chunk"]:
        out["hidden"] = now[:, :P].contiguous()
    return out
