"""Timing cases of the segmented training path, through its public entry points.

Five kinds of work, each a call sequence of a training program:

- ``layout``: size and build the packed layout of a batch (every batch does it);
- ``attn``: the segmented attention forward and, with ``grad``, its backward;
- ``logprob``: the fused log-prob and clipped-ratio loss of the action rows,
  with gradients (``grad``) or as the forward-only reference pass;
- ``layer``: one decoder layer forward and backward;
- ``step``: a whole policy-update step (layout, attention forward, loss with
  gradients, attention backward).

A case fixes the batch geometry (its span lists come from ``spans``, a seed
that is part of the case); the seed given to ``prepare`` draws the values.
Only the layout cases let that seed move the text lengths, between turns of
one segment, so that every array keeps its size.
"""
import math

import numpy as np
import torch

from paper_2607_11185_amd import seg as S
from paper_2607_11185_amd import workload as WL

DEV = "cuda"
IMAGE, TEXT = WL.KIND_IMAGE, WL.KIND_TEXT


def _geo(traj, turns, prompt, img, text, action, window, seg_steps, mode="sliding", max_seg=0,
         buffer=0, spans=0):
    return dict(traj=traj, turns_lo=turns[0], turns_hi=turns[1], prompt=prompt, img=img,
                text_lo=text[0], text_hi=text[1], action=action, window=window,
                seg_steps=seg_steps, mode=mode, max_seg=max_seg, buffer=buffer, spans=spans)


def _of(cfg, **kw):
    """Geometry of one of the repository's workloads."""
    g = _geo(cfg.num_traj, cfg.steps, cfg.prompt_len, cfg.img_len, cfg.text_len, cfg.action_len,
             cfg.window, cfg.seg_steps, cfg.mode, cfg.max_seg_tokens, cfg.buffer_tokens)
    g.update(kw)
    return g


def _heads(cfg):
    return dict(hq=cfg.hq, hkv=cfg.hkv, d=cfg.head_dim)


def listed():
    return [
        # the smallest attention call, fp32 tensors: latency and launches count
        dict(name="attn_tiny_f32", kind="attn", **_of(WL.TINY), **_heads(WL.TINY), dtype="f32",
             grad=True, kscale=1.0),
        # every batch builds its layout: host plan, upload and a few small kernels
        dict(name="layout_7b", kind="layout", **_of(WL.SEVEN_B)),
        # an ordinary batch of short trajectories, GQA 8:1: the chip is filled
        # only a few times over
        dict(name="attn_small", kind="attn", **_of(WL.SMALL), **_heads(WL.SMALL), dtype="bf16",
             grad=True, kscale=1.0),
        # head dimension 64, ragged turn counts, buffers with padded tails
        dict(name="attn_d64_buffers", kind="attn",
             **_geo(6, (5, 25), 100, 1000, (20, 333), 17, 4, 6, max_seg=16384, buffer=16384),
             hq=12, hkv=4, d=64, dtype="bf16", grad=True, kscale=1.0),
        # the reference-policy forward over the anchored segments of one long
        # trajectory, keys of large norm (peaked scores)
        dict(name="attn_ref_anchored", kind="attn", **_of(WL.SEVEN_B_ANCHORED, traj=1),
             **_heads(WL.SEVEN_B), dtype="bf16", grad=False, kscale=6.0),
        # the smallest loss call, fp32 tensors
        dict(name="logprob_tiny_f32", kind="logprob", rows=64, hidden=128, vocab=1024, dtype="f32",
             grad=True, kl=0.0, dual=0.0),
        # the loss of a small batch: the dH product has few output tiles and a
        # long contraction over the vocabulary
        dict(name="logprob_small", kind="logprob", rows=1024, hidden=2048, vocab=32000,
             dtype="bf16", grad=True, kl=0.0, dual=3.0),
        # the loss of the 7B-class batch with the KL penalty
        dict(name="logprob_7b", kind="logprob", rows=7680, hidden=3584, vocab=151936, dtype="bf16",
             grad=True, kl=1e-4, dual=3.0),
        # forward-only log-probs on one tensor-parallel rank's vocabulary shard
        dict(name="logprob_ref_shard", kind="logprob", rows=7680, hidden=3584, vocab=37984,
             dtype="bf16", grad=False, kl=0.0, dual=0.0),
        # a decoder layer at the small width, one short trajectory
        dict(name="layer_small", kind="layer", **_of(WL.SMALL, traj=1), **_heads(WL.SMALL),
             hidden=2048, inter=5504),
        # a decoder layer at the 7B-class width, one trajectory as a micro-batch
        dict(name="layer_7b", kind="layer", **_of(WL.SEVEN_B, traj=1), **_heads(WL.SEVEN_B),
             hidden=3584, inter=18944),
        # the whole policy-update step of the benchmark's batch
        dict(name="step_7b", kind="step", **_of(WL.SEVEN_B), **_heads(WL.SEVEN_B), hidden=3584,
             vocab=151936, kl=1e-4, dual=0.0),
    ]


HEADS = [(4, 1, 64), (8, 8, 64), (12, 4, 64), (16, 2, 128), (28, 4, 128), (7, 1, 128), (6, 6, 128)]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_geo(rng, most_rows):
    """A random batch whose segments hold at most about `most_rows` rows."""
    lo = rng.randint(2, 20)
    g = _geo(rng.randint(1, 6), (lo, lo + rng.randint(0, 15)), rng.choice([0, rng.randint(1, 600)]),
             _log(rng, 30, 4096), (16, 16 + _log(rng, 8, 500)), rng.randint(1, 16),
             rng.randint(1, 8), rng.randint(1, 10), rng.choice(["sliding", "sliding", "anchored"]),
             spans=rng.randrange(1 << 20))
    while sum(s["len"] for s in _segments(g)) > most_rows:
        if g["traj"] > 1:
            g["traj"] -= 1
        elif g["turns_hi"] > 4 and g["turns_hi"] * 100 > g["img"]:
            g["turns_lo"], g["turns_hi"] = 2, max(4, g["turns_hi"] * 2 // 3)
        elif g["img"] > 30:
            g["img"] = max(30, int(g["img"] * 0.7))
        elif g["text_hi"] > 40:
            g["text_hi"] = max(40, int(g["text_hi"] * 0.7))
        else:
            g["prompt"] = 0
            break
    if g["mode"] == "sliding" and rng.random() < 0.3:
        g["buffer"] = max(s["len"] for s in _segments(g)) + rng.randint(0, 3000)
    return g


def draw(rng):
    kind = rng.choice(["attn"] * 4 + ["logprob"] * 3 + ["layer"] * 3 + ["layout"] * 2)
    if kind == "layout":
        g = _draw_geo(rng, 2000000)
        g["seg_steps"], g["buffer"] = max(3, g["seg_steps"]), 0
        return dict(kind=kind, **g)
    if kind == "attn":
        g = _draw_geo(rng, _log(rng, 500, 150000))
        hq, hkv, d = rng.choice(HEADS)
        return dict(kind=kind, **g, hq=hq, hkv=hkv, d=d,
                    dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]), grad=rng.random() < 0.75,
                    kscale=rng.choice([1.0, 1.0, 6.0]))
    if kind == "logprob":
        c = dict(kind=kind, rows=_log(rng, 16, 8192), hidden=8 * _log(rng, 16, 512),
                 vocab=_log(rng, 1000, 152064), dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]),
                 grad=rng.random() < 0.75, kl=rng.choice([0.0, 1e-4]), dual=rng.choice([0.0, 3.0]))
        return c
    g = _draw_geo(rng, _log(rng, 500, 40000))
    hq, hkv, d = rng.choice(HEADS)
    hidden = 8 * _log(rng, 32, 448)
    return dict(kind="layer", **g, hq=hq, hkv=hkv, d=d, hidden=hidden,
                inter=8 * int(hidden * rng.uniform(2.0, 5.3) / 8))


# ------------------------------------------------------------------ geometry

def _spans(c, mix=None):
    """Span lists of a case; `mix` shuffles text lengths within each run of
    seg_steps turns (segment sizes do not change)."""
    rng = np.random.default_rng([c["spans"], 11])
    T = rng.integers(c["turns_lo"], c["turns_hi"] + 1, size=c["traj"])
    n = int(T.sum())
    text = rng.integers(c["text_lo"], c["text_hi"] + 1, size=n)
    off = np.concatenate([[0], np.cumsum(T)])
    if mix is not None:
        rng = np.random.default_rng([mix, 12])
        for t in range(c["traj"]):
            a = int(off[t])
            first = c["window"] + c["seg_steps"] if c["mode"] == "anchored" else c["seg_steps"]
            while a < off[t + 1]:
                b = min(int(off[t + 1]), a + first)
                text[a:b] = rng.permutation(text[a:b])
                a, first = b, c["seg_steps"]
    return WL.Spans(off.astype(np.int32), np.full(c["traj"], c["prompt"], np.int32),
                    np.full(n, c["img"], np.int32), text.astype(np.int32),
                    np.minimum(c["action"], text).astype(np.int32))


def _problem(c, spans):
    return S.Problem.from_spans(spans, c["window"], c["seg_steps"], c["max_seg"], c["buffer"], 128,
                                c["mode"])


def _segments(c):
    """Segments of the batch in packed order: start, len and the runs of
    tokens (turn, kind, length); independent of the library."""
    sp, out, pos, fill, buf = _spans(c), [], 0, 0, 0
    anch = c["mode"] == "anchored"
    keep = c["window"] + 1 if anch else c["window"]
    for t in range(sp.num_traj):
        o = int(sp.step_offsets[t])
        T = int(sp.step_offsets[t + 1]) - o

        def runs(a, b):
            r = [(0, WL.KIND_PROMPT, int(sp.prompt_len[t]))]
            for j in range(1, b):
                if j > a - keep:
                    r.append((j, IMAGE, int(sp.img_len[o + j - 1])))
                r.append((j, TEXT, int(sp.text_len[o + j - 1])))
            return r
        a = 1
        while a <= T:
            b, most = a + 1, c["window"] + c["seg_steps"] if anch and a == 1 else c["seg_steps"]
            while b - a < most and b <= T and not (
                    c["max_seg"] and sum(r[2] for r in runs(a, b + 1)) > c["max_seg"]):
                b += 1
            r = runs(a, b)
            n = sum(x[2] for x in r)
            if c["buffer"]:
                if buf == 0 or fill + n > c["buffer"]:
                    pos, fill, buf = buf * c["buffer"], 0, buf + 1
                fill += n
            out.append(dict(start=pos, len=n, runs=r, a=a, b=b))
            pos += n
            a = b
    return out


def _packed(c, segs):
    if c["buffer"]:
        return -(-(segs[-1]["start"] + segs[-1]["len"]) // c["buffer"]) * c["buffer"]
    return segs[-1]["start"] + segs[-1]["len"]


def _pairs(c, segs):
    """Visible (query, key) pairs per head."""
    total = 0
    for s in segs:
        total += s["len"] * (s["len"] + 1) // 2
        if c["mode"] == "anchored":
            continue
        img = {}
        rows = {}
        for turn, kind, n in s["runs"]:
            rows[turn] = rows.get(turn, 0) + n
            if kind == IMAGE:
                img[turn] = img.get(turn, 0) + n
        for turn, n in rows.items():
            total -= n * sum(m for j, m in img.items() if j <= turn - c["window"])
    return total


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _randn(g, *shape, std=1.0, dtype=torch.bfloat16):
    x = torch.randn(*shape, generator=g, device=DEV, dtype=dtype)
    return x if std == 1.0 else x.mul_(std)


def _attn_inputs(c, seed, P):
    """q, k, v and dO as a projection gives them: unit variance, keys scaled
    by `kscale`."""
    g = _gen(seed)
    dt = torch.float32 if c.get("dtype") == "f32" else torch.bfloat16
    q = _randn(g, P, c["hq"], c["d"], dtype=dt)
    k = _randn(g, P, c["hkv"], c["d"], std=c.get("kscale", 1.0), dtype=dt)
    v = _randn(g, P, c["hkv"], c["d"], dtype=dt)
    do = _randn(g, P, c["hq"], c["d"], dtype=dt) if c.get("grad", True) else None
    return q, k, v, do


def _loss_inputs(c, seed, rows, h_rows, index=None):
    """Hidden states, projection, targets and rollout log-probs: the current
    log-probs (in float32) plus N(0, 0.1) noise."""
    g = _gen(seed + 1000003)
    dt = torch.float32 if c.get("dtype") == "f32" else torch.bfloat16
    h = _randn(g, h_rows, c["hidden"], dtype=dt)
    w = _randn(g, c["vocab"], c["hidden"], std=0.02, dtype=dt)
    tgt = torch.randint(0, c["vocab"], (rows,), generator=g, device=DEV, dtype=torch.int32)
    ntraj = c.get("traj", 8)
    adv = torch.randn(ntraj, generator=g, device=DEV)
    cur = torch.empty(rows, device=DEV)
    wt = w.float().t()
    for a in range(0, rows, 1024):
        b = min(rows, a + 1024)
        hr = (h[a:b] if index is None else h[index[a:b].long()]).float()
        z = torch.log_softmax(hr @ wt, dim=1)
        cur[a:b] = z.gather(1, tgt[a:b].long()[:, None])[:, 0]
        del z
    noise = 0.1 * torch.randn(rows, generator=g, device=DEV)
    traj = torch.arange(rows, device=DEV, dtype=torch.int64).mul_(ntraj).div_(
        rows, rounding_mode="floor").to(torch.int32)
    return dict(h=h, w=w, tgt=tgt, adv=adv, old=cur + noise, ref=cur - noise, traj=traj)


def _loss_cfg(c, rows):
    return S.LossCfg(0.2, 0.28, c["dual"], 1.0 / rows, 1.0, c.get("grad", True), c["kl"])


def _layer_inputs(c, seed, P):
    g = _gen(seed)
    w = {}
    for n, shp in WL.layer_shapes(c["hidden"], c["inter"], c["hq"], c["hkv"], c["d"]).items():
        if len(shp) == 1:
            w[n] = (1 + 0.1 * torch.randn(shp, generator=g, device=DEV)).to(torch.bfloat16)
        else:
            w[n] = _randn(g, *shp, std=1.0 / math.sqrt(shp[1]))
    return w, _randn(g, P, c["hidden"]), _randn(g, P, c["hidden"])


def prepare(case, seed):
    c, kind = case, case["kind"]
    st = {"c": c}
    if kind == "logprob":
        R = c["rows"]
        st.update(_loss_inputs(c, seed, R, R), cfg=_loss_cfg(c, R))
        return st
    if kind == "layout":
        p = st["problem"] = _problem(c, _spans(c, mix=seed))
        # the arrays of the batch before, reused; zeros past the listed tiles
        lay = st["lay"] = S.Layout(S.seg_layout_query(p), torch.device(DEV))
        for f in S.Layout.FIELDS:
            getattr(lay, f).zero_()
        return st
    p = st["problem"] = _problem(c, _spans(c))
    lay = st["lay"] = S.seg_build_layout(p, device=DEV)
    P = lay.sizes.packed_tokens
    if kind == "layer":
        st["cfg"] = S.LayerCfg(c["hidden"], c["inter"], c["hq"], c["hkv"], c["d"])
        st["w"], st["x"], st["dy"] = _layer_inputs(c, seed, P)
        # padding rows of the saved log-sum-exp stay unwritten; y is undefined there
        return st
    st["q"], st["k"], st["v"], st["do"] = _attn_inputs(c, seed, P)
    st["scale"] = 1.0 / math.sqrt(c["d"])
    # output buffers, kept over the steps; padding rows are not written
    st["o"] = torch.zeros_like(st["q"])
    st["lse"] = torch.zeros(c["hq"], P, device=DEV)
    if c.get("grad", True):
        st["dq"], st["dk"], st["dv"] = (torch.zeros_like(st[n]) for n in "qkv")
    if kind == "step":
        R = lay.sizes.loss_rows
        st.update(_loss_inputs(c, seed, R, P, lay.loss_pred_row[:R]))
        st["cfg"] = _loss_cfg(c, R)
    return st


# ------------------------------------------------------------------ the calls

def _run_loss(st, index=None):
    out = S.seg_logprob_loss(st["h"], index, st["w"], st["tgt"], st["old"], st["adv"], st["traj"],
                             st["cfg"], ref_logp=st["ref"])
    names = ["logp", "loss_tok", "clipped", "kl_tok", "loss_sum"]
    return {n: out[n] for n in names + (["dh", "dw"] if st["cfg"].want_grad else [])}


def run(st):
    c = st["c"]
    kind = c["kind"]
    if kind == "logprob":
        return _run_loss(st)
    if kind == "layout":
        sz = S.seg_layout_query(st["problem"])
        lay = S.seg_build_layout(st["problem"], sz, DEV, out=st["lay"])
        r = {f: getattr(lay, f) for f in S.Layout.FIELDS}
        r["xcd"] = np.array(list(lay.c.xcd_rows) + list(lay.c.xcd_cols), np.int32)
        return r
    if kind == "layer":
        y, saved = S.seg_layer_fwd(st["lay"], st["cfg"], st["w"], st["x"])
        dx, grads = S.seg_layer_bwd(st["lay"], st["cfg"], st["w"], st["x"], saved, st["dy"])
        if c["buffer"]:  # outputs of padding rows are undefined
            y = y * (st["lay"].tok_src >= 0)[:, None]
        return {"y": y, "dx": dx, **grads}
    lay = st["lay"]
    if kind == "step":
        sz = S.seg_layout_query(st["problem"])
        S.seg_build_layout(st["problem"], sz, DEV, out=lay)
    S.seg_attn_fwd(lay, st["q"], st["k"], st["v"], st["scale"], o=st["o"], lse=st["lse"])
    r = {"o": st["o"], "lse": st["lse"]}
    if kind == "step":
        r.update(_run_loss(st, lay.loss_pred_row))
    if c.get("grad", True):
        S.seg_attn_bwd(lay, st["q"], st["k"], st["v"], st["o"], st["lse"], st["do"], st["scale"],
                       dq=st["dq"], dk=st["dk"], dv=st["dv"])
        r.update(dq=st["dq"], dk=st["dk"], dv=st["dv"])
    return r


# ------------------------------------------------------------------ needed work

def work(case):
    c, kind = case, case["kind"]
    if kind == "logprob":
        return _loss_work(c, c["rows"])
    segs = _segments(c)
    P, pairs = _packed(c, segs), _pairs(c, segs)
    rows = sum(s["len"] for s in segs)
    if kind == "layout":
        listed_tiles = sum(-(-s["len"] // 128) for s in segs) + pairs / 128 ** 2
        return {"bytes": 8 * P + 18 * listed_tiles + 12 * _loss_rows(c, segs), "flops": 0}
    e = 4 if c.get("dtype") == "f32" else 2
    QD, KD, grad = c["hq"] * c["d"], c["hkv"] * c["d"], c.get("grad", True)
    flops = (12 if grad else 4) * c["d"] * pairs * c["hq"]
    if kind == "layer":
        H, I = c["hidden"], c["inter"]
        params = 2 * H * QD + 2 * H * KD + 3 * H * I
        return {"bytes": rows * H * 2 * 4 + params * (2 + 4), "flops": flops + 6 * rows * params}
    # q, k, v, dO in; o, lse, dq, dk, dv out
    nbytes = rows * e * (2 * QD + 2 * KD + (2 * QD + 2 * KD if grad else 0)) + 4 * rows * c["hq"]
    if kind == "step":
        lw = _loss_work(c, _loss_rows(c, segs))
        nbytes, flops = nbytes + lw["bytes"], flops + lw["flops"]
    return {"bytes": nbytes, "flops": flops}


def _loss_rows(c, segs):
    return int(_spans(c).action_len.sum())


def _loss_work(c, R):
    e = 4 if c.get("dtype") == "f32" else 2
    H, V, grad = c["hidden"], c["vocab"], c.get("grad", True)
    return {"bytes": e * (R * H + V * H) + (e * R * H + 4 * V * H if grad else 0) + 40 * R,
            "flops": (6 if grad else 2) * V * H * R}


def tolerance(case):
    kind = case["kind"]
    if kind == "layout":
        return "exact"
    if kind == "logprob" and not case["grad"]:
        # fp32 sums of exact bf16 products: 1e-5 from the 64-bit result (the
        # KL term, an e^x - 1 - x of small x, is the furthest)
        return {"rel": 4e-5, "differ": 2e-3}
    # bf16 operands, probabilities, activations and score gradients with fp32
    # sums: 2e-3 to 7e-3 from the 64-bit result, and two orders of the sums
    # differ by no more.  A clip decision may fall the other way where the
    # ratio sits on its bound.
    return {"rel": 1e-2, "differ": 2e-3}


# ------------------------------------------------------------------ 64-bit results

def _attn64(c, segs, q, k, v, do):
    """Attention and its gradients in float64, query rows in chunks."""
    scale, grp = 1.0 / math.sqrt(c["d"]), c["hq"] // c["hkv"]
    f = dict(dtype=torch.float64, device=DEV)
    o, lse = torch.zeros(q.shape, **f), torch.zeros(c["hq"], q.shape[0], **f)
    dq, dk, dv = ((torch.zeros(x.shape, **f) for x in (q, k, v)) if do is not None else (None,) * 3)
    for s in segs:
        a, n = s["start"], s["len"]
        turn = torch.cat([torch.full((m,), t) for t, _, m in s["runs"]]).to(DEV)
        img = torch.cat([torch.full((m,), kd == IMAGE) for _, kd, m in s["runs"]]).to(DEV)
        step = max(1, min(n, (1 << 27) // n))
        for r0 in range(0, n, step):
            r1 = min(n, r0 + step)
            hide = torch.arange(r1, device=DEV)[None, :] > torch.arange(r0, r1, device=DEV)[:, None]
            if c["mode"] == "sliding":
                hide |= img[None, :r1] & (turn[None, :r1] <= turn[r0:r1, None] - c["window"])
            for h in range(c["hq"]):
                kh, vh = (x[a:a + r1, h // grp].double() for x in (k, v))
                qh = q[a + r0:a + r1, h].double()
                z = (qh @ kh.t()).mul_(scale).masked_fill_(hide, -math.inf)
                l = torch.logsumexp(z, 1)
                p = z.sub_(l[:, None]).exp_()
                oh = p @ vh
                o[a + r0:a + r1, h], lse[h, a + r0:a + r1] = oh, l
                if do is None:
                    continue
                doh = do[a + r0:a + r1, h].double()
                dv[a:a + r1, h // grp] += p.t() @ doh
                ds = (doh @ vh.t()).sub_((doh * oh).sum(1, keepdim=True)).mul_(p).mul_(scale)
                dq[a + r0:a + r1, h] = ds @ kh
                dk[a:a + r1, h // grp] += ds.t() @ qh
    return o, lse, dq, dk, dv


class _Attn64(torch.autograd.Function):
    @staticmethod
    def forward(ctx, q, k, v, c, segs):
        ctx.save_for_backward(q, k, v)
        ctx.more = c, segs
        return _attn64(c, segs, q, k, v, None)[0]

    @staticmethod
    def backward(ctx, do):
        return (*_attn64(*ctx.more, *ctx.saved_tensors, do)[2:], None, None)


def _layer64(c, segs, w, x, dy):
    P, d = x.shape[0], c["d"]
    pos = torch.zeros(P, dtype=torch.float64, device=DEV)
    own = torch.zeros(P, 1, dtype=torch.float64, device=DEV)
    for s in segs:
        pos[s["start"]:s["start"] + s["len"]] = torch.arange(s["len"], device=DEV).double()
        own[s["start"]:s["start"] + s["len"]] = 1
    ang = pos[:, None] * 1e6 ** (-2 * torch.arange(d // 2, device=DEV).double() / d)
    cos, sin = ang.cos()[:, None], ang.sin()[:, None]

    def rms(t, g):
        return t * torch.rsqrt((t * t).mean(1, keepdim=True) + 1e-6) * g

    def rope(t):
        a, b = t[..., :d // 2], t[..., d // 2:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

    w = {n: t.double().requires_grad_() for n, t in w.items()}
    x = x.double().requires_grad_()
    a = rms(x, w["g1"])
    q, k, v = ((a @ w[n].t()).view(P, -1, d) for n in ("wq", "wk", "wv"))
    o = _Attn64.apply(rope(q), rope(k), v, c, segs).view(P, -1)
    y1 = x + o @ w["wo"].t()
    b = rms(y1, w["g2"])
    y = y1 + (torch.nn.functional.silu(b @ w["wg"].t()) * (b @ w["wu"].t())) @ w["wd"].t()
    names = list(w)
    g = torch.autograd.grad((y * own * dy.double()).sum(), [x] + [w[n] for n in names])
    return {"y": (y * own).detach(), "dx": g[0], **dict(zip(names, g[1:]))}


def _loss64(c, st):
    h, w, R = st["h"].double(), st["w"].double(), c["rows"]
    tgt, traj = st["tgt"].long(), st["traj"].long()
    z = h @ w.t()
    lp = torch.log_softmax(z, 1) if R * c["vocab"] < 1 << 28 else None
    lse = torch.logsumexp(z, 1) if lp is None else None
    logp = (z.gather(1, tgt[:, None])[:, 0] - lse) if lp is None else lp.gather(1, tgt[:, None])[:, 0]
    del lp
    A, rho = st["adv"].double()[traj], (logp - st["old"].double()).exp()
    lo, hi = 1 - 0.2, 1 + 0.28
    obj = torch.minimum(rho * A, rho.clamp(lo, hi) * A)
    clip = ((A > 0) & (rho > hi)) | ((A < 0) & (rho < lo))
    if c["dual"] > 0:
        obj = torch.where(A < 0, torch.maximum(obj, c["dual"] * A), obj)
        clip |= (A < 0) & (rho > c["dual"])
    x = st["ref"].double() - logp
    tok = -obj + c["kl"] * (torch.expm1(x) - x)
    r = {"logp": logp, "loss_tok": tok, "clipped": clip.to(torch.uint8),
         "kl_tok": torch.expm1(x) - x, "loss_sum": tok.mean().view(1)}
    if c["grad"]:
        g = (torch.where(clip, 0.0, -rho * A) - c["kl"] * torch.expm1(x)) / R
        dz = z.sub_(torch.logsumexp(z, 1, keepdim=True)).exp_().mul_(-g[:, None])
        dz.scatter_add_(1, tgt[:, None], g[:, None])
        r["dh"] = dz @ w
        r["dw"] = dz.t() @ h
    return r


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind in ("layout", "step"):
        return None
    if kind == "logprob":
        return _loss64(c, _loss_inputs(c, seed, c["rows"], c["rows"]))
    segs = _segments(c)
    # float64 work of the dense products: about 20 s on the card at 1e14
    dense = 20 * c["d"] * c["hq"] * sum(s["len"] ** 2 for s in segs)
    if kind == "layer":
        dense += 6 * _packed(c, segs) * c["hidden"] * (3 * c["inter"] + 2 * c["hq"] * c["d"])
    if dense > 1e14:
        return None
    if kind == "layer":
        return _layer64(c, segs, *_layer_inputs(c, seed, _packed(c, segs)))
    o, lse, dq, dk, dv = _attn64(c, segs, *_attn_inputs(c, seed, _packed(c, segs)))
    return {"o": o, "lse": lse, **(dict(dq=dq, dk=dk, dv=dv) if c["grad"] else {})}
