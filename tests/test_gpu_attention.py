"""GPU masked GQA attention (seg_attn_fwd / seg_attn_bwd through the C ABI)
against the float64 oracle.

Full parity on workloads the oracle finishes in seconds (several tiles per
segment, ragged tails, GQA ratios, head_dim 64 and 128, fp32 inputs,
buffer padding) and on ten seeded random shapes (span lengths, empty
prompts, window, segment length, head shape, buffers, anchored mode);
sampled rows plus exact identities at the 7B-class size;
bitwise run-to-run determinism; and the segment == step-wise invariant of
the action rows (Sec. 3.3)."""
import math

import numpy as np
import pytest

from oracle import attention as OA
from oracle import layout as OL
from paper_2607_11185_amd import _lib
from paper_2607_11185_amd import seg as S
from paper_2607_11185_amd import workload as WL
from tests.gpu_helpers import TOL, GpuRun, rel, say, vis_window

pytestmark = pytest.mark.gpu
LOG2E = 1.0 / math.log(2.0)

MED = WL.Config("med", 2, (4, 7), 48, 150, (30, 90), 6, 2, 3, 4, 2, 128, 128, 1000)
CASES = {
    "med_d128": MED,
    "med_d64_gqa4": MED.with_(hq=8, hkv=2, head_dim=64, seed=1),
    "med_mha_w1_l2": MED.with_(hq=2, hkv=2, window=1, seg_steps=2, seed=2),
    "med_f32": MED.with_(dtype="f32", seed=3),
    "med_buffers": MED.with_(buffer_tokens=1400, seed=4, steps=(3, 5)),
    "stepwise_small": MED.with_(seg_steps=1, seed=5, steps=(3, 4)),
    # the long-window end of the W = L sweep
    "med_w8_l8": MED.with_(window=8, seg_steps=8, seed=11, steps=(9, 12)),
    "med_w15_l15": MED.with_(window=15, seg_steps=15, seed=12, steps=(16, 17), img_len=60),
    # the App. D algorithm as printed (window anchored at the segment start)
    "med_anchored_k2_d3": MED.with_(mode="anchored", window=2, seg_steps=3, seed=13, steps=(8, 11)),
    "med_anchored_k1_d1_d64": MED.with_(mode="anchored", window=1, seg_steps=1, hq=8, hkv=2,
                                        head_dim=64, seed=14),
    # segments of exactly 5 and 5.5 tiles (640 and 704 rows): no ragged rows,
    # and a last tile that is exactly one 64-row half
    "exact_tiles": MED.with_(steps=(4, 8), prompt_len=128, img_len=64, text_len=(64, 64),
                             action_len=8, window=4, seg_steps=4, seed=15),
    # the benchmarked head shape: 7 query heads per kv head, d = 128
    "med_gqa7_28q4kv": MED.with_(hq=28, hkv=4, seed=17, steps=(4, 5)),
    # keys scaled up along each segment (x1, x4, x16 per 128 rows): the
    # forward's running max moves by more than 8 log2 units after it is
    # finite, so the online-softmax rescale runs (asserted from the inputs)
    "med_ramped_keys": MED.with_(seed=16),
    "med_mixed_offset": MED.with_(seed=21, hq=8, hkv=2),
    # no prompt: rows whose first listed 64-key unit is an expired screenshot
    # (fully masked for them) and whose first visible key comes later
    "med_no_prompt": MED.with_(prompt_len=0, seed=19, steps=(5, 7)),
    # fewer tiles than the chip's eight dies: most launch-schedule ranges are
    # empty (one trajectory of two turns, a single 2-tile segment)
    "few_tiles": MED.with_(num_traj=1, steps=(2, 2), seed=20),
    "tiny": WL.TINY,
}
RAMPED = {"med_ramped_keys"}
# queries of every third 32-row group scaled by 8: in one launch some waves
# have every score bounded by |q| max|k| within 64 log2 units (fixed offset,
# no running max) and others do not (running max)
MIXED = {"med_mixed_offset"}


def _key_factors(ref, P):
    """Per packed row: 4 ** min(2, row-in-segment // 128) (powers of two, so
    scaling bf16 keys is exact on both sides); padding rows 1."""
    f = np.ones(P)
    for sg in ref.segments:
        f[sg.start:sg.start + sg.length] = 4.0 ** np.minimum(2, np.arange(sg.length) // 128)
    return f


def _query_factors(ref, P):
    """Per packed row: 8 for every third group of 32 rows of a segment
    (a power of two, so scaling bf16 queries is exact), else 1."""
    f = np.ones(P)
    for sg in ref.segments:
        f[sg.start:sg.start + sg.length] = np.where(np.arange(sg.length) // 32 % 3 == 0, 8.0, 1.0)
    return f


def _offset_waves(q, k, scale, grp):
    """(waves with every row's bound |q| max|k| * scale * log2 e <= 64, waves
    without), a wave being 32 consecutive rows of the segment for one query
    head and max|k| running over the segment's keys of its kv head."""
    kmax = np.sqrt((k.astype(np.float64) ** 2).sum(-1).max(0))  # [hkv]
    qn = np.sqrt((q.astype(np.float64) ** 2).sum(-1))           # [len, hq]
    bound = qn * kmax[np.arange(q.shape[1]) // grp][None, :] * scale * np.log2(np.e)
    fixed = other = 0
    for w0 in range(0, q.shape[0], 32):
        ok = (bound[w0:w0 + 32] <= 64).all(0)
        fixed += int(ok.sum())
        other += int((~ok).sum())
    return fixed, other


def _unit_scores(q, k, mask, scale, h, grp):
    """Scores in log2 units of query head h, invisible pairs -inf, padded to
    whole 64-key units: [rows, units, 64]."""
    s = (q[:, h] @ k[:, h // grp].T) * (scale * LOG2E)
    s = np.where(mask, s, -np.inf)
    n, nk = s.shape
    nu = (nk + 63) // 64
    out = np.full((n, nu * 64), -np.inf)
    out[:, :nk] = s
    return out.reshape(n, nu, 64)


def _rescale_events(q, k, mask, scale, hq, hkv, margin=9.0):
    """Rows x units where a 64-key unit's max exceeds a finite running max by
    more than `margin` log2 units, the running max following the forward
    kernel's rule (it moves only when a unit max exceeds it by more than 8).
    Units are taken in ascending key order; units of skipped tiles hold no
    visible key and never move the running max, so the count is the
    kernel's."""
    n = 0
    for h in range(hq):
        um = _unit_scores(q, k, mask, scale, h, hq // hkv).max(-1)
        run = np.full(um.shape[0], -np.inf)
        for u in range(um.shape[1]):
            x = um[:, u]
            n += int((np.isfinite(run) & (x > run + margin)).sum())
            run = np.where(x > run + 8.0, x, run)
    return n


def _masked_first_units(mask):
    """Rows whose first 64-key unit among the k-tiles listed for their q-tile
    (tiles with any visible pair in the q-tile) has no visible key while a
    later unit has one."""
    n = mask.shape[0]
    cnt = 0
    for qt in range((n + 127) // 128):
        m = mask[qt * 128:(qt + 1) * 128]
        listed = [kt for kt in range(qt + 1) if m[:, kt * 128:(kt + 1) * 128].any()]
        units = [kt * 128 + h * 64 for kt in listed for h in (0, 1) if kt * 128 + h * 64 < n]
        vis = np.stack([m[:, u:u + 64].any(1) for u in units], 1)
        cnt += int((~vis[:, 0] & vis.any(1)).sum())
    return cnt


def _ref_layout(run):
    c = run.cfg
    return OL.build(run.spans, c.window, c.seg_steps, 128, c.max_seg_tokens, c.buffer_tokens,
                    with_tiles=False, mode=c.mode)


@pytest.mark.parametrize("name", list(CASES))
def test_fwd_bwd_full_parity(name):
    _full_parity(name, CASES[name])


def _random_config(i):
    """Seeded random workload of a few thousand packed rows: trajectory count,
    turn counts, prompt (possibly empty), span lengths, window and segment
    length, head shape (GQA ratios 1-7, d 64 or 128), buffer packing and the
    anchored mode all drawn from one generator per case."""
    rng = np.random.default_rng(1000 + i)
    hq, hkv, d = [(2, 1, 64), (4, 2, 128), (8, 8, 64), (6, 3, 128), (7, 1, 128),
                  (14, 2, 64)][rng.integers(6)]
    lo = int(rng.integers(1, 6))
    t_lo = int(rng.integers(1, 60))
    cfg = MED.with_(name=f"random{i}", num_traj=int(rng.integers(1, 4)),
                    steps=(lo, lo + int(rng.integers(0, 4))),
                    prompt_len=int(rng.choice([0, int(rng.integers(1, 200))])),
                    img_len=int(rng.integers(1, 260)),
                    text_len=(t_lo, t_lo + int(rng.integers(0, 120))),
                    action_len=int(rng.integers(0, t_lo + 1)),
                    window=int(rng.integers(1, 6)), seg_steps=int(rng.integers(1, 6)),
                    hq=hq, hkv=hkv, head_dim=d, seed=2000 + i,
                    mode="anchored" if rng.random() < 0.25 else "sliding")
    if cfg.mode == "sliding" and rng.random() < 0.4:
        # buffer packing: room for the longest segment plus a random slack
        ref = OL.build(WL.Inputs(cfg).spans, cfg.window, cfg.seg_steps, 128, with_tiles=False)
        longest = max(sg.length for sg in ref.segments)
        cfg = cfg.with_(buffer_tokens=longest + int(rng.integers(0, 700)))
    return cfg


@pytest.mark.parametrize("i", range(10))
def test_random_shapes_full_parity(i):
    cfg = _random_config(i)
    say(f"random case {i}: {cfg}")
    _full_parity(cfg.name, cfg)


def _full_parity(name, cfg):
    say(f"case {name}")
    import torch
    run = GpuRun(cfg).packed_inputs()
    ref = _ref_layout(run)
    assert np.array_equal(run.host["tok_src"], ref.tok_src)
    fac = _key_factors(ref, run.P) if name in RAMPED else None
    if fac is not None:
        run.k = run.k * torch.from_numpy(fac).to(run.dev, torch.bfloat16)[:, None, None]
    qfac = _query_factors(ref, run.P) if name in MIXED else None
    if qfac is not None:
        run.q = run.q * torch.from_numpy(qfac).to(run.dev, torch.bfloat16)[:, None, None]
    waves = [0, 0]
    run.fwd()
    run.bwd()
    torch.cuda.synchronize()
    o, lse = run.o.float().cpu().numpy(), run.lse.cpu().numpy()
    dq, dk, dv = (t.float().cpu().numpy() for t in (run.dq, run.dk, run.dv))
    acc = {n: [[], []] for n in ("o", "lse", "dq", "dk", "dv")}
    events = masked_first = 0
    for sg in ref.segments:
        q, k, v, dout = run.seg_np(sg)
        mask = OL.visibility(sg, vis_window(cfg))
        if fac is not None:
            k = k * fac[sg.start:sg.start + sg.length, None, None]
            events += _rescale_events(q, k, mask, run.scale, cfg.hq, cfg.hkv)
        if name == "med_no_prompt":
            masked_first += _masked_first_units(mask)
        if qfac is not None:
            q = q * qfac[sg.start:sg.start + sg.length, None, None]
            fx, ot = _offset_waves(q, k, run.scale, cfg.hq // cfg.hkv)
            waves[0] += fx
            waves[1] += ot
        o_r, lse_r = OA.forward(q, k, v, mask, run.scale)
        dq_r, dk_r, dv_r = OA.backward(q, k, v, mask, run.scale, dout)
        rows = slice(sg.start, sg.start + sg.length)
        for n, g, r in (("o", o[rows], o_r), ("lse", lse[:, rows], lse_r), ("dq", dq[rows], dq_r),
                        ("dk", dk[rows], dk_r), ("dv", dv[rows], dv_r)):
            e = rel(g, r)
            assert e < TOL, (name, n, sg.start, e)
            acc[n][0].append(g.ravel())
            acc[n][1].append(r.ravel())
    for n, (g, r) in acc.items():
        e = rel(np.concatenate(g), np.concatenate(r))
        say(f"  {n}: rel err {e:.2e}")
        assert e < TOL, (name, n, e)
    if cfg.dtype == "f32":
        # fp32 inputs are rounded to bf16 at load: the error against the
        # oracle on the unrounded values, reported next to the one above
        for sg in ref.segments:
            q, k, v = (run.inp.q_np(sg.canon), run.inp.k_np(sg.canon), run.inp.v_np(sg.canon))
            dout = run.inp.dout_np(np.arange(sg.start, sg.start + sg.length))
            mask = OL.visibility(sg, vis_window(cfg))
            o_r, lse_r = OA.forward(q, k, v, mask, run.scale)
            dq_r, dk_r, dv_r = OA.backward(q, k, v, mask, run.scale, dout)
            rows = slice(sg.start, sg.start + sg.length)
            for n, g, r in (("o", o[rows], o_r), ("lse", lse[:, rows], lse_r),
                            ("dq", dq[rows], dq_r), ("dk", dk[rows], dk_r), ("dv", dv[rows], dv_r)):
                e = rel(g, r)
                say(f"  {n} vs unrounded fp32 inputs (segment at {sg.start}): rel err {e:.2e}")
                assert e < TOL, (name, "unrounded", n, e)
    if fac is not None:
        say(f"  running-max moves of > 9 log2 units after a finite max: {events}")
        assert events > 0
    if name == "med_no_prompt":
        say(f"  rows whose first listed unit is fully masked: {masked_first}")
        assert masked_first > 0
    if qfac is not None:
        say(f"  waves with bounded scores {waves[0]}, without {waves[1]}")
        assert waves[0] > 0 and waves[1] > 0


def test_padding_rows_hold_nan():
    """Buffer padding after ragged segment ends, with o, lse and dO of every
    padding row set to NaN before the backward (the forward does not write
    padding rows): dQ, dK and dV stay finite and match the oracle."""
    import torch
    cfg = MED.with_(buffer_tokens=1400, seed=18, steps=(3, 5), hq=8, hkv=2)
    run = GpuRun(cfg).packed_inputs()
    ref = _ref_layout(run)
    pad = torch.from_numpy(run.host["tok_src"] < 0).to(run.dev)
    say(f"  padding rows {int(pad.sum())} of {run.P}")
    assert bool(pad.any())
    run.fwd()
    run.o[pad] = float("nan")
    run.lse[:, pad] = float("nan")
    run.dout[pad] = float("nan")
    run.bwd()
    torch.cuda.synchronize()
    rows = ~pad
    for t in (run.dq, run.dk, run.dv):
        assert bool(torch.isfinite(t[rows].float()).all())
    dq, dk, dv = (t.float().cpu().numpy() for t in (run.dq, run.dk, run.dv))
    for sg in ref.segments:
        q, k, v, dout = run.seg_np(sg)
        mask = OL.visibility(sg, vis_window(cfg))
        dq_r, dk_r, dv_r = OA.backward(q, k, v, mask, run.scale, dout)
        r = slice(sg.start, sg.start + sg.length)
        for n, g, want in (("dq", dq[r], dq_r), ("dk", dk[r], dk_r), ("dv", dv[r], dv_r)):
            e = rel(g, want)
            assert e < TOL, (n, sg.start, e)


def test_determinism_bitwise():
    import torch
    run = GpuRun(MED.with_(seed=7)).packed_inputs()
    a = [t.clone() for t in run.fwd()] + [t.clone() for t in run.bwd()]
    b = list(run.fwd()) + list(run.bwd())
    torch.cuda.synchronize()
    for x, y in zip(a, b):
        assert torch.equal(x, y)


def _segment_of_rows(ref, rows):
    out = {}
    for r in rows:
        for si, sg in enumerate(ref.segments):
            if sg.start <= r < sg.start + sg.length:
                out.setdefault(si, []).append(r)
    return out


@pytest.mark.parametrize("cfg", [WL.SMALL, WL.SEVEN_B, WL.SEVEN_B_ANCHORED, WL.LONG],
                         ids=lambda c: c.name)
def test_full_size_sampled_rows_and_identities(cfg):
    """Full-size launch: O, LSE and dQ of sampled rows against the oracle
    computed row by row; dK and dV through exact identities of every segment
    and kv head: sum over keys of dV = sum over rows and group heads of dO
    (softmax rows sum to one) and sum over keys of dK = 0 (each row of dS sums
    to zero)."""
    import torch
    say(f"full-size {cfg.name}")
    run = GpuRun(cfg).packed_inputs()
    run.fwd()
    run.bwd()
    torch.cuda.synchronize()
    ref = _ref_layout(run)
    rng = np.random.default_rng(0)
    picks = [0, len(ref.segments) // 2, len(ref.segments) - 1]
    for si in picks:
        sg = ref.segments[si]
        say(f"  segment {si}: {sg.length} tokens")
        k = run.inp.k_np(sg.canon)
        v = run.inp.v_np(sg.canon)
        loc = np.unique(np.concatenate([rng.integers(0, sg.length, 24), [0, sg.length - 1]]))
        q = run.inp.q_np(sg.canon[loc])
        dout = run.inp.dout_np(sg.start + loc)
        mask = OL.visibility_rows(sg, vis_window(cfg), loc)
        o_r, lse_r = OA.forward_generic(q, k, v, mask, run.scale)
        rows = sg.start + loc
        o_g = run.o[torch.from_numpy(rows).cuda()].float().cpu().numpy()
        lse_g = run.lse[:, torch.from_numpy(rows).cuda()].cpu().numpy()
        assert rel(o_g, o_r) < TOL and rel(lse_g, lse_r) < 1e-3
        # dQ of the sampled rows: dS_ij = P_ij (dO_i . v_j - dO_i . O_i)
        hq, hkv = cfg.hq, cfg.hkv
        dq_r = np.zeros_like(q)
        for h in range(hq):
            g = h // (hq // hkv)
            s = run.scale * (q[:, h] @ k[:, g].T)
            s = np.where(mask, s, -np.inf)
            p = np.exp(s - lse_r[h][:, None])
            dp = dout[:, h] @ v[:, g].T
            ds = p * (dp - (dout[:, h] * o_r[:, h]).sum(1, keepdims=True))
            dq_r[:, h] = run.scale * (ds @ k[:, g])
        dq_g = run.dq[torch.from_numpy(rows).cuda()].float().cpu().numpy()
        assert rel(dq_g, dq_r) < TOL
        # identities over the whole segment
        seg_rows = slice(sg.start, sg.start + sg.length)
        dv_sum = run.dv[seg_rows].double().sum(0).cpu().numpy()         # [hkv, d]
        do_sum = run.dout[seg_rows].double().sum(0).cpu().numpy()       # [hq, d]
        grp = hq // hkv
        want = do_sum.reshape(hkv, grp, -1).sum(1)
        dv_fro = float(run.dv[seg_rows].double().pow(2).sum().sqrt())
        assert np.linalg.norm(dv_sum - want) < TOL * max(np.linalg.norm(want), dv_fro)
        # random per-key errors add up to about err * ||dK||_F; a systematic
        # error would grow with the segment length
        dk_seg = run.dk[seg_rows].double()
        dk_sum = dk_seg.sum(0).cpu().numpy()
        assert np.linalg.norm(dk_sum) < TOL * float(dk_seg.pow(2).sum().sqrt())


def _tail_keys(sg, turn, n, span, rng):
    """n screenshot keys of `turn` among the last `span` rows of its screenshot
    (always its last row)."""
    img = np.nonzero((sg.kind == OL.KIND_IMAGE) & (sg.step == turn))[0][-span:]
    return np.unique(np.concatenate([img[-1:], rng.choice(img, n - 1, replace=False)]))


# (workload, also sample keys of the second-to-last turn)
KEY_CASES = [(WL.SEVEN_B, True), (WL.SEVEN_B_ANCHORED, False), (WL.LONG, False)]


@pytest.mark.parametrize("cfg,prev_turn", KEY_CASES, ids=[c.name for c, _ in KEY_CASES])
def test_full_size_key_gradients(cfg, prev_turn):
    """Full-size launch (28q/4kv, d = 128: seven query heads per kv head):
    dK and dV of sampled screenshot keys, key by key, against the oracle, on
    the last kv head.  Keys lie in the tail of the last turn's screenshot of
    the shortest segment with two or more turns (two 128-row tiles), and for
    the 7B-class batch also in the tail of the turn before, which the last
    turn's rows still see; only rows at or after a key can see it, and each
    such row's softmax (its LSE and Delta) is the oracle's over every key it
    sees."""
    import torch
    say(f"full-size key gradients {cfg.name}")
    run = GpuRun(cfg).packed_inputs()
    run.fwd()
    run.bwd()
    torch.cuda.synchronize()
    ref = _ref_layout(run)
    multi = [sg for sg in ref.segments if len(np.unique(sg.step[sg.step > 0])) >= 2]
    sg = min(multi, key=lambda s: s.length)
    turns = np.unique(sg.step[sg.step > 0])
    rng = np.random.default_rng(1)
    keys = [_tail_keys(sg, turns[-1], 10, 192, rng)]
    if prev_turn:
        keys.append(_tail_keys(sg, turns[-2], 4, 64, rng))
    keys = np.unique(np.concatenate(keys))
    rows = np.arange(keys.min(), sg.length)
    mask = OL.visibility_rows(sg, vis_window(cfg), rows)
    sees = mask[:, keys].any(1)
    rows, mask = rows[sees], mask[sees]
    say(f"  segment at {sg.start}: {sg.length} tokens, {len(keys)} keys, {len(rows)} rows")
    grp = cfg.hq // cfg.hkv
    g = cfg.hkv - 1
    hs = slice(g * grp, (g + 1) * grp)
    k_all = run.inp.k_np(sg.canon)[:, g:g + 1]
    v_all = run.inp.v_np(sg.canon)[:, g:g + 1]
    q = run.inp.q_np(sg.canon[rows])[:, hs]
    dout = run.inp.dout_np(sg.start + rows)[:, hs]
    idx = torch.from_numpy(sg.start + keys).cuda()
    dk_g = run.dk[idx, g].float().cpu().numpy()
    dv_g = run.dv[idx, g].float().cpu().numpy()
    dk_r, dv_r = OA.key_grads(q, k_all, v_all, mask, run.scale, dout, keys)
    e_k, e_v = rel(dk_g, dk_r[:, 0]), rel(dv_g, dv_r[:, 0])
    say(f"  kv head {g}: dK rel err {e_k:.2e}, dV rel err {e_v:.2e}")
    assert e_k < TOL and e_v < TOL, (e_k, e_v)
    for i in range(len(keys)):   # and no single key off
        assert rel(dk_g[i], dk_r[i, 0]) < TOL, ("dk", int(keys[i]))
        assert rel(dv_g[i], dv_r[i, 0]) < TOL, ("dv", int(keys[i]))


def test_action_rows_segment_equals_stepwise():
    """Attention outputs of the action-predicting rows agree between the
    segmented layout and the step-wise decomposition of the same canonical
    tensors (both see the same keys)."""
    import torch
    cfg = MED.with_(seed=9, steps=(5, 6))
    seg_run = GpuRun(cfg).packed_inputs(with_dout=False)
    sw_run = GpuRun(cfg.with_(seg_steps=1)).packed_inputs(with_dout=False)
    o1, l1 = seg_run.fwd()
    o2, l2 = sw_run.fwd()
    torch.cuda.synchronize()

    def by_target(run, o, lse):
        h = run.host
        rows = torch.from_numpy(h["loss_pred_row"].astype(np.int64)).cuda()
        order = np.argsort(h["loss_tgt_src"])
        return (o[rows].float().cpu().numpy()[order], lse[:, rows].cpu().numpy()[:, order],
                np.sort(h["loss_tgt_src"]))

    a_o, a_l, a_t = by_target(seg_run, o1, l1)
    b_o, b_l, b_t = by_target(sw_run, o2, l2)
    assert np.array_equal(a_t, b_t)
    assert rel(a_o, b_o) < 1e-2 and rel(a_l, b_l) < 1e-3


# (kv heads, image tokens, turns): tiles x kv heads per eighth of the dK/dV
# launch below and above the 32 blocks that run at once, and above the 512
# tiles that the longest-first classes take
@pytest.mark.parametrize("hkv,img,turns", [(1, 150, 5), (8, 150, 12), (5, 700, 9), (2, 40, 2)])
def test_dkdv_block_order_covers_every_key(hkv, img, turns):
    import torch
    n_traj = 4 if turns != 2 else 4400
    cfg = WL.Config("order", n_traj, (turns, turns), 30, img, (20, 90), 4, 2, 3, hkv, hkv, 64, 64, 100,
                    seed=77)
    run = GpuRun(cfg).packed_inputs()
    cols = np.diff(run.host["xcd_cols"])
    say(f"P={run.P} tiles per eighth {cols.min()}..{cols.max()} x {hkv}")
    assert {1: cols.max() * hkv <= 32, 2: cols.max() > 512}.get(hkv, cols.max() * hkv > 32)
    run.fwd()
    dk, dv = (torch.full_like(t, float("nan")) for t in (run.k, run.v))
    S.seg_attn_bwd(run.lay, run.q, run.k, run.v, run.o, run.lse, run.dout, run.scale, dk=dk, dv=dv)
    assert bool(torch.isfinite(dk).all()) and bool(torch.isfinite(dv).all())
    ref = OL.build(run.spans, cfg.window, cfg.seg_steps, 128, with_tiles=False, mode=cfg.mode)
    segs = ref.segments if len(ref.segments) < 100 else ref.segments[::400]
    for sg in segs:
        hide = torch.from_numpy(~OL.visibility(sg, vis_window(cfg))).to(run.dev)
        rows = slice(sg.start, sg.start + sg.length)
        for h in range(hkv):
            q, k, v, do, o = (x[rows, h].double() for x in (run.q, run.k, run.v, run.dout, run.o))
            p = torch.softmax((q @ k.t() * run.scale).masked_fill(hide, float("-inf")), 1)
            ds = p * (do @ v.t() - (do * o).sum(1, keepdim=True)) * run.scale
            for name, got, want in (("dk", dk, ds.t() @ q), ("dv", dv, p.t() @ do)):
                e = float((got[rows, h].double() - want).norm() / want.norm())
                assert e < TOL, (name, sg.start, h, e)


class _Spans:
    """Attention over segments of given lengths (one turn of text each), on the
    GPU: inputs, forward outputs and the float64 dk and dv."""

    def __init__(self, lens, hq, hkv, d, dtype="bf16", buffer=0, seed=0):
        import torch
        n = len(lens)
        sp = WL.explicit_spans([1] * n, [1] * n, [0] * n, [x - 1 for x in lens], [1] * n)
        self.lay = S.seg_build_layout(S.Problem.from_spans(sp, 1, 1, 0, buffer), device="cuda")
        self.P = self.lay.sizes.packed_tokens
        info = self.lay.host()["seg_info"]
        self.rows = [slice(int(a), int(a) + int(b)) for a, b in info[:, 3:5]]
        self.grp, self.hkv, self.scale = hq // hkv, hkv, d ** -0.5
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        dt = torch.bfloat16 if dtype == "bf16" else torch.float32
        self.q, self.k, self.v, self.dout = (
            torch.randn(self.P, h, d, generator=g, device="cuda", dtype=torch.float32).to(dt)
            for h in (hq, hkv, hkv, hq))
        self.o, self.lse = S.seg_attn_fwd(self.lay, self.q, self.k, self.v, self.scale)

    def bwd(self, ws=None, noalloc=False):
        """dq, dk, dv over NaN: what no kernel writes stays NaN."""
        import torch
        out = [torch.full_like(t, float("nan")) for t in (self.q, self.k, self.v)]
        a = (self.lay, self.q, self.k, self.v, self.o, self.lse, self.dout, self.scale)
        if noalloc:
            S.seg_attn_bwd_noalloc(*a, *out)
        else:
            S.seg_attn_bwd(*a, *out, ws=ws)
        torch.cuda.synchronize()
        return out

    def check(self, dk, dv):
        import torch
        real = torch.zeros(self.P, dtype=torch.bool, device="cuda")
        for r in self.rows:
            real[r] = True
        for t in (dk, dv):
            assert bool(torch.isfinite(t[real]).all()) and bool(torch.isnan(t[~real]).all())
        bf = lambda t: t.to(torch.bfloat16).double()  # the kernels round fp32 inputs
        for r in self.rows[::max(1, len(self.rows) // 12)]:
            n = r.stop - r.start
            hide = torch.ones(n, n, dtype=torch.bool, device="cuda").triu(1)
            for h in range(self.hkv):
                wk, wv = 0, 0
                for j in range(h * self.grp, (h + 1) * self.grp):
                    q, do, o = bf(self.q[r, j]), bf(self.dout[r, j]), self.o[r, j].double()
                    k, v = bf(self.k[r, h]), bf(self.v[r, h])
                    p = torch.softmax((q @ k.t() * self.scale).masked_fill(hide, float("-inf")), 1)
                    ds = p * (do @ v.t() - (do * o).sum(1, keepdim=True)) * self.scale
                    wk, wv = wk + ds.t() @ q, wv + p.t() @ do
                for name, got, want in (("dk", dk[r, h], wk), ("dv", dv[r, h], wv)):
                    e = float((got.double() - want).norm() / want.norm())
                    assert e < TOL, (name, r.start, h, e)


# (tiles of a segment, segments, kv heads, query heads of each): more blocks of
# an eighth than run at once, on both sides of the rule that sorts them (at
# least two tiles, and four tiles x heads)
@pytest.mark.parametrize("tiles,segs,hkv,grp", [(1, 50, 8, 1), (1, 50, 8, 8), (3, 33, 8, 1), (4, 25, 8, 1),
                                                (2, 50, 4, 2)])
def test_dkdv_short_walks_cover_every_key(tiles, segs, hkv, grp):
    run = _Spans([tiles * 128 - 7 * (i % 11) for i in range(segs)], hkv * grp, hkv, 64)
    cols = np.diff(run.lay.host()["xcd_cols"])
    assert cols.max() * hkv > 32
    run.check(*run.bwd()[1:])


# (rows of each segment, kv heads, query heads of each, d, dtype, buffer rows, parts):
# even and uneven shares of the heads, ragged last tiles, padding rows
@pytest.mark.parametrize("lens,hkv,grp,d,dtype,buffer,parts", [
    ([300], 1, 2, 64, "bf16", 0, 2), ([257, 500, 90], 2, 3, 128, "bf16", 0, 3),
    ([400, 130, 700], 1, 7, 128, "f32", 800, 7), ([1000] * 3, 4, 7, 64, "bf16", 0, 3),
    ([1000] * 3, 2, 8, 128, "f32", 1100, 4), ([128] * 60, 1, 8, 64, "bf16", 0, 4)])
def test_dkdv_parts(lens, hkv, grp, d, dtype, buffer, parts):
    """dk and dv summed in parts: against float64, repeated, through the
    allocation-free entry point, and with a workspace that has no room for the
    parts (one byte short of them, and none at all), which sums in one part."""
    import torch
    run = _Spans(lens, hkv * grp, hkv, d, dtype, buffer)
    ws = S.attn_workspace(run.lay, S._dtype_code(run.q), hkv * grp, hkv, d, True)
    held = parts * run.P * hkv * d * 2 * 4
    base = (ws.numel() - held) // 256 * 256
    assert base >= 8 * run.P * hkv * grp and base + held <= ws.numel() < base + held + 256
    ws.fill_(255)  # NaN wherever the call reads what it has not written
    whole = run.bwd(ws)
    run.check(*whole[1:])
    for other in (run.bwd(ws), run.bwd(noalloc=True)):
        assert all(torch.equal(a.nan_to_num(7), b.nan_to_num(7)) for a, b in zip(whole, other))
    short = run.bwd(ws[:ws.numel() - 1])
    run.check(*short[1:])
    least = run.bwd(ws[:base])
    assert all(torch.equal(a.nan_to_num(7), b.nan_to_num(7)) for a, b in zip(short, least))
    assert torch.equal(short[0].nan_to_num(7), whole[0].nan_to_num(7))
    for a, b in zip(short[1:], whole[1:]):  # the same sum in another order, then rounded
        e = float((a.double() - b.double()).nan_to_num(0).norm() / b.double().nan_to_num(0).norm())
        assert e < (2 ** -8 if dtype == "bf16" else 1e-5), e
    with pytest.raises(_lib.SegError):
        run.bwd(ws[:base - 1])
