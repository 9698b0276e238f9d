"""GPU fused log-prob + clipped-ratio loss with its KL penalty
(seg_logprob_loss through the C ABI) against the float64 oracle (Eq. loss):
full parity on the tiny and small heads (also with the KL penalty on), on
eight seeded random problems (rows, hidden, vocabulary, clip range, dual
clip, KL, input dtype), the 7B-class head at full vocabulary and hidden size
on a reduced row count, and
the full 7B-class row count on sampled rows plus the identity
sum_v dW[v] = 0 (each dz row sums to zero)."""
import numpy as np
import pytest

from oracle import layout as OL
from oracle import loss as OLS
from paper_2607_11185_amd import seg as S
from paper_2607_11185_amd import workload as WL
from tests.gpu_helpers import TOL, GpuRun, as_model_dtype, rel, say

pytestmark = pytest.mark.gpu


def _inputs(run, rows_idx=None):
    """Oracle-side inputs of the loss rows (optionally a subset)."""
    c = run.cfg
    hst = run.host
    R = len(hst["loss_pred_row"])
    sel = np.arange(R) if rows_idx is None else np.asarray(rows_idx)
    pred_canon = hst["tok_src"][hst["loss_pred_row"][sel]]
    h = as_model_dtype(run.inp.h_np(pred_canon), c)
    tgt = run.inp.tgt_np(hst["loss_tgt_src"][sel])
    adv = run.inp.adv_np().astype(np.float32)
    return sel, h, tgt, adv[hst["loss_traj"][sel]].astype(np.float64)


def _run_gpu(run, old_logp, cfg_loss, w=None, ref_logp=None):
    import torch
    dev = run.dev
    hst = run.host
    src = torch.from_numpy(hst["tok_src"].astype(np.int64)).to(dev)
    h = run.inp.h_torch(dev)[src].contiguous()
    w = run.inp.w_torch(dev) if w is None else w
    tgt = torch.from_numpy(run.inp.tgt_np(hst["loss_tgt_src"])).to(dev)
    adv = torch.from_numpy(run.inp.adv_np().astype(np.float32)).to(dev)
    ref_t = None if ref_logp is None else torch.from_numpy(ref_logp.astype(np.float32)).to(dev)
    out = S.seg_logprob_loss(h, run.lay.loss_pred_row, w, tgt,
                             torch.from_numpy(old_logp.astype(np.float32)).to(dev), adv,
                             run.lay.loss_traj, cfg_loss, ref_logp=ref_t)
    torch.cuda.synchronize()
    return out


def _full_case(cfg, dual=0.0, want_grad=True, kl=None):
    """kl: None (no reference log-probs) or the KL coefficient; the reference
    log-probs are the current ones plus a reversed copy of the rollout noise."""
    run = GpuRun(cfg)
    R = run.lay.sizes.loss_rows
    sel, h, tgt, adv = _inputs(run)
    w = as_model_dtype(run.inp.w_np(), cfg)
    logp_cur, _, _ = OLS.logprob(h, w, tgt)
    noise = run.inp.old_noise_np(run.host["loss_tgt_src"])
    old = (logp_cur + noise).astype(np.float32)
    refl = None if kl is None else (logp_cur + 2.0 * noise[::-1]).astype(np.float32)
    lc = S.LossCfg(cfg.eps_low, cfg.eps_high, dual, 1.0 / R, 1.0, want_grad, kl or 0.0)
    ref = OLS.loss_and_grads(h, w, tgt, old.astype(np.float64), adv, cfg.eps_low, cfg.eps_high,
                             loss_scale=1.0 / R, dual_clip_c=dual, want_grad=want_grad,
                             ref_logp=None if refl is None else refl.astype(np.float64),
                             kl_coef=kl or 0.0)
    out = _run_gpu(run, old, lc, ref_logp=refl)
    return run, ref, out, old


@pytest.mark.parametrize("cfg,dual", [(WL.TINY, 0.0), (WL.SMALL, 0.0), (WL.SMALL, 1.15),
                                     (WL.TINY.with_(vocab=1001, action_len=5, steps=(7, 7), old_noise_std=0.3,
                                                  seed=5), 0.0)],
                         ids=["tiny", "small", "small_dualclip", "tiny_odd_vocab_rows"])
def test_full_parity(cfg, dual):
    say(f"logprob {cfg.name} dual={dual}")
    run, ref, out, old = _full_case(cfg, dual)
    _check_full(run, ref, out, old, cfg, dual, both_branches=True)


def _random_case(i):
    """Seeded random loss problem: row count (through turn and action
    counts), hidden size, vocabulary, clip range (possibly asymmetric), dual
    clip, KL penalty and logit dtype drawn from one generator per case."""
    rng = np.random.default_rng(3000 + i)
    hidden = 8 * int(rng.integers(1, 97))
    cfg = WL.TINY.with_(name=f"lp_random{i}", num_traj=int(rng.integers(1, 4)),
                        steps=(1, int(rng.integers(1, 9))), text_len=(40, 40),
                        action_len=int(rng.integers(1, 33)), hidden=hidden,
                        vocab=int(rng.integers(1, 6000)),
                        eps_low=float(rng.uniform(0.05, 0.3)), eps_high=float(rng.uniform(0.05, 0.3)),
                        old_noise_std=float(rng.uniform(0.05, 0.4)),
                        dtype="bf16" if rng.random() < 0.7 else "f32", seed=4000 + i)
    dual = float(rng.uniform(1.5, 3.5)) if rng.random() < 0.4 else 0.0
    kl = float(rng.uniform(1e-4, 0.1)) if rng.random() < 0.5 else None
    return cfg, dual, kl


@pytest.mark.parametrize("i", range(8))
def test_random_shapes_parity(i):
    cfg, dual, kl = _random_case(i)
    say(f"logprob random case {i}: hidden={cfg.hidden} vocab={cfg.vocab} dtype={cfg.dtype} "
        f"eps=({cfg.eps_low:.3f},{cfg.eps_high:.3f}) dual={dual} kl={kl}")
    run, ref, out, old = _full_case(cfg, dual, kl=kl)
    _check_full(run, ref, out, old, cfg, dual, both_branches=False)
    if kl is not None:
        R = run.lay.sizes.loss_rows
        assert rel(out["loss_tok"][:R].cpu().numpy(), ref["loss_tok"]) < TOL


def _check_full(run, ref, out, old, cfg, dual, both_branches):
    R = run.lay.sizes.loss_rows
    logp = out["logp"][:R].cpu().numpy()
    assert np.abs(logp - ref["logp"]).max() < 2e-2 * max(1.0, np.abs(ref["logp"]).max())
    assert rel(logp, ref["logp"]) < TOL
    assert rel(out["loss_tok"][:R].cpu().numpy(), ref["loss_tok"]) < TOL
    # Clip decisions.  (1) The kernel decides from its own log-prob: its flag
    # equals the decision recomputed from that log-prob, except within 1e-5
    # of a bound in ln(rho) (the float32 ratio's rounding).  (2) A flag that
    # differs from the oracle's needs the row's ratio to lie nearer a bound
    # than the row's own log-prob error (plus that 1e-5).
    cl = out["clipped"][:R].cpu().numpy().astype(bool)
    adv_rows = _inputs(run)[3]
    bounds = [np.log(1 - cfg.eps_low), np.log(1 + cfg.eps_high)] + ([np.log(dual)] if dual else [])

    def near(log_rho, width):
        return np.any([np.abs(log_rho - b) <= width for b in bounds], axis=0)

    _, _, _, own = OLS.clipped_objective(logp.astype(np.float64), old.astype(np.float64), adv_rows,
                                         cfg.eps_low, cfg.eps_high, dual)
    lr_gpu = logp.astype(np.float64) - old
    assert (cl == own)[~near(lr_gpu, 1e-5)].all()
    err = np.abs(logp.astype(np.float64) - ref["logp"])
    lr_ref = ref["logp"] - old
    flips = cl != ref["clipped"]
    say(f"  clip flags differing from the oracle: {int(flips.sum())} of {R}")
    assert near(lr_ref, err + 1e-5)[flips].all()
    if both_branches:
        assert ref["clipped"].any() and (~ref["clipped"]).any()
    assert abs(float(out["loss_sum"][0]) - ref["loss_sum"]) < TOL * max(1e-3, abs(ref["loss_sum"]))
    e_dh = rel(out["dh"][:R].float().cpu().numpy(), ref["dh"])
    e_dw = rel(out["dw"].cpu().numpy(), ref["dw"])
    say(f"  dh {e_dh:.2e} dw {e_dw:.2e}")
    assert e_dh < TOL and e_dw < TOL
    # the last row of dh and the last vocabulary row of dW sit in the ragged
    # tails of the gradient GEMMs (output edge and reduction edge)
    dh = out["dh"][:R].float().cpu().numpy()
    dw = out["dw"].cpu().numpy()
    for i in (0, R - 1):
        assert rel(dh[i], ref["dh"][i]) < TOL, ("dh row", i)
    for v in (0, dw.shape[0] - 1):
        assert rel(dw[v], ref["dw"][v]) < TOL, ("dw row", v)


def test_tiny_against_unrounded_fp32_inputs():
    """The tiny workload's fp32 h and W are rounded to bf16 at load; report
    (and bound) the error against the oracle on the unrounded values, next to
    the error against the oracle on the rounded ones."""
    cfg = WL.TINY
    run, ref, out, old = _full_case(cfg)
    R = run.lay.sizes.loss_rows
    hst = run.host
    h = run.inp.h_np(hst["tok_src"][hst["loss_pred_row"]])
    w = run.inp.w_np()
    _, _, tgt, adv = _inputs(run)
    raw = OLS.loss_and_grads(h, w, tgt, old.astype(np.float64), adv, cfg.eps_low, cfg.eps_high,
                             loss_scale=1.0 / R)
    for n, g in (("logp", out["logp"][:R].cpu().numpy()),
                 ("loss_tok", out["loss_tok"][:R].cpu().numpy()),
                 ("dh", out["dh"][:R].float().cpu().numpy()), ("dw", out["dw"].cpu().numpy())):
        e_round, e_raw = rel(g, ref[n]), rel(g, raw[n])
        say(f"  {n}: rel err {e_round:.2e} vs bf16-rounded inputs, {e_raw:.2e} vs unrounded fp32")
        assert e_round < TOL and e_raw < TOL, (n, e_round, e_raw)


@pytest.mark.parametrize("cfg,kl", [(WL.TINY, 0.5), (WL.SMALL, 0.5), (WL.SMALL, 1e-4)],
                         ids=["tiny_kl0.5", "small_kl0.5", "small_kl1e-4"])
def test_kl_penalty_parity(cfg, kl):
    """Loss, per-token KL and gradients with the KL penalty on."""
    say(f"logprob {cfg.name} kl={kl}")
    run, ref, out, old = _full_case(cfg, kl=kl)
    R = run.lay.sizes.loss_rows
    e_kl = rel(out["kl_tok"][:R].cpu().numpy(), ref["kl_tok"])
    e_loss = rel(out["loss_tok"][:R].cpu().numpy(), ref["loss_tok"])
    e_dh = rel(out["dh"][:R].float().cpu().numpy(), ref["dh"])
    e_dw = rel(out["dw"].cpu().numpy(), ref["dw"])
    say(f"  kl {e_kl:.2e} loss {e_loss:.2e} dh {e_dh:.2e} dw {e_dw:.2e}")
    assert (out["kl_tok"][:R].cpu().numpy() >= 0).all()
    assert e_kl < TOL and e_loss < TOL and e_dh < TOL and e_dw < TOL
    assert abs(float(out["loss_sum"][0]) - ref["loss_sum"]) < TOL * max(1e-3, abs(ref["loss_sum"]))


def test_kl_zero_coefficient_matches_plain_loss():
    """kl_coef = 0 with reference log-probs given: the same loss and
    gradients, bitwise, as without them."""
    import torch
    run, _, out_kl, old = _full_case(WL.TINY, kl=0.0)
    R = run.lay.sizes.loss_rows
    lc = S.LossCfg(WL.TINY.eps_low, WL.TINY.eps_high, 0.0, 1.0 / R, 1.0, True)
    out = _run_gpu(run, old, lc)
    for k in ("logp", "loss_tok", "loss_sum", "dh", "dw"):
        assert torch.equal(out[k], out_kl[k]), k


def test_forward_only():
    run, ref, out, _ = _full_case(WL.TINY, want_grad=False)
    R = run.lay.sizes.loss_rows
    assert rel(out["logp"][:R].cpu().numpy(), ref["logp"]) < TOL


def test_seven_b_head_reduced_rows():
    """Full vocabulary and hidden size of the 7B-class head, 96 rows."""
    cfg = WL.SEVEN_B.with_(num_traj=1, steps=(3, 3))
    say("logprob 7B head, one trajectory of 3 turns")
    run, ref, out, _ = _full_case(cfg)
    R = run.lay.sizes.loss_rows
    assert rel(out["logp"][:R].cpu().numpy(), ref["logp"]) < TOL
    assert rel(out["dh"][:R].float().cpu().numpy(), ref["dh"]) < TOL
    assert rel(out["dw"].cpu().numpy(), ref["dw"]) < TOL


def test_seven_b_full_rows_sampled():
    """All 7,680 action rows of the 7B-class batch; sampled rows against the
    oracle and the dW column-sum identity."""
    import torch
    cfg = WL.SEVEN_B
    say("logprob 7B full rows")
    run = GpuRun(cfg)
    R = run.lay.sizes.loss_rows
    rng = np.random.default_rng(0)
    sel = np.unique(rng.integers(0, R, 12))
    _, h, tgt, adv = _inputs(run, sel)
    w = run.inp.w_np()
    logp_cur, _, _ = OLS.logprob(h, w, tgt)
    # rollout log-probs: oracle value + noise on the sampled rows, a fixed
    # offset elsewhere (any value is a valid input there)
    old = np.full(R, -np.log(cfg.vocab), np.float64)
    old += run.inp.old_noise_np(run.host["loss_tgt_src"])
    old[sel] = logp_cur + run.inp.old_noise_np(run.host["loss_tgt_src"][sel])
    lc = S.LossCfg(cfg.eps_low, cfg.eps_high, 0.0, 1.0 / R, 1.0, True)
    out = _run_gpu(run, old, lc)
    ref = OLS.loss_and_grads(h, w, tgt, old[sel].astype(np.float32).astype(np.float64), adv,
                             cfg.eps_low, cfg.eps_high, loss_scale=1.0 / R)
    assert rel(out["logp"][sel].cpu().numpy(), ref["logp"]) < TOL
    assert rel(out["loss_tok"][sel].cpu().numpy(), ref["loss_tok"]) < TOL
    assert rel(out["dh"][torch.from_numpy(sel).cuda()].float().cpu().numpy(), ref["dh"]) < TOL
    dw = out["dw"].double()
    assert float(dw.sum(0).norm()) < TOL * float(dw.norm())


def test_no_loss_rows():
    """A batch without action rows: zero loss and a zero weight gradient
    (the outputs are cleared by a kernel, so this also holds under graph
    capture)."""
    import torch
    dev = "cuda"
    H, V = 64, 300
    h = torch.randn(5, H, device=dev).to(torch.bfloat16)
    w = torch.randn(V, H, device=dev).to(torch.bfloat16)
    e32 = torch.empty(0, dtype=torch.int32, device=dev)
    ef = torch.empty(0, dtype=torch.float32, device=dev)
    out = {"logp": torch.empty(1, device=dev), "loss_tok": torch.empty(1, device=dev),
           "clipped": torch.empty(1, dtype=torch.uint8, device=dev),
           "kl_tok": torch.empty(1, device=dev), "loss_sum": torch.full((1,), 7.0, device=dev),
           "dh": torch.empty((1, H), dtype=torch.bfloat16, device=dev),
           "dw": torch.full((V, H), 7.0, device=dev)}
    S.seg_logprob_loss(h, e32, w, e32, ef, torch.zeros(1, device=dev), e32, S.LossCfg(), out=out)
    torch.cuda.synchronize()
    assert float(out["loss_sum"][0]) == 0.0
    assert torch.count_nonzero(out["dw"]).item() == 0


# rows, hidden and vocabulary at the edges of the products' 256 x 256 and
# 128 x 256 tiles, 64-wide steps and 8-element chunks; the last four cut dH's
# contraction over the vocabulary into parts (few output tiles, a long K)
GEMM_EDGES = [(1, 8, 1), (31, 8, 127), (33, 24, 129), (127, 56, 256), (128, 64, 255), (129, 72, 384),
              (255, 248, 257), (257, 264, 513), (64, 328, 2049), (40, 520, 16401), (300, 256, 12288),
              (257, 136, 9001)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("R,H,V", GEMM_EDGES)
def test_gemm_edges(R, H, V, dtype):
    import torch
    rng = np.random.default_rng([R, H, V])
    cfg = WL.TINY.with_(dtype="bf16")
    h, w = (as_model_dtype(WL.bf16_bits_to_f64(WL.bf16_round_np(x.astype(np.float32))), cfg)
            for x in (rng.standard_normal((R, H)), 0.3 * rng.standard_normal((V, H))))
    tgt = rng.integers(0, V, R).astype(np.int32)
    adv = rng.standard_normal(3).astype(np.float32)
    traj = rng.integers(0, 3, R).astype(np.int32)
    cur, _, _ = OLS.logprob(h, w, tgt)
    old = (cur + 0.05 * rng.standard_normal(R)).astype(np.float32)
    ref = OLS.loss_and_grads(h, w, tgt, old.astype(np.float64), adv[traj].astype(np.float64), 0.5, 0.5,
                             loss_scale=1.0, dual_clip_c=0.0, want_grad=True, ref_logp=None, kl_coef=0.0)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    t = [torch.from_numpy(x).to("cuda") for x in (tgt, old, adv, traj)]
    out = S.seg_logprob_loss(torch.from_numpy(h).to("cuda").to(dt), None,
                             torch.from_numpy(w).to("cuda").to(dt), *t, S.LossCfg(0.5, 0.5))
    torch.cuda.synchronize()
    # fp32 sums of H exact products of values below 16: 1e-5 of the largest
    lp = out["logp"].cpu().numpy()
    assert np.abs(lp - ref["logp"]).max() < 1e-5 * max(1.0, np.abs(ref["logp"]).max())
    # one bf16 rounding (2^-9) of each dz (and of dH on output): the errors of a
    # sum are independent, so its relative error stays below 2^-8
    for n in ("dh", "dw"):
        if np.linalg.norm(ref[n]) > 1e-6:
            assert rel(out[n].float().cpu().numpy(), ref[n]) < 2.0 ** -8, n


def test_probabilities_of_the_score_gradient():
    """Every bf16 dz is the rounding of a probability as exact as a fp32
    exponential gives it, far from the maximum too.  Rows of h are one-hot in
    their own column and carry two more values, so dW holds dz itself, and z =
    w1 h1 + w2 (16 bits at most) is exact in fp32; with a zero row of W as the
    target, logp = -lse, and old_logp = logp, A = -1 make dz = -exp(z - lse)."""
    import torch
    rng = np.random.default_rng(8)
    R, H, V = 32, 40, 32768
    h = np.zeros((R, H), np.float32)
    h[np.arange(R), np.arange(R)] = 1
    h[:, R] = 1 + rng.permutation(R) / 128
    h[:, R + 1] = 1
    w = np.zeros((V, H), np.float32)
    w[1:, R] = -(32 + rng.integers(0, 128, V - 1) / 4)
    w[1:, R + 1] = rng.integers(0, 256, V - 1) / 256
    z = w[:, R:R + 1].astype(np.float64) * h[:, R].astype(np.float64) + w[:, R + 1:R + 2]
    assert np.array_equal(z, z.astype(np.float32).astype(np.float64))
    t = lambda x, d: torch.from_numpy(x).to("cuda").to(d)
    hb, wb = t(h, torch.bfloat16), t(w, torch.bfloat16)
    assert np.array_equal(wb.float().cpu().numpy(), w) and np.array_equal(hb.float().cpu().numpy(), h)
    zero = t(np.zeros(R, np.int32), torch.int32)
    args = lambda old: (hb, None, wb, zero, old, t(-np.ones(1, np.float32), torch.float32), zero,
                        S.LossCfg(0.2, 0.2))
    old = S.seg_logprob_loss(*args(torch.zeros(R, device="cuda")))["logp"].clone()
    out = S.seg_logprob_loss(*args(old))
    assert torch.equal(out["logp"], old) and not out["clipped"].any()
    lse = -old.cpu().numpy()
    x = (z[1:].astype(np.float32) - lse).astype(np.float64)  # the kernel's own exponent
    want = torch.from_numpy(-np.exp(x)).to(torch.float32).to(torch.bfloat16).float().numpy()
    got = out["dw"].cpu().numpy()[1:, :R]
    assert np.abs(got / want - 1).max() < 2.0 ** -6
    # an fp32 exponential is within one unit in the last place: a relative error
    # of p of at most 2^-23, which takes it over a rounding boundary of bf16 (one
    # per relative step of 2^-8 or more) with a probability of at most 2^-15
    off = float((got != want).mean())
    say(f"  dz off the rounded exact value: {off:.1e} of {got.size}")
    assert off < 2.0 ** -15


def test_log_probs_with_a_logit_scale():
    """The softmax statistics are those of the scaled logits: no error that
    grows with them beyond the rounding of log2(e) and ln(2) to fp32 (1.6e-8
    together).  Products of two bf16 numbers and a six-bit scale are exact in
    fp32, a zero row of W as the target leaves logp = -lse, and the roundings of
    single rows (up to 2^-23) average out over 4,096 rows."""
    import torch
    rng = np.random.default_rng(9)
    R, H, V, scale = 4096, 8, 512, 45 / 16
    h, w = np.zeros((R, H), np.float32), np.zeros((V, H), np.float32)
    h[:, 0] = rng.integers(64, 192, R) / 128
    w[1:, 0] = rng.integers(64, 256, V - 1) / 16
    z = scale * h[:, :1].astype(np.float64) * w[:, 0].astype(np.float64)
    assert np.array_equal(z, z.astype(np.float32).astype(np.float64))
    zi = torch.zeros(R, dtype=torch.int32, device="cuda")
    t = lambda x: torch.from_numpy(x).to("cuda").to(torch.bfloat16)
    out = S.seg_logprob_loss(t(h), None, t(w), zi, torch.zeros(R, device="cuda"),
                             torch.ones(1, device="cuda"), zi,
                             S.LossCfg(0.2, 0.2, logit_scale=scale, want_grad=False))
    m = z.max(1, keepdims=True)
    lse = (m + np.log(np.exp(z - m).sum(1, keepdims=True)))[:, 0]
    bias = float((-out["logp"].cpu().numpy().astype(np.float64) / lse - 1).mean())
    say(f"  mean relative error of lse (up to {lse.max():.0f}): {bias:.1e}")
    assert abs(bias) < 2.5e-8
