"""Calls with more rows or samples than one launch can have a workgroup for (2^32 lanes): they go through in slabs.  The
inputs repeat every 4099 rows, so that a period of the outputs is checked against float64 and all others against it, bit
for bit."""

import numpy as np
import pytest
import torch

from paper_2605_17862_amd import binding as fb
from paper_2605_17862_amd.loss_pass import LossPass

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
HP = (1.0, 1.0, 0.05, 0.1)
PERIOD, V, K = 4099, 8, 2


def _inputs(T, B, seed=1):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    rnd = lambda *shape: torch.randn(*shape, generator=gen, device=DEV)
    base = {"logits": rnd(PERIOD, V), "second": rnd(PERIOD, V),
            "token_ids": torch.randint(0, V, (PERIOD,), generator=gen, device=DEV).int(),
            "mask": (torch.rand(PERIOD, generator=gen, device=DEV) < 0.8).to(torch.uint8)}
    lp = torch.log_softmax(base["logits"], 1).gather(1, base["token_ids"].long()[:, None])[:, 0]
    base["behav_logp"] = (lp + 0.1 * rnd(PERIOD)).clamp(max=0.0)
    base["teacher_logp"] = (lp + 0.3 * rnd(PERIOD)).clamp(max=0.0)
    q = torch.log_softmax(base["second"], 1)
    base["list_ids"], base["list_logp"] = torch.topk(q, K, 1).indices.int(), torch.topk(q, K, 1).values
    at = torch.arange(T, device=DEV) % PERIOD
    w = {k: v[at].contiguous() for k, v in base.items()}
    w["teacher_logp_stale"] = None
    lens = torch.full((B,), T // B, dtype=torch.int32, device=DEV)
    lens[-1] += T - (T // B) * B
    w.update(seq_lens=lens, lag=torch.ones(B, dtype=torch.int32, device=DEV))
    return base, w


def _repeats(out):
    """Every row is that of the first period."""
    T = out.shape[0]
    whole = T // PERIOD * PERIOD
    assert torch.equal(out[:whole].view(T // PERIOD, PERIOD, -1), out[:PERIOD].reshape(1, PERIOD, -1).expand(
        T // PERIOD, -1, -1))
    assert torch.equal(out[whole:], out[:T - whole])


def _call(op, w, p, T):
    per_row = torch.full((T,), 7.0, device=DEV)
    ws = p.workspace
    if op == "topk":
        n = fb.fopd_topk_workspace_bytes(T, 1, K)
        ws = torch.empty(n + 256, dtype=torch.uint8, device=DEV)
        ws = ws[(-ws.data_ptr()) % 256:][:n]
        fb.fopd_workspace_init(ws)
    ins = (w["token_ids"], w["mask"])
    outs = (1.0, p.loss, p.freshness, p.weights, p.logp)
    rest = (w["seq_lens"], w["lag"], 1, HP)
    none4 = (None, None, None, 0, None, None, None, None)
    if op == "step":
        p.loss_fwd_bwd(w, HP)
    elif op == "minibatch":
        fb.fopd_loss_fwd_bwd(w["logits"], p.dt, T, V, V, *ins, w["behav_logp"], w["teacher_logp"], None, *rest,
                             torch.full((1,), 0.4, device=DEV), None, None, 0, None, None, *outs, p.dlogits, ws)
    elif op == "unit":
        fb.fopd_loss_fwd_bwd_unit(w["logits"], p.dt, T, V, V, *ins, w["behav_logp"], w["teacher_logp"], None, *rest,
                                  *outs, p.dlogits, ws)
    elif op == "full_kl":
        fb.fopd_loss_fwd_bwd_full_kl(w["logits"], w["second"], p.dt, T, V, V, V, *ins, w["teacher_logp"], None, *rest,
                                     *none4, *outs, per_row, p.dlogits, ws)
    elif op == "teacher":
        fb.fopd_loss_fwd_bwd_full_teacher(w["logits"], w["second"], p.dt, T, V, V, V, *ins, w["behav_logp"], None, *rest,
                                          *none4, *outs, per_row, p.dlogits, ws)
    else:
        fb.fopd_loss_fwd_bwd_topk_teacher(w["logits"], p.dt, T, V, V, *ins, w["behav_logp"], w["list_ids"],
                                          w["list_logp"], K, 1e-4, w["teacher_logp"], None, *rest, None, None, None, 0,
                                          None, None, *outs, per_row, p.dlogits, ws)
    assert fb.fopd_workspace_status(ws) == (0, 0)
    return per_row


@pytest.mark.parametrize("T,op", [(2 ** 21 + 5, op) for op in ("step", "minibatch", "unit", "full_kl", "teacher", "topk")]
                         + [(T, op) for T in (2 ** 24 - 6, 2 ** 24 + 9) for op in ("step", "minibatch", "full_kl")])
def test_rows_beyond_one_launch(T, op):
    base, w = _inputs(T, 1)
    p = LossPass(T, V, 1, "f32")
    p.dlogits.fill_(7.0)
    p.logp.fill_(7.0)
    per_row = _call(op, w, p, T)
    for out in (p.dlogits, p.logp) + ((per_row,) if op in ("full_kl", "teacher", "topk") else ()):
        assert not bool((out == 7.0).any())
        _repeats(out)
    z = base["logits"].double()
    live = (base["mask"] != 0).double()
    logp = torch.log_softmax(z, 1).gather(1, base["token_ids"].long()[:, None])[:, 0]
    assert float((p.logp[:PERIOD].double() - logp * live).abs().max()) <= 1e-5
    if op in ("step", "minibatch"):
        # c_t of the first period; 2e-5 of the largest entry, as for every fp32 gradient
        n = float((w["mask"] != 0).sum())
        delta = logp - base["behav_logp"].double()
        c = float(p.weights) * (base["teacher_logp"].double() - logp - HP[3] * torch.exp(delta) * delta) / n * live
        ref = c[:, None] * (torch.softmax(z, 1) - torch.nn.functional.one_hot(base["token_ids"].long(), V))
        assert float((p.dlogits[:PERIOD].double() - ref).abs().max()) <= 2e-5 * float(ref.abs().max())
    assert float(p.dlogits[:PERIOD].abs().max()) > 0.0


def test_samples_beyond_one_launch():
    B = 2 ** 23 + 3                            # one row each, four of five trained on
    base, w = _inputs(B, B)
    p = LossPass(B, V, B, "f32")
    for out in (p.freshness, p.D_roll, p.weights):
        out.fill_(7.0)
    p.token_logprobs(w)
    p.freshness_score(w, HP)
    delta = (p.logp - w["behav_logp"]).double()
    k = (torch.exp(delta) * delta - torch.exp(delta) + 1.0) * (w["mask"] != 0)
    assert float((p.D_roll.double() - k).abs().max()) <= 1e-6 * float(k.max())
    f = torch.where(w["mask"] != 0, 0.5 * torch.exp(-torch.sqrt(k)), torch.zeros_like(k))
    assert float((p.freshness.double() - f).abs().max()) <= 1e-6
    assert torch.equal(p.n_train, w["mask"].int()) and torch.equal(p.cu_seqlens, torch.arange(B + 1, device=DEV))
    # counts taken from the mask
    fb.fopd_loss_fwd_bwd(w["logits"], p.dt, B, V, V, w["token_ids"], w["mask"], w["behav_logp"], w["teacher_logp"], None,
                         w["seq_lens"], w["lag"], B, HP, p.freshness, None, None, 0, None, None, 1.0, p.loss, None,
                         p.weights, p.logp, p.dlogits, p.workspace)
    assert p.status() == (0, 0)
    assert float((p.weights.double() - torch.clamp(f - HP[2], min=0.0)).abs().max()) <= 1e-6
    _repeats(p.dlogits)


def test_masked_rows_beyond_one_launch_through_the_projection():
    T, d, vocab = 2 ** 21 + 5, 64, 64
    gen = torch.Generator(device=DEV)
    gen.manual_seed(2)
    hidden = torch.randn(T, d, generator=gen, device=DEV).bfloat16()
    weight = torch.randn(vocab, d, generator=gen, device=DEV).bfloat16()
    mask = torch.zeros(T, dtype=torch.uint8, device=DEV)
    mask[::65536] = 1
    mask[-2] = 1
    tok = torch.randint(0, vocab, (T,), generator=gen, device=DEV).int()
    logp, lse, loss, weights = (torch.full((n,), 7.0, device=DEV) for n in (T, T, 1, 1))
    dh, dw = torch.full((T, d), 7.0, device=DEV), torch.empty(vocab, d, device=DEV)
    n = fb.fopd_lm_head_loss_workspace_bytes(T, vocab, d, 1, 1048576)
    ws = torch.empty(n + 256, dtype=torch.uint8, device=DEV)
    ws = ws[(-ws.data_ptr()) % 256:][:n]
    fb.fopd_workspace_init(ws)
    lens, lag = torch.full((1,), T, dtype=torch.int32, device=DEV), torch.ones(1, dtype=torch.int32, device=DEV)
    bl = torch.full((T,), -4.0, device=DEV)
    fb.fopd_lm_head_loss_fwd_bwd(hidden, d, weight, d, T, vocab, d, tok, mask, bl, bl + 0.5, lens, lag, 1, HP,
                                 torch.full((1,), 0.4, device=DEV), None, None, 1.0, 1048576, loss, weights, logp, lse, dh, d,
                                 dw, d, False, ws)
    assert fb.fopd_workspace_status(ws) == (0, 0)
    out = mask == 0
    assert not bool(dh[out].any()) and not bool(logp[out].any()) and not bool(lse[out].any())
    z = hidden[~out].double() @ weight.double().t()
    ref = torch.log_softmax(z, 1).gather(1, tok[~out].long()[:, None])[:, 0]
    assert float((logp[~out].double() - ref).abs().max()) <= 1e-4
    assert bool((dh[~out].abs().sum(1) > 0).all()) and np.isfinite(float(loss))
