"""Numbers of samples and rows around the lines where a call forms the samples' offsets (1024 samples) and the row
coefficients (2048 rows) inside the statistics kernel and where that takes 512 or 1024 lanes a sample, against float64; the
error flags of the offsets there; rows kept in the caches between the two passes of a call."""

import numpy as np
import pytest
import torch

from harness import workloads as wl
from paper_2605_17862_amd import binding as fb
from test_gpu_parity import HP, _compare_everything, _pass_for

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("B,length,staged", [(1, 1, True), (1, 1025, True), (1, 2048, False), (1, 2049, False),
                                             (3, 700, True), (1024, 2, True), (1024, 4, False), (1025, 3, True)])
def test_offsets_and_coefficients_at_the_edges(B, length, staged):
    w = wl.generate("reasoning", DEV, seed=B + length, B=B, len_lo=length, len_hi=length, V=264)
    w["mask"][::5] = 0
    if B > 2:                                   # an empty sample, its rows with the one after it
        seq = w["seq_lens_host"].copy()
        seq[2] += seq[1]
        seq[1] = 0
        w["seq_lens"] = torch.from_numpy(seq).to(DEV)
    _compare_everything(w, HP, staged=staged)


@pytest.mark.parametrize("B,length", [(1, 4095), (1, 4096), (3, 4096), (256, 4096), (257, 4096), (256, 4095), (1025, 5)])
def test_scores_at_the_line_between_the_lane_counts(B, length):
    """1024 lanes a sample for up to 256 samples of 4096 rows or more on average, else 512.  1e-6: scores are fp32 results of
    fp64 sums."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(B + length)
    lens = torch.full((B,), length, dtype=torch.int32, device=DEV)
    if B > 2:                                    # ragged; the same total
        lens[0] += length // 2
        lens[1] -= length // 2
    T = B * length
    p = _pass_for(dict(T=T, V=8, B=B, dtype="bf16", ld=8), alloc_dlogits=False)
    p.logp.copy_(-torch.rand(T, generator=gen, device=DEV))
    w = dict(behav_logp=p.logp + 0.1 * torch.randn(T, generator=gen, device=DEV), teacher_logp=p.logp - 0.1,
             teacher_logp_stale=p.logp - 0.15, mask=(torch.rand(T, generator=gen, device=DEV) < 0.7).to(torch.uint8),
             seq_lens=lens, lag=torch.ones(B, dtype=torch.int32, device=DEV))
    p.freshness_score(w, HP)
    assert p.status() == (0, 0)
    at, live = torch.repeat_interleave(torch.arange(B, device=DEV), lens.long()), (w["mask"] != 0).double()
    mean = lambda x: torch.zeros(B, dtype=torch.float64, device=DEV).index_add_(0, at, x * live) / n
    est = lambda d: torch.exp(d) * d - torch.exp(d) + 1.0
    n = torch.zeros(B, dtype=torch.float64, device=DEV).index_add_(0, at, live)
    assert torch.equal(p.n_train, n.int()) and torch.equal(p.cu_seqlens[1:], torch.cumsum(lens, 0))
    roll = mean(est(p.logp.double() - w["behav_logp"].double()))
    sup = mean(est(w["teacher_logp"].double() - w["teacher_logp_stale"].double()))
    f = 0.5 * torch.exp(-torch.sqrt(roll) - torch.sqrt(sup))
    for got, ref in ((p.D_roll, roll), (p.D_sup, sup), (p.freshness, f), (p.cover, n / lens),
                     (p.ell, mean(p.logp.double() - w["teacher_logp"].double()))):
        assert float(((got.double() - ref) / ref).abs().max()) <= 1e-6


@pytest.mark.parametrize("B", [3, 1024, 1025])
@pytest.mark.parametrize("what", ["short", "long", "negative length", "negative lag"])
def test_flags_of_the_offsets(B, what):
    w = wl.generate("reasoning", DEV, seed=1, B=B, len_lo=4, len_hi=4, V=264)
    lens, lag = w["seq_lens_host"].copy(), w["lag_host"].copy()
    if what == "negative lag":
        lag[B - 2] = -1
    else:
        lens[B - 2] = {"short": 1, "long": 9, "negative length": -4}[what]
    w["seq_lens"], w["lag"] = torch.from_numpy(lens).to(DEV), torch.from_numpy(lag).to(DEV)
    lp = _pass_for(w)
    lp.dlogits.fill_(1.0)
    lp.loss_fwd_bwd(w, HP)
    st, flags = lp.status()
    assert st != 0 and flags != 0
    cu = np.minimum(np.concatenate([[0], np.cumsum(np.maximum(lens, 0))]), w["T"])
    rest = lp.dlogits[int(cu[-1]):]              # rows that belong to no sample
    assert not bool(rest.any())
    if what == "negative lag":
        assert not bool(lp.dlogits[int(cu[B - 2]):int(cu[B - 1])].any()) and float(lp.weights[B - 2]) == 0.0


CACHED, CACHED_TOTAL = 240 << 20, 640 << 20       # bytes of rows: read by ordinary loads the first time; no more than this in all


@pytest.mark.parametrize("T,V,two", [(1203, 151936, False), (2207, 151936, False), (9, 4104, False), (2403, 151936, False),
                                     (1203, 151936, True), (5001, 32000, True), (9, 4104, True)])
def test_rows_kept_in_the_caches_between_the_passes(T, V, two):
    """All rows (9), the last ones only (1203 and 2207) and, in a one-tensor call past the line, none of them (2403) read by
    ordinary loads the first time, the second pass from the last row and there from the first; rows not a multiple of eight.
    The log-probs are those of the scoring call bit for bit, every gradient row is written, and sampled rows have the
    properties of c (softmax - onehot)."""
    if not two:
        nbytes = T // 3 * 3 * V * 2
        assert (nbytes <= CACHED) == (T == 9) and (nbytes > CACHED_TOTAL) == (T == 2403)
    B = 3
    w = wl.generate("reasoning", DEV, seed=T, B=B, len_lo=T // B, len_hi=T // B, V=V, **(dict(stale_logit_sigma=0.05) if two else {}))
    lens = w["seq_lens_host"].copy()
    T = int(lens.sum())
    lp, st = _pass_for(w), _pass_for(w, alloc_dlogits=False)
    lp.dlogits.fill_(7.0)
    if two:
        kl, ref = torch.empty(T, device=DEV), torch.empty(T, device=DEV)
        f32 = [torch.empty(T, device=DEV) for _ in range(3)]
        fb.fopd_loss_fwd_bwd_full_kl(w["logits"], w["logits_stale"], lp.dt, T, V, lp.ld, lp.ld, w["token_ids"], w["mask"],
                                     w["teacher_logp"], w["teacher_logp_stale"], w["seq_lens"], w["lag"], B, HP, None, None,
                                     None, 0, None, None, None, None, 1.0, lp.loss, lp.freshness, lp.weights, lp.logp, kl,
                                     lp.dlogits, lp.workspace)
        fb.fopd_rollout_kl(w["logits"], w["logits_stale"], lp.dt, T, V, lp.ld, lp.ld, w["token_ids"], w["mask"], ref,
                           f32[0], f32[1], f32[2], None, st.workspace)
        assert torch.equal(kl, ref) and torch.equal(lp.logp, f32[0])
    else:
        lp.loss_fwd_bwd(w, HP)
        st.token_logprobs(w)
        assert torch.equal(lp.logp, st.logp)
    assert lp.status() == (0, 0)
    rows = lp.dlogits[:, :V].float()
    assert not bool((rows == 7.0).any())
    # a row of c (softmax - onehot), or of p (d - E d), sums to zero up to the rounding of its bf16 entries (2^-9 each)
    assert bool((rows.sum(dim=1).abs() <= 2.0 ** -8 * rows.abs().sum(dim=1) + 1e-30).all())
    live = torch.repeat_interleave(lp.weights, w["seq_lens"].long()) > 0
    assert bool((rows.abs().sum(dim=1)[live & (w["mask"] != 0)] > 0).all())


@pytest.mark.parametrize("T,V", [(2403, 151936), (1203, 151936), (25011, 16384), (9, 4104)])
def test_both_gradient_kernels_on_both_sides_of_the_line(T, V):
    """The kernel of one 256-lane workgroup a row (the only one for rows of at most 2048 vectors: 25,011 x 16,384, which is
    past the line) and the one that holds a row in registers: the same bits, from the first row and from the last."""
    assert (T * V * 2 > CACHED_TOTAL) == (T > 2400)
    w = wl.generate("reasoning", DEV, seed=T, B=3, len_lo=T // 3, len_hi=T // 3, V=V)
    w["mask"][::5] = 0
    lp, st = _pass_for(w), _pass_for(w, alloc_dlogits=False)
    lp.dlogits.fill_(7.0)
    try:
        fb.fopd_set_option("k4_regs", 0)
        lp.loss_fwd_bwd(w, HP)
        rows, loss = lp.dlogits.clone(), lp.loss.clone()
        fb.fopd_set_option("k4_regs", 1)
        lp.dlogits.fill_(7.0)
        lp.loss_fwd_bwd(w, HP)
    finally:
        fb.fopd_set_option("k4_regs", 1)
    assert lp.status() == (0, 0)
    assert torch.equal(rows, lp.dlogits) and torch.equal(loss, lp.loss) and not bool((rows == 7.0).any())
    st.token_logprobs(w)
    assert torch.equal(lp.logp, st.logp)
    # sampled rows against c (softmax - onehot) in float64: bf16 entries (2^-9 each) of fp32 values
    live = torch.nonzero(torch.repeat_interleave(lp.weights, w["seq_lens"].long()) * (w["mask"] != 0))[:, 0]
    for t in live[[0, 1, len(live) // 2, -2, -1]].tolist() if len(live) > 4 else live.tolist():
        p = torch.softmax(w["logits"][t, :V].double(), 0)
        p[w["token_ids"][t].long()] -= 1.0
        g = rows[t, :V].double()
        c = (g * p).sum() / (p * p).sum()
        assert float((g - c * p).abs().max()) <= 2.0 ** -8 * float((c * p).abs().max())
