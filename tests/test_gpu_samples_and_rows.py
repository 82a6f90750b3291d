"""Numbers of samples and rows around the lines where a call forms the samples' offsets (1024 samples) and the row
coefficients (2048 rows) inside the statistics kernel, against float64, and the error flags of the offsets there."""

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


@pytest.mark.parametrize("T,V,two", [(1203, 151936, False), (2207, 151936, False), (9, 4104, False), (1203, 151936, True),
                                     (5001, 32000, True), (9, 4104, True)])
def test_rows_kept_in_the_caches_between_the_passes(T, V, two):
    """All rows, the last ones only and none of them read by ordinary loads the first time, the second pass from the last row
    and from the first; rows not a multiple of eight.  The log-probs are those of the scoring call bit for bit, every gradient
    row is written, and sampled rows have the properties of c (softmax - onehot)."""
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
