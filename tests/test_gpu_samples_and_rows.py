"""Numbers of samples and rows around the lines where a call forms the samples' offsets (1024 samples) and the row
coefficients (2048 rows) inside the statistics kernel, against float64, and the error flags of the offsets there."""

import numpy as np
import pytest
import torch

from harness import workloads as wl
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
