"""The projection kernels at few rows, where a launch is made of short work items: token counts around the edges of
the 256-row tiles and of the groups of tiles (1, 2, 3, 4, 5 tiles), with and without masked rows, against float64."""

import numpy as np
import pytest
import torch

from harness import workloads as wl
from oracle import fopd_oracle as orc
from paper_2605_17862_amd import binding as fb
from parity_util import np64
from projection_cases import STRIPS_OF_SEVERAL_TILES
from test_gpu_projection_loss import _compare, _run, _scores_from_the_oracle

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _aligned(nbytes):
    ws = torch.empty(nbytes + 256, dtype=torch.uint8, device=DEV)
    off = (-ws.data_ptr()) % 256
    ws = ws[off:off + nbytes]
    fb.fopd_workspace_init(ws)
    return ws


@pytest.mark.parametrize("T", [1, 255, 256, 257, 512, 513, 1024, 1029])
@pytest.mark.parametrize("masked_every", [0, 3])
def test_log_probs_at_the_edges_of_tiles_and_groups(T, masked_every):
    # 79 vocabulary tiles, the last with 33 entries; 1e-4 as everywhere for log-probs of fp32 sums over bf16 products
    w = wl.generate_lm_head(T, 64, 20001, DEV, seed=T, masked_every=masked_every)
    ws = _aligned(fb.fopd_lm_head_workspace_bytes(T))
    ref_lse, ref_lp = orc.lm_head_token_logprobs(np64(w["hidden"].float()), np64(w["weight"].float()),
                                                 w["token_ids"].cpu().numpy(), w["mask"].cpu().numpy())
    for mask in ([w["mask"]] if masked_every else [w["mask"], None]):
        logp = torch.full((T,), 7.0, device=DEV)
        lse = torch.full((T,), 7.0, device=DEV)
        fb.fopd_lm_head_token_logprobs(w["hidden"], w["ldh"], w["weight"], w["ldw"], T, w["V"], w["d"],
                                       w["token_ids"], mask, logp, lse, ws)
        assert fb.fopd_workspace_status(ws) == (0, 0)
        assert np.max(np.abs(np64(lse) - ref_lse)) <= 1e-4 and np.max(np.abs(np64(logp) - ref_lp)) <= 1e-4


@pytest.mark.parametrize("T", [64, 128, 129, 300, 384, 385, 600, 1100])
@pytest.mark.parametrize("d,V", [(64, 20001), (192, 20001), (128, 100), (64, 385)])
def test_log_probs_with_a_last_tile_of_few_tokens(T, d, V):
    """A last tile of up to 128 tokens alone, beside 2 whole ones with the same strips and, with 20,001 entries, beside 4 with strips
    of its own, and one token more; beside one, all tokens in one tile, one vocabulary tile a strip; one to three steps a
    vocabulary tile, vocabularies of less than a tile and of an entry more than whole ones.  Half of the rows masked moves the
    last tile to another place than the launch was made for."""
    w = wl.generate_lm_head(T, d, V, DEV, seed=T + d)
    ws = _aligned(fb.fopd_lm_head_workspace_bytes(T))
    half = torch.ones(T, dtype=torch.uint8, device=DEV)
    half[::2] = 0
    for mask in (None, half):
        ref_lse, ref_lp = orc.lm_head_token_logprobs(np64(w["hidden"].float()), np64(w["weight"].float()),
                                                     w["token_ids"].cpu().numpy(), None if mask is None else mask.cpu().numpy())
        logp = torch.full((T,), 7.0, device=DEV)
        lse = torch.full((T,), 7.0, device=DEV)
        fb.fopd_lm_head_token_logprobs(w["hidden"], w["ldh"], w["weight"], w["ldw"], T, w["V"], w["d"],
                                       w["token_ids"], mask, logp, lse, ws)
        assert fb.fopd_workspace_status(ws) == (0, 0)
        assert np.max(np.abs(np64(lse) - ref_lse)) <= 1e-4 and np.max(np.abs(np64(logp) - ref_lp)) <= 1e-4


@pytest.mark.parametrize("T,masked_every", [(300, 2), (600, 2), (600, 3), (1100, 9)])
def test_masked_rows_left_out_or_projected_give_the_same_bits(T, masked_every):
    """All tokens in one tile (300 rows), three tiles with the same strips (600) and four with a last one with strips of its own,
    which has no unmasked row (1100): an unmasked row is summed over the same strips whether the masked rows are projected or
    not.  Unmasked rows in the last one's own strips: the next test."""
    w = wl.generate_lm_head(T, 64, 20001, DEV, seed=T, masked_every=masked_every)
    ws = _aligned(fb.fopd_lm_head_workspace_bytes(T))
    out = {}
    try:
        for compact in (0, 1):
            fb.fopd_set_option("lm_head_compact", compact)
            logp, lse = torch.full((T,), 7.0, device=DEV), torch.full((T,), 7.0, device=DEV)
            fb.fopd_lm_head_token_logprobs(w["hidden"], w["ldh"], w["weight"], w["ldw"], T, w["V"], w["d"],
                                           w["token_ids"], w["mask"], logp, lse, ws)
            out[compact] = (logp, lse)
    finally:
        fb.fopd_set_option("lm_head_compact", 1)
    assert not bool(out[0][0][w["mask"] == 0].any())
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("T,V,form,whole", STRIPS_OF_SEVERAL_TILES)
@pytest.mark.parametrize("d,sigma", [(64, 3.0), (192, 40.0)])
def test_log_probs_of_strips_with_several_vocabulary_tiles(T, V, form, whole, d, sigma):
    """In every form of the token tiles the requests run on from one vocabulary tile into the next, after one or after three steps,
    and the running pair of a token is carried over; with a spread of 40 its reference rises by tens on the way.  No mask, and
    every 20th row masked, which leaves unmasked rows in a last tile with strips of its own; the same bits where the masked rows
    are projected too."""
    w = wl.generate_lm_head(T, d, V, DEV, seed=T + d, logit_sigma=sigma, masked_every=20)
    ws = _aligned(fb.fopd_lm_head_workspace_bytes(T))
    some = w["mask"]
    assert form != "own" or int(some.sum()) > whole
    ref_lse, ref_lp = orc.lm_head_token_logprobs(np64(w["hidden"].float()), np64(w["weight"].float()),
                                                 w["token_ids"].cpu().numpy(), None)

    def call(mask):
        logp, lse = torch.full((T,), 7.0, device=DEV), torch.full((T,), 7.0, device=DEV)
        fb.fopd_lm_head_token_logprobs(w["hidden"], w["ldh"], w["weight"], w["ldw"], T, V, d, w["token_ids"], mask, logp, lse, ws)
        assert fb.fopd_workspace_status(ws) == (0, 0)
        return logp, lse

    # fp32 sums of d products: a few 1e-6 on a logit of the ordinary spread, a few 1e-5 on one of magnitude 150
    atol = 1e-4 if sigma <= 3.0 else 2e-4
    try:
        for mask in (None, some):
            fb.fopd_set_option("lm_head_compact", 1)
            logp, lse = call(mask)
            live = np.ones(T, dtype=bool) if mask is None else mask.cpu().numpy() != 0
            assert np.all(np.abs(np64(lse) - ref_lse)[live] <= atol + 2e-6 * np.abs(ref_lse)[live])
            assert np.all(np.abs(np64(logp) - ref_lp)[live] <= atol + 2e-6 * np.abs(ref_lp)[live])
            assert not np64(lse)[~live].any() and not np64(logp)[~live].any()
            fb.fopd_set_option("lm_head_compact", 0)
            again = call(mask)
            assert torch.equal(logp, again[0]) and torch.equal(lse, again[1])
    finally:
        fb.fopd_set_option("lm_head_compact", 1)


@pytest.mark.parametrize("seq,d,pad_h", [((1,), 64, 0), ((40, 25), 64, 2), ((100, 157), 320, 4), ((300, 214), 512, 3),
                                          ((500, 260), 320, 4), ((700, 500), 128, 0)])
def test_gradients_with_the_vocabulary_cut_into_runs(seq, d, pad_h):
    """One to six result tiles of dL/dhidden, one to five along the rows: the contraction over 20,001 entries is cut into
    runs and the scatter sums them, into rows whose pitch is and is not a multiple of four."""
    T = sum(seq)
    h = wl.generate_lm_head(T, d, 20001, DEV, seed=T, masked_every=4 if T > 1 else 0)
    w = wl.attach_loss_inputs(h, seq, [1, 3][:len(seq)], seed=T)
    scores = _scores_from_the_oracle(w, (1.0, 1.0, 0.05, 0.1))
    out = _run(w, (1.0, 1.0, 0.05, 0.1), 1.0, (T + 63) // 64 * 64, scores, pad_h=pad_h)
    _compare(w, (1.0, 1.0, 0.05, 0.1), 1.0, out, scores)


@pytest.mark.parametrize("T", [4096, 4097])
@pytest.mark.parametrize("V,d", [(129, 64), (200, 192)])
def test_gradients_at_the_line_between_the_two_layouts_of_the_projection_matrix(T, V, d):
    """4096 rows take dL/dhidden from the matrix as it is, its last step with fewer rows than 64; 4097 from a transposed
    copy.  A pitch wider than the rows of the matrix in both."""
    h = wl.generate_lm_head(T, d, V, DEV, seed=T, masked_every=5, ldw=d + 8)
    w = wl.attach_loss_inputs(h, (T - 1500, 1500), [1, 3], seed=T)
    scores = _scores_from_the_oracle(w, (1.0, 1.0, 0.05, 0.1))
    out = _run(w, (1.0, 1.0, 0.05, 0.1), 1.0, 4160, scores)
    _compare(w, (1.0, 1.0, 0.05, 0.1), 1.0, out, scores)


@pytest.mark.parametrize("seq,d", [((40, 23), 64), ((40, 24), 128), ((70, 58, 1), 64), ((90, 110), 192), ((330, 200), 64)])
def test_gradients_with_more_result_tiles_than_workgroups(seq, d):
    """274 vocabulary tiles, the last with 113 entries: workgroups walk from one tile to the next, which changes after every step
    (64 hidden elements, 64 rows), every second or third, or later.  A third of the rows masked, the first sample gated out: the
    hidden rows of the others are gathered and transposed, 64 to 128 of them or a few more than 128."""
    T = sum(seq)
    h = wl.generate_lm_head(T, d, 70001, DEV, seed=T + d, masked_every=3)
    w = wl.attach_loss_inputs(h, seq, [45] + [1] * (len(seq) - 1), seed=T)
    scores = _scores_from_the_oracle(w, (1.0, 1.0, 0.05, 0.1))
    out = _run(w, (1.0, 1.0, 0.05, 0.1), 1.0, (T + 63) // 64 * 64, scores, pad_w=4)
    _compare(w, (1.0, 1.0, 0.05, 0.1), 1.0, out, scores)
    first = torch.zeros(70001, d, device=DEV)
    again = _run(w, (1.0, 1.0, 0.05, 0.1), 1.0, (T + 63) // 64 * 64, scores, accumulate=True, dweight=first)
    assert torch.equal(again["dweight"], out["dweight"])


@pytest.mark.parametrize("T", [4096, 4097])
def test_gradients_with_more_tiles_of_dhidden_than_workgroups(T):
    """Four steps over 200 vocabulary entries, the last one of 8, and 16 or 17 times 18 tiles of dL/dhidden, the last one of 64
    hidden elements: workgroups walk from tile to tile in both layouts of the projection matrix (4096 and 4097 rows)."""
    h = wl.generate_lm_head(T, 4416, 200, DEV, seed=T, masked_every=7)
    w = wl.attach_loss_inputs(h, (T - 700, 700), [1, 2], seed=T)
    scores = _scores_from_the_oracle(w, (1.0, 1.0, 0.05, 0.1))
    out = _run(w, (1.0, 1.0, 0.05, 0.1), 1.0, 4160, scores)
    _compare(w, (1.0, 1.0, 0.05, 0.1), 1.0, out, scores)


@pytest.mark.parametrize("T,d,V", [(2304, 1024, 3000), (4096, 576, 200), (1100, 1856, 3001)])
def test_dhidden_of_few_and_of_many_tiles_has_the_same_bits(T, d, V):
    """40 to 72 tiles of dL/dhidden in one chunk, 3 to 8 a chunk of 256 rows, which go through the other matrix instruction: a
    row's sum is the same.  The last tile of 64 hidden elements or of few rows, the last step of 8, 56 or 57 vocabulary entries.
    (Entries are bounded one by one, two units in the last place of each bf16 gradient entry; one alone, 2^-8 of it, is more than
    2e-3 of the largest result where a single entry makes that.)"""
    h = wl.generate_lm_head(T, d, V, DEV, seed=T, masked_every=5)
    w = wl.attach_loss_inputs(h, (T - 300, 300), [1, 3], seed=T)
    scores = _scores_from_the_oracle(w, (1.0, 1.0, 0.05, 0.1))
    out = _run(w, (1.0, 1.0, 0.05, 0.1), 1.0, (T + 63) // 64 * 64, scores)
    _compare(w, (1.0, 1.0, 0.05, 0.1), 1.0, out, scores, check_scale=False)
    chunks = _run(w, (1.0, 1.0, 0.05, 0.1), 1.0, 256, scores)
    _compare(w, (1.0, 1.0, 0.05, 0.1), 1.0, chunks, scores, check_scale=False)
    assert torch.equal(out["dhidden"], chunks["dhidden"])
