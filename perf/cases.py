"""What a training or scoring program has this library do, as cases that can be timed.

Each case is one call (or the two calls that belong together) of the public entry points on inputs of the kind that
buffered rollouts give: logits of a language model in HBM, or its last hidden states and output projection, ragged
samples, masked observation spans, stored behaviour and teacher log-probabilities, lags.  The shapes are those of the
repository's own workloads (a tiny batch in fp32; reasoning, tool use and coding rollouts at a vocabulary of 151,936;
262,144 entries for the large vocabulary; hidden size 4096 for the projection), cut to batches of which three fit a
card, plus a vocabulary of 32,000, a common size between the two.
"""

import functools
import math
import random

import numpy as np
import torch

from paper_2605_17862_amd import binding as fb
from paper_2605_17862_amd.loss_pass import LossPass

DEV = "cuda:0"
HP = (1.0, 1.0, 0.05, 0.1)          # alpha, beta, xi, lambda: the defaults of the repository's benchmark
REST_FLOOR = 1e-4                   # least teacher probability of "any other token" with a listed teacher

# op        step       everything in one call: log-probs, scores, weights, loss, gradient (fopd_loss_fwd_bwd)
#           minibatch  the same with the scores of an earlier scoring loop (freshness_in)
#           unit       the whole pass with the logits read once (fopd_loss_fwd_bwd_unit)
#           score      the scoring loop: log-probs with token entropy, then the samples' scores
#           full_kl    drift from the stale checkpoint's logits (a second [T, V] tensor)
#           teacher    distribution-level loss against the teacher's logits (a second [T, V] tensor)
#           topk       distribution-level loss against a teacher stored as k tokens per row
#           lm_logps   log-probs straight from hidden states, projection fused
#           lm_loss    loss and both gradients through the projection; scored: scores supplied or formed inside
# T rows, B samples, V vocabulary, dtype of the stored logits, d hidden size, spans: plain (every row trains), turns
# (masked observation, then response) or coding (long responses and observations in turn), max_lag, k listed tokens


def listed():
    return [
        # the repository's tiny configuration: four short samples in fp32.  Latency and launches are what counts.
        dict(name="step_tiny_f32", op="step", dtype="f32", T=512, B=4, V=4096, spans="plain", max_lag=3),
        # many short rows of a mid-sized vocabulary, an odd number of them
        dict(name="step_short_rows", op="step", dtype="bf16", T=12289, B=24, V=32000, spans="plain", max_lag=4),
        # a fifth of the benchmark's reasoning batch: the ordinary training step on stored logits
        dict(name="step_reasoning", op="step", dtype="bf16", T=32768, B=13, V=151936, spans="plain", max_lag=4),
        # the large vocabulary: a row does not fit one compute unit's registers; half the samples very stale, some gated
        dict(name="step_largevocab", op="step", dtype="bf16", T=8192, B=8, V=262144, spans="plain", max_lag=32),
        # a minibatch of tool-use rollouts after the scoring loop: a third of the rows is masked
        dict(name="minibatch_tooluse", op="minibatch", dtype="bf16", T=15602, B=2, V=151936, spans="turns", max_lag=8),
        # one chunk of the scoring loop over long coding trajectories, stale teacher context present
        dict(name="score_coding", op="score", dtype="bf16", T=16384, B=2, V=151936, spans="coding", max_lag=16),
        # drift diagnostic from the stale checkpoint's full logits
        dict(name="full_kl_reasoning", op="full_kl", dtype="bf16", T=8192, B=4, V=151936, spans="plain", max_lag=4),
        # teacher stored as 64 tokens per row
        dict(name="topk_reasoning", op="topk", dtype="bf16", T=8192, B=4, V=151936, spans="plain", max_lag=4, k=64),
        # log-probs of one short rollout from its hidden states
        dict(name="lm_logps_one_rollout", op="lm_logps", T=300, B=1, V=151936, d=4096, spans="plain", max_lag=4),
        # log-probs of a scoring batch from hidden states
        dict(name="lm_logps_reasoning", op="lm_logps", T=16384, B=7, V=151936, d=4096, spans="plain", max_lag=4),
        # one micro-batch of a short rollout through the projection, scores formed inside
        dict(name="lm_loss_one_rollout", op="lm_loss", scored=False, T=512, B=1, V=151936, d=4096, spans="plain",
             max_lag=0),
        # a training batch through the projection after the scoring loop
        dict(name="lm_loss_reasoning", op="lm_loss", scored=True, T=16384, B=7, V=151936, d=4096, spans="plain",
             max_lag=4),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["step", "step", "minibatch", "unit", "score", "full_kl", "teacher", "topk", "lm_logps", "lm_loss"])
    if op in ("lm_logps", "lm_loss"):
        V = rng.choice([32000, 151936, _log_uniform(rng, 32000, 151936)])
        d = rng.choice([4096, 64 * rng.randint(16, 64)])
        T = _log_uniform(rng, 256, 16384)
        case = dict(op=op, V=V, d=d)
        if op == "lm_loss":
            case["scored"] = rng.random() < 0.5
    else:
        dtype = "f32" if rng.random() < 0.25 else "bf16"
        V = rng.choice([4096, 32000, 151936, 262144, _log_uniform(rng, 4096, 262144), _log_uniform(rng, 4096, 262144)])
        most = 4.9e9 if op in ("step", "minibatch", "unit") else 2.4e9        # entries x 2 bytes: as the listed cases
        T = _log_uniform(rng, 256, max(257, min(32768, int(most / (V * (2 if dtype == "f32" else 1))))))
        case = dict(op=op, dtype=dtype, V=V)
        if op == "topk":
            case["k"] = rng.choice([16, 64, 100])
    case.update(T=T, B=rng.randint(1, max(1, min(32, T // 64))), spans=rng.choice(["plain", "turns", "coding"]),
                max_lag=rng.choice([4, 8, 16]))
    return case


# ---- what the batch looks like: a function of the case alone, so that the work is the case's --------------------

@functools.lru_cache(maxsize=64)
def _structure_of(key):
    case = dict(key)
    rs = random.Random("%d %d %s %d" % (case["T"], case["B"], case["spans"], case["max_lag"]))
    T, B = case["T"], case["B"]
    parts = [rs.uniform(0.25, 1.75) for _ in range(B)]               # ragged, as U{512..4096} is
    lens = [max(1, int(p / sum(parts) * T)) for p in parts]
    lens[-1] += T - sum(lens)
    mask = np.ones(T, dtype=np.uint8)
    if case["spans"] != "plain":
        (obs_lo, obs_hi), (resp_lo, resp_hi) = (((128, 512), (256, 1024)) if case["spans"] == "turns"
                                                else ((256, 1536), (512, 2048)))
        at = 0
        for n in lens:
            here, train = 0, case["spans"] == "coding" or n <= obs_hi          # tool use starts with an observation
            while here < n:
                span = min(n - here, rs.randint(resp_lo, resp_hi) if train else rs.randint(obs_lo, obs_hi))
                if not train:
                    mask[at + here:at + here + span] = 0
                here += span
                train = not train
            at += n
    lag = [rs.randint(0, case["max_lag"]) for _ in range(B)]
    lag[0] = max(lag[0], min(1, case["max_lag"]))                    # drift of an all-fresh batch is rounding noise
    if case["max_lag"] >= 32:                                        # half fresh, half very stale: some are gated
        lag = [0 if i < B // 2 else rs.randint(8, 32) for i in range(B)]
    return np.array(lens, dtype=np.int32), mask, np.array(lag, dtype=np.int32)


def _structure(case):
    return _structure_of(tuple(sorted((k, case[k]) for k in ("T", "B", "spans", "max_lag"))))


def _ld(case):
    per = 4 if case["dtype"] == "f32" else 8
    return (case["V"] + per - 1) // per * per                        # rows are 16-byte aligned


def _row_gated(case):
    """Rows of samples whose lag alone puts the score 1 / (lag + 1) under the gate (their gradient rows are zeros)."""
    lens, mask, lag = _structure(case)
    return np.repeat(1.0 / (lag + 1.0) <= HP[2], lens)


def _logit_rows(z, gen):
    """Raw logits in place: N(0, 3^2) with 32 strongly preferred tokens per row."""
    z.normal_(0.0, 3.0, generator=gen)
    n, V = z.shape
    at = torch.randint(0, V, (n, 32), generator=gen, device=z.device)
    z.scatter_add_(1, at, torch.full((n, 32), 8.0, device=z.device))
    return z


def _draw_tokens(z, gen):
    """Tokens from softmax(z) (by exponential races) and their log-probabilities."""
    u = torch.empty_like(z).exponential_(1.0, generator=gen)
    y = torch.argmax(z - u.clamp_(min=1e-30).log_(), dim=1)
    return y, z.gather(1, y[:, None])[:, 0] - torch.logsumexp(z, dim=1)


def _workspace(nbytes):
    ws = torch.empty(nbytes + 256, dtype=torch.uint8, device=DEV)
    off = (-ws.data_ptr()) % 256
    ws = ws[off:off + nbytes]
    fb.fopd_workspace_init(ws)
    return ws


def prepare(case, seed):
    T, B, V, op = case["T"], case["B"], case["V"], case["op"]
    lens, mask, lag = _structure(case)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed) * 1000003 + 17)
    s = dict(case=case, mask=torch.from_numpy(mask).to(DEV), seq_lens=torch.from_numpy(lens).to(DEV),
             lag=torch.from_numpy(lag).to(DEV), seq_lens_host=lens,
             token_ids=torch.empty(T, dtype=torch.int32, device=DEV))
    logp = torch.empty(T, device=DEV)
    rows = max(64, min(T, (1 << 27) // V))
    if op in ("lm_logps", "lm_loss"):
        d = case["d"]
        s["hidden"] = torch.randn(T, d, generator=gen, device=DEV).to(torch.bfloat16)
        s["weight"] = (torch.randn(V, d, generator=gen, device=DEV) * (3.0 / d ** 0.5)).to(torch.bfloat16)
        for a in range(0, T, rows):
            b = min(a + rows, T)
            y, logp[a:b] = _draw_tokens((s["hidden"][a:b] @ s["weight"].t()).float(), gen)
            s["token_ids"][a:b] = y.to(torch.int32)
    else:
        ld = _ld(case)
        dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
        s["logits"] = torch.zeros(T, ld, dtype=dtype, device=DEV) if ld > V else torch.empty(T, ld, dtype=dtype, device=DEV)
        if op in ("full_kl", "teacher"):
            s["second"] = torch.zeros_like(s["logits"]) if ld > V else torch.empty_like(s["logits"])
        if op == "topk":
            s["list_ids"] = torch.empty(T, case["k"], dtype=torch.int32, device=DEV)
            s["list_logp"] = torch.empty(T, case["k"], device=DEV)
        row_lag = torch.from_numpy(np.repeat(lag, lens).astype(np.float32)).to(DEV)
        for a in range(0, T, rows):
            b = min(a + rows, T)
            raw = _logit_rows(torch.empty(b - a, V, device=DEV), gen)
            s["logits"][a:b, :V] = raw
            z = s["logits"][a:b, :V].float()
            y, logp[a:b] = _draw_tokens(z, gen)
            s["token_ids"][a:b] = y.to(torch.int32)
            if op in ("full_kl", "teacher"):      # a few updates apart: 0.03 per update; the teacher further away
                sigma = (0.03 * row_lag[a:b, None]) if op == "full_kl" else 0.3
                s["second"][a:b, :V] = torch.randn(b - a, V, generator=gen, device=DEV).mul_(sigma).add_(raw)
            if op == "topk":
                zq = torch.randn(b - a, V, generator=gen, device=DEV).mul_(0.3).add_(z)
                top = torch.topk(zq, case["k"], dim=1)
                s["list_ids"][a:b] = top.indices.to(torch.int32)
                s["list_logp"][a:b] = top.values - torch.logsumexp(zq, dim=1, keepdim=True)
    # what the rollout and the teacher left in the buffer
    per_row = torch.from_numpy(np.repeat(lag, lens).astype(np.float32)).to(DEV)
    noise = torch.randn(3, T, generator=gen, device=DEV)
    s["behav_logp"] = torch.clamp(logp + 0.05 * per_row * noise[0], max=0.0)
    s["teacher_logp"] = torch.clamp(logp - 0.2 + 0.4 * noise[1], max=0.0)
    s["teacher_logp_stale"] = (torch.clamp(s["teacher_logp"] + 0.1 * per_row * noise[2], max=0.0)
                               if case["spans"] == "coding" else None)

    # buffers and workspaces that a program keeps from step to step
    f32 = dict(dtype=torch.float32, device=DEV)
    if op in ("lm_logps", "lm_loss"):
        s["logp"], s["lse"] = torch.empty(T, **f32), torch.empty(T, **f32)
        if op == "lm_logps":
            s["ws"] = _workspace(fb.fopd_lm_head_workspace_bytes(T))
            return s
        s["loss"], s["weights"], s["freshness"] = torch.empty(1, **f32), torch.empty(B, **f32), torch.empty(B, **f32)
        s["dhidden"], s["dweight"] = torch.empty(T, d, **f32), torch.empty(V, d, **f32)
        s["rows_chunk"] = min(16384, (T + 63) // 64 * 64)
        s["ws"] = _workspace(fb.fopd_lm_head_loss_workspace_bytes(T, V, d, B, s["rows_chunk"]))
    else:
        s["lp"] = LossPass(T, V, B, case["dtype"], ld=ld, device=DEV, alloc_dlogits=(op != "score"))
        if op == "score":
            s["lp"].entropy = torch.empty(T, **f32)
        if op in ("full_kl", "teacher", "topk"):
            s["token_term"] = torch.empty(T, **f32)
        if op == "topk":
            s["ws"] = _workspace(fb.fopd_topk_workspace_bytes(T, B, case["k"]))
        if ld > V and op != "score":
            s["lp"].dlogits.zero_()                                  # padding columns are never written
    if op == "minibatch" or (op == "lm_loss" and case["scored"]):    # the scoring loop before the minibatch loop
        p = s["lp"] if op == "minibatch" else LossPass(T, 8, B, "bf16", device=DEV, alloc_dlogits=False)
        p.logp.copy_(torch.where(s["mask"] != 0, logp, torch.zeros_like(logp)))
        p.freshness_score(s, HP)
        s["freshness_in"] = p.freshness.clone()
        s["n_train"], s["n_roll"] = p.n_train.clone(), p.n_roll.clone()
    return s


def run(s):
    case = s["case"]
    T, B, V, op = case["T"], case["B"], case["V"], case["op"]
    if op == "lm_logps":
        fb.fopd_lm_head_token_logprobs(s["hidden"], case["d"], s["weight"], case["d"], T, V, case["d"], s["token_ids"],
                                       s["mask"], s["logp"], s["lse"], s["ws"])
        return {"logp": s["logp"], "lse": s["lse"]}
    if op == "lm_loss":
        d, scored = case["d"], case["scored"]
        fb.fopd_lm_head_loss_fwd_bwd(s["hidden"], d, s["weight"], d, T, V, d, s["token_ids"], s["mask"],
                                     s["behav_logp"], s["teacher_logp"], s["seq_lens"], s["lag"], B, HP,
                                     s["freshness_in"] if scored else None, s["n_train"] if scored else None,
                                     s["n_roll"] if scored else None, 1.0, s["rows_chunk"], s["loss"], s["weights"],
                                     s["logp"], s["lse"], s["dhidden"], d, s["dweight"], d, False, s["ws"],
                                     seq_lens_host=None if scored else s["seq_lens_host"], freshness=s["freshness"])
        return {k: s[k] for k in ("loss", "weights", "freshness", "logp", "lse", "dhidden", "dweight")}
    p = s["lp"]
    if op == "score":
        p.token_logprobs(s, want_entropy=True)
        p.freshness_score(s, HP)
        return {k: getattr(p, k) for k in ("logp", "lse", "gather_idx", "entropy", "cu_seqlens", "n_train", "n_roll",
                                           "D_roll", "D_sup", "ell", "cover", "cover_roll", "freshness", "agg")}
    out = {"loss": p.loss, "freshness": p.freshness, "weights": p.weights, "logp": p.logp, "grad": p.dlogits}
    if op == "step":
        p.loss_fwd_bwd(s, HP)
    elif op == "minibatch":
        fb.fopd_loss_fwd_bwd(s["logits"], p.dt, T, V, p.ld, s["token_ids"], s["mask"], s["behav_logp"],
                             s["teacher_logp"], s["teacher_logp_stale"], s["seq_lens"], s["lag"], B, HP,
                             s["freshness_in"], s["n_train"], s["n_roll"], 0, None, None, 1.0, p.loss, p.freshness,
                             p.weights, p.logp, p.dlogits, p.workspace)
    elif op == "unit":
        fb.fopd_loss_fwd_bwd_unit(s["logits"], p.dt, T, V, p.ld, s["token_ids"], s["mask"], s["behav_logp"],
                                  s["teacher_logp"], s["teacher_logp_stale"], s["seq_lens"], s["lag"], B, HP, 1.0,
                                  p.loss, p.freshness, p.weights, p.logp, p.dlogits, p.workspace)
    elif op == "full_kl":
        out["token_term"] = s["token_term"]
        fb.fopd_loss_fwd_bwd_full_kl(s["logits"], s["second"], p.dt, T, V, p.ld, p.ld, s["token_ids"], s["mask"],
                                     s["teacher_logp"], s["teacher_logp_stale"], s["seq_lens"], s["lag"], B, HP, None,
                                     None, None, 0, None, None, None, None, 1.0, p.loss, p.freshness, p.weights, p.logp,
                                     s["token_term"], p.dlogits, p.workspace)
    elif op == "teacher":
        out["token_term"] = s["token_term"]
        fb.fopd_loss_fwd_bwd_full_teacher(s["logits"], s["second"], p.dt, T, V, p.ld, p.ld, s["token_ids"], s["mask"],
                                          s["behav_logp"], s["teacher_logp_stale"], s["seq_lens"], s["lag"], B, HP,
                                          None, None, None, 0, None, None, None, None, 1.0, p.loss, p.freshness,
                                          p.weights, p.logp, s["token_term"], p.dlogits, p.workspace)
    elif op == "topk":
        out["token_term"] = s["token_term"]
        fb.fopd_loss_fwd_bwd_topk_teacher(s["logits"], p.dt, T, V, p.ld, s["token_ids"], s["mask"], s["behav_logp"],
                                          s["list_ids"], s["list_logp"], case["k"], REST_FLOOR, s["teacher_logp"],
                                          s["teacher_logp_stale"], s["seq_lens"], s["lag"], B, HP, None, None, None, 0,
                                          None, None, 1.0, p.loss, p.freshness, p.weights, p.logp, s["token_term"],
                                          p.dlogits, s["ws"])
    else:
        raise ValueError(op)
    return out


def work(case):
    """Bytes: each input read once and each output written once; rows that are masked are not read, their gradient
    rows are written as zeros.  Flops: the contractions of the rows that take part in them."""
    lens, mask, lag = _structure(case)
    T, V, op = case["T"], case["V"], case["op"]
    live = int((mask != 0).sum())
    with_grad = int(((mask != 0) & ~_row_gated(case)).sum())
    per_row = 4 * T * 6
    if op in ("lm_logps", "lm_loss"):
        d = case["d"]
        io = 2 * V * d + 2 * live * d + per_row
        if op == "lm_logps":
            return {"bytes": io, "flops": 2 * live * V * d}
        return {"bytes": io + 4 * T * d + 4 * V * d, "flops": 2 * V * d * (live + 2 * with_grad)}
    e = 4 if case["dtype"] == "f32" else 2
    row = V * e
    total = live * row + per_row
    if op != "score":
        total += T * row
    if op in ("full_kl", "teacher"):
        total += live * row
    if op == "topk":
        total += live * case["k"] * 8
    return {"bytes": total, "flops": 0}


def tolerance(case):
    """Four times the distance measured between the library and the same pass in float64 rounded where the path stores
    (several seeds and sizes; rel / max): log-probs and scores 4e-7 / 2.3e-6; with an fp32 gradient 2e-6 (listed
    teacher's token loss) / 5e-4 (gradient rows whose coefficient nearly cancels); with a bf16 one 9.4e-5 / one unit in
    its last place; sums of bf16 gradient rows through the projection 1.2e-4 / 9e-3."""
    op = case["op"]
    if op == "lm_loss":
        return {"rel": 5e-4, "max": 0.036}
    if op in ("lm_logps", "score"):
        return {"rel": 1.6e-6, "max": 1e-5}
    if case["dtype"] == "f32":
        return {"rel": 8e-6, "max": 2e-3}
    return {"rel": 4e-4, "max": 0.03}
