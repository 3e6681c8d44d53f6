"""The calls whose time matters: one training, audit or analysis step through the library's
public entry points, on rollouts that look like a trained policy's.

Every case is a plain dict; `path` says which entry point it takes.

* fused  -- adwin_opd_fused: hidden states and LM heads in, losses and gradients out.
  `job` is what the caller wants of it: "train" (prefix window, gradient to the hidden
  states), "probe" (every position, prefix and full gradients, alignment and the candidate
  windows), "head" (train plus the gradient of the student LM head), "stats" (every position,
  losses and the teacher diagnostics, no gradient).
* logits -- adwin_opd_from_logits: logits in, losses and logit gradient out; `job` "train" or
  "diag" (train plus the teacher diagnostics).

`api`: "handle" keeps the marshalled call with its outputs and workspace and runs it again, as
a loop over batches of one shape does; "function" is the one-call form, which a program whose
rollouts differ from step to step uses; "static" (logits) is the form that takes no workspace.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2605_28396_amd import binding as B
from paper_2605_28396_amd import synth

V_FULL = 151936                                     # vocabulary of the benchmark configurations
CANDIDATES = (64, 128, 256, 512, 1024, 1536, 2048)  # candidate windows of the scheduler
TOPK = 20                                           # rejection depth of the drift diagnostics


def _fused(name, job, B_, lens, window, V=V_FULL, H_s=2048, H_t=4096, estimator="expected", dh="f32",
           api="handle"):
    return {"name": name, "path": "fused", "job": job, "B": B_, "len_lo": lens[0], "len_hi": lens[1],
            "window": window, "V": V, "H_s": H_s, "H_t": H_t, "estimator": estimator, "dh": dh, "api": api}


def _logits(name, job, B_, lens, window, V=V_FULL, estimator="expected", api="handle"):
    return {"name": name, "path": "logits", "job": job, "B": B_, "len_lo": lens[0], "len_hi": lens[1],
            "window": window, "V": V, "estimator": estimator, "api": api}


def listed():
    return [
        # a toy vocabulary and two short rollouts: what a unit test or a debugging run calls all
        # day; nothing but launches and latency
        _fused("fused_tiny", "train", 2, (96, 128), "uniform", V=4096, H_s=256, H_t=384, api="function"),
        # small ragged audit: odd vocabulary, hidden sizes that are no multiple of a tile
        _fused("fused_ragged_probe", "probe", 9, (1, 700), "uniform", V=11912, H_s=512, H_t=640, api="function"),
        # one rollout supervised as soon as it arrives
        _fused("fused_one_rollout", "train", 1, (337, 337), 256, api="function"),
        # the start of the schedule: the benchmark's batch at the shortest candidate window
        _fused("fused_first_window", "train", 64, (1024, 8192), 64, dh="bf16"),
        # the benchmark's headline batch
        _fused("fused_strong_to_weak", "train", 64, (1024, 8192), 1024),
        # student and teacher of one family, a window per rollout, the sampled-token estimator
        _fused("fused_same_family_sampled", "train", 32, (512, 4096), "mixed", H_s=2560, estimator="sampled", dh="bf16"),
        # the probe audit over whole long rollouts with the candidate list
        _fused("fused_probe_alignment", "probe", 16, (8192, 16384), 2048),
        # training of the LM head itself
        _fused("fused_head_grad", "head", 16, (512, 4096), 512, dh="bf16"),
        # drift analysis of finished rollouts: statistics only
        _fused("fused_stats", "stats", 8, (1024, 8192), 1024),
        # a few rows of logits from a serving loop that owns no workspace
        _logits("logits_few_rows", "train", 1, (37, 37), 29, api="static"),
        # the benchmark's bandwidth-bound batch
        _logits("logits_given", "train", 32, (256, 1792), "uniform"),
        # diagnostics and gradient at a smaller vocabulary that is no multiple of a tile
        _logits("logits_diag", "diag", 24, (64, 1024), "uniform", V=32776, estimator="sampled"),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(max(lo, hi))))))

    # the benchmark's vocabulary half the time, otherwise any multiple of 8
    V = V_FULL if rng.random() < 0.5 else 8 * log(256, 19000)
    window = ("shared", "uniform", "mixed")[rng.randrange(3)]
    est = "sampled" if rng.random() < 0.3 else "expected"
    if rng.random() < 0.4:
        T = log(8, min(32768, 32768 * V_FULL // V))
        n = log(max(1, T // 4096), min(64, T))
        mean = max(1, T // n)
        lens = (max(1, mean // 3), max(1, (5 * mean) // 3))
        w = max(1, int(mean * rng.uniform(0.3, 1.2))) if window == "shared" else window
        api = ("handle", "function", "static")[rng.randrange(3 if T * 4 < 900000 else 2)]
        return {k: v for k, v in _logits("", "diag" if rng.random() < 0.3 else "train", n, lens, w, V, est, api).items()
                if k != "name"}
    H_s, H_t = 64 * log(2, 56), 64 * log(2, 72)
    job = ("train", "train", "train", "probe", "head", "stats")[rng.randrange(6)]
    if job == "stats":
        est = "expected"
    rows = log(16, 65536)
    while rows * V * (2.0 * H_s + H_t) > 65536.0 * V_FULL * 8192:     # no dearer than the headline batch
        rows //= 2
    n = log(max(1, rows // 4096), min(64, rows))
    mean = max(1, rows // n)
    if job in ("probe", "stats"):       # every position is computed
        lens, w = (max(1, mean // 2), max(1, (3 * mean) // 2)), max(1, mean // 4)
    else:                               # the window is computed
        lens, w = (max(1, mean // 2), 4 * mean), mean
    w = w if window == "shared" or mean > 2048 else window
    return {k: v for k, v in _fused("", job, n, lens, w, V, H_s, H_t, est, "bf16" if rng.random() < 0.5 else "f32",
                                    "function" if rng.random() < 0.5 else "handle").items() if k != "name"}


def _ragged(case):
    """Offsets and windows; they belong to the case, so that every seed has the same work."""
    g = np.random.default_rng([case["B"], case["len_lo"], case["len_hi"]])
    lens = g.integers(case["len_lo"], case["len_hi"], size=case["B"], endpoint=True)
    off = np.zeros(case["B"] + 1, np.int64)
    off[1:] = np.cumsum(lens)
    if case["window"] == "uniform":
        win = np.array([g.integers((l + 3) // 4, l, endpoint=True) for l in lens])
    elif case["window"] == "mixed":
        win = np.minimum(g.choice(np.array(CANDIDATES), size=case["B"]), lens)
    else:
        win = np.full(case["B"], int(case["window"]))
    return off, win.astype(np.int32)


def _counts(case):
    off, win = _ragged(case)
    T = int(off[-1])
    n_adm = int(np.minimum(win, np.diff(off)).sum())
    return T, n_adm, (T if case["job"] in ("probe", "stats") else n_adm)


def _token_logit(T, V, key):
    """Logit of the sampled token of each position: a trained policy samples tokens that it finds
    likely, from barely (a small share of the softmax) to almost certain."""
    u = torch.rand(T, generator=torch.Generator("cuda").manual_seed(key), device="cuda")
    return (0.4 + 0.8 * u) * (math.log(V) + 0.4)


def _hidden_inputs(case, T, seed):
    V, H_s, H_t = case["V"], case["H_s"], case["H_t"]
    W = {"s": synth.normal_bf16((V, H_s), 0.02, ("W_s", seed), "cuda"),
         "t": synth.normal_bf16((V, H_t), 0.02, ("W_t", seed), "cuda")}
    h = {"s": synth.normal_bf16((T, H_s), 1.0, ("h_s", seed), "cuda"),
         "t": synth.normal_bf16((T, H_t), 1.0, ("h_t", seed), "cuda")}
    ids = torch.randint(0, V, (T,), generator=torch.Generator("cuda").manual_seed(seed), device="cuda",
                        dtype=torch.int32)
    z = _token_logit(T, V, seed + 1)
    dz = torch.randn(T, generator=torch.Generator("cuda").manual_seed(seed + 2), device="cuda")
    for m, H, target in (("s", H_s, z), ("t", H_t, z + dz)):
        # h += a W[y] with a |W[y]|^2 = the token's logit
        for lo in range(0, T, 16384):
            rows = W[m][ids[lo:lo + 16384].long()].float()
            a = target[lo:lo + 16384] / rows.square().sum(1)
            h[m][lo:lo + 16384] = (h[m][lo:lo + 16384].float() + a[:, None] * rows).to(torch.bfloat16)
    return h["s"], h["t"], W["s"], W["t"], ids


def _logit_inputs(case, T, seed):
    V = case["V"]
    ids = torch.randint(0, V, (T,), generator=torch.Generator("cuda").manual_seed(seed), device="cuda",
                        dtype=torch.int32)
    z_s = synth.normal_bf16((T, V), 1.0, ("z_s", seed), "cuda")
    z_t = synth.normal_bf16((T, V), 1.0, ("z_t", seed), "cuda")
    z = _token_logit(T, V, seed + 1)
    dz = torch.randn(T, generator=torch.Generator("cuda").manual_seed(seed + 2), device="cuda")
    z_s.scatter_(1, ids.long()[:, None], z.to(torch.bfloat16)[:, None])
    z_t.scatter_(1, ids.long()[:, None], (z + dz).to(torch.bfloat16)[:, None])
    return z_s, z_t, ids


def prepare(case, seed):
    off, win = _ragged(case)
    T = int(off[-1])
    est = B.ADWIN_EST_SAMPLED if case["estimator"] == "sampled" else B.ADWIN_EST_EXPECTED
    if case["path"] == "logits":
        args = (*_logit_inputs(case, T, seed), off, win)
        kw = {"estimator": est,
              "want": ("kl", "c", "dz", "loss_prefix", "batch", "n_out", "n_adm_out", "status_dev")}
        if case["job"] == "diag":
            kw["want"] += ("t_logp", "t_entropy", "t_rank", "t_first_reject", "t_logp_mean")
            kw["topk"] = TOPK
        kind, functions = B.LogitsCall, {"function": B.adwin_opd_from_logits, "static": B.adwin_opd_from_logits_static}
    else:
        args = (*_hidden_inputs(case, T, seed), off, win)
        kw = {"estimator": est, "dh_dtype": B.ADWIN_DT_BF16 if case["dh"] == "bf16" else B.ADWIN_DT_F32,
              "want": B.FusedCall.DEFAULT_OUTPUTS}
        if case["job"] == "head":
            kw["want"] += ("dW_prefix",)
        elif case["job"] == "probe":
            kw.update(mode=B.ADWIN_PREFIX_AND_FULL, candidates=CANDIDATES)
        elif case["job"] == "stats":
            kw.update(mode=B.ADWIN_PREFIX_AND_FULL, candidates=CANDIDATES, cand_outputs=False, topk=TOPK,
                      want=("kl", "c", "loss_prefix", "loss_full", "n_out", "n_adm_out", "status_dev", "t_logp",
                            "t_entropy", "t_rank", "t_first_reject", "t_logp_mean", "cand_loss_share"))
        kind, functions = B.FusedCall, {"function": B.adwin_opd_fused}
    if case["api"] == "handle":
        return {"call": kind(*args, **kw)}
    return {"function": functions[case["api"]], "args": args, "kw": kw}


def run(state):
    if "call" in state:
        status = state["call"].run()
        if status != B.ADWIN_OK:
            raise B.AdwinError(status)
        return state["call"].out
    return state["function"](*state["args"], **state["kw"])


def work(case):
    T, n_adm, rows = _counts(case)
    V = case["V"]
    if case["path"] == "logits":
        # both logit rows of an admitted position in, a gradient row of every position out
        return {"bytes": 4.0 * V * n_adm + 2.0 * V * T, "flops": 0.0}
    H_s, H_t, job = case["H_s"], case["H_t"], case["job"]
    flops = 2.0 * V * (H_s + H_t) * rows
    nbytes = 2.0 * (H_s + H_t) * (V + rows)
    dh = (2.0 if case["dh"] == "bf16" else 4.0) * H_s * T
    if job != "stats":
        flops += 2.0 * V * H_s * rows
        nbytes += dh * (2 if job == "probe" else 1)
    if job == "head":
        flops += 2.0 * V * H_s * rows
        nbytes += 4.0 * V * H_s
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Measured against the oracle in 64 bits: 2-norm of the difference over that of the result,
    # and the largest difference over the larger of the value and the result's rms, of the worst
    # output; about four times that is allowed.
    if case["path"] == "fused" and case["job"] == "stats":
        # fp32 sums (KL 3.1e-6, largest 3.7e-5); a rank may differ where a logit ties with the
        # sampled token's within rounding
        return {"rel": 1.2e-5, "max": 2e-4, "differ": 5e-3}
    if case["job"] == "head":
        return {"rel": 9e-3, "max": 0.12}       # three bf16 roundings per summand: 2.1e-3, largest 0.028
    # bf16 logit gradient or bf16 storage: 1.7e-3, largest 7e-3 (fp32 hidden-state gradients of
    # batches with likely tokens 2e-4: their few heavy entries are taken in fp32)
    return {"rel": 7e-3, "max": 0.03}
