"""The calls this library is timed on: what a training job and an evaluation job have it do.

Two programs use the library.  A rollout collects trajectories: every decode step is one
`espo_step` on the [B, V] logits of that step (plain draws for training, filtered draws for
evaluation), from a handful of rows to a full batch, early in a batch with every row live and
late in it with most rows done.  The batch boundary then turns the finished trajectories into
what the policy update reads: `espo_batch_stats` on the regrets, an advantage pass in the layout
and reward form the trainer keeps, and the whitening of the advantages.  Every pass here is
written as such a program writes it: buffers, workspaces and parameters are made once, the calls
run on the current stream, and nothing waits for the GPU in between.

Logits, critic values, rewards, lengths and regrets come from the package's seeded generators
(`paper_2605_29860_amd.workloads`): rows shaped like a language-model head's, lengths uniform.
"""
from __future__ import annotations

import math

import torch

import paper_2605_29860_amd as espo
from paper_2605_29860_amd import workloads as W

DEVICE = "cuda"
MOST_BYTES = 190e6          # what a drawn case moves at most (the largest listed one moves a little more)

# An `espo_step` case: rows B, vocabulary V, logit type, temperature, share of rows that are done,
# outputs asked for ("token": no log-probability, "logprob", "entropy": both) and filter on the draw.
_STEP = {"kind": "step", "B": 1, "V": 1, "dtype": "bf16", "tau": 0.6, "done": 0.0, "out": "logprob", "top_p": 0.0, "top_k": 0}
# An advantage case: B trajectories of at most T tokens (shortest `lo`), reward form, layout, value
# targets, and the whitening that follows ("two": espo_whiten, "ws": through the workspace of the pass).
_ADV = {"kind": "adv", "B": 1, "T": 1, "lo": 1, "form": "dense", "layout": "padded", "returns": False, "fill": True, "whiten": "two"}
_STATS = {"kind": "stats", "B": 1, "T": 1, "lo": 1}


def _step(name, **kw):
    return {"name": name, **_STEP, **kw}


def _adv(name, **kw):
    return {"name": name, **_ADV, **kw}


def listed():
    return [
        # The smallest call: the four-row fp32 reference rollout (one prompt's few samples), where a
        # decode step is latency and nothing else.
        _step("step_f32_b4", B=4, V=32768, dtype="f32", tau=1.0),
        # One decode step of a small rollout batch, 64 prompts with one sample each.
        _step("step_bf16_b64", B=64, V=W.QWEN_VOCAB),
        # The training rollout in the middle of a batch: 8 rollouts x 64 prompts, an eighth of them done.
        _step("step_bf16_b512", B=512, V=W.QWEN_VOCAB, done=0.13),
        # A large training batch near its end: most trajectories stopped or finished.
        _step("step_bf16_b1024_late", B=1024, V=W.QWEN_VOCAB, done=0.58),
        # An engine that hands out fp32 logits, with the policy entropy tracked, odd vocabulary.
        _step("step_f32_b320_entropy", B=320, V=150001, dtype="f32", out="entropy"),
        # Evaluation of a small model (odd vocabulary) with top-k draws, a hundred samples at a time.
        _step("step_top_k_b100", B=100, V=50003, tau=1.0, top_k=50),
        # Evaluation as the paper runs it: nucleus 0.7 at temperature 1.
        _step("step_top_p_b512", B=512, V=W.QWEN_VOCAB, tau=1.0, top_p=0.7),
        # The batch boundary of the four-row reference rollout: latency of two calls.
        _adv("adv_b4_t128", B=4, T=128, lo=32),
        # The batch boundary of a large batch with a dense reward array: advantages, then whitening,
        # with the workspace between them.
        _adv("adv_dense_b1024_t16384", B=1024, T=16384, lo=512, whiten="ws"),
        # The boundary of the training batch with the paper's rewards (one per trajectory) and the
        # critic's targets, padded arrays, then whitening.
        _adv("adv_terminal_b512_t8192", B=512, T=8192, lo=64, form="terminal", returns=True),
        # The same for a trainer that stores trajectories back to back.
        _adv("adv_packed_b512", B=512, T=8192, lo=65, layout="packed", returns=True),
        # Regret statistics and threshold controller at the boundary of the training batch.
        {"name": "stats_b512_t8192", **_STATS, "B": 512, "T": 8192, "lo": 64},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    while True:
        what = rng.random()
        if what < 0.6:
            case = dict(_STEP, B=_log_int(rng, 1, 1024), V=_log_int(rng, 8000, 200000), dtype=rng.choice(("bf16", "bf16", "f32")),
                        tau=rng.choice((0.6, 0.8, 1.0)), done=rng.choice((0.0, 0.0, 0.13, 0.5)),
                        out=rng.choice(("token", "logprob", "logprob", "entropy")))
            flt = rng.choice(("", "", "top_p", "top_k"))
            if flt == "top_p":
                case["top_p"] = rng.choice((0.7, 0.7, 0.9))
            elif flt == "top_k":
                case["top_k"] = rng.choice((1, 20, 50))
        elif what < 0.9:
            case = dict(_ADV, B=_log_int(rng, 1, 1024), T=_log_int(rng, 100, 16384), form=rng.choice(("dense", "terminal")),
                        layout=rng.choice(("padded", "padded", "packed")), returns=rng.random() < 0.5)
            case["lo"] = max(1, case["T"] // rng.choice((2, 8, 32)))
            if rng.random() < 0.5:
                case["T"] = (case["T"] + 3) // 4 * 4      # trainers often round the horizon up
            if case["layout"] == "padded":
                case["fill"] = case["form"] == "dense" or rng.random() < 0.5
                case["whiten"] = rng.choice(("two", "ws"))
            if case["form"] == "dense" and case["layout"] == "padded":
                case["returns"] = False                   # that call has no such output
        else:
            case = dict(_STATS, B=_log_int(rng, 8, 1024), T=_log_int(rng, 200, 16384))
            case["lo"] = max(1, case["T"] // 16)
        if work(case)["bytes"] <= MOST_BYTES:
            return case


# --------------------------------------------------------------------------- inputs
def _tokens(case):
    """Valid tokens of a batch: lengths are uniform over [lo, T]."""
    return case["B"] * (min(case["lo"], case["T"]) + case["T"]) // 2


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _prepare_step(case, seed):
    B, V, dt = case["B"], case["V"], _dtype(case)
    pitch = 16 // (2 if dt == torch.bfloat16 else 4)
    stride = (V + pitch - 1) // pitch * pitch             # rows start at multiples of 16 bytes
    logits = torch.zeros(B, stride, dtype=dt, device=DEVICE)
    W.ZipfLogits(V=V, seed=seed, device=DEVICE, dtype=dt).rows(B, out=logits[:, :V])
    z, alive, stop_step = W.seeded_state(B, seed, device="cpu", dead_every=0)
    z = z * 0.5
    g = torch.Generator().manual_seed(seed)
    alive[torch.randperm(B, generator=g)[:int(round(B * case["done"]))]] = 0
    new = lambda dtype: torch.zeros(B, dtype=dtype, device=DEVICE)
    nws = espo.espo_step_workspace_bytes(B, V, dt)
    p = W.RolloutParams().as_dict()
    return {"case": case, "logits": logits, "V": V, "seed": seed, "t": 0,
            # a critic that expects success: the stop rule is on and tested, and no row reaches its threshold,
            # so every pass over the same state has the same live rows
            "values": W.step_values(B, seed, 0, 0.5, 1.0, device=DEVICE),
            "params": espo.EspoParams(**p, top_p=case["top_p"], top_k=case["top_k"]),
            "z": z.to(DEVICE), "alive": alive.to(DEVICE), "stop_step": stop_step.to(DEVICE),
            "tokens": new(torch.int32), "regret": new(torch.float32),
            "logprob": new(torch.float32) if case["out"] != "token" else None,
            "entropy": new(torch.float32) if case["out"] == "entropy" else None,
            "ws": torch.zeros(nws, dtype=torch.uint8, device=DEVICE) if nws else None}


def _with_total(lengths, total, lo, hi):
    """`lengths` moved by as little as it takes to have the given sum: packed arrays then have one size per case."""
    while (off := total - int(lengths.sum())) != 0:
        n = lengths.numel()
        step = torch.full((n,), int(off / n), dtype=lengths.dtype)
        step[:abs(off) % n] += 1 if off > 0 else -1
        lengths = (lengths + step).clamp(lo, hi)
    return lengths


def _prepare_adv(case, seed):
    B, T, lo = case["B"], case["T"], min(case["lo"], case["T"])
    rewards, values, lengths, stopped = W.advantage_batch(B=B, T=T, len_lo=lo, len_hi=T, seed=seed, device=DEVICE)
    terminal = rewards[torch.arange(B, device=DEVICE), (lengths.long() - 1).clamp(min=0)].contiguous()
    s = {"case": case, "stopped": stopped, "terminal": terminal, "wstats": torch.zeros(3, dtype=torch.float64, device=DEVICE)}
    if case["layout"] == "packed":
        lengths = _with_total(lengths.long().cpu(), _tokens(case), lo, T).to(DEVICE)
        s["cu"] = torch.zeros(B + 1, dtype=torch.int64, device=DEVICE)
        s["cu"][1:] = lengths.cumsum(0)
        s["values"] = values[torch.arange(T, device=DEVICE)[None, :] < lengths[:, None]]
        s["rewards"] = torch.zeros_like(s["values"])
        s["rewards"][s["cu"][1:] - 1] = terminal
        shape = (s["values"].numel(),)
        s["lengths"] = torch.tensor(shape, dtype=torch.int32, device=DEVICE)   # one span for the whitening
        nws = espo.espo_whiten_workspace_bytes(1, shape[0])
    else:
        s["rewards"], s["values"], s["lengths"] = rewards, values, lengths
        shape = (B, T)
        nws = espo.espo_advantages_ws_bytes(B) if case["whiten"] == "ws" else espo.espo_whiten_workspace_bytes(B, T)
    s["td"] = torch.zeros(shape, device=DEVICE)
    s["adv"] = torch.zeros(shape, device=DEVICE)
    s["returns"] = torch.zeros(shape, device=DEVICE) if case["returns"] else None
    s["ws"] = torch.zeros(nws, dtype=torch.uint8, device=DEVICE)
    return s


def _prepare_stats(case, seed):
    regret, lengths, stopped = W.regret_batch(B=case["B"], T=case["T"], len_lo=case["lo"], seed=seed, device=DEVICE)
    out = torch.zeros(espo.BATCH_RESULT_BYTES, dtype=torch.uint8, device=DEVICE)
    return {"case": case, "regret": regret, "lengths": lengths, "stopped": stopped, "out": out,
            "ws": torch.zeros(espo.espo_batch_stats_workspace_bytes(case["B"], case["T"]), dtype=torch.uint8, device=DEVICE),
            # the fields of the result, as views of the buffer it is written to
            "fields": {"batch": out[:24].view(torch.float64), "tokens": out[24:32].view(torch.int64),
                       "next": out[32:44].view(torch.float32), "stopped": out[44:48].view(torch.int32)}}


def prepare(case, seed):
    return {"step": _prepare_step, "adv": _prepare_adv, "stats": _prepare_stats}[case["kind"]](case, seed)


# --------------------------------------------------------------------------- one pass
def _run_step(s):
    t = s["t"]
    s["t"] = t + 1
    espo.espo_step(s["logits"], s["case"]["tau"], s["seed"], t, s["values"], s["params"], s["z"], s["alive"], s["stop_step"],
                   s["tokens"], s["regret"], s["logprob"], V=s["V"], workspace=s["ws"], entropy=s["entropy"])
    return {k: s[k] for k in ("tokens", "regret", "logprob", "entropy", "z", "alive", "stop_step")}


def _run_adv(s):
    c = s["case"]
    args = (-1.0, 1.0, 0.95, s["td"], s["adv"])           # r_fail, gamma, lambda and the outputs
    if c["layout"] == "packed":
        form = {"rewards": s["rewards"]} if c["form"] == "dense" else {"terminal_reward": s["terminal"]}
        espo.espo_advantages_packed(s["values"], s["cu"], s["stopped"], *args, returns=s["returns"], **form)
    elif c["form"] == "dense":
        if c["whiten"] == "ws":
            espo.espo_advantages_ws(s["rewards"], s["values"], s["lengths"], s["stopped"], *args, s["ws"])
        else:
            espo.espo_advantages(s["rewards"], s["values"], s["lengths"], s["stopped"], *args)
    else:
        kw = {"returns": s["returns"], "zero_padding": c["fill"]}
        if c["whiten"] == "ws":
            espo.espo_advantages_terminal_ws(s["values"], s["lengths"], s["stopped"], s["terminal"], *args, s["ws"], **kw)
        else:
            espo.espo_advantages_terminal(s["values"], s["lengths"], s["stopped"], s["terminal"], *args, **kw)
    whiten = espo.espo_whiten_from_ws if c["whiten"] == "ws" and c["layout"] == "padded" else espo.espo_whiten
    whiten(s["adv"], s["lengths"], s["adv"], s["ws"], stats=s["wstats"])   # in place
    return {"td": s["td"], "adv": s["adv"], "returns": s["returns"], "moments": s["wstats"]}


def _run_stats(s):
    p = W.RolloutParams
    espo.espo_batch_stats(s["regret"], s["lengths"], s["stopped"], p.mu_g, p.var_g, p.beta, s["out"], s["ws"])
    return s["fields"]


def run(state):
    return {"step": _run_step, "adv": _run_adv, "stats": _run_stats}[state["case"]["kind"]](state)


# --------------------------------------------------------------------------- what a pass cannot do without
def work(case):
    B = case["B"]
    if case["kind"] == "step":
        live = B - int(round(B * case["done"]))
        scalars = 22 + (4 if case["out"] != "token" else 0) + (4 if case["out"] == "entropy" else 0)
        return {"bytes": live * (case["V"] * (2 if case["dtype"] == "bf16" else 4) + scalars) + (B - live) * 9,
                "flops": live * case["V"] * (4 if case["out"] == "logprob" else 6 if case["out"] == "entropy" else 2)}
    tokens = _tokens(case)
    if case["kind"] == "stats":
        return {"bytes": tokens * 4 + B * 5 + 48, "flops": tokens * 4}
    outputs = 3 if case["returns"] else 2
    written = B * case["T"] if case["layout"] == "padded" and case["fill"] else tokens
    return {"bytes": tokens * (8 if case["form"] == "dense" else 4) + written * 4 * outputs + B * 9, "flops": tokens * 12}


# Whole numbers (tokens, flags, stop steps, counts) do not depend on the order of any sum.  Of the floats,
# regret and state are single rounded operations; the softmax sums, the scan and the moments are sums whose
# order is free.  Against the same path in double, on the listed cases: log-probability 8e-8 and entropy 7e-7
# (largest single error 1.9e-6) of the result's norm; td 2e-8, whitened advantages 1.6e-7 (1.4e-6) and value
# targets, which cancel against the critic's values, 9e-7 (9e-6); the statistics are sums in double that are
# rounded to float once.  The bounds are about four times that.
TOLERANCE = {"step": {"rel": 3e-6, "max": 1e-5}, "adv": {"rel": 4e-6, "max": 4e-5}, "stats": {"rel": 5e-7, "max": 1e-6}}


def tolerance(case):
    return TOLERANCE[case["kind"]]
