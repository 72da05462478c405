"""The work a user of shared-prompt attention has it do, as measurable cases.

A case names one pass through the public entry points of ``paper_2511_18871_amd.binding``:

  train   one attention layer of a training step: forward, then backward (o, lse, dq, dk, dv)
  score   log-probability passes without a backward: the forward of one tensor set, or of several sets
          (policy / old policy / reference) that share a packing, in one call
  micro   a micro-batch whose prompt was computed by an earlier one: response rows only, forward and
          backward, dk / dv accumulated
  rope    position encoding of q and k at the restarted positions (or of their gradients, inverse)
  loss    logits -> log-probabilities -> GRPO objective -> gradient of the logits

and a packing: ``groups`` prompts of ``prompt_lo .. prompt_hi`` tokens, each with ``responses`` answers of
``resp_lo .. resp_hi`` tokens (seeded ragged lengths), plus the head geometry and the element type.  Callers
use the default arguments: outputs and workspaces are allocated by the binding, as in a plain training loop.
"""
from __future__ import annotations

import math

import torch

from paper_2511_18871_amd import binding as B
from paper_2511_18871_amd import workloads as W

ROPE_BASE = 1e6
HEADS = ((4, 2), (28, 4), (32, 8), (40, 8))     # q / kv heads of the model shapes this repository names


def _case(kind, groups, prompt_lo, prompt_hi, responses, resp_lo, resp_hi, hq, hkv, head_dim=128, dtype="bf16",
          pack_seed=1, **more):
    return {"kind": kind, "groups": groups, "prompt_lo": prompt_lo, "prompt_hi": prompt_hi, "responses": responses,
            "resp_lo": resp_lo, "resp_hi": resp_hi, "hq": hq, "hkv": hkv, "head_dim": head_dim, "dtype": dtype,
            "pack_seed": pack_seed, **more}


def listed():
    named = {
        # the smallest call: one group of 192 tokens in float32, the cross-checking path of a unit-sized model
        "tiny_group_f32": _case("train", 1, 64, 64, 4, 32, 32, 2, 2, head_dim=64, dtype="f32"),
        # a small batch of ragged groups of a small model: launches and host time count
        "small_ragged_groups": _case("train", 2, 70, 333, 7, 1, 200, 4, 2, pack_seed=7),
        # scoring one short prompt with four answers under the old policy: a single forward call
        "short_group_scoring": _case("score", 1, 203, 203, 4, 30, 75, 28, 4, pack_seed=11, sets=1),
        # one GRPO group of a 7B-class model per micro-batch
        "single_group": _case("train", 1, 1024, 1024, 8, 256, 256, 28, 4),
        # four long prompts with 16 ragged answers each
        "long_prompt_ragged": _case("train", 4, 4096, 4096, 16, 128, 512, 32, 8, pack_seed=3000),
        # the forwards of policy, old policy and reference over eight groups, one call
        "tri_model_scoring": _case("score", 8, 2048, 2048, 8, 1024, 1024, 28, 4, sets=3),
        # the headline workload: one 16K prompt, 32 short answers, some keys with large logits
        "extreme_sharing": _case("train", 1, 16384, 16384, 32, 64, 256, 40, 8, pack_seed=5000, stress=0.01),
        # grade-school maths GRPO at 1K context: many groups of a short prompt and 16 answers
        "many_short_answers": _case("train", 64, 64, 192, 16, 96, 416, 28, 4, pack_seed=6000),
        # many groups of about 1000 tokens, mostly prompt
        "many_short_groups": _case("train", 64, 560, 840, 4, 40, 111, 32, 8, pack_seed=9000),
        # the second micro-batch of a long-prompt group: its prompt rows are already done
        "response_rows": _case("micro", 1, 8192, 8192, 16, 64, 256, 40, 8, pack_seed=5100),
        # rotary encoding of q and k of a long-prompt group
        "rope_long_prompt": _case("rope", 1, 16384, 16384, 32, 64, 256, 40, 8, pack_seed=5000, inverse=False),
        # the response-token loss of one GRPO group over a 152K vocabulary
        "vocabulary_loss": _case("loss", 1, 1024, 1024, 8, 256, 256, 1, 1, vocab=151936),
    }
    return [dict(case, name=name) for name, case in named.items()]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges the listed ones stand for."""
    while True:
        kind = rng.choice(("train", "train", "train", "score", "micro", "rope", "loss"))
        hq, hkv = rng.choice(HEADS)
        prompt = _log_int(rng, 48, 16384)
        resp = _log_int(rng, 24, 1024)
        case = _case(kind, _log_int(rng, 1, 64), max(1, int(prompt * rng.uniform(0.3, 1.0))), prompt,
                     rng.randint(1, 32), max(1, int(resp * rng.uniform(0.1, 1.0))), resp, hq, hkv,
                     pack_seed=rng.randint(1, 10 ** 6))
        if kind == "train":
            if rng.random() < 0.15:                 # the float32 path serves small problems
                case.update(dtype="f32", hq=4, hkv=rng.choice((2, 4)), head_dim=rng.choice((64, 128)))
            elif rng.random() < 0.25:
                case["stress"] = 0.01
        elif kind == "score":
            case["sets"] = rng.choice((1, 1, 2, 3))
        elif kind == "rope":
            case["inverse"] = rng.random() < 0.5
        elif kind == "loss":
            vocab = _log_int(rng, 1000, 151936)
            case.update(hq=1, hkv=1, vocab=vocab if rng.random() < 0.3 else (vocab + 63) // 64 * 64,
                        dtype=rng.choice(("bf16", "bf16", "f32")))
        tokens = sum(g.total for g in _groups(case))
        flops, size = work(case)["flops"], work(case)["bytes"]
        if case["dtype"] == "f32" and kind == "train":
            fits = tokens <= 2500
        elif kind == "loss":
            fits = tokens * case["vocab"] <= 3072 * 151936
        else:                                       # well inside the largest listed case's time at any packing
            fits = flops <= 4.0e12 and size <= 4.0e9
        if fits:
            return case


def _groups(case):
    """Ragged lengths from the workload module's seeded stream."""
    out = []
    for g in range(case["groups"]):
        prompt = W.ragged_lengths(case["pack_seed"] + 100000 + g, 1, case["prompt_lo"], case["prompt_hi"])[0]
        out.append(W.Group(prompt, W.ragged_lengths(case["pack_seed"] + g, case["responses"], case["resp_lo"],
                                                    case["resp_hi"])))
    return out


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def prepare(case, seed):
    groups = _groups(case)
    dev, dt = torch.device("cuda"), _dtype(case)
    T, Hq, Hkv, d = sum(g.total for g in groups), case["hq"], case["hkv"], case["head_dim"]
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)

    def normal(*shape, dtype=dt, std=1.0):
        return torch.empty(*shape, dtype=dtype, device=dev).normal_(0.0, std, generator=gen)

    s = {"case": case, "pl": [g.prompt_len for g in groups], "Gs": [len(g.resp_lens) for g in groups],
         "rl": [n for g in groups for n in g.resp_lens], "scale": d ** -0.5}
    kind = case["kind"]
    if kind == "loss":
        V = case["vocab"]
        s["logits"] = normal(T, V, std=2.0)
        s["labels"] = torch.randint(0, V, (T,), generator=gen, device=dev, dtype=torch.int32)
        logp = torch.empty(T, device=dev)
        for a in range(0, T, 256):                  # the policy's own values, from which the other two differ a little
            z = s["logits"][a:a + 256].float()
            logp[a:a + 256] = z.gather(1, s["labels"][a:a + 256, None].long())[:, 0] - torch.logsumexp(z, 1)
        s["old"] = logp + 0.1 * normal(T, dtype=torch.float32)
        s["ref"] = logp + 0.1 * normal(T, dtype=torch.float32)
        s["adv"] = normal(len(s["rl"]), dtype=torch.float32)
        return s
    if kind == "score":
        s["q"] = [normal(T, Hq, d) for _ in range(case["sets"])]
        s["k"] = [normal(T, Hkv, d) for _ in range(case["sets"])]
        s["v"] = [normal(T, Hkv, d) for _ in range(case["sets"])]
        return s
    s["q"], s["k"] = normal(T, Hq, d), normal(T, Hkv, d)
    if kind == "rope":
        return s
    s["v"], s["d_o"] = normal(T, Hkv, d), normal(T, Hq, d)
    if case.get("stress"):
        s["k"][torch.rand(T, generator=gen, device=dev) < case["stress"]] *= 8.0
    if kind == "micro":                             # what the micro-batch that ran in full left behind
        s["o"], s["lse"] = normal(T, Hq, d), torch.zeros(Hq, T, device=dev)
        s["dq"] = torch.zeros_like(s["q"])
    return s


def run(state):
    s = state
    case, pack = s["case"], (s["pl"], s["Gs"], s["rl"])
    kind = case["kind"]
    if kind == "train":
        if case["groups"] == 1:
            o, lse = B.sp_attn_fwd(s["q"], s["k"], s["v"], s["pl"][0], s["rl"], s["scale"])
            dq, dk, dv = B.sp_attn_bwd(s["q"], s["k"], s["v"], o, lse, s["d_o"], s["pl"][0], s["rl"], s["scale"])
        else:
            o, lse = B.sp_attn_fwd_batched(s["q"], s["k"], s["v"], *pack, s["scale"])
            dq, dk, dv = B.sp_attn_bwd_batched(s["q"], s["k"], s["v"], o, lse, s["d_o"], *pack, s["scale"])
        return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    if kind == "score":
        if case["sets"] == 1:
            o, lse = B.sp_attn_fwd_batched(s["q"][0], s["k"][0], s["v"][0], *pack, s["scale"])
            return {"o": o, "lse": lse}
        os, lses = B.sp_attn_fwd_multi(s["q"], s["k"], s["v"], *pack, s["scale"])
        return {"o": os, "lse": lses}
    if kind == "micro":
        o, lse = B.sp_attn_fwd_batched_ex(s["q"], s["k"], s["v"], *pack, s["scale"], B.SP_FLAG_RESPONSE_ROWS,
                                          o=s["o"], lse=s["lse"])
        dk, dv = torch.zeros_like(s["k"]), torch.zeros_like(s["v"])
        dq, dk, dv = B.sp_attn_bwd_batched_ex(s["q"], s["k"], s["v"], o, lse, s["d_o"], *pack, s["scale"],
                                              B.SP_FLAG_RESPONSE_ROWS | B.SP_FLAG_ACCUMULATE_DKDV, dq=s["dq"],
                                              dk=dk, dv=dv)
        return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    if kind == "rope":
        q, k = B.sp_attn_rope_qk(s["q"], s["k"], *pack, ROPE_BASE, inverse=case["inverse"])
        return {"q": q, "k": k}
    logp, lse = B.sp_attn_logprob_fwd(s["logits"], s["labels"], *pack)
    loss, g = B.sp_attn_grpo_loss(logp, s["old"], s["ref"], s["adv"], *pack)
    dlogits = B.sp_attn_logprob_bwd(s["logits"], s["labels"], lse, g, *pack)
    return {"logp": logp, "lse": lse, "loss": loss, "g": g, "dlogits": dlogits}


def work(case):
    groups = _groups(case)
    T, Hq, Hkv, d = sum(g.total for g in groups), case["hq"], case["hkv"], case["head_dim"]
    resp = sum(sum(g.resp_lens) for g in groups)
    e = 2 if case["dtype"] == "bf16" else 4
    kind = case["kind"]
    if kind == "loss":
        # response rows of the logits read once and their gradient written, zeros on the gradient's prompt rows;
        # an exponential, a scaling and a subtraction each way
        V = case["vocab"]
        return {"bytes": float(e) * V * (resp + T) + 4.0 * (8 * resp + 3 * T), "flops": 6.0 * resp * V}
    if kind == "rope":
        return {"bytes": 2.0 * e * T * (Hq + Hkv) * d, "flops": 3.0 * T * (Hq + Hkv) * d}
    pairs = sum(W.allowed_pairs(g) for g in groups)
    q_rows = T
    if kind == "micro":
        pairs -= sum(g.prompt_len * (g.prompt_len + 1) // 2 for g in groups)
        q_rows = resp
    fwd_bytes = e * d * (2.0 * q_rows * Hq + 2.0 * T * Hkv) + 4.0 * q_rows * Hq        # q, o, k, v, lse
    if kind == "score":
        return {"bytes": case["sets"] * fwd_bytes, "flops": 4.0 * d * pairs * Hq * case["sets"]}
    bwd_bytes = e * d * (2.0 * q_rows * Hq + 2.0 * T * Hkv)                             # d_o, dq, dk, dv
    return {"bytes": fwd_bytes + bwd_bytes, "flops": 14.0 * d * pairs * Hq}


def tolerance(case):
    # About four times what the path shows against float64 evaluations of the same inputs (largest of ragged groups,
    # short prompts and large-logit keys: bf16 attention 2.5e-3 in the 2-norm and 6.2e-2 at one element, where dS
    # cancels; float32 attention 7.9e-7 and 1.0e-5; bf16 logit gradients and rotations 1.7e-3 and 3.9e-3, their
    # rounding; float32 losses 4.8e-7, and 1.6e-5 for a scalar objective whose advantages nearly cancel).
    bf16 = case["dtype"] == "bf16"
    if case["kind"] == "loss":
        return {"rel": 7e-3} if bf16 else {"rel": 7e-5}
    if case["kind"] == "rope":
        return {"rel": 7e-3, "max": 1.6e-2}
    return {"rel": 1e-2, "max": 0.25} if bf16 else {"rel": 4e-6, "max": 4e-5}
