"""The work a user of this package has it do, as measurable cases.

Four families, all through the public calls of ``paper_2602_01744_amd``:

* ``decode``  one generated token for a batch of sequences (``decode_step``), the state updated in place;
* ``prefill`` the forward over whole sequences (``forward``), as prompt processing and evaluation run it;
* ``train``   one training step of the mixer: the prologue the variant has (gate projections; for the delta rule also
  the short convolutions), the forward, the backward and the prologue's backward;
* ``packed``  forward and backward over sequences of different lengths laid end to end (``forward_varlen``,
  ``backward_varlen``, ``backward_gdn_varlen``).

Values follow the package's synthetic workloads: q, k ~ N(0,1) / sqrt(dk) (L2-normalised for the delta rule), v ~ N(0,1),
head logits ~ N(0,1) (or from the gate matrices), GLA log-decay logsigmoid(N(0,1)) / 16 per key dimension, RetNet
gamma_h = 1 - 2^(-5-h), delta rule log-decay logsigmoid(N(0,1)) / 8 and beta = sigmoid(N(0,1)).
"""
from __future__ import annotations

import math
import random

import torch
import torch.nn.functional as F

import paper_2602_01744_amd as sla

RETNET, GLA, GDN = sla.RETNET, sla.GLA, sla.GDN
VARIANT = {"retnet": RETNET, "gla": GLA, "gdn": GDN}

# The most one drawn case may touch: token-heads times (bytes per token-head), below the long-context prefill's.
MOST_BYTES = 2.0e9


def _case(name, kind, variant, dtype, B, T, H, dk, dv, **more):
    c = dict(name=name, kind=kind, variant=variant, dtype=dtype, B=B, T=T, H=H, dk=dk, dv=dv,
             segments=1, states=False, layout="bthd", prologue=False, decay_shift=0.0, logit_std=1.0, peaked=0, mix=0)
    c.update(more)
    return c


def listed():
    return [
        # One user generating text: a single token of a single sequence, 4 wide heads, the gate projection fused in.
        _case("decode_single", "decode", "gla", "bf16", 1, 1, 4, 128, 256, prologue=True),
        # A serving batch: one token for each of 64 sequences, delta rule.
        _case("decode_batch", "decode", "gdn", "bf16", 64, 1, 16, 128, 128),
        # A short prompt in fp32: few small heads, the smallest forward in use.
        _case("prefill_short_f32", "prefill", "gla", "f32", 1, 256, 4, 64, 64),
        # A small batch of 2K prompts with few sequences, sharp gates; the library chooses the schedule.
        _case("prefill_retnet", "prefill", "retnet", "bf16", 4, 2048, 8, 128, 128, segments=0, logit_std=2.0),
        # The forward at the training shape (16 heads of width 128), GLA.
        _case("prefill_gla", "prefill", "gla", "bf16", 8, 2048, 16, 128, 128),
        # The same for the delta rule at 4K context.
        _case("prefill_gdn", "prefill", "gdn", "bf16", 8, 4096, 16, 128, 128),
        # Long-context evaluation: one document of 64K tokens, 32 heads, long memory, one dominant head per passage.
        _case("prefill_long", "prefill", "gla", "bf16", 1, 65536, 32, 128, 128, segments=0, decay_shift=2.0, peaked=512),
        # A training step at 2K context.
        _case("train_gla", "train", "gla", "bf16", 8, 2048, 16, 128, 128, prologue=True),
        # A training step of the delta rule at 4K context, with its short convolutions.
        _case("train_gdn", "train", "gdn", "bf16", 8, 4096, 16, 128, 128, prologue=True),
        # A training step of the 4-head, 4K-context model shape (keys 128, values 256).
        _case("train_gla_wide", "train", "gla", "bf16", 8, 4096, 4, 128, 256, segments=0),
        # A training step on packed documents of 64 to 4096 tokens, 16K tokens in all.
        _case("train_packed_retnet", "packed", "retnet", "bf16", 0, 16384, 16, 128, 128, mix=1),
        # A training step in fp32 on a ragged length with states passed in and out (truncated backpropagation).
        _case("train_ragged_f32", "train", "gla", "f32", 2, 1021, 8, 64, 128, states=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["decode", "prefill", "prefill", "train", "train", "packed"])
    variant = rng.choice(["retnet", "gla", "gdn"])
    dtype = "f32" if rng.random() < 0.15 else "bf16"
    # Head widths as the model shapes have them; (32, 64) is the many-narrow-heads shape.
    dk, dv = rng.choice([(128, 128), (128, 128), (128, 256), (64, 128), (64, 64), (32, 64)])
    H = rng.choice([2, 4, 5, 8, 12, 16, 16, 32])
    if kind == "decode":
        c = _case("", kind, variant, dtype, _log_int(rng, 1, 256), 1, H, dk, dv, prologue=rng.random() < 0.5)
    elif kind == "packed":
        c = _case("", kind, variant, dtype, 0, _log_int(rng, 512, 16384), H, dk, dv, mix=rng.randrange(1, 1000))
    else:
        T = _log_int(rng, 17, 16384 if kind == "prefill" else 8192)
        few = rng.random() < 0.5  # let the library cut sequences into segments
        c = _case("", kind, variant, dtype, _log_int(rng, 1, 16), T, H, dk, dv, states=rng.random() < 0.25)
        if kind == "prefill":
            c["segments"] = 0 if few and variant != "gdn" else 1
            c["layout"] = "bhtd" if rng.random() < 0.2 else "bthd"
            c["logit_std"] = rng.choice([1.0, 2.0])
            c["decay_shift"] = rng.choice([0.0, 2.0])
        else:
            c["segments"] = 0 if few and variant != "gdn" and dtype == "bf16" and dk > 32 else 1
            c["prologue"] = rng.random() < 0.5
    del c["name"]
    # Too large: fewer tokens. fp32 passes and the delta rule's backward are the slow ones; they are cut first.
    limit = MOST_BYTES * (0.15 if dtype == "f32" else 0.6 if kind in ("train", "packed") and variant == "gdn" else 1.0)
    while work(c)["bytes"] > limit:
        if c["B"] > 1:
            c["B"] = max(1, c["B"] * 2 // 3)
        else:
            c["T"] = max(17, c["T"] * 2 // 3)
    return c


def lengths(case):
    """Document lengths of a packed case: spread over their logarithm between 64 and 4096 tokens, longest first."""
    rng = random.Random(case["mix"])
    left, out = case["T"], []
    while left > 0:
        n = min(left, _log_int(rng, 64, 4096))
        out.append(n)
        left -= n
    return sorted(out, reverse=True)


def _element(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def prepare(case, seed):
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    kind, var, el = case["kind"], VARIANT[case["variant"]], _element(case)
    B, T, H, dk, dv = (case[n] for n in ("B", "T", "H", "dk", "dv"))
    s = {"case": case, "variant": var}
    if kind == "decode":
        lead = (B, H)
    elif kind == "packed":
        lens = lengths(case)
        B = len(lens)
        s["cu"] = torch.tensor([sum(lens[:i]) for i in range(B + 1)], dtype=torch.int32, device=dev)
        lead = (T, H)
    else:
        lead = (B, H, T) if case["layout"] == "bhtd" else (B, T, H)
    small = (B, T, H) if kind in ("prefill", "train") else lead  # logits and per-token scalars

    def normal(*shape):
        return torch.randn(shape, generator=g, device=dev, dtype=torch.float32)

    def keys():
        x = normal(*lead, dk)
        return (F.normalize(x, dim=-1) if var == GDN else x * dk ** -0.5).to(el)

    conv = kind == "train" and var == GDN and case["prologue"]
    if conv:  # what the projections emit; q, k, v come out of the short convolutions
        for n, d in (("q", dk), ("k", dk), ("v", dv)):
            s["x" + n] = normal(B, T, H * d).to(el)
            s["c" + n] = normal(H * d, 4) * 0.5
    else:
        s["q"], s["k"] = keys(), keys()
        s["v"] = normal(*lead, dv).to(el)
    if case["prologue"]:
        s["wq"], s["wk"] = normal(H, dk), normal(H, dk)
    else:
        ql, kl = normal(*small) * case["logit_std"], normal(*small) * case["logit_std"]
        if case["peaked"]:  # one head per passage dominates both gates
            n = (T + case["peaked"] - 1) // case["peaked"]
            win = torch.randint(0, H, (B, n), generator=g, device=dev).repeat_interleave(case["peaked"], dim=1)[:, :T]
            bump = 6.0 * F.one_hot(win, H).float()
            ql, kl = ql + bump, kl + bump
        s["ql"], s["kl"] = ql, kl
    s["beta"] = None
    if var == RETNET:
        s["decay"] = torch.log1p(-torch.pow(2.0, -5.0 - torch.arange(H, dtype=torch.float64))).float().to(dev)
    elif var == GLA:
        s["decay"] = (F.logsigmoid(normal(*lead, dk) + case["decay_shift"]) / 16.0).to(el)
    else:
        s["decay"] = F.logsigmoid(normal(*small) + case["decay_shift"]) / 8.0
        s["beta"] = torch.sigmoid(normal(*small))
    s["initial"] = s["d_final"] = None
    if kind == "decode":
        s["state"] = normal(B, H, dk, dv) * 0.5
    elif case["states"]:
        s["initial"] = normal(B, H, dk, dv) * 0.5
    if kind in ("train", "packed"):
        s["d_out"] = normal(*lead, dv).to(el)
        if case["states"]:
            s["d_final"] = normal(B, H, dk, dv) * 0.5
    return s


def run(s):
    return {"decode": _decode, "prefill": _prefill, "train": _train, "packed": _packed}[s["case"]["kind"]](s)


def _decode(s):
    if s["case"]["prologue"]:
        out = sla.decode_step(s["variant"], s["q"], s["k"], s["v"], None, None, s["decay"], s["beta"], s["state"],
                              w_gq=s["wq"], w_gk=s["wk"])
    else:
        out = sla.decode_step(s["variant"], s["q"], s["k"], s["v"], s["ql"], s["kl"], s["decay"], s["beta"], s["state"])
    return {"out": out, "state": s["state"]}


def _prefill(s):
    c = s["case"]
    out, fin = sla.forward(s["variant"], s["q"], s["k"], s["v"], s["ql"], s["kl"], s["decay"], s["beta"], s["initial"],
                           segments=c["segments"], head_major=c["layout"] == "bhtd")
    return {"out": out, "final": fin}


def _train(s):
    c, var = s["case"], s["variant"]
    B, T, H, dk, dv = (c[n] for n in ("B", "T", "H", "dk", "dv"))
    conv = "xq" in s
    if conv:
        q = sla.short_conv_silu_l2(s["xq"], s["cq"], dk).view(B, T, H, dk)
        k = sla.short_conv_silu_l2(s["xk"], s["ck"], dk).view(B, T, H, dk)
        v = sla.short_conv_silu(s["xv"], s["cv"]).view(B, T, H, dv)
    else:
        q, k, v = s["q"], s["k"], s["v"]
    ql, kl = sla.gate_logits(q, k, s["wq"], s["wk"], dv=dv) if c["prologue"] else (s["ql"], s["kl"])
    out, fin = sla.forward(var, q, k, v, ql, kl, s["decay"], s["beta"], s["initial"], segments=c["segments"])
    if var == GDN:
        g = sla.backward_gdn(q, k, v, ql, kl, s["decay"], s["beta"], s["d_out"], s["initial"], s["d_final"],
                             want_d_initial_state=c["states"])
    else:
        g = sla.backward(var, q, k, v, ql, kl, s["decay"], s["d_out"], s["initial"], s["d_final"],
                         want_d_initial_state=c["states"], segments=c["segments"])
    r = {"out": out, "final": fin}
    if c["prologue"]:
        r["dwq"] = sla.gate_logits_backward(q, s["wq"], g["dq_head_logits"], g["dq"])
        r["dwk"] = sla.gate_logits_backward(k, s["wk"], g["dk_head_logits"], g["dk"])
    if conv:
        r["dxq"], r["dcq"] = sla.short_conv_silu_l2_backward(s["xq"], s["cq"], g["dq"].view(B, T, H * dk), dk)
        r["dxk"], r["dck"] = sla.short_conv_silu_l2_backward(s["xk"], s["ck"], g["dk"].view(B, T, H * dk), dk)
        r["dxv"], r["dcv"] = sla.short_conv_silu_l2_backward(s["xv"], s["cv"], g["dv"].view(B, T, H * dv))
    r.update({n: t for n, t in g.items() if t is not None})
    return r


def _packed(s):
    var = s["variant"]
    out, fin = sla.forward_varlen(var, s["q"], s["k"], s["v"], s["ql"], s["kl"], s["decay"], s["beta"], s["cu"])
    if var == GDN:
        g = sla.backward_gdn_varlen(s["q"], s["k"], s["v"], s["ql"], s["kl"], s["decay"], s["beta"], s["d_out"], s["cu"])
    else:
        g = sla.backward_varlen(var, s["q"], s["k"], s["v"], s["ql"], s["kl"], s["decay"], s["d_out"], s["cu"])
    r = {"out": out, "final": fin}
    r.update({n: t for n, t in g.items() if t is not None})
    return r


def work(case):
    """Each call of the pass reads its inputs once and writes its outputs once; products as the recurrence needs them."""
    kind, var = case["kind"], VARIANT[case["variant"]]
    H, dk, dv = case["H"], case["dk"], case["dv"]
    es = 2 if case["dtype"] == "bf16" else 4
    n = (case["T"] if kind == "packed" else case["B"] * case["T"]) * H
    seqs = (len(lengths(case)) if kind == "packed" else case["B"]) * H
    decay = {RETNET: 0, GLA: dk * es, GDN: 8}[var]
    state = seqs * dk * dv * 4
    mixer = (2 * dk + dv) * es + decay  # q, k, v and the decay (and beta)
    if kind == "decode":
        gates = 2 * H * dk * 4 if case["prologue"] else n * 8
        return {"bytes": n * (mixer + dv * es) + gates + 2 * state, "flops": n * (4 * dk * dv + (4 * H * dk if case["prologue"] else 0))}
    held = state * (2 if case["states"] else 1)
    total = n * (mixer + 8 + dv * es) + held
    flops = n * (4 * dk * dv + 65 * (dk + dv))
    if kind in ("train", "packed"):
        # inputs again and d_out; one gradient for every input
        total += n * (2 * (mixer + 8) + dv * es) + (3 * state if case["states"] else 0)
        flops += n * (10 * dk * dv + 3 * 65 * (dk + dv))
    if kind == "train" and case["prologue"]:
        total += n * (2 * dk * es + 8) + n * (6 * dk * es + 8)  # projections; theirs backward updates dq, dk in place
        flops += n * 12 * dk
        if var == GDN:
            total += n * (2 * dk + dv) * es * 5  # convolution in and out; x and dy in, dx out
            flops += n * (2 * dk + dv) * 40
    return {"bytes": int(total), "flops": int(flops)}


def tolerance(case):
    """Four times the differences measured between this path and the same call on fp32 tensors (bf16 cases) or the fp64
    oracle (fp32 cases): out and states 3.7e-3, gradients 5e-3 after the prologue's backward; fp32 1.4e-6 and less.  The
    decay gradient is a running sum of differences of large terms: 1.8e-2 (GLA) to 3.2e-2 (delta rule) in bf16."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    if case["kind"] in ("decode", "prefill"):
        return {"rel": 1.5e-2}
    return {"rel": 2e-2 if case["variant"] == "retnet" else 3e-2}
