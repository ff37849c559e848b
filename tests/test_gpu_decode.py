"""GPU parity of the recurrent decode step (sla_decode_step through the C ABI) against the CPU oracle."""
import numpy as np
import pytest

import sla_inputs as si
from gpu_util import GDN, GLA, RETNET, TOL, rel_err, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

VARIANTS = [RETNET, GLA, GDN]


def _name(v):
    return si.VARIANT_NAMES[v]


def _dev(a, dtype, narrow):
    import torch

    if a is None:
        return None
    x = torch.from_numpy(np.ascontiguousarray(a))
    if narrow and dtype == "bf16":
        y = x.to(torch.bfloat16)
        assert torch.equal(y.to(torch.float32), x), "inputs must be bf16-representable"
        x = y
    return x.cuda().contiguous()


def decode_chain(variant, d, dtype, state0):
    """Feeds the T tokens of d one at a time; returns (out [B,T,H,dv], final state) as float64."""
    import torch
    import paper_2602_01744_amd as sla

    B, T, H, dk = d["q"].shape
    state = torch.from_numpy(np.ascontiguousarray(state0, dtype=np.float32)).cuda()
    outs = []
    ld_all = d["log_decay"]
    for t in range(T):
        q, k, v = (_dev(d[n][:, t], dtype, True) for n in ("q", "k", "v"))
        ql = _dev(d["q_logits"][:, t], dtype, False)
        kl = None if d["k_logits"] is None else _dev(d["k_logits"][:, t], dtype, False)
        ld = _dev(ld_all if variant == RETNET else ld_all[:, t], dtype, variant == GLA)
        beta = None if d["beta"] is None else _dev(d["beta"][:, t], dtype, False)
        o = sla.decode_step(variant, q, k, v, ql, kl, ld, beta, state)
        outs.append(o.to(torch.float32).cpu().numpy().astype(np.float64))
    torch.cuda.synchronize()
    return np.stack(outs, 1), state.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("dk,dv", [(128, 128), (64, 64), (64, 128), (128, 64), (128, 256), (64, 256), (32, 64), (32, 128),
                                   (32, 256)])
def test_single_step_matches_oracle(variant, dtype, dk, dv):
    d = si.custom(variant, dtype, B=3, T=1, H=5, dk=dk, dv=dv, seed=2100 + variant + dk + dv)
    s0 = si.initial_state(3, 5, dk, dv, seed=21)
    o, f = decode_chain(variant, d, dtype, s0)
    ro, rf = run_oracle(variant, d, s0)
    eo, ef = rel_err(o, ro), rel_err(f, rf)
    print(f"[parity] decode {_name(variant)} {dtype} dk={dk} dv={dv} out_err={eo:.3e} state_err={ef:.3e}", flush=True)
    assert eo <= TOL[dtype] and ef <= 1e-5  # the state stays fp32 end to end


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("H", [1, 2, 7, 16, 33, 64])
def test_head_counts(variant, H):
    d = si.custom(variant, "bf16", B=2, T=1, H=H, dk=64, dv=64, seed=2200 + H)
    s0 = si.initial_state(2, H, 64, 64, seed=22)
    o, f = decode_chain(variant, d, "bf16", s0)
    ro, rf = run_oracle(variant, d, s0)
    assert rel_err(o, ro) <= TOL["bf16"] and rel_err(f, rf) <= 1e-5


@pytest.mark.parametrize("variant", VARIANTS)
def test_chain_of_steps_equals_the_sequence_forward(variant):
    """24 decode steps from a given state: every output and the final state against the oracle's forward over
    the same 24 tokens, and against the chunked GPU forward."""
    T = 24
    d = si.custom(variant, "bf16", B=2, T=T, H=4, dk=128, dv=128, seed=2300 + variant)
    s0 = si.initial_state(2, 4, 128, 128, seed=23)
    o, f = decode_chain(variant, d, "bf16", s0)
    ro, rf = run_oracle(variant, d, s0)
    assert rel_err(o, ro) <= TOL["bf16"]
    assert rel_err(f, rf) <= 1e-5
    go, gf = run_gpu(variant, d, "bf16", s0)
    assert rel_err(go, o) <= TOL["bf16"] and rel_err(gf, f) <= TOL["bf16"]


@pytest.mark.parametrize("variant", VARIANTS)
def test_read_gate_only_and_saturated_gates(variant):
    H, sel = 4, 2
    d = si.custom(variant, "bf16", B=2, T=3, H=H, dk=64, dv=128, seed=2400, dual_gates=False)
    s0 = si.initial_state(2, H, 64, 128, seed=24)
    o, f = decode_chain(variant, d, "bf16", s0)
    ro, rf = run_oracle(variant, d, s0)
    assert rel_err(o, ro) <= TOL["bf16"] and rel_err(f, rf) <= 1e-5
    # a saturated read gate selects one head: the others output exact zeros (Thm 4.2 limit)
    sat = np.zeros_like(d["q_logits"]); sat[..., sel] = 1e4
    d["q_logits"] = sat
    o, f = decode_chain(variant, d, "bf16", s0)
    assert np.all(o[:, :, [h for h in range(H) if h != sel]] == 0.0)
    assert np.abs(o[:, :, sel]).max() > 0


def test_zero_decay_zero_beta_leaves_the_state_alone():
    """Delta rule with beta = 0 and log-decay 0: the state must come back bit for bit."""
    d = si.custom(GDN, "f32", B=1, T=2, H=2, dk=64, dv=64, seed=2500)
    d["beta"] = np.zeros_like(d["beta"]); d["log_decay"] = np.zeros_like(d["log_decay"])
    s0 = si.initial_state(1, 2, 64, 64, seed=25)
    o, f = decode_chain(GDN, d, "f32", s0)
    np.testing.assert_array_equal(f, s0.astype(np.float64))


def test_full_size_decode_batch():
    """The shape bench.py times for the decode step (B=64, H=16, d=128, bf16): sampled heads against the oracle."""
    import torch
    import paper_2602_01744_amd as sla

    B, H, dk, dv = 64, 16, 128, 128
    d = si.custom(GLA, "bf16", B=B, T=1, H=H, dk=dk, dv=dv, seed=2600)
    s0 = si.initial_state(B, H, dk, dv, seed=26)
    o, f = decode_chain(GLA, d, "bf16", s0)
    ro, rf = run_oracle(GLA, d, s0)
    assert rel_err(o, ro) <= TOL["bf16"] and rel_err(f, rf) <= 1e-5


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("H,dk,dv,both", [(16, 128, 128, True), (5, 64, 256, True), (33, 128, 64, False), (1, 64, 64, True),
                                          (16, 32, 64, True), (40, 32, 128, True)])
def test_fused_gate_projection_matches_oracle(variant, dtype, H, dk, dv, both):
    """sla_decode_step_fused: logits formed in the kernel from q, k and the gate matrices.  The reference is the
    oracle's projection (q . W_GQ per head) followed by the oracle's forward on those logits."""
    import torch
    import paper_2602_01744_amd as sla
    from oracle import sla_numpy

    B = 3
    d = si.custom(variant, dtype, B=B, T=1, H=H, dk=dk, dv=dv, seed=2700 + variant + H + dk)
    w = si.gate_weights(H, dk, seed=2701 + H)
    d["q_logits"] = sla_numpy.gate_logits(d["q"], w["w_gq"])
    d["k_logits"] = sla_numpy.gate_logits(d["k"], w["w_gk"]) if both else None
    s0 = si.initial_state(B, H, dk, dv, seed=27)
    ro, rf = run_oracle(variant, d, s0)
    state = torch.from_numpy(np.ascontiguousarray(s0, dtype=np.float32)).cuda()
    q, k, v = (_dev(d[n][:, 0], dtype, True) for n in ("q", "k", "v"))
    ld = _dev(d["log_decay"] if variant == RETNET else d["log_decay"][:, 0], dtype, variant == GLA)
    beta = None if d["beta"] is None else _dev(d["beta"][:, 0], dtype, False)
    wq = torch.from_numpy(w["w_gq"]).cuda()
    wk = torch.from_numpy(w["w_gk"]).cuda() if both else None
    o = sla.decode_step(variant, q, k, v, None, None, ld, beta, state, w_gq=wq, w_gk=wk)
    torch.cuda.synchronize()
    eo = rel_err(o.to(torch.float32).cpu().numpy().astype(np.float64)[:, None], ro)
    ef = rel_err(state.cpu().numpy().astype(np.float64), rf)
    print(f"[parity] fused decode {_name(variant)} {dtype} H={H} dk={dk} dv={dv} out_err={eo:.3e} state_err={ef:.3e}",
          flush=True)
    assert eo <= TOL[dtype] and ef <= 1e-5


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("B,H,dk,dv", [(64, 4, 32, 64), (43, 6, 32, 64), (32, 2, 128, 256), (13, 5, 64, 256)])
def test_slice_widths(variant, B, H, dk, dv):
    """Both sides of the rule for the slice width: 256 and 258, 256 and 260 workgroups of 64 columns."""
    d = si.custom(variant, "bf16", B=B, T=2, H=H, dk=dk, dv=dv, seed=2600 + variant + B)
    s0 = si.initial_state(B, H, dk, dv, seed=26)
    o, f = decode_chain(variant, d, "bf16", s0)
    ro, rf = run_oracle(variant, d, s0)
    assert rel_err(o, ro) <= TOL["bf16"] and rel_err(f, rf) <= 1e-5


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("B,H,dk,dv", [(32, 4, 128, 64), (43, 3, 128, 64), (16, 4, 64, 64), (13, 5, 64, 64), (5, 26, 32, 128),
                                       (13, 5, 32, 256), (33, 4, 64, 128), (5, 33, 128, 128), (9, 33, 128, 128),
                                       (60, 17, 128, 128), (21, 48, 128, 128)])
def test_fused_slice_widths(variant, B, H, dk, dv):
    """Both sides of the fused step's rules: dk and dk + 1 workgroups of 64 columns; past 256, slices of 128 and 256 for
    narrow keys; past 512, 128 columns for a small state or (GLA) many heads; states past 60 MB."""
    import torch
    import paper_2602_01744_amd as sla
    from oracle import sla_numpy

    d = si.custom(variant, "bf16", B=B, T=1, H=H, dk=dk, dv=dv, seed=2800 + variant + B)
    w = si.gate_weights(H, dk, seed=2801)
    d["q_logits"], d["k_logits"] = sla_numpy.gate_logits(d["q"], w["w_gq"]), sla_numpy.gate_logits(d["k"], w["w_gk"])
    s0 = si.initial_state(B, H, dk, dv, seed=28)
    ro, rf = run_oracle(variant, d, s0)
    state = torch.from_numpy(np.ascontiguousarray(s0, dtype=np.float32)).cuda()
    q, k, v = (_dev(d[n][:, 0], "bf16", True) for n in ("q", "k", "v"))
    ld = _dev(d["log_decay"] if variant == RETNET else d["log_decay"][:, 0], "bf16", variant == GLA)
    beta = None if d["beta"] is None else _dev(d["beta"][:, 0], "bf16", False)
    o = sla.decode_step(variant, q, k, v, None, None, ld, beta, state, w_gq=torch.from_numpy(w["w_gq"]).cuda(),
                        w_gk=torch.from_numpy(w["w_gk"]).cuda())
    eo = rel_err(o.float().cpu().numpy().astype(np.float64), ro[:, 0])
    ef = rel_err(state.cpu().numpy().astype(np.float64), rf)
    assert eo <= TOL["bf16"] and ef <= 1e-5


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("B,H,dk,dv", [(16, 4, 32, 64), (13, 5, 32, 64), (32, 4, 64, 64), (43, 3, 64, 64)])
def test_slice_widths_of_narrow_keys(variant, B, H, dk, dv):
    """2 dk workgroups of 64 columns and one more."""
    test_slice_widths(variant, B, H, dk, dv)


@pytest.mark.parametrize("variant", VARIANTS)
@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("B,H,d", [(2, 3, 64), (40, 16, 128)])
def test_out_may_be_an_input(variant, fused, B, H, d):
    """out in the memory of an input: one workgroup then owns a whole head, and reads all of it before it writes.  The
    outputs agree with those in a tensor of their own up to the order of fp32 sums (a last bit of bf16, 2^-8)."""
    import torch
    import paper_2602_01744_amd as sla

    x = si.custom(variant, "bf16", B=B, T=1, H=H, dk=d, dv=d, seed=2900 + variant)
    s0 = torch.from_numpy(si.initial_state(B, H, d, d, seed=29).astype(np.float32)).cuda()
    ql, kl = (_dev(x[n][:, 0], "bf16", False) for n in ("q_logits", "k_logits"))
    w = torch.from_numpy(si.gate_weights(H, d, seed=29)["w_gq"]).cuda()

    def step(alias):
        t = {n: _dev(x[n][:, 0], "bf16", True) for n in ("q", "k", "v")}
        t["log_decay"] = _dev(x["log_decay"] if variant == RETNET else x["log_decay"][:, 0], "bf16", variant == GLA)
        beta = None if x["beta"] is None else _dev(x["beta"][:, 0], "bf16", False)
        state = s0.clone()
        gates = dict(w_gq=w, w_gk=w) if fused else {}
        o = sla.decode_step(variant, t["q"], t["k"], t["v"], None if fused else ql, None if fused else kl, t["log_decay"], beta,
                            state, out=t.get(alias), **gates)
        return o.float(), state

    want, ws = step(None)
    for alias in ["v"] if fused else ["q", "k", "v"] + ["log_decay"] * (variant == GLA):
        got, gs = step(alias)
        assert float((got - want).norm() / want.norm()) <= 2.0**-8, alias
        assert float((gs - ws).norm() / ws.norm()) <= 1e-6, alias
