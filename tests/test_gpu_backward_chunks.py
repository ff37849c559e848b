"""GPU parity of the chunk-parallel backward of RetNet and GLA on bf16 tensors (sla_backward with the workspace that
sla_backward_chunks_workspace_bytes asks for), at the edges of its 64-token chunks and 16-token blocks, for every key
width's split over the waves, against the gradient oracle; and the schedules it can run in against each other.
Tolerance: the bf16 bar of test_gpu_backward.py."""
import numpy as np
import pytest

import sla_inputs as si
from gpu_util import GDN, GLA, RETNET
from test_gpu_backward import check_backward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", [RETNET, GLA])
@pytest.mark.parametrize("T,dk,dv", [(1, 128, 128), (15, 64, 64), (16, 32, 64), (17, 128, 64), (33, 64, 128), (48, 32, 256),
                                     (63, 128, 256), (64, 64, 64), (65, 128, 128), (80, 32, 128), (129, 64, 256), (191, 128, 128)])
def test_edges_of_chunks_and_blocks(variant, T, dk, dv):
    d = si.custom(variant, "bf16", B=2, T=T, H=3, dk=dk, dv=dv, seed=3000 + T)
    cot = si.cotangents(2, T, 3, dk, dv, seed=3001 + T, final_state=True)
    check_backward(variant, d, cot, si.initial_state(2, 3, dk, dv, seed=3002 + T), want_ds0=True, label=f"chunks T={T} {dk}x{dv}")


def _tensors(variant, B, T, H, dk, dv, seed):
    import torch

    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    n = lambda *s: torch.randn(s, generator=g, device="cuda")
    q, k = ((n(B, T, H, dk) * dk ** -0.5).bfloat16() for _ in range(2))
    v, do = n(B, T, H, dv).bfloat16(), n(B, T, H, dv).bfloat16()
    ld = (torch.nn.functional.logsigmoid(n(B, T, H, dk)) / 16).bfloat16() if variant == GLA else -0.02 * torch.arange(1, H + 1, device="cuda")
    return q, k, v, n(B, T, H), n(B, T, H), ld.contiguous(), do


@pytest.mark.parametrize("variant,B,T,H,dk,dv", [(GLA, 3, 1500, 24, 128, 128), (RETNET, 40, 130, 24, 64, 128), (GLA, 1, 2048, 20, 128, 256)])
def test_parts_give_the_same_bits(variant, B, T, H, dk, dv):
    """A workspace too small for the states of the whole batch: the call works it off in parts (whole rows, or heads of one
    row), each result exactly as in one part.  The smallest workspace of all runs the sweeps, to the bf16 bar."""
    import torch
    import paper_2602_01744_amd as sla

    x = _tensors(variant, B, T, H, dk, dv, seed=3100)
    p = sla.SlaParams(variant, sla.BF16, B, T, H, dk, dv, 0, 0, 1)
    want, least = sla.sla_backward_chunks_workspace_bytes(p), 4 * 4 * B * T * H + (64 << 20)
    assert least < want  # the shape has more states than the smallest part's 64 MiB
    whole = sla.backward(variant, *x)
    parts = sla.backward(variant, *x, workspace=torch.empty(least, dtype=torch.uint8, device="cuda"))
    sweeps = sla.backward(variant, *x, workspace=torch.empty(min(sla.sla_backward_workspace_bytes(p), least - 16), dtype=torch.uint8, device="cuda"))
    for n, t in whole.items():
        if t is not None:
            assert torch.equal(t, parts[n]), n
            rel = ((t.double() - sweeps[n].double()).norm() / sweeps[n].double().norm()).item()
            assert rel <= (4e-2 if n == "dlog_decay" else 2e-2), (n, rel)  # the bar of each side


@pytest.mark.parametrize("variant", [RETNET, GLA])
@pytest.mark.parametrize("layout", ["packed", "head-major"])
def test_parts_of_packed_and_head_major_batches(monkeypatch, variant, layout):
    """The same in the other two layouts: some heads of all sequences at a time, and rows of [B,H,T,d] tensors; with and
    without the states' gradients, which GLA's decay gradient takes another area of the workspace for."""
    import torch
    import paper_2602_01744_amd as sla
    from paper_2602_01744_amd import binding

    B, T, H, dk, dv = 3, 1500, 24, 128, 128
    q, k, v, ql, kl, ld, do = _tensors(variant, B, T, H, dk, dv, seed=3150)
    ds = torch.randn(B, H, dk, dv, device="cuda")
    if layout == "packed":
        x = [t.reshape(B * T, *t.shape[2:]) if t.dim() > 2 else t for t in (q, k, v, ql, kl, ld, do)]
        cu = torch.tensor([0, 1000, 1007, B * T], dtype=torch.int32, device="cuda")
        call = lambda: sla.backward_varlen(variant, *x, cu, None, ds, want_d_initial_state=True)
    else:
        hm = lambda t: t.transpose(1, 2).contiguous() if t.dim() == 4 else t
        x = [hm(t) for t in (q, k, v)] + [ql, kl] + [hm(t) for t in (ld, do)]
        call = lambda: sla.backward(variant, *x, None, ds, want_d_initial_state=True, head_major=True)
    whole = call()
    least, plain = 4 * 4 * B * T * H + (64 << 20), binding.sla_backward_chunks_workspace_bytes
    p = sla.SlaParams(variant, sla.BF16, B, B * T if layout == "packed" else T, H, dk, dv, 0, 0, 1)
    assert least < plain(p, layout == "packed")
    monkeypatch.setattr(binding, "sla_backward_chunks_workspace_bytes", lambda p, packed=False: least)
    parts = call()
    for n, t in whole.items():
        assert t is None or torch.equal(t, parts[n]), n


@pytest.mark.parametrize("T,dk,dv", [(100, 64, 64), (64, 128, 128), (200, 128, 256), (130, 32, 64)])
def test_strongest_decay_with_states(T, dk, dv):
    """Log-decay down to the bound of -5 a token, whole blocks of it among them, with states in and out."""
    d = si.custom(GLA, "bf16", B=2, T=T, H=2, dk=dk, dv=dv, seed=3900 + T)
    r = np.random.default_rng(3901)
    ld = (-5.0 * r.random(size=d["log_decay"].shape)).astype(np.float32)
    ld[:, 16:48, :, : dk // 2] = -5.0
    ld[:, :, :, 0] = -5.0
    d["log_decay"] = si.round_to_bf16(ld)
    cot = si.cotangents(2, T, 2, dk, dv, seed=3902, final_state=True)
    check_backward(GLA, d, cot, si.initial_state(2, 2, dk, dv, seed=3903), want_ds0=True, label=f"decay in [-5, 0] T={T} {dk}x{dv}")


@pytest.mark.parametrize("variant", [RETNET, GLA])
def test_layouts_and_packing_give_the_same_bits(variant):
    """[B,H,T,d] tensors, and the rows as a packed batch with empty sequences in between, against the rectangular call."""
    import torch
    import paper_2602_01744_amd as sla

    B, T, H, dk, dv = 3, 201, 5, 128, 128
    q, k, v, ql, kl, ld, do = _tensors(variant, B, T, H, dk, dv, seed=3200)
    ref = sla.backward(variant, q, k, v, ql, kl, ld, do, want_d_initial_state=True)
    hm = lambda t: t.transpose(1, 2).contiguous()
    got = sla.backward(variant, hm(q), hm(k), hm(v), ql, kl, hm(ld) if variant == GLA else ld, hm(do), head_major=True,
                       want_d_initial_state=True)
    for n, t in ref.items():
        if t is not None:
            assert torch.equal(t, got[n] if t.dim() == 3 or n == "d_initial_state" else got[n].transpose(1, 2)), n
    flat = lambda t: t.reshape(B * T, *t.shape[2:])
    cu = torch.tensor([0, 0, T, 2 * T, 2 * T, 2 * T, 3 * T], dtype=torch.int32, device="cuda")
    got = sla.backward_varlen(variant, flat(q), flat(k), flat(v), flat(ql), flat(kl), flat(ld) if variant == GLA else ld,
                              flat(do), cu, want_d_initial_state=True)
    for n, t in ref.items():
        if n == "d_initial_state":
            assert torch.equal(t, got[n][[1, 2, 5]]) and not got[n][[0, 3, 4]].any()
        elif t is not None:
            assert torch.equal(flat(t), got[n]), n


@pytest.mark.parametrize("T,dk,dv", [(1, 128, 128), (16, 32, 64), (63, 64, 256), (64, 128, 64), (65, 64, 128), (130, 128, 256), (200, 32, 128)])
def test_decay_gradient_behind_the_last_token(T, dk, dv):
    """dlog_decay of the last token is rowsum(d_final_state * S_T), here with states so large that nothing else counts, plus
    one token's q dq - k dk.  Formed in fp32 and rounded once, to bf16 (ulp / sqrt(12), 1.6e-3 of the norm for mantissas spread
    over their logarithm); every state rounded to bf16 on the way adds as much: sqrt(2) of it with one, 2.8e-3 with both."""
    d = si.custom(GLA, "bf16", B=2, T=T, H=4, dk=dk, dv=dv, seed=3600 + T)
    d["log_decay"] = si.round_to_bf16((d["log_decay"] * 0.02).astype(np.float32))
    cot = si.cotangents(2, T, 4, dk, dv, seed=3601 + T, final_state=True)
    cot["d_final_state"] = cot["d_final_state"] * np.float32(8)
    s0 = si.initial_state(2, 4, dk, dv, seed=3602 + T) * np.float32(32)
    got, ref = check_backward(GLA, d, cot, s0, want_ds0=True, label=f"last token T={T} {dk}x{dv}")
    e = got["dlog_decay"][:, -1] - ref["dlog_decay"][:, -1]
    err = np.linalg.norm(e) / np.linalg.norm(ref["dlog_decay"][:, -1])
    print(f"[last token] {err:.2e}", flush=True)
    assert err <= 2.0e-3  # between none and one


@pytest.mark.parametrize("variant", [RETNET, GLA, GDN])
@pytest.mark.parametrize("B", [63, 65, 4097])
def test_many_packed_sequences(monkeypatch, variant, B):
    """More sequences than one, and than two, steps of the search for a chunk's sequence look at, empty ones among them, the
    first and last tokens in none: against the sweeps, to the bar of both sides."""
    import torch
    import paper_2602_01744_amd as sla
    from paper_2602_01744_amd import binding

    r = np.random.default_rng(3800 + B)
    lens = r.integers(0, 4, B) * r.integers(0, 3, B)
    lens[r.integers(0, B, 3)] = [64, 65, 200]
    cu = np.concatenate([[5], 5 + np.cumsum(lens)])
    T, H, dk, dv = int(cu[-1]) + 9, 2, 128, 64
    q, k, v, ql, kl, ld, do = (t[0].contiguous() if t.dim() > 1 else t for t in _tensors(min(variant, GLA), 1, T, H, dk, dv, 3801))
    cu = torch.tensor(cu, dtype=torch.int32, device="cuda")
    if variant == GDN:
        k = torch.nn.functional.normalize(k.float(), dim=-1).bfloat16()
        call = lambda: sla.backward_gdn_varlen(q, k, v, ql, kl, ld.float().mean(-1), torch.sigmoid(ql + kl), do, cu, want_d_initial_state=True)
        names, least = ("sla_backward_gdn_chunks_workspace_bytes", sla.sla_backward_gdn_varlen_workspace_bytes)
    else:
        call = lambda: sla.backward_varlen(variant, q, k, v, ql, kl, ld, do, cu, want_d_initial_state=True)
        names, least = ("sla_backward_chunks_workspace_bytes", sla.sla_backward_varlen_workspace_bytes)
    got = call()
    p = sla.SlaParams(variant, sla.BF16, B, T, H, dk, dv, 0, 0, 1)
    assert getattr(sla, names)(p, True) > least(p)
    monkeypatch.setattr(binding, names, lambda p, packed=False: least(p))
    ref = call()
    inside = slice(int(cu[0]), int(cu[-1]))
    for n, t in got.items():
        if t is not None:
            x, y = (t, ref[n]) if n == "d_initial_state" else (t[inside], ref[n][inside])
            rel = ((x.double() - y.double()).norm() / y.double().norm()).item()
            assert rel <= (4e-2 if n == "dlog_decay" else 2e-2), (n, rel)
