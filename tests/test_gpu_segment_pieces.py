"""The segment schedule's pre-pass on pieces of segments: against the oracle, and against the pre-pass on whole segments,
which a workspace of sla_workspace_bytes still gets."""
import pytest
import torch

import paper_2602_01744_amd as sla
import sla_inputs as si
from gpu_util import GLA, RETNET, check, rel_err

# T, segments: segments of 576 tokens in 2 pieces (288), 768 in 3 (256), 1088 in 4 (272), 2048 in 8 (256); ragged ends
# pieces in several segments: three segments of 576 in 2, four of 768 in 3 (the chain takes four pieces at a time, so that
# segments end inside of a group)
CHAINS = [(3 * 576 - 9, 3), (4 * 768 - 7, 4)]
SHAPES = [(1100, 2), (2 * 768 - 1, 2), (2065, 2), (2 * 2048 - 3, 2)]


def _params(variant, dtype, T, segments, B=1, H=2, dk=64, dv=64):
    return sla.SlaParams(variant, {"f32": sla.F32, "bf16": sla.BF16}[dtype], B, T, H, dk, dv, 0, 0, segments)


@pytest.mark.parametrize("T,segments", SHAPES)
def test_workspace_holds_the_pieces(T, segments):
    p = _params(GLA, "bf16", T, segments)
    m = {1100: 2, 1535: 3, 2065: 4, 4093: 8}[T]
    n = (sla.sla_segments(p, 256) - 1) * m
    want = 4 * 2 * ((n + 1) * 64 * 64 + n * 8 * 64)
    assert sla.sla_forward_workspace_bytes(p, 256) == sla.sla_workspace_bytes(p, 256) + want
    whole = _params(GLA, "bf16", 500, 2)  # 256 tokens: too short to cut
    assert sla.sla_forward_workspace_bytes(whole, 256) == sla.sla_workspace_bytes(whole, 256) > 0
    assert sla.sla_forward_workspace_bytes(_params(GLA, "bf16", T, 1), 256) == 0
    assert sla.sla_forward_workspace_bytes(_params(sla.GDN, "bf16", T, 0), 256) == 0


WIDTHS = [(2, 4096, 8, 128, 128, 2), (1, 65536, 32, 128, 128, 0), (1, 1100, 2, 64, 64, 2), (4, 8192, 4, 128, 256, 0), (3, 2065, 5, 32, 128, 2)]


@pytest.mark.parametrize("B,T,H,dk,dv,segments", WIDTHS)
def test_slice_width_does_not_choose_the_pieces(B, T, H, dk, dv, segments):
    """dv_split is a schedule, not a result: the pieces, whose chaining orders the sums, are the same for every width."""
    sizes = set()
    for width in (0, 16, 32, 64):
        p = _params(GLA, "bf16", T, segments, B, H, dk, dv)
        p.dv_split = width
        sizes.add(sla.sla_forward_workspace_bytes(p, 256))
    assert len(sizes) == 1 and sizes.pop() > 0


@pytest.mark.gpu
@pytest.mark.parametrize("variant", [RETNET, GLA])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,T,H,dk,dv,segments", [(2, 1152, 8, 128, 128, 2), (1, 1100, 2, 64, 64, 2), (1, 3100, 3, 32, 256, 3)])
def test_slice_width_keeps_the_bits(variant, dtype, B, T, H, dk, dv, segments):
    d = si.custom(variant, dtype, B=B, T=T, H=H, dk=dk, dv=dv, seed=1800 + T)
    g, _ = si.to_device(d, dtype, variant)
    args = [g[n] for n in ("q", "k", "v", "q_logits", "k_logits", "log_decay", "beta")]
    ref, fin = sla.forward(variant, *args, segments=segments)
    for width in (16, 32, 64):
        o, f = sla.forward(variant, *args, segments=segments, dv_split=width)
        assert torch.equal(o, ref) and torch.equal(f, fin), width


@pytest.mark.gpu
@pytest.mark.parametrize("variant", [RETNET, GLA])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T,segments", SHAPES + CHAINS)
def test_pieces(variant, dtype, T, segments):
    d = si.custom(variant, dtype, B=1, T=T, H=2, dk=64, dv=64, seed=1700 + T)
    s0 = si.initial_state(1, 2, 64, 64, seed=1701)
    check(variant, d, dtype, s0, label=f"{si.VARIANT_NAMES[variant]} T={T} in pieces", segments=segments)
    g, _ = si.to_device(d, dtype, variant)
    args = [g[n] for n in ("q", "k", "v", "q_logits", "k_logits", "log_decay", "beta")] + [torch.from_numpy(s0).cuda()]
    o1, f1 = sla.forward(variant, *args, segments=segments)
    ws = torch.empty(sla.sla_workspace_bytes(_params(variant, dtype, T, segments), 256), dtype=torch.uint8, device="cuda")
    o2, f2 = sla.forward(variant, *args, segments=segments, workspace=ws)
    # the states differ by the order of fp32 sums; out, rounded to bf16 from it, by a rounding of single elements
    assert rel_err(f1.cpu().numpy(), f2.cpu().numpy()) <= 2e-5
    assert rel_err(o1.float().cpu().numpy(), o2.float().cpu().numpy()) <= (2e-5 if dtype == "f32" else 4e-3)
