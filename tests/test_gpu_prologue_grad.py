"""GPU parity of the prologue's backward and of the feature map's L2 option against oracle/sla_prologue.py."""
import numpy as np
import pytest

import sla_inputs as si
from gpu_util import GLA, rel_err
from oracle import sla_prologue as op

pytestmark = pytest.mark.gpu

# fp32 tensors: fp32 accumulation against fp64, hardware exp2 / rsq (1 ulp); bf16 tensors: one rounding of the output
TOL = {"f32": 1e-5, "bf16": 6e-3}


def _dev(a, dtype):
    import torch

    t = torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    return t.to(torch.bfloat16) if dtype == "bf16" else t


def _host(t):
    import torch

    return t.to(torch.float32).cpu().numpy().astype(np.float64)


def _round(a, dtype):
    return si.round_to_bf16(a.astype(np.float32)) if dtype == "bf16" else a.astype(np.float32)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("head_width,C", [(0, 72), (32, 128), (64, 256), (128, 384)])
@pytest.mark.parametrize("K", [1, 4])
def test_feature_map_l2_forward_and_backward(dtype, head_width, C, K):
    import paper_2602_01744_amd as sla

    rng = np.random.default_rng(3000 + C + K)
    B, T = 2, 150  # three segments of 64 tokens, the last ragged
    x = _round(rng.normal(size=(B, T, C)), dtype)
    w = rng.normal(size=(C, K)).astype(np.float32) * 0.5
    dy = _round(rng.normal(size=(B, T, C)), dtype)
    eps = 1e-6
    xd, wd, dyd = _dev(x, dtype), _dev(w, "f32"), _dev(dy, dtype)
    y = sla.short_conv_silu_l2(xd, wd, head_width, eps)
    dx, dw = sla.short_conv_silu_l2_backward(xd, wd, dyd, head_width, eps)
    ry = op.short_conv_silu_l2(x, w, head_width, eps)
    rdx, rdw = op.short_conv_silu_l2_backward(x, w, dy, head_width, eps)
    ey, ex, ew = rel_err(_host(y), ry), rel_err(_host(dx), rdx), rel_err(_host(dw), rdw)
    print(f"[feature map] {dtype} C={C} head={head_width} K={K}: y {ey:.2e} dx {ex:.2e} dw {ew:.2e}", flush=True)
    assert ey <= TOL[dtype] and ex <= TOL[dtype] and ew <= 1e-5, (ey, ex, ew)
    if head_width == 0:  # the plain entry point is the same function
        y0 = sla.short_conv_silu(xd, wd)
        assert rel_err(_host(y0), ry) <= TOL[dtype]
    # the two-stage sum over tokens is bitwise reproducible
    dx2, dw2 = sla.short_conv_silu_l2_backward(xd, wd, dyd, head_width, eps)
    assert bool((dw2 == dw).all()) and bool((dx2 == dx).all())


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("H,dk", [(1, 64), (5, 128), (16, 32), (16, 128), (64, 64)])
def test_gate_logits_backward(dtype, H, dk):
    import paper_2602_01744_amd as sla

    rng = np.random.default_rng(3100 + H + dk)
    B, T = 2, 333
    x = _round(rng.normal(size=(B, T, H, dk)), dtype)
    w = si.gate_weights(H, dk, seed=3101)["w_gq"]
    dl = rng.normal(size=(B, T, H)).astype(np.float32)
    dx0 = _round(rng.normal(size=(B, T, H, dk)), dtype)  # what the mixer's backward left in dq
    dxd = _dev(dx0, dtype)
    dw = sla.gate_logits_backward(_dev(x, dtype), _dev(w, "f32"), _dev(dl, "f32"), dxd)
    rdx, rdw = op.gate_logits_backward(x, w, dl)
    ex, ew = rel_err(_host(dxd), dx0.astype(np.float64) + rdx), rel_err(_host(dw), rdw)
    print(f"[gate logits bwd] {dtype} H={H} dk={dk}: dx {ex:.2e} dw {ew:.2e}", flush=True)
    assert ex <= TOL[dtype] and ew <= 1e-5, (ex, ew)


def test_prologue_and_mixer_gradients_chain():
    """Gate logits -> forward -> backward -> gate projections' backward on one small GLA problem: the logit
    cotangents that sla_backward returns, pushed through the projections, against the two oracles chained."""
    import torch

    import paper_2602_01744_amd as sla
    from gpu_util import to_device
    from oracle import sla_backward as ob
    from oracle import sla_numpy as on

    B, T, H, dk, dv = 1, 100, 4, 128, 128
    d = si.custom(GLA, "bf16", B=B, T=T, H=H, dk=dk, dv=dv, seed=3200)
    gw = si.gate_weights(H, dk, seed=3201)
    cot = si.cotangents(B, T, H, dk, dv, seed=3202)
    g, _ = to_device(d, "bf16", GLA)
    wq, wk = torch.from_numpy(gw["w_gq"]).cuda(), torch.from_numpy(gw["w_gk"]).cuda()
    ql, kl = sla.gate_logits(g["q"], g["k"], wq, wk)
    dout = torch.from_numpy(cot["d_out"]).to(torch.bfloat16).cuda()
    gr = sla.backward(GLA, g["q"], g["k"], g["v"], ql, kl, g["log_decay"], dout)
    dwq = sla.gate_logits_backward(g["q"], wq, gr["dq_head_logits"], gr["dq"])
    dwk = sla.gate_logits_backward(g["k"], wk, gr["dk_head_logits"], gr["dk"])
    torch.cuda.synchronize()
    # oracle chain on the same (bf16-representable) inputs, logits in fp64 rounded to the fp32 the GPU passes on
    rql = on.gate_logits(d["q"], gw["w_gq"]).astype(np.float32)
    rkl = on.gate_logits(d["k"], gw["w_gk"]).astype(np.float32)
    ref = ob.backward(GLA, d["q"], d["k"], d["v"], rql, rkl, d["log_decay"], cot["d_out"])
    pq, rwq = op.gate_logits_backward(d["q"], gw["w_gq"], ref["dq_logits"])
    pk, rwk = op.gate_logits_backward(d["k"], gw["w_gk"], ref["dk_logits"])
    assert rel_err(_host(gr["dq"]), ref["dq"] + pq) <= 2e-2
    assert rel_err(_host(gr["dk"]), ref["dk"] + pk) <= 2e-2
    assert rel_err(_host(dwq), rwq) <= 2e-2 and rel_err(_host(dwk), rwk) <= 2e-2


@pytest.mark.parametrize("C", [1024, 2048])
def test_feature_map_segment_lengths_agree(C):
    """How many tokens a thread walks depends on the size of the batch (here 32 and 64, a row alone: 16); every token's
    arithmetic is the same, so rows of a batch equal the rows run alone, bit for bit; dw differs by summation order."""
    import torch

    import paper_2602_01744_amd as sla

    B, T = 40, 1160  # 19 segments of 64 tokens, the last of 8
    gen = torch.Generator(device="cuda").manual_seed(3300 + C)
    x, dy = (torch.randn(B, T, C, generator=gen, device="cuda").bfloat16() for _ in range(2))
    w = torch.randn(C, 4, generator=gen, device="cuda") * 0.5
    y = sla.short_conv_silu_l2(x, w, 128)
    dx, dw = sla.short_conv_silu_l2_backward(x, w, dy, 128)
    rows = [sla.short_conv_silu_l2_backward(x[b : b + 1], w, dy[b : b + 1], 128) for b in range(B)]
    for b in range(B):
        assert torch.equal(sla.short_conv_silu_l2(x[b : b + 1], w, 128)[0], y[b])
        assert torch.equal(rows[b][0][0], dx[b])
    total = torch.stack([r[1].double() for r in rows]).sum(0)
    assert float((dw.double() - total).abs().max() / total.abs().max()) <= 1e-5


def test_feature_map_saturates():
    """SiLU far out: exactly 0 (not NaN) where e^-s overflows, s itself on the other side; gradients 0 and dy."""
    import torch

    import paper_2602_01744_amd as sla

    x = torch.tensor([-3e38, -1e4, -100.0, 100.0, 1e4, 3e38, 0.0, -0.0], device="cuda").repeat(1, 5, 1)
    w = torch.ones(8, 1, device="cuda")
    dy = torch.full_like(x, 2.0)
    want = torch.where(x > 0, x, torch.zeros_like(x))
    assert torch.equal(sla.short_conv_silu(x, w), want)
    dx, _ = sla.short_conv_silu_l2_backward(x, w, dy)
    assert torch.equal(dx[..., :6], torch.where(x > 0, dy, torch.zeros_like(x))[..., :6])
    assert torch.equal(dx[..., 6:], torch.ones_like(dx[..., 6:]))


def test_silu_is_a_correctly_rounded_division():
    """silu(s) = s / (1 + e^-s) with one rounding of the quotient.  Where s * log2(e) rounds to a whole number n the
    hardware's power of two is exact and so is 1 + 2^-n for |n| <= 23, which leaves the division as the only rounding:
    equality with numpy's.  Where 1 / (1 + e^-s) is subnormal the quotient is not: 88 units of fp32 rounding in the
    exponent, e^-s off by 88 * 2^-23 at most."""
    import torch

    import paper_2602_01744_amd as sla

    log2e, s, want = np.float32(1.4426950408889634), [], []
    for n in range(-23, 24):
        near = np.float32(n / 1.4426950408889634)
        for x in {near, np.nextafter(near, np.float32(-99)), np.nextafter(near, np.float32(99))}:
            if np.float32(x * log2e) == n:
                s.append(x)
                want.append(np.float32(x) / np.float32(1.0 + 2.0**-n))
    s, want = np.array(s, np.float32), np.array(want, np.float32)
    assert len(s) >= 47
    one = lambda a: torch.from_numpy(np.resize(a, -(-len(a) // 8) * 8)).cuda().view(1, -1, 8)
    w = torch.ones(8, 1, device="cuda")
    assert torch.equal(sla.short_conv_silu(one(s), w), one(want))
    s = np.linspace(-88.6, -87.4, 64).astype(np.float32)
    got = sla.short_conv_silu(one(s), w).cpu().double().numpy().ravel()
    exact = s.astype(np.float64) / (1.0 + np.exp(-s.astype(np.float64)))
    assert np.abs(got / exact - 1.0).max() <= 88 * 2.0**-23 + 2.0**-22


def test_short_division_equals_the_division():
    """A group of eight values with one below -87 takes the compiler's divisions, any other the short form: the same
    values with and without such a neighbour, bit for bit (every 509th bit pattern, infinities and both zeros)."""
    import torch

    import paper_2602_01744_amd as sla

    bits = torch.arange(-(1 << 31), 1 << 31, 509, dtype=torch.int64, device="cuda")
    bits = torch.cat([bits, torch.tensor([0, -(1 << 31), 0x7F800000], device="cuda")]).to(torch.int32)
    x = bits[len(bits) % 7 :].view(torch.float32).view(-1, 7)
    w = torch.ones(8, 1, device="cuda")
    run = lambda first: torch.cat([torch.full_like(x[:, :1], first), x], 1).view(1, -1, 8).contiguous()
    for f in (lambda z: sla.short_conv_silu(z, w),
              lambda z: sla.short_conv_silu_l2_backward(z, w, torch.ones_like(z))[0]):
        a, b = (f(run(first))[0, :, 1:] for first in (1.0, -90.0))
        differ = a.contiguous().view(torch.int32) != b.contiguous().view(torch.int32)
        assert int((differ & ~(torch.isnan(a) & torch.isnan(b))).sum()) == 0


@pytest.mark.parametrize("B,T,C,head", [(3, 1000, 128, 128), (70, 4000, 128, 128), (140, 4000, 72, 0), (300, 4000, 64, 0)])
def test_feature_map_backward_with_few_channels(B, T, C, head):
    """Waves that hold several segments of few channels each, walked by four, two and one threads: dx of sampled rows
    equals those rows run alone, bit for bit, and dw the sum over parts of the batch."""
    import torch

    import paper_2602_01744_amd as sla

    gen = torch.Generator(device="cuda").manual_seed(3400 + C)
    x, dy = (torch.randn(B, T, C, generator=gen, device="cuda").bfloat16() for _ in range(2))
    w = torch.randn(C, 4, generator=gen, device="cuda") * 0.5
    dx, dw = sla.short_conv_silu_l2_backward(x, w, dy, head)
    for b in {0, B // 2, B - 1}:
        assert torch.equal(sla.short_conv_silu_l2_backward(x[b : b + 1], w, dy[b : b + 1], head)[0][0], dx[b])
    total = sum(sla.short_conv_silu_l2_backward(x[b : b + 2].contiguous(), w, dy[b : b + 2].contiguous(), head)[1].double()
                for b in range(0, B, 2))
    assert float((dw.double() - total).abs().max() / total.abs().max()) <= 1e-5
