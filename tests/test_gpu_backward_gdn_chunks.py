"""The chunk-parallel backward of the delta rule on bf16 tensors (sla_backward_gdn with the workspace that
sla_backward_gdn_chunks_workspace_bytes asks for): what that query asks for; at the edges of the 64-token chunks and their
32-token blocks against the gradient oracle, to the bf16 bar of test_gpu_backward_gdn.py; against the sweeps; packed."""
import pytest

import paper_2602_01744_amd as sla
import sla_inputs as si


def _params(dtype=sla.BF16, B=2, T=100, H=4, dk=128, dv=128, variant=sla.GDN):
    return sla.SlaParams(variant, dtype, B, T, H, dk, dv, 0, 0, 1)


@pytest.mark.parametrize("packed", [False, True])
def test_size(packed):
    least = sla.sla_backward_gdn_varlen_workspace_bytes if packed else sla.sla_backward_gdn_workspace_bytes
    for B, T, H, dk, dv in ((2, 100, 4, 128, 128), (1, 1, 1, 64, 64), (8, 4096, 4, 128, 256), (3, 65, 7, 64, 128)):
        rows = T if packed else B * T
        slots, blocks = ((T // n + B + 1) if packed else B * ((T + n - 1) // n) for n in (64, 32))
        four = lambda n: (n + 3) // 4 * 4
        # gates, their gradients and the decay's scalar; the ends of 512-token spans as eight sums, of sequences as one for each
        # 16 value columns; two bf16 states per chunk, and the rest of two per span; res and du; 8 x 32 floats and a bf16
        # matrix per block
        spans = rows // 512 + 1
        want = (5 * four(rows * H) + 8 * spans * H + B * H * dv // 16 + (slots + spans) * H * dk * dv + 3 * rows * H * dv // 2
                + blocks * H * (256 + 512))
        p = _params(B=B, T=T, H=H, dk=dk, dv=dv)
        assert sla.sla_backward_gdn_chunks_workspace_bytes(p, packed) == max(4 * want, least(p))
    for p in (_params(dtype=sla.F32), _params(dk=32), _params(T=0), _params(B=0), _params(B=8, T=65536, H=16)):
        assert sla.sla_backward_gdn_chunks_workspace_bytes(p, packed) == least(p)
    assert sla.sla_backward_gdn_chunks_workspace_bytes(_params(variant=sla.GLA), packed) == 0
    # 256 workgroups of long rows in the sweeps: they keep a rectangular batch
    full = _params(B=8, T=4096, H=16)
    assert (sla.sla_backward_gdn_chunks_workspace_bytes(full, packed) == least(full)) == (not packed)


def test_which_calls_run_chunk_parallel():
    def chunks(B, T, H, dk=128, dv=128, packed=False):
        p = _params(B=B, T=T, H=H, dk=dk, dv=dv)
        least = sla.sla_backward_gdn_varlen_workspace_bytes if packed else sla.sla_backward_gdn_workspace_bytes
        return sla.sla_backward_gdn_chunks_workspace_bytes(p, packed) > least(p)

    # one full round of the sweeps' workgroups on long rows; not a round and a part, nor two, nor short rows
    assert not chunks(8, 4096, 16) and chunks(8, 4096, 15) and chunks(10, 4096, 16) and chunks(16, 4096, 16) and chunks(8, 1024, 16)
    assert chunks(16, 4096, 16, 128, 64) and chunks(8, 2048, 32, 64, 128) and chunks(16, 4096, 16, 64, 64)
    # heads of 256 values: where the sweeps fill three quarters of the chip in every round
    assert chunks(5, 1024, 16, 128, 256) and not chunks(7, 1024, 16, 128, 256) and not chunks(8, 512, 16, 128, 256)
    assert chunks(10, 1024, 16, 128, 256) and not chunks(16, 1024, 16, 128, 256) and chunks(7, 256, 16, 128, 256)
    assert not chunks(32, 32 * 256, 16, 128, 256, packed=True) and chunks(32, 32 * 64, 16, 128, 256, packed=True)
    assert not chunks(16, 1024, 16, 64, 256) and chunks(24, 1024, 16, 64, 256) and chunks(16, 16384, 16, 64, 256, packed=True)


@pytest.mark.gpu
@pytest.mark.parametrize("T,dk,dv", [(1, 128, 128), (16, 64, 64), (31, 128, 64), (33, 64, 128), (48, 128, 256), (63, 64, 256),
                                     (64, 128, 128), (65, 64, 64), (96, 128, 128), (97, 128, 128), (129, 64, 128), (200, 128, 256)])
def test_edges_of_chunks_and_blocks(T, dk, dv):
    from test_gpu_backward_gdn import check_backward_gdn

    d = si.custom(sla.GDN, "bf16", B=2, T=T, H=3, dk=dk, dv=dv, seed=3300 + T)
    cot = si.cotangents(2, T, 3, dk, dv, seed=3301 + T, final_state=True)
    check_backward_gdn(d, cot, si.initial_state(2, 3, dk, dv, seed=3302 + T), want_ds0=True, label=f"chunks T={T} {dk}x{dv}")


def _tensors(B, T, H, dk, dv, seed, dtype):
    import torch

    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    n = lambda *s: torch.randn(s, generator=g, device="cuda")
    norm = lambda x: torch.nn.functional.normalize(x, dim=-1)
    wide = [norm(n(B, T, H, dk)), norm(n(B, T, H, dk)), n(B, T, H, dv)]
    small = [n(B, T, H), n(B, T, H), torch.nn.functional.logsigmoid(n(B, T, H)) / 8, torch.sigmoid(n(B, T, H))]
    return [x.bfloat16().to(dtype) for x in wide] + small + [n(B, T, H, dv).bfloat16().to(dtype)]


@pytest.mark.gpu
@pytest.mark.parametrize("B,T,H,dk,dv", [(2, 1000, 5, 128, 128), (3, 333, 4, 64, 256)])
def test_no_further_from_fp32_than_the_sweeps(B, T, H, dk, dv):
    """Both schedules against the same call on fp32 tensors of the same values."""
    import torch

    x = _tensors(B, T, H, dk, dv, 3400, torch.bfloat16)
    ref = sla.backward_gdn(*_tensors(B, T, H, dk, dv, 3400, torch.float32), want_d_initial_state=True)
    p = _params(B=B, T=T, H=H, dk=dk, dv=dv)
    small = torch.empty(sla.sla_backward_gdn_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    large = torch.empty(sla.sla_backward_gdn_chunks_workspace_bytes(p) + (64 << 20), dtype=torch.uint8, device="cuda")
    assert sla.sla_backward_gdn_chunks_workspace_bytes(p) >= small.numel()
    out = [sla.backward_gdn(*x, want_d_initial_state=True, workspace=w) for w in (large, small)]
    for n, t in ref.items():
        if t is not None:
            err = [((o[n].double() - t.double()).norm() / t.double().norm()).item() for o in out]
            print(f"[chunks] {n} {err[0]:.3e}, sweeps {err[1]:.3e}", flush=True)
            # the bf16 bar; the decay gradient, a sum of rounding errors of up to 512 tokens, to the bar of a sum of
            # that many.  1.15: the two round independently, and their errors scatter by 10 % from shape to shape.
            assert err[0] <= (4e-2 if n == "dlog_decay" else 2e-2) and err[0] <= 1.15 * err[1], (n, err)


@pytest.mark.gpu
def test_packing_gives_the_same_bits():
    """The rows as a packed batch with empty sequences in between, against the rectangular call."""
    import torch

    B, T, H, dk, dv = 3, 201, 5, 128, 128
    x = _tensors(B, T, H, dk, dv, 3500, torch.bfloat16)
    ref = sla.backward_gdn(*x, want_d_initial_state=True)
    flat = lambda t: t.reshape(B * T, *t.shape[2:])
    cu = torch.tensor([0, 0, T, 2 * T, 2 * T, 2 * T, 3 * T], dtype=torch.int32, device="cuda")
    got = sla.backward_gdn_varlen(*[flat(t) for t in x], cu, want_d_initial_state=True)
    for n, t in ref.items():
        if n == "d_initial_state":
            assert torch.equal(t, got[n][[1, 2, 5]]) and not got[n][[0, 3, 4]].any()
        elif t is not None:
            assert torch.equal(flat(t), got[n]), n


@pytest.mark.gpu
@pytest.mark.parametrize("B,T,dk,dv", [(2, 1, 128, 128), (1, 8, 64, 64), (2, 64, 128, 256), (1, 200, 64, 128), (2, 512, 64, 256), (1, 1025, 128, 128), (2, 1600, 128, 64)])
def test_decay_gradient_at_anchors(B, T, dk, dv):
    """dlog_decay of a row's last token, and of every 512th, is <X, S> behind it plus one token's scalar, here with states so
    large that <X, S> is nearly all of it.  It is formed from the states as the sweeps carry them: 2^-17 of a product's
    terms, and the rounding of the tokens' own operands, 2^-9 of what they add to states that are 64 times as large: 1e-4.
    States in bf16 would give 2e-3."""
    import numpy as np
    from test_gpu_backward_gdn import check_backward_gdn

    H = 3
    d = si.custom(sla.GDN, "bf16", B=B, T=T, H=H, dk=dk, dv=dv, seed=3700 + T)
    d["log_decay"] = (d["log_decay"] * 1e-3).astype(np.float32)
    d["beta"] = (d["beta"] * 1e-3).astype(np.float32)  # the rule erases what it reads: keep the states for 1600 tokens
    cot = si.cotangents(B, T, H, dk, dv, seed=3701 + T, final_state=True)
    cot["d_final_state"] = cot["d_final_state"] * np.float32(64)
    s0 = si.initial_state(B, H, dk, dv, seed=3702 + T) * np.float32(64)
    got, ref = check_backward_gdn(d, cot, s0, want_ds0=True, label=f"anchors T={T} {dk}x{dv}")
    for t in [T - 1] + list(range(511, T - 1, 512)):
        e = got["dlog_decay"][:, t] - ref["dlog_decay"][:, t]
        # on the scale of the products' root sum of squares, which <X, S> itself may be small against
        scale = np.linalg.norm(s0, axis=(2, 3)) * np.linalg.norm(cot["d_final_state"], axis=(2, 3)) / np.sqrt(dk * dv)
        err = np.abs(e / scale).max()
        print(f"[anchor] t={t} {err:.2e}", flush=True)
        assert err <= 5e-4
