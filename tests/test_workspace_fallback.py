"""The binding allocates the workspace that a call runs fastest with; where there is no room for it, the one it needs."""
import pytest
import torch

import paper_2602_01744_amd as sla
from paper_2602_01744_amd import binding


def _full_above(monkeypatch, limit):
    """Memory with room for tensors of up to `limit` bytes; returns the sizes asked for above 16 KiB."""
    asked, empty = [], torch.empty

    def fake(*shape, **kw):
        if kw.get("dtype") is torch.uint8 and shape[0] > 1 << 14:
            asked.append(shape[0])
            if shape[0] > limit:
                raise torch.cuda.OutOfMemoryError("no room")
        return empty(*shape, **kw)

    monkeypatch.setattr(torch, "empty", fake)
    return asked


def test_falls_back_to_what_is_needed(monkeypatch):
    asked = _full_above(monkeypatch, 1 << 16)
    assert binding._workspace("cpu", 1 << 20, lambda: 1 << 15).numel() == 1 << 15 and asked == [1 << 20, 1 << 15]
    assert binding._workspace("cpu", 1 << 15, lambda: 1 << 15).numel() == 1 << 15
    assert binding._workspace("cpu", 0, lambda: 0).numel() == 16
    for least in (1 << 17, 1 << 20):  # no room for that either; nothing smaller to ask for
        with pytest.raises(torch.cuda.OutOfMemoryError):
            binding._workspace("cpu", 1 << 20, lambda: least)


@pytest.mark.gpu
@pytest.mark.parametrize("call", ["backward", "backward_varlen", "backward_gdn", "backward_gdn_varlen", "forward"])
def test_calls_run_with_little_memory(monkeypatch, call):
    gdn, packed = "gdn" in call, "varlen" in call
    B, T, H, d = (1, 4096, 2, 64) if call == "forward" else (2, 300, 3, 128)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    n = lambda *s: torch.randn(s, generator=g, device="cuda")
    q, k, v, do = (n(B, T, H, d).mul(d ** -0.5).bfloat16() for _ in range(4))
    ql, kl = n(B, T, H), n(B, T, H)
    ld = -torch.rand(B, T, H, generator=g, device="cuda") / 8 if gdn else (-torch.rand(B, T, H, d, generator=g, device="cuda") / 16).bfloat16()
    beta = (torch.rand(B, T, H, generator=g, device="cuda"),) if gdn else ()
    p = sla.SlaParams(sla.GDN if gdn else sla.GLA, sla.BF16, B, B * T if packed else T, H, d, d, 0, 0, 2 if call == "forward" else 1)
    if call == "forward":
        most, least = sla.sla_forward_workspace_bytes(p, 256), sla.sla_workspace_bytes(p, 256)
        run = lambda: sla.forward(sla.GLA, q, k, v, ql, kl, ld, None, segments=2)
    else:
        most = (sla.sla_backward_gdn_chunks_workspace_bytes if gdn else sla.sla_backward_chunks_workspace_bytes)(p, packed)
        least = {"backward": sla.sla_backward_workspace_bytes, "backward_varlen": sla.sla_backward_varlen_workspace_bytes,
                 "backward_gdn": sla.sla_backward_gdn_workspace_bytes,
                 "backward_gdn_varlen": sla.sla_backward_gdn_varlen_workspace_bytes}[call](p)
        x = [q, k, v, ql, kl, ld, *beta, do]
        if packed:
            x = [t.reshape(B * T, *t.shape[2:]) for t in x] + [torch.tensor([0, T, B * T], dtype=torch.int32, device="cuda")]
        run = lambda: getattr(sla, call)(*(() if gdn else (sla.GLA,)), *x)
    assert most > least
    ref = run()
    asked = _full_above(monkeypatch, least)
    got = run()
    assert asked == [most, least]
    pairs = zip(ref, got) if call == "forward" else ((t, got[n]) for n, t in ref.items() if t is not None)
    for a, b in pairs:
        rel = ((a.double() - b.double()).norm() / a.double().norm()).item()
        assert rel <= 4e-2  # the bf16 bar of two schedules
