"""sla_backward_chunks_workspace_bytes (host side, no GPU): what it asks for and that it never is less than the plain queries."""
import pytest

import paper_2602_01744_amd as sla


def _params(variant=sla.GLA, dtype=sla.BF16, B=2, T=100, H=4, dk=128, dv=128, flags=0, segments=1):
    return sla.SlaParams(variant, dtype, B, T, H, dk, dv, 0, flags, segments)


@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("variant", [sla.RETNET, sla.GLA])
def test_size(variant, packed):
    least = sla.sla_backward_varlen_workspace_bytes if packed else sla.sla_backward_workspace_bytes
    for B, T, H, dk, dv in ((2, 100, 4, 128, 128), (1, 1, 1, 64, 64), (8, 4096, 4, 128, 256), (3, 64, 64, 32, 64)):
        rows = T if packed else B * T
        slots = T // 64 + B + 1 if packed else B * ((T + 63) // 64)
        # gates and their gradients, rounded to 16 bytes; two bf16 states per chunk and head; GLA: rowsum(d_final * S) in
        # fp32, a sum for each 32 value columns
        want = 4 * 4 * ((rows * H + 3) // 4 * 4) + 4 * slots * H * dk * dv + (4 * B * H * dk * dv // 32 if variant == sla.GLA else 0)
        p = _params(variant, B=B, T=T, H=H, dk=dk, dv=dv)
        assert sla.sla_backward_chunks_workspace_bytes(p, packed) == max(want, least(p))
    # no more than 1 GiB of states at a time, however long the batch
    p = _params(variant, B=8, T=65536, H=16)
    n = 65536 * (1 if packed else 8) * 16 * 16 + 8 * 16 * 128 * 4 * 4
    assert sla.sla_backward_chunks_workspace_bytes(p, packed) <= max(n + (1 << 30), least(p))

    # batches whose states are a GiB to the byte are worked off at once
    for B, T, H, dk, dv in ((4, 32768, 8, 128, 128), (1, 32768, 64, 64, 128)):
        p = _params(variant, B=B, T=T, H=H, dk=dk, dv=dv)
        assert sla.sla_backward_chunks_workspace_bytes(p) >= 4 * 4 * B * T * H + (1 << 30)


def test_where_the_other_queries_hold():
    for p in (_params(dtype=sla.F32), _params(T=0), _params(B=0)):
        assert sla.sla_backward_chunks_workspace_bytes(p) == sla.sla_backward_workspace_bytes(p)
        assert sla.sla_backward_chunks_workspace_bytes(p, True) == sla.sla_backward_varlen_workspace_bytes(p)
    assert sla.sla_backward_chunks_workspace_bytes(_params(sla.GDN)) == 0
    assert sla.sla_backward_chunks_workspace_bytes(_params(dk=96)) == 0
    assert sla.sla_backward_chunks_workspace_bytes(_params(dk=32, segments=2)) == 0
