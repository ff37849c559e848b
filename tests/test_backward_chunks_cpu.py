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


@pytest.mark.parametrize("variant", [sla.RETNET, sla.GLA])
def test_which_calls_run_chunk_parallel(variant):
    """A call that the other schedules are faster for is told so by the query, which then asks for what these want."""
    def chunks(B, T, H, dk=128, dv=128, segments=0, packed=False):
        p = _params(variant, B=B, T=T, H=H, dk=dk, dv=dv)
        if segments == 0 and not packed:
            segments = sla.sla_backward_segments(p, 256)
        p.segments = max(segments, 1)
        least = sla.sla_backward_varlen_workspace_bytes if packed else sla.sla_backward_workspace_bytes
        return sla.sla_backward_chunks_workspace_bytes(p, packed) > least(p)

    # few heads: up to a length that grows with their number
    assert chunks(1, 2048, 2) and not chunks(1, 16384, 2)
    assert chunks(1, 4096, 8) and not chunks(1, 32768, 8)
    assert chunks(4, 16384, 8) and chunks(4, 32768, 8)
    assert not chunks(1, 131072, 8, 64, 64) and not chunks(1, 65536, 4) and not chunks(1, 65536, 32, segments=8)
    assert chunks(1, 131072, 8, 64, 64, segments=1)  # the sweeps would be slower still
    # one part however long, or as many as the chip is full in; not one for each of a few heads
    assert chunks(1, 65536, 32, segments=1) and not chunks(1, 1 << 20, 5, segments=1)
    assert chunks(8, 4096, 16) and chunks(128, 1024, 16) and chunks(8, 4096, 4, 128, 256)
    # sequences of a block: not in numbers that fill the chip once
    assert chunks(32, 32 * 40, 16, packed=True) and not chunks(32, 32 * 12, 16, packed=True)
    assert chunks(2, 2 * 12, 16, packed=True)
    assert chunks(64, 64 * 12, 16, 128, 256, packed=True) == (variant == sla.RETNET)
    assert chunks(1024, 1024 * 12, 16, 64, 128, packed=True) == (variant == sla.RETNET)
    # RetNet's widest values, where the sweeps fill the chip in every round
    assert chunks(16, 640, 16, 64, 256) == chunks(32, 2048, 16, 64, 256) == (variant == sla.GLA)
    assert chunks(16, 448, 16, 64, 256) and chunks(24, 2048, 16, 64, 256) and chunks(16, 1024, 16, 64, 128)
    assert chunks(4096, 4096 * 12, 16, packed=True)


@pytest.mark.parametrize("variant", [sla.RETNET, sla.GLA])
@pytest.mark.parametrize("packed", [False, True])
def test_narrow_keys_never_need_more_than_the_plain_workspace(variant, packed):
    """bf16 calls with keys of 32 run chunk-parallel in any workspace that is accepted at all: the states fit into what the
    plain query asks for."""
    least = sla.sla_backward_varlen_workspace_bytes if packed else sla.sla_backward_workspace_bytes
    for B in (1, 3, 64, 16384):
        for T in (1, 63, 64, 65, 1000, 65536):
            for H, dv in ((1, 64), (4, 256), (64, 128)):
                p = _params(variant, B=B, T=T, H=H, dk=32, dv=dv)
                rows, slots = (T, T // 64 + B + 1) if packed else (B * T, B * ((T + 63) // 64))
                need = 16 * ((rows * H + 3) // 4 * 4) + 4 * slots * H * 32 * dv + (4 * B * H * dv if variant == sla.GLA else 0)
                if least(p) > 0:  # 0: tensors beyond what the library takes
                    assert need <= least(p) == sla.sla_backward_chunks_workspace_bytes(p, packed)
