import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


def pytest_collection_modifyitems(config, items):
    # GPU tests are selected explicitly with -m gpu; without a device they are skipped.
    try:
        import torch

        have_gpu = torch.cuda.is_available()
    except Exception:  # pragma: no cover
        have_gpu = False
    if have_gpu:
        return
    skip = pytest.mark.skip(reason="no GPU in this environment")
    for item in items:
        if "gpu" in item.keywords:
            item.add_marker(skip)


@pytest.fixture(params=["largest workspace", "plain workspace"])
def backward_workspace(request, monkeypatch):
    """Runs a test with both sizes of workspace that the binding's backward calls may get: the one it allocates, in which most
    bf16 calls run chunk-parallel, and the plain queries', in which those of key heads of 64 and 128 run in the segments
    asked for, or in the sweeps."""
    if request.param == "plain workspace":
        from paper_2602_01744_amd import binding as b

        monkeypatch.setattr(b, "sla_backward_chunks_workspace_bytes", lambda p, packed=False: (
            b.sla_backward_varlen_workspace_bytes if packed else b.sla_backward_workspace_bytes)(p))
        monkeypatch.setattr(b, "sla_backward_gdn_chunks_workspace_bytes", lambda p, packed=False: (
            b.sla_backward_gdn_varlen_workspace_bytes if packed else b.sla_backward_gdn_workspace_bytes)(p))
    return request.param
