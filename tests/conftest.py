import pytest

import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the built HIP library")


@pytest.fixture(params=["packed", "plain"])
def both_routes(request, monkeypatch):
    """Runs a test twice: with the workspaces that the binding passes, under which calls
    over dense patterns and long batches pack their operands (and the adaptive update
    keeps its dense result), and with those of the plain routes, whose kernels other
    sizes and callers with smaller workspaces still run."""
    import paper_1905_07931_amd as L1
    if request.param == "plain":
        sizes, packed = L1.workspace_bytes, (L1.OP_WGRAD_PACKED, L1.OP_SDDMM_PACKED, L1.OP_SPMM_PACKED, L1.OP_PROX_DENSE)
        monkeypatch.setattr(L1, "workspace_bytes", lambda op, *a: 0 if op in packed else sizes(op, *a))
    return request.param
