import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="session")
def gpu_device():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.fixture(params=["as_told", "work_list"])
def both_forms(request, monkeypatch):
    """A test that uses this runs twice: with its bf16 extend_attention calls as they are, small batches without a work list, and
    with every call told of 1,000,000 keys more than it has, so that it builds a list; the header of the workspace has to say so."""
    if request.param == "as_told":
        return
    import torch
    from paper_2407_00023_amd import binding
    real = binding.extend_attention

    def told_of_more(q, k, v, *rest, max_kv_len, workspace=None, **kw):
        B, T, Hq, D = rest[3].numel(), q.shape[0], q.shape[1], q.shape[2]
        max_kv_len += 1000000
        ws = torch.full((binding.extend_workspace_bytes(B, T, max_kv_len, Hq, k.shape[1], D, q.dtype),), 255, dtype=torch.uint8, device=q.device)
        out = real(q, k, v, *rest, max_kv_len=max_kv_len, workspace=ws, **kw)
        if q.dtype == torch.bfloat16 and B and T:
            assert ws[20:24].view(torch.int32).item() == 0
            if workspace is not None:  # (the test may look at the header)
                workspace[:256].copy_(ws[:256])
        return out

    monkeypatch.setattr(binding, "extend_attention", told_of_more)
