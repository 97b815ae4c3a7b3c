"""The binding's workspaces from PyTorch's allocator (no GPU: the allocator is stood in for)."""
import pytest

from paper_2603_15780_amd import sg

torch = pytest.importorskip("torch")


@pytest.fixture
def allocated(monkeypatch):
    seen, empty = [], torch.empty

    def record(n, dtype, device):
        seen.append((n, device))
        return empty(n, dtype=dtype)

    monkeypatch.setattr(torch, "empty", record)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    return seen


def test_workspace_on_the_current_device(allocated):
    dev = torch.device("cuda", 0)
    o = sg.opts()
    w, ws = sg._with_workspace(o, 4096, dev)
    assert allocated == [(4096, dev)] and w.workspace == ws.data_ptr() and w.workspace_bytes == 4096
    assert not o.workspace


def test_none_for_another_device(allocated):
    """A call's launches go to the current device's stream, which does not order the other device's blocks."""
    o = sg.opts()
    assert sg._with_workspace(o, 4096, torch.device("cuda", 1)) == (o, None) and not allocated


def test_none_where_none_is_needed_or_the_caller_has_one(allocated):
    dev = torch.device("cuda", 0)
    o = sg.opts(workspace=256, workspace_bytes=4096)
    assert sg._with_workspace(o, 4096, dev) == (o, None)
    assert sg._with_workspace(sg.opts(), 0, dev)[1] is None and not allocated
