"""When the binding brings scratch along for a linear: its Python path on stand-ins for the device, which need no GPU."""
import pytest
import torch

from paper_2506_04985_amd import binding as fptq

M, N, K = 4096, 8192, 4096      # takes scratch on a device with 256 compute units, which the library assumes without one


class OnDevice(torch.Tensor):
    """A tensor that says it lies on device `where`."""
    where = 0
    is_cuda = True
    device = property(lambda self: torch.device("cuda", self.where))


@pytest.fixture
def taken(monkeypatch):
    """Makes device 0 the current one and returns the list of allocations."""
    made = []

    def empty(n, dtype, device):
        made.append((n, dtype, device))
        return "scratch"
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: False)
    monkeypatch.setattr(torch, "empty", empty)
    return made


def operand(where):
    t = torch.zeros(1, dtype=torch.uint8).as_subclass(OnDevice)
    t.where = where
    return t


def test_only_on_the_current_device(taken):
    """The launch goes to the current device's stream; scratch of another device's stream could be given out again under it."""
    assert fptq._scratch(M, N, K, operand(0)) == "scratch" and taken[0][2] == torch.device("cuda", 0)
    assert fptq._scratch(M, N, K, operand(1)) is None and len(taken) == 1


def test_not_under_capture_and_not_where_it_does_not_pay(taken, monkeypatch):
    assert fptq._scratch(64, N, K, operand(0)) is None and fptq._scratch(M, 64, 64, operand(0)) is None
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: True)
    assert fptq._scratch(M, N, K, operand(0)) is None and taken == []


@pytest.mark.parametrize("error", [torch.cuda.OutOfMemoryError, RuntimeError])
def test_a_failing_allocation_refuses_no_call(taken, monkeypatch, error):
    """No memory, or an allocator that may not allocate now (a capture going on in another thread): the call goes without."""
    def empty(n, dtype, device):
        raise error("no")
    monkeypatch.setattr(torch, "empty", empty)
    assert fptq._scratch(M, N, K, operand(0)) is None
