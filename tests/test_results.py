"""Reading a build's sizes back: what the error word and a failing device are
reported as, on the CPU (the reads are torch's, on whatever device)."""
import contextlib

import pytest
import torch

from paper_1604_04689_amd import binding
from paper_1604_04689_amd.binding import MeshError, Status


@pytest.fixture
def cpu_streams(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: None)
    monkeypatch.setattr(torch.cuda, "stream", lambda s: contextlib.nullcontext())


def _workspace(err):
    return torch.tensor([err, 77], dtype=torch.int32).view(torch.uint8)


def test_sizes(cpu_streams):
    a, b = torch.tensor([0, 3, 9], dtype=torch.int32), torch.tensor([0], dtype=torch.int32)
    assert binding._sizes(_workspace(0), None, "cpu", a, b) == [9, 0]


@pytest.mark.parametrize("err", range(1, 8))
def test_errors_as_mesh_check_reports_them(cpu_streams, err):
    want = Status.INTERNAL if err & 4 else Status.INDEX_RANGE if err & 1 else Status.CAPACITY
    with pytest.raises(MeshError) as e:
        binding._sizes(_workspace(err), None, "cpu", torch.zeros(2, dtype=torch.int32))
    assert e.value.status == want


def test_a_failing_device(cpu_streams, monkeypatch):
    def fails(*a, **k):
        raise RuntimeError("HIP error")
    monkeypatch.setattr(torch, "cat", fails)
    with pytest.raises(MeshError) as e:
        binding._sizes(_workspace(0), None, "cpu", torch.zeros(2, dtype=torch.int32))
    assert e.value.status == Status.HIP
