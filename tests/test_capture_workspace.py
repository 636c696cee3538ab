"""Which workspace the tensor calls take, on the CPU: a stream that is being
captured has its graph's own, which is not kept for eager calls."""
import pytest
import torch

from paper_1502_02389_amd import lift as B


@pytest.fixture
def streams(monkeypatch):
    monkeypatch.setattr(B, "_WS", {})
    monkeypatch.setattr(B, "_stream_handle", lambda device: 77)
    captured = {}
    monkeypatch.setattr(B, "lift_capture_workspace", lambda stream: (B.LIFT_OK, captured.get(stream)))
    return captured


def test_captured_calls_take_the_graphs(streams):
    cpu = torch.device("cpu")
    streams[77] = 0x1000
    assert B._call_workspace(cpu, 77) == (0x1000, B.lift_workspace_bytes())
    assert B._WS == {}
    streams.clear()
    at, size = B._call_workspace(cpu, 77)
    assert at == B._WS[(None, 77)].data_ptr() and size == B.lift_workspace_bytes()
    streams[77] = 0x2000
    assert B._call_workspace(cpu, 77)[0] == 0x2000
    streams.clear()
    assert B._call_workspace(cpu, 77)[0] == at


def test_the_null_stream_is_not_asked(monkeypatch):
    assert B.lift_capture_workspace(0) == (B.LIFT_OK, None)
    assert B._lib().lift_capture_workspace(None, None) == B.LIFT_EINVAL
