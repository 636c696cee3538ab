"""The native route of the tensor calls and the binding's own code, one beside
the other in one test: the same bits for every form, on any stream, and in a
captured graph."""
import pytest
import torch

import paper_1502_02389_amd as L
from paper_1502_02389_amd import lift as B
from tests.gpu_util import banner
from tests.test_gpu_native_calls import _calls, _inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _bits(t):
    return t.contiguous().reshape(-1).view(torch.uint8)


@pytest.mark.parametrize("own_stream", [False, True])
def test_both_routes(gpu_device, monkeypatch, own_stream):
    assert B._native() is not B._NoNative, "the native route is not built"
    s = torch.cuda.Stream(device=DEV) if own_stream else torch.cuda.current_stream()
    banner("both routes", own_stream)
    with torch.cuda.stream(s):
        d = _inputs()
        s.synchronize()
        native = _calls(d)
        with monkeypatch.context() as m:
            m.setattr(B, "_NATIVE", B._NoNative)
            general = _calls(d)
        s.synchronize()
    assert len(native) == len(general)
    for i, (a, b) in enumerate(zip(native, general)):
        assert a.dtype == b.dtype and a.shape == b.shape and torch.equal(_bits(a), _bits(b)), i


def test_both_routes_captured(gpu_device, monkeypatch):
    d = _inputs()
    x = d["f32"]
    s = torch.cuda.Stream(device=DEV)
    s.wait_stream(torch.cuda.current_stream())
    got = []
    banner("both routes captured")
    for route in (B._native(), B._NoNative):
        with monkeypatch.context() as m, torch.cuda.stream(s):
            m.setattr(B, "_NATIVE", route)
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s):
                r = [L.asum(x), L.dot(x[1:], x[:-1], acc="comp"), L.scal(2.5, x)]
            for _ in range(2):
                g.replay()
            s.synchronize()
            got.append([v.clone() for v in r])
    for a, b in zip(*got):
        assert torch.equal(_bits(a), _bits(b))
