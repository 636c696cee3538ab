"""Calls captured into a graph have a workspace of the graph's own: graphs
captured on one stream run next to each other and to eager calls, the eager
calls' own workspace is ready whether or not it was first asked for in a
capture, and a captured gemv of few long rows is split as the eager one is.
"""
import ctypes

import pytest
import torch

import paper_1502_02389_amd as L
import workloads as W
from paper_1502_02389_amd import lift as B
from tests.gpu_util import banner

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(params=["native", "general"])
def route(request, monkeypatch):
    if request.param == "general":
        monkeypatch.setattr(B, "_NATIVE", B._NoNative)
    return request.param


def _at(stream):
    st, at = L.lift_capture_workspace(stream.cuda_stream)
    assert st == L.LIFT_OK
    return at


def test_graphs_of_one_stream_side_by_side(gpu_device, route):
    n = (1 << 22) + 3
    x = [W.uniform(n, W.gen(i)).to(DEV) for i in range(3)]
    s, others = torch.cuda.Stream(), [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    graphs, got = [], []
    with torch.cuda.stream(s):
        want = [(L.asum(v), L.dot(v, x[0], acc="comp")) for v in x]
        s.synchronize()
        for v in x[:2]:
            graphs.append(torch.cuda.CUDAGraph())
            with torch.cuda.graph(graphs[-1], stream=s):
                got.append([(L.asum(v), L.dot(v, x[0], acc="comp")) for _ in range(8)])
    banner("graphs side by side", route)
    for _ in range(20):
        for r in got:
            for a, b in r:
                a.fill_(float("nan")), b.fill_(float("nan"))
        torch.cuda.synchronize()
        for g, o in zip(graphs, others):
            with torch.cuda.stream(o):
                g.replay()
        with torch.cuda.stream(s):                     # eager calls of the capture's stream meanwhile
            eager = [(L.asum(x[2]), L.dot(x[2], x[0], acc="comp")) for _ in range(8)]
        torch.cuda.synchronize()
        for r, w in zip(got + [eager], want):
            for a, b in r:
                assert torch.equal(a, w[0]) and torch.equal(b, w[1])


def test_a_stream_first_used_in_a_capture(gpu_device, route):
    """Eager calls between the capture and its first replay."""
    n = (1 << 20) + 7
    x = torch.ones(n, device=DEV)
    s = torch.cuda.ExternalStream(_new_stream())
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            r = L.asum(x)
            ws = L.workspace(x.device)                 # asked for while capturing: ready all the same
        assert not ws.any().item()
        assert L.asum(x).item() == n and L.dot(x, x).item() == n
        g.replay()
        assert r.item() == n and L.asum(x).item() == n
        assert not ws.any().item()


def _new_stream():
    hip = ctypes.CDLL("libamdhip64.so")
    h = ctypes.c_void_p()
    assert hip.hipStreamCreateWithFlags(ctypes.byref(h), ctypes.c_uint(1)) == 0
    return h.value


@pytest.mark.parametrize("m, n, dtype", [(32, 300_001, "f32"), (3, 1_000_003, "bf16"), (1, 70_000, "f16")])
def test_captured_long_rows_have_the_eager_bits(gpu_device, route, m, n, dtype):
    g = W.gen(m)
    A = (torch.rand((m, n), generator=torch.Generator().manual_seed(5)) - 0.5).to(W.STORAGE[dtype]).to(DEV)
    x, y = W.uniform(n, g).to(DEV), W.uniform(m, g).to(DEV)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        want = L.gemv(1.5, A, x, 0.5, y.clone())
        out = y.clone()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            L.gemv(1.5, A, x, 0.5, out)
        for _ in range(3):
            out.copy_(y)
            graph.replay()
            assert torch.equal(out, want)


def test_owned_by_the_graph(gpu_device):
    x = torch.ones(100_000, device=DEV)
    s, side = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    assert _at(s) is None and L.lift_capture_workspace(0) == (L.LIFT_OK, None)
    alive, seen = [], []
    with torch.cuda.stream(s):
        eager = L.workspace(x.device).data_ptr()
        for _ in range(3):
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s):
                first = _at(s)
                r = L.asum(x)
                side.wait_stream(s)
                with torch.cuda.stream(side):
                    L.asum(x)
                    branch = _at(side)
                s.wait_stream(side)
                assert _at(s) == first                 # one per capture and stream
            alive.append((g, r))
            seen += [first, branch]
    assert None not in seen and len(set(seen + [eager])) == 7
    for g, r in alive:
        g.replay()
        torch.cuda.synchronize()
        assert r.item() == x.numel()
    # graphs that end give theirs back to later ones
    later = set()
    with torch.cuda.stream(s):
        for _ in range(60):
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=s):
                later.add(_at(s))
                r = L.asum(x)
            g.replay()
            s.synchronize()
            assert r.item() == x.numel()
            g.reset()
    assert not later & set(seen) and len(later) <= 10, len(later)
