"""The tensor conveniences' native route against the binding's own code.

Every ordinary call must give the same bits both ways, on the current stream;
everything else (unusual tensors, numbers, errors) must end as it does in the
binding's own code: same result or same exception.
"""
import numpy as np
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
    native = B._native()
    assert native is not B._NoNative, "the native route is not built"
    if request.param == "general":
        monkeypatch.setattr(B, "_NATIVE", B._NoNative)
    return request.param


def _inputs():
    g = W.gen(5)
    n = 70_003
    d = {k: W.uniform(n, g, k).to(DEV) for k in ("f32", "bf16", "f16")}
    d.update(A=W.normal((37, 1001), g).to(DEV), gx=W.normal(1001, g).to(DEV), gy=W.normal(37, g).to(DEV),
             s=W.blackscholes_prices(1003)[0].to(DEV))
    pos, nbr, _ = W.md_system(box=(5, 6, 7), slots=24)
    d.update(pos=pos.to(DEV), nbr=nbr.to(DEV))
    return d


def _calls(d):
    out = []
    for k in ("f32", "bf16", "f16"):
        x = d[k]
        for acc in ("f32", "comp", "f64combine", 1):
            for rt in (None, torch.float32, torch.float64):
                out += [L.asum(x, acc, rt), L.dot(x[1:], x[:-1], acc=acc, result_dtype=rt)]
    x = d["f32"]
    for alpha in (2.5, 3, np.float32(0.1), torch.tensor(1.5)):
        out += [L.scal(alpha, x), L.scal(alpha, x[3:], out=torch.empty(x.numel() - 3, device=DEV))]
    out.append(L.scal(2, torch.nn.Parameter(x.clone())))
    out.append(L.scal(2.0, x.clone().requires_grad_()))
    for acc in ("f32", "comp", "f64combine"):
        out.append(L.gemv(1, d["A"], d["gx"], 0.5, d["gy"].clone(), acc))
        out.append(L.gemv(1.5, d["A"], d["gx"][:900].contiguous(), 0, d["gy"].clone(), acc=acc, lda=1001))
    out += [L.blackscholes(d["s"], 20, 0.02, 0.3, 1.0),
            L.blackscholes(d["s"], 20.0, 0.02, 0.3, 1.0, out=torch.empty((1003, 2), device=DEV)),
            L.md(d["pos"], d["nbr"], 2.5, 1, 1.0), L.md(d["pos"], d["nbr"], 2.5, 1.0, 1.0, out=torch.empty_like(d["pos"]))]
    empty = torch.empty(0, device=DEV)
    out += [L.asum(empty), L.dot(empty, empty), L.scal(1.0, empty)]
    return out


_GOT = {}


def test_same_bits(gpu_device, route):
    banner("native calls", route)
    got = _calls(_inputs())
    s = torch.cuda.Stream(device=DEV)
    with torch.cuda.stream(s):                 # another stream: its own workspace
        d = _inputs()
        s.synchronize()
        got += _calls(d)
        s.synchronize()
    assert not any(t.requires_grad for t in got)
    _GOT[route] = [(t.dtype, t.shape, t.cpu()) for t in got]
    if len(_GOT) == 2:
        for a, b in zip(_GOT["native"], _GOT["general"]):
            assert a[:2] == b[:2] and torch.equal(a[2].view(torch.uint8) if a[2].dim() else a[2].reshape(1).view(torch.uint8),
                                                  b[2].view(torch.uint8) if b[2].dim() else b[2].reshape(1).view(torch.uint8))


def test_same_refusals(gpu_device, route):
    d = _inputs()
    x = d["f32"]
    banner("native refusals", route)
    for exc, call in [
        (ValueError, lambda: L.asum(x.cpu())), (TypeError, lambda: L.asum(x.double())), (TypeError, lambda: L.asum([1.0])),
        (ValueError, lambda: L.asum(x[::2])), (KeyError, lambda: L.asum(x, "exact")), (ValueError, lambda: L.dot(x, x[1:])),
        (TypeError, lambda: L.dot(x, d["bf16"])), (L.LiftError, lambda: L.asum(x, result_dtype=torch.float16)),
        (TypeError, lambda: L.scal(1.0, d["f16"])), (ValueError, lambda: L.scal(1.0, x, out=x[1:])),
        (L.LiftError, lambda: L.scal(1.0, x[1:], out=x[:-1])), (ValueError, lambda: L.scal("a", x, out=x)),
        (ValueError, lambda: L.gemv(1.0, x, x, 0.0, x)), (ValueError, lambda: L.gemv(1.0, d["A"], x, 0.0, d["gy"])),
        (L.LiftError, lambda: L.gemv(1.0, d["A"], d["gx"], 0.0, d["A"].view(-1)[:37])),
        (ValueError, lambda: L.md(d["pos"][:, :3].contiguous(), d["nbr"], 2.5, 1.0, 1.0)),
        (L.LiftError, lambda: L.md(d["pos"], d["nbr"], -1.0, 1.0, 1.0)),
        (L.LiftError, lambda: L.blackscholes(d["s"], 0.0, 0.02, 0.3, 1.0)),
    ]:
        with pytest.raises(Exception) as e:
            call()
        assert isinstance(e.value, exc), (exc, e.value)


@pytest.mark.parametrize("m, n", [(1, 32769), (8, 32768), (8, 32769), (22, 60184), (512, 33001), (513, 33001)])
@pytest.mark.parametrize("captured", [False, True])
def test_few_long_rows(gpu_device, m, n, captured):
    """gemv on both sides of where rows are split through the stream's
    workspace, on a stream of its own; under capture they are not."""
    g = W.gen(97)
    A, x, y = W.integers((m, n), -1, 1, g, "bf16"), W.integers(n, -1, 1, g), W.integers(m, -8, 8, g)
    want = 2.0 * (A.double() @ x.double()) + 0.5 * y.double()
    Ad, xd, yd, first = A.cuda(), x.cuda(), y.cuda(), y.cuda()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        if captured:
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=s):
                L.gemv(2.0, Ad, xd, 0.5, yd)
        for _ in range(3):
            yd.copy_(first)
            graph.replay() if captured else L.gemv(2.0, Ad, xd, 0.5, yd)
            s.synchronize()
            assert torch.equal(yd.double().cpu(), want)
