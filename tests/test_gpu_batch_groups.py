"""Wavefront tiles of batches whose problems are few and large, or tall and
narrow: reductions of more than 64 tiles, folded group by group, and gemv
problems cut by the rounds of loads that their rows take.  Integers, exact, run
after run on the same counters and replayed from a graph.
"""
import pytest
import torch

import paper_1502_02389_amd as L
import workloads as W
from tests.gpu_util import banner, o_asum, o_dot
from tests.test_gpu_batch_wave import _gemv, _run_and_check

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("storage", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("acc", ["f32", "comp", "f64combine"])
def test_around_the_groups(gpu_device, storage, acc):
    eb = 4 if storage == "f32" else 2
    per = {"asum": 8192 // eb, "dot": 4096 // eb}          # elements per tile of a small batch
    g = W.gen(17)
    banner("batch groups", storage, acc)
    for kind in ("asum", "dot"):
        problems, wants = [], []
        for tiles, more in ((63, 0), (64, 0), (64, 1), (65, 0), (127, 5), (128, 0), (129, 0), (200, 77)):
            n = tiles * per[kind] + more
            x = W.integers(n + 3, -4, 4, g, storage)
            y = W.integers(n, -3, 3, g, storage)
            xd = x.to(DEV)
            problems.append(("dot", xd[3:], y.to(DEV)) if kind == "dot" else ("asum", xd[3:]))
            wants.append(o_dot(x[3:], y)[0] if kind == "dot" else o_asum(x[3:]))
        _run_and_check(problems, wants, [None] * len(problems), acc, runs=3)


@pytest.mark.parametrize("acc", ["f32", "comp", "f64combine"])
def test_one_large_problem_in_a_graph(gpu_device, acc):
    n = 4_000_003
    g = W.gen(18)
    x, y = W.integers(n, -2, 2, g, "bf16"), W.integers(n, -2, 2, g, "bf16")
    b = L.Batch([("dot", x.to(DEV), y.to(DEV)), ("asum", x.to(DEV)[:70]), ("asum", x.to(DEV))], acc=acc)
    want = [o_dot(x, y)[0], o_asum(x[:70]), o_asum(x)]
    assert b.tiles > 1000
    banner("batch one large problem", acc)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        b.run()
        s.synchronize()
        assert [r.item() for r in b.results] == want
        with torch.cuda.graph(graph, stream=s):
            b.run()
        for _ in range(4):
            for r in b.results:
                r.fill_(float("nan"))
            graph.replay()
            assert [r.item() for r in b.results] == want
    graph.reset()
    b.close()


@pytest.mark.parametrize("storage", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("m, n, at_least", [(3370, 1, 100), (40_000, 2, 1000), (5000, 7, 150), (3871, 33, 100), (23, 72_268, 23),
                                            (2735, 5245, 1300), (7767, 1074, 1000), (589, 486, 100)])
def test_tall_and_wide(gpu_device, storage, m, n, at_least):
    g = W.gen(m)
    p, want, buf = _gemv(m, n, n, storage, g, m % 3, 0.5)
    banner("batch tall and wide", storage, m, n)
    b = L.Batch([p])
    assert b.tiles >= at_least, b.tiles
    b.close()
    y = p[5].clone()
    for acc in ("f32", "comp", "f64combine"):
        p[5].copy_(y)
        _run_and_check([p], [want], [buf], acc)
