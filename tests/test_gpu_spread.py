"""scal, asum and dot without knobs where the launch goes by size: around one
work-group's reach, around one step on every compute unit for each number of
loads, and around scal's largest vector-per-thread size; aligned and shifted.

Integers bounded so that every partial sum is exact: no tolerance.
"""
import pytest
import torch

import paper_1502_02389_amd as L
import workloads as W
from tests.gpu_util import banner, o_asum, o_dot

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _edges(storage):
    """Elements at which the loads per thread change, one to each side."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    E = 4 if storage == "f32" else 8
    at = [256 * E * u for u in (1, 2, 4, 8)] + [256 * E * u * cus for u in (1, 2, 4)]
    return [n + d for n in at for d in (-1, 0, 1, E)]


@pytest.mark.parametrize("storage", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("acc", ["f32", "comp", "f64combine"])
def test_reductions_around_the_edges(gpu_device, storage, acc):
    g = W.gen(95)
    sizes = _edges(storage)
    n = max(sizes) + 3
    x, y = W.integers(n, -2, 2, g, storage), W.integers(n, -1, 1, g, storage)
    xd, yd = x.to(DEV), y.to(DEV)
    for off in (0, 1):
        banner("spread", storage, acc, off)
        for m in sizes:
            a, b = xd[off:off + m], yd[off:off + m]
            assert L.asum(a, acc=acc).item() == o_asum(x[off:off + m]), (m, off)
            assert L.dot(a, b, acc=acc).item() == o_dot(x[off:off + m], y[off:off + m])[0], (m, off)


@pytest.mark.parametrize("n", [1, 3, 4, 255, 1023, 1024, 1025, 3000001, (1 << 22) - 1, 1 << 22, (1 << 22) + 1])
@pytest.mark.parametrize("ox, oo", [(0, 0), (1, 1), (0, 1), (3, 2)])
def test_scal_around_the_edges(gpu_device, n, ox, oo):
    x = torch.randn(n + ox, device=DEV)[ox:]
    buf = torch.full((n + oo + 5,), float("nan"), device=DEV)
    out = buf[oo:oo + n]
    banner("scal spread", n, ox, oo)
    L.scal(2.5, x, out=out)
    assert torch.equal(out, x * 2.5)
    assert torch.isnan(buf[:oo]).all() and torch.isnan(buf[oo + n:]).all()
    L.scal(2.5, x, out=x)
    assert torch.equal(out, x)
