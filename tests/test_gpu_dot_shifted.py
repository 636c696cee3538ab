"""dot of operands that do not share a 16-byte phase, without knobs.

x's vectors are read aligned and y's from wherever they then start.  Every
pair of phases, sizes around a work-group's step (1024 vectors) and the grid's
(256 steps), every storage and accumulation, integer inputs: bit-exact; normal
inputs within 1e-5 of sum |x y| (compensated: 1e-6).
"""
import pytest
import torch

import paper_1502_02389_amd as L
import workloads as W
from tests.gpu_util import banner, o_dot

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _at(t, off):
    """t on the GPU, `off` elements past a 16-byte boundary, NaN around it."""
    buf = torch.full((t.numel() + off + 8,), float("nan"), dtype=t.dtype, device=DEV)
    buf[off:off + t.numel()] = t.to(DEV)
    return buf[off:off + t.numel()]


@pytest.mark.parametrize("storage", ["f32", "bf16", "f16"])
def test_every_phase_and_size_integer_exact(gpu_device, storage):
    E = 4 if storage == "f32" else 8
    step = 1024 * E
    for n in (1, E - 1, E, 2 * E + 1, step - 1, step, step + E + 3, 3 * step + 5, 256 * step + 1, 300 * step + 7):
        g = W.gen(n)
        x, y = W.integers(n, -4, 4, g, storage), W.integers(n, -3, 3, g, storage)
        want, _ = o_dot(x, y)
        pairs = [(i, j) for i in range(E) for j in range(E) if i != j] if n < 4 * step else [(0, 1), (1, 0), (E - 1, 2)]
        banner("dot shifted", storage, n)
        for ox, oy in pairs:
            xd, yd = _at(x, ox), _at(y, oy)
            for acc in ("f32", "comp", "f64combine") if (ox + oy) % 3 == 0 or n >= 4 * step else ("f32",):
                assert L.dot(xd, yd, acc=acc, result_dtype=torch.float64).item() == want, (n, ox, oy, acc)


@pytest.mark.parametrize("storage", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("acc", ["f32", "comp", "f64combine"])
def test_lag_product_within_bound(gpu_device, storage, acc):
    n = (1 << 21) + 13
    x = W.normal(n, W.gen(17), storage)
    xd = x.to(DEV)
    want, mass = o_dot(x[1:].contiguous(), x[:-1].contiguous())
    banner("lag product", storage, acc)
    got = L.dot(xd[1:], xd[:-1], acc=acc)
    assert abs(got.item() - want) <= (1e-6 if acc == "comp" else 1e-5) * mass
    assert torch.equal(got, L.dot(xd[1:], xd[:-1], acc=acc))
