"""Short dots of operands in different 16-byte phases: the work-group has as
many threads as take the vectors in one step, 64 to 512.  Integers, exact, on
both sides of every size; what lies around the operands is NaN."""
import pytest
import torch

import paper_1502_02389_amd as L
import workloads as W
from tests.gpu_util import banner, o_dot

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("storage", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("acc", ["f32", "comp", "f64combine"])
def test_around_every_work_group_size(gpu_device, storage, acc):
    E = 4 if storage == "f32" else 8
    edges = [64 * E, 128 * E, 256 * E, 512 * E, 1024 * E]
    g = W.gen(E)
    banner("short shifted dots", storage, acc)
    for n in [0, 1, 2, E - 1, E, E + 1, 3 * E] + [e + d for e in edges for d in (-E - 1, -1, 0, 1, E, 2 * E + 1)]:
        x, y = W.integers(n, -4, 4, g, storage), W.integers(n, -4, 4, g, storage)
        want = o_dot(x, y)[0]
        for ox, oy in ((0, 1), (1, 0), (E - 1, 1)):
            bx = torch.full((n + 2 * E,), float("nan"), dtype=x.dtype, device=DEV)
            by = bx.clone()
            bx[ox:ox + n] = x.to(DEV)
            by[oy:oy + n] = y.to(DEV)
            for rt in (torch.float32, torch.float64):
                assert L.dot(bx[ox:ox + n], by[oy:oy + n], acc=acc, result_dtype=rt).item() == want, (n, ox, oy)
