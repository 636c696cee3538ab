"""scal of x and out in different 16-byte phases around the sizes where the
loads per thread change: bit-exact, nothing written beside out."""
import pytest
import torch

import paper_1502_02389_amd as L
import workloads as W
from tests.gpu_util import banner

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n", [1, 1023, (1 << 20) - 1, 1 << 20, (1 << 20) + 1025, (1 << 21) - 1, 1 << 21, (1 << 22) + 3])
def test_out_of_phase(gpu_device, n):
    x = W.uniform(n + 4, W.gen(n)).to(DEV)
    banner("scal phases", n)
    for ox, oo in ((1, 0), (0, 3), (2, 1), (1, 1)):
        buf = torch.full((n + 8,), float("nan"), device=DEV)
        L.scal(1.7, x[ox:ox + n], out=buf[oo:oo + n])
        assert torch.equal(buf[oo:oo + n], x[ox:ox + n] * 1.7)
        assert torch.isnan(buf[:oo]).all() and torch.isnan(buf[oo + n:]).all()
