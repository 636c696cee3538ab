"""The batch without knobs on both sides of its size line, and which form it
took: wavefront tiles (many, one launch) up to 64 KiB per wavefront that the
device holds, work-group tiles above."""
import pytest
import torch

import paper_1502_02389_amd as L
from tests.gpu_util import banner

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("storage", [torch.float32, torch.bfloat16])
def test_form_by_size(gpu_device, storage):
    eb = torch.empty(0, dtype=storage).element_size()
    x = torch.zeros((1 << 28) + (1 << 20), dtype=storage, device=DEV)
    x[::11] = 1.0                                  # sums below 2^24 elements of which one in 11 counts
    small = L.Batch([("asum", x[:1 << 24])])
    groups = small.grid                            # as many as the device holds
    small.close()
    line = 65536 * 4 * groups // eb
    banner("batch line", storage, groups)
    for n in (line, line + 1):
        # parts of 2^24 elements, so that every sum is exact
        parts = [x[i:min(i + (1 << 24), n)] for i in range(0, n, 1 << 24)]
        b = L.Batch([("asum", p) for p in parts])
        if n == line:
            assert b.grid == groups and b.tiles >= 3 * groups
        else:
            assert b.tiles <= n // 65536 + 2 * len(parts)
        b.run()
        torch.cuda.synchronize()
        for i, (p, r) in enumerate(zip(parts, b.results)):
            start = i << 24
            assert r.item() == -(-(start + p.numel()) // 11) - -(-start // 11)
        b.close()
