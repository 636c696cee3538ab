"""MD without knobs by the length of the lists: short lists take one launch
however many particles there are, long ones the passes over slices of the
positions, in each index width and number of slices; a periodic lattice in its
own order is done by the first launch of those, boundary particles included.
"""
import pytest
import torch

import paper_1502_02389_amd as L
import workloads as W
from tests.gpu_util import banner
from tests.test_gpu_md import _large_system, check

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
PARAMS = (W.MD_CUTOFF, W.MD_EPSILON, W.MD_SIGMA)


def _same(a, b):
    return torch.equal(a.view(torch.int32), b.view(torch.int32))


@pytest.mark.parametrize("n, k, lanes, unroll", [
    (600_001, 95, 16, 2), (600_001, 64, 8, 2), (600_001, 16, 8, 1), (700_001, 63, 16, 2), (1_048_576, 60, 8, 2),
    (1_048_576, 40, 8, 2), (1_048_576, 18, 8, 2), (1_048_576, 2, 8, 1), (1_300_003, 32, 8, 1)])
def test_short_lists_take_one_launch(gpu_device, n, k, lanes, unroll):
    pos, nbr = _large_system(n, k, "random", n % 1000, DEV)
    banner("md short lists", n, k)
    kn = L.knobs(block=256, vec_bytes=16, unroll=unroll, lanes_per_item=lanes)
    assert _same(L.md(pos, nbr, *PARAMS), L.md(pos, nbr, *PARAMS, knobs=kn))


@pytest.mark.parametrize("n, k, order", [(468_753, 97, "random"), (500_001, 98, "mixed"), (520_000, 96, "lattice"),
                                         (700_002, 66, "random"), (710_003, 65, "mixed"), (1_100_007, 64, "random")])
def test_long_lists_take_passes(gpu_device, n, k, order):
    pos, nbr = _large_system(n, k, order, n % 1000, DEV)
    i = torch.arange(n, device=DEV)[:, None]
    hole = (torch.arange(k, device=DEV)[None, :] * 7 + i) % 5 == 0      # holes, empty rows, rows by index
    nbr = torch.where((i // 8 % 6 == 1) & hole, -1, nbr)
    nbr = torch.where(i // 4 % 24 == 6, -1, nbr)
    nbr = torch.where(i // 8 % 6 == 4, nbr.sort(1).values, nbr)
    nbr = torch.where(i // 8 % 6 == 5, nbr.sort(1, descending=True).values, nbr).contiguous()
    banner("md long lists", n, k, order)
    out = torch.full((n, 4), float("nan"), device=DEV)
    L.md(pos, nbr, *PARAMS, out=out)
    first = out.clone()
    L.md(pos, nbr, *PARAMS, out=out)
    assert _same(first, out)
    check(out, pos.cpu(), nbr.cpu(), PARAMS)


@pytest.mark.parametrize("nx, k, lanes, unroll", [(512, 96, 8, 4), (700, 124, 8, 4), (700, 65, 16, 2), (1100, 66, 16, 2)])
def test_periodic_lattice_in_its_own_order(gpu_device, nx, k, lanes, unroll):
    """nx planes of 1024 particles, neighbours across the periodic faces."""
    n = nx * 1024
    pos, _ = _large_system(n, 1, "lattice", 3, DEV)
    i = torch.arange(n, device=DEV)
    offs = sorted((a * a + b * b + d * d, a, b, d) for a in range(-3, 4) for b in range(-3, 4) for d in range(-3, 4)
                  if (a, b, d) != (0, 0, 0))[:k]
    nbr = torch.stack([((i // 1024 + a) % nx * 32 + (i // 32 % 32 + b) % 32) * 32 + (i % 32 + d) % 32
                       for _, a, b, d in offs], 1).to(torch.int32)
    banner("md periodic lattice", nx, k)
    kn = L.knobs(block=256, vec_bytes=16, unroll=unroll, lanes_per_item=lanes)
    assert _same(L.md(pos, nbr, *PARAMS), L.md(pos, nbr, *PARAMS, knobs=kn))
