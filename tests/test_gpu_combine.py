"""The cross-work-group combine of asum / dot at the edges of its rounds.

The last work-group folds the others' partials as they arrive: 4 loads per
lane up to 256 of them, 8 beyond, in rounds.  Grids from 2 work-groups to
the largest, every accumulation and result type, on one workspace shared with
the kernels that use it otherwise (small lane forms, split gemv rows), its
slots filled with 0xff or left as the calls before left them.
"""
import math

import pytest
import torch

import paper_1502_02389_amd as L
import workloads as W
from tests.gpu_util import banner, o_asum, o_dot

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
STEP = 64 * 4 * 1            # elements per work-group: block 64, one 16-byte load
CODE = {"f32": L.LIFT_F32, "bf16": L.LIFT_BF16}


def _red(op, x, y, acc, rt, ws, knobs):
    res = torch.full((), float("nan"), dtype=torch.float64 if rt == L.LIFT_F64 else torch.float32, device=DEV)
    s = torch.cuda.current_stream().cuda_stream
    code = CODE["f32" if x.dtype == torch.float32 else "bf16"]
    args = (x.numel(), code, x.data_ptr()) + ((y.data_ptr(),) if op == "dot" else ())
    fn = L.lift_dot_ex if op == "dot" else L.lift_asum_ex
    assert fn(*args, L.ACC[acc], rt, res.data_ptr(), ws.data_ptr(), ws.numel(), knobs, s) == 0
    return res.item()


@pytest.mark.parametrize("acc", ["f32", "comp", "f64combine"])
@pytest.mark.parametrize("grid", [2, 3, 64, 65, 66, 256, 257, 258, 513, 1025, 8192])
def test_grids_integer_exact_on_a_shared_workspace(gpu_device, acc, grid):
    ws = torch.zeros(L.lift_workspace_bytes(), dtype=torch.uint8, device=DEV)
    hdr = L.lift_workspace_bytes() - 16 * L.lift_max_workgroups()
    n = STEP * (grid - 1) + 5
    g = W.gen(grid)
    x, y = W.integers(n, -4, 4, g), W.integers(n, -4, 4, g)
    ra, (rd, _) = o_asum(x), o_dot(x, y)
    xd, yd = x.to(DEV), y.to(DEV)
    A, gx = torch.ones((3, 70_000), device=DEV), torch.ones(70_000, device=DEV)
    s = torch.cuda.current_stream().cuda_stream
    kn = L.knobs(block=64, vec_bytes=16, unroll=1, split=STEP, interleave=L.LIFT_INTERLEAVE_CHUNK)
    banner("combine", acc, grid)
    for turn in range(3):
        for rt in (L.LIFT_F32, L.LIFT_F64):
            assert _red("asum", xd, None, acc, rt, ws, kn) == ra
            assert _red("dot", xd, yd, acc, rt, ws, kn) == rd
        assert _red("asum", xd, None, "f32", L.LIFT_F32, ws, L.knobs(block=16, split=1 << 10, lane_form=3)) == ra
        gy = torch.zeros(3, device=DEV)
        assert L.lift_gemv_ex_ws(3, 70_000, 1.0, L.LIFT_F32, A.data_ptr(), 70_000, gx.data_ptr(), 0.0, gy.data_ptr(),
                                 L.ACC[acc], ws.data_ptr(), ws.numel(), None, s) == 0
        assert gy.tolist() == [70_000.0] * 3
        assert int(ws[:hdr].count_nonzero().item()) == 0
        if turn == 0:
            ws[hdr:].fill_(0xFF)


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("acc", ["f32", "comp", "f64combine"])
def test_zero_and_nonfinite_partials_arrive(gpu_device, storage, acc):
    """Partials of every special value: zeros, infinities, NaNs (quiet and signalling inputs)."""
    ws = torch.zeros(L.lift_workspace_bytes(), dtype=torch.uint8, device=DEV)
    kn = L.knobs(block=64, vec_bytes=16, unroll=1, split=512, interleave=L.LIFT_INTERLEAVE_CHUNK)
    n = 512 * 300
    dt = W.STORAGE[storage]
    zero = torch.zeros(n, dtype=dt, device=DEV)
    banner("combine specials", storage, acc)
    assert _red("asum", zero, None, acc, L.LIFT_F32, ws, kn) == 0.0
    assert _red("dot", -zero, zero, acc, L.LIFT_F32, ws, kn) == 0.0
    inf = zero.clone()
    inf[700] = float("-inf")
    got = _red("asum", inf, None, acc, L.LIFT_F32, ws, kn)
    assert got == math.inf or (acc == "comp" and math.isnan(got))     # inf - inf in the error term
    for bits in ((0x7FC00001, 0x7FA5C3E1, 0xFFA00001) if storage == "f32" else (0x7FC1, 0x7FA5, 0xFFA0)):
        nan = torch.zeros(n, dtype=torch.int32 if storage == "f32" else torch.int16, device=DEV)
        top = 32 if storage == "f32" else 16
        nan[1500] = bits - (1 << top) if bits >= 1 << (top - 1) else bits
        assert math.isnan(_red("asum", nan.view(dt), None, acc, L.LIFT_F32, ws, kn))
        assert math.isnan(_red("dot", nan.view(dt), zero + 1, acc, L.LIFT_F64, ws, kn))
    assert _red("asum", zero + 1, None, acc, L.LIFT_F32, ws, kn) == float(n)
