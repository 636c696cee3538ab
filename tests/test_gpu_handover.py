"""The combine handed over: the last work-group's wait cut to no wait at all,
so that a work-group that comes later folds in its place.  Bits, workspace and
result types as without, in every accumulation, for asum, dot and split gemv.
"""
import pytest
import torch

import paper_1502_02389_amd as L
import workloads as W
from tests.gpu_util import banner

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CODE = {"f32": L.LIFT_F32, "bf16": L.LIFT_BF16}


def _ws():
    return torch.zeros(L.lift_workspace_bytes(), dtype=torch.uint8, device=DEV)


def _red(op, x, y, storage, acc, rt, ws, knobs):
    res = torch.full((1,), float("nan"), dtype=torch.float64 if rt == L.LIFT_F64 else torch.float32, device=DEV)
    s = torch.cuda.current_stream().cuda_stream
    args = (x.numel(), CODE[storage], x.data_ptr()) + ((y.data_ptr(),) if op == "dot" else ())
    fn = L.lift_dot_ex if op == "dot" else L.lift_asum_ex
    assert fn(*args, L.ACC[acc], rt, res.data_ptr(), ws.data_ptr(), ws.numel(), knobs, s) == 0
    return res


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("acc", ["f32", "comp", "f64combine"])
@pytest.mark.parametrize("grid, split", [(2, 1 << 20), (3, 1 << 20), (65, 1 << 18), (257, 1 << 16), (258, 256), (1025, 1 << 14),
                                         (8192, 256)])
def test_reductions(gpu_device, storage, acc, grid, split):
    """The last work-group has 5 elements, the others `split`."""
    n = split * (grid - 1) + 5
    g = W.gen(grid)
    x, y = W.uniform(n, g, storage).to(DEV), W.uniform(n, g, storage).to(DEV)
    kn = L.knobs(block=64, vec_bytes=16, unroll=1, split=split, interleave=L.LIFT_INTERLEAVE_CHUNK)
    ws = _ws()
    banner("handover", storage, acc, grid)
    for op in ("asum", "dot"):
        for rt in (L.LIFT_F32, L.LIFT_F64):
            want = _red(op, x, y, storage, acc, rt, ws, kn)
            for rounds in (0, 0, 1, 40):
                assert L.lift_combine_rounds_next_launch(rounds) == L.LIFT_OK
                got = _red(op, x, y, storage, acc, rt, ws, kn)
                assert torch.equal(got.view(torch.uint8), want.view(torch.uint8)), (op, rt, rounds, got, want)
                assert not ws.any().item(), (op, rt, rounds)


def test_another_work_group_combines(gpu_device):
    """Of 64 work-groups with a MiB each and one with 20 bytes, the last does
    not wait: the stamps name another one as the one that combined."""
    split = 1 << 18
    x = torch.ones(split * 64 + 5, device=DEV)
    kn = L.knobs(block=256, vec_bytes=16, unroll=4, split=split, interleave=L.LIFT_INTERLEAVE_CHUNK)
    want = L.asum(x, knobs=kn).item()
    banner("handover stamps")
    for rounds, handed in ((0, True), (1 << 20, False)):
        stamps = torch.zeros((65, 8), dtype=torch.int64, device=DEV)
        assert L.lift_stamp_next_launch(stamps.data_ptr(), 65)[0] == L.LIFT_OK
        assert L.lift_combine_rounds_next_launch(rounds) == L.LIFT_OK
        assert L.asum(x, knobs=kn).item() == want
        combined = torch.nonzero((stamps[:, 6].cpu() >> 32) & 1).flatten().tolist()
        assert len(combined) == 1 and (combined != [64]) == handed, (rounds, combined)


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("acc", ["f32", "comp", "f64combine"])
@pytest.mark.parametrize("m, n", [(1, 70_001), (1, 4_000_001), (3, 400_003), (32, 200_001), (57, 262_144), (256, 40_001)])
def test_split_gemv(gpu_device, storage, acc, m, n):
    g = W.gen(m)
    A = torch.rand((m, n), generator=torch.Generator().manual_seed(n)).mul_(2).sub_(1).to(W.STORAGE[storage]).to(DEV)
    x, y = W.uniform(n, g).to(DEV), W.uniform(m, g).to(DEV)
    ws = _ws()
    s = torch.cuda.current_stream().cuda_stream
    banner("handover gemv", storage, acc, m, n)

    def call():
        out = y.clone()
        assert L.lift_gemv_ex_ws(m, n, 1.5, CODE[storage], A.data_ptr(), n, x.data_ptr(), 0.5, out.data_ptr(), L.ACC[acc],
                                 ws.data_ptr(), ws.numel(), None, s) == 0
        return out

    want = call()
    exact = 1.5 * (A.double() @ x.double()) + 0.5 * y.double()
    mass = 1.5 * (A.double().abs() @ x.double().abs()) + 0.5 * y.double().abs()
    assert ((want.double() - exact).abs() <= 1e-5 * mass).all()
    for rounds in (0, 0, 1, 40):
        assert L.lift_combine_rounds_next_launch(rounds) == L.LIFT_OK
        assert torch.equal(call(), want), rounds
        assert not ws.any().item(), rounds
