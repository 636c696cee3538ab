"""Panels of one, two and four whole rows of gemv's long rows: both sides of the
row counts where the panel grows, rows that start alike and alternately on and
between dwords, a last group that is not full, in every storage and
accumulation.  Integers, exact.
"""
import pytest
import torch

import paper_1502_02389_amd as L
from tests.gpu_util import banner

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
CODE = {"f32": L.LIFT_F32, "bf16": L.LIFT_BF16, "f16": L.LIFT_F16}


@pytest.mark.parametrize("per_cu, more", [(1, 0), (1, 1), (6, 0), (6, 1), (8, 1), (8, 3)])
@pytest.mark.parametrize("storage, n, pad, start", [
    ("bf16", 32769, 0, 0), ("f16", 33001, 0, 1), ("bf16", 32784, 0, 0), ("f16", 32775, 1, 1), ("f32", 16389, 0, 1), ("f32", 16400, 0, 0)])
def test_whole_rows(gpu_device, storage, n, pad, start, per_cu, more):
    m = torch.cuda.get_device_properties(0).multi_processor_count * per_cu + more
    g = torch.Generator(DEV).manual_seed(m + n)
    lda = n + pad
    # one entry in 16 is not zero: sums stay below 2^24 in any order
    buf = torch.full((m * lda + 16,), float("nan"), dtype=DTYPE[storage], device=DEV)
    A = buf[start:start + m * lda].view(m, lda)
    v = torch.randint(-3, 4, (m, n), generator=g, device=DEV, dtype=torch.int8)
    v *= torch.randint(0, 16, (m, n), generator=g, device=DEV, dtype=torch.int8) == 0
    A[:, :n] = v.to(DTYPE[storage])
    x = torch.randint(-3, 4, (n + 1,), generator=g, device=DEV).float()[1:]
    y = torch.randint(-8, 9, (m,), generator=g, device=DEV).float()
    want = 2.0 * (v.float() @ x) + 0.5 * y
    banner("gemv panel", storage, m, n, lda, start)
    s = torch.cuda.current_stream().cuda_stream
    for acc in ("f32", "comp", "f64combine"):
        for beta in (0.5, 0.0):
            out = y.clone() if beta else torch.full_like(y, float("nan"))
            assert L.lift_gemv_ex(m, n, 2.0, CODE[storage], A.data_ptr(), lda, x.data_ptr(), beta, out.data_ptr(), L.ACC[acc],
                                  None, s) == 0
            assert torch.equal(out, want if beta else want - 0.5 * y), (acc, beta)
