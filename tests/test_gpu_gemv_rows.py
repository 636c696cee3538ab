"""gemv calls that leave the launch to the library, over every row length
class, row start, pitch and storage, against the binary64 oracle.

The launch goes by row length: element loads below one 16-byte vector, 8 to
64 lanes x up to 8 vectors, a work-group of 3 to 8 wavefronts, panels of long
rows (split over work-groups when there is a workspace).  Sizes sit on both
sides of each boundary; rows start at every 2-byte phase (odd pitches, odd
views of A), x and y are misaligned views, padding columns hold NaN.  Integer
inputs whose partial sums stay below 2^24 must be bit-exact in every variant;
normal inputs meet the row bound 1e-5 (|alpha| sum |A x| + |beta y|).
"""
import numpy as np
import pytest
import torch

import paper_1502_02389_amd as L
import workloads as W
from tests.gpu_util import banner, o_gemv

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
ACCS = ["f32", "comp", "f64combine"]
CODE = {"f32": L.LIFT_F32, "bf16": L.LIFT_BF16, "f16": L.LIFT_F16}


def _view(t, off):
    """t on the GPU, starting `off` elements into a buffer of NaN (the bytes around it too)."""
    buf = torch.full((t.numel() + off + 16,), float("nan"), dtype=t.dtype, device=DEV)
    buf[off:off + t.numel()] = t.reshape(-1).to(DEV)
    return buf[off:off + t.numel()], buf


def _call(m, n, lda, storage, acc, ad, xd, yd, alpha, beta, ws):
    s = torch.cuda.current_stream().cuda_stream
    args = (m, n, alpha, CODE[storage], ad.data_ptr(), lda, xd.data_ptr(), beta, yd.data_ptr(), L.ACC[acc])
    if ws is None:
        return L.lift_gemv_ex(*args, None, s)
    return L.lift_gemv_ex_ws(*args, ws.data_ptr(), ws.numel(), None, s)


# columns around the class boundaries (in elements of 16-byte vectors: E = 4 or 8)
def _columns(E):
    return [1, 2, E - 1, E, E + 1, 8 * E, 8 * E + 1, 16 * E + 3, 64 * E - 1, 64 * E + 1, 128 * E + 2, 64 * 5 * E + 1,
            64 * 8 * E, 64 * 8 * E + 1, 64 * 17 * E + 5, 64 * 49 * E - 3, 64 * 64 * E, 64 * 64 * E + 1,
            64 * 64 * E + 7 * E + 3]


@pytest.mark.parametrize("storage", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("pad", [0, 1, 2])
@pytest.mark.parametrize("off", [0, 1])
def test_rows_integer_bitexact(gpu_device, storage, pad, off):
    E = 4 if storage == "f32" else 8
    ws = torch.zeros(L.lift_workspace_bytes(), dtype=torch.uint8, device=DEV)
    hdr = L.lift_workspace_bytes() - 16 * L.lift_max_workgroups()
    for n in _columns(E):
        lda = n + pad
        for m in (1, 2, 3, 37) + ((2051,) if n < 64 * 17 * E else ()):
            g = W.gen(n * 31 + m + pad + off)
            A = W.integers((m, lda), -4, 4, g, storage)
            x = W.integers(n, -4, 4, g)
            y = W.integers(m, -8, 8, g)
            want, _ = o_gemv(2.0, A, x, 0.5, y)
            A[:, n:] = float("nan")               # padding columns are never part of a sum
            ad, _ka = _view(A, off)
            xd, _kx = _view(x, 1)
            banner("gemv rows", storage, m, n, lda, off)
            for acc in ACCS:
                for w in (None, ws):
                    yd, buf = _view(y, 3)
                    assert _call(m, n, lda, storage, acc, ad, xd, yd, 2.0, 0.5, w) == 0
                    assert np.array_equal(yd.cpu().numpy().astype(np.float64), want), (m, n, acc, w is not None)
                    assert torch.isnan(buf[:3]).all() and torch.isnan(buf[3 + m:]).all()
    assert int(ws[:hdr].count_nonzero().item()) == 0


@pytest.mark.parametrize("storage", ["f32", "bf16", "f16"])
def test_split_rows_integer_bitexact_and_repeatable(gpu_device, storage):
    """Few long rows: chunks on several work-groups, a ragged last chunk."""
    ws = torch.zeros(L.lift_workspace_bytes(), dtype=torch.uint8, device=DEV)
    for m, n in [(1, 300_001), (3, 262_144), (5, 100_003), (32, 131_072 + 9), (257, 70_001)]:
        g = W.gen(n + m)
        A = W.integers((m, n), -2, 2, g, storage)
        x = W.integers(n, -2, 2, g)
        y = W.integers(m, -8, 8, g)
        want, _ = o_gemv(1.0, A, x, -0.5, y)
        ad, _ka = _view(A, 1)
        xd, _kx = _view(x, 2)
        banner("gemv split rows", storage, m, n)
        for acc in ACCS:
            for _ in range(3):
                yd, _ky = _view(y, 1)
                assert _call(m, n, n, storage, acc, ad, xd, yd, 1.0, -0.5, ws) == 0
                assert np.array_equal(yd.cpu().numpy().astype(np.float64), want), (m, n, acc)


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("m,n", [(700, 33), (300, 1001), (64, 4099), (9, 33_333), (4, 200_000)])
def test_rows_normal_within_bound_and_nonfinite_stay_in_their_row(gpu_device, storage, m, n):
    g = W.gen(m + n)
    A, x, y = W.normal((m, n), g, storage), W.normal(n, g), W.normal(m, g)
    r, mass = o_gemv(1.25, A, x, 0.0, torch.zeros(m))
    banner("gemv rows normal", storage, m, n)
    yd = torch.full((m,), float("nan"), device=DEV)      # beta 0: not read
    L.gemv(1.25, A.to(DEV), x.to(DEV), 0.0, yd)
    err = np.abs(yd.cpu().numpy().astype(np.float64) - r) / mass
    assert float(err.max()) <= 1e-5
    A[1, n - 1] = float("inf")                            # the end of a row, next to the following row
    A[2, 0] = float("nan")
    yd = y.to(DEV)
    L.gemv(1.25, A.to(DEV), x.abs().to(DEV), 0.5, yd)
    got = yd.cpu().numpy()
    bad = ~np.isfinite(got)
    assert list(np.nonzero(bad)[0]) == [1, 2] and np.isposinf(got[1]) and np.isnan(got[2])


def test_ws_entry_rejects_bad_workspace(gpu_device):
    ws = torch.zeros(L.lift_workspace_bytes(), dtype=torch.uint8, device=DEV)
    A, x, y = torch.ones((2, 8), device=DEV), torch.ones(8, device=DEV), torch.ones(2, device=DEV)
    s = torch.cuda.current_stream().cuda_stream
    args = (2, 8, 1.0, L.LIFT_F32, A.data_ptr(), 8, x.data_ptr(), 0.0, y.data_ptr(), 0)
    assert L.lift_gemv_ex_ws(*args, 0, ws.numel(), None, s) == L.LIFT_EWORKSPACE
    assert L.lift_gemv_ex_ws(*args, ws.data_ptr(), ws.numel() - 1, None, s) == L.LIFT_EWORKSPACE
    assert L.lift_gemv_ex_ws(*args, ws.data_ptr() + 4, ws.numel(), None, s) == L.LIFT_EINVAL


@pytest.mark.parametrize("m, n, storage", [(4096, 4096, "f32"), (4090, 4100, "f32"), (2100, 8188, "f32"), (8200, 8192, "f32"),
                                           (7000, 9600, "f32"), (16385, 16384, "bf16"), (16000, 16392, "bf16"),
                                           (9000, 30000, "f16")])
def test_both_sides_of_the_tuned_rows(gpu_device, m, n, storage):
    """Aligned rows of a power of two (a tuned entry's) and just off it, in the
    size buckets that have tuned entries: exact on small integers."""
    g = torch.Generator(DEV)
    g.manual_seed(m + n)
    dt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[storage]
    A = torch.randint(-1, 2, (m, n), generator=g, device=DEV, dtype=torch.int8).to(dt)
    x = torch.randint(-3, 4, (n,), generator=g, device=DEV).float()
    y = torch.randint(-8, 9, (m,), generator=g, device=DEV).float()
    want = torch.cat([2.0 * (a.double() @ x.double()) for a in A.split(2048)]) + 0.5 * y.double()
    banner("tuned rows", m, n, storage)
    L.gemv(2.0, A, x, 0.5, y)
    assert torch.equal(y.double(), want)
