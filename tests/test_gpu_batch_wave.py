"""The batch without knobs (wavefront tiles, one launch) over every class of
tile: rows on both sides of each row-length class and of each storage, starts
at any element, reductions around a tile's and a step's size, problems of one
and of many tiles, more tiles than wavefronts (drawn) and fewer (not).

Integer inputs bit-exact in every accumulation; what lies around the operands
is NaN, what lies around the outputs stays as it was.
"""
import pytest
import torch

import paper_1502_02389_amd as L
import workloads as W
from tests.gpu_util import banner, o_asum, o_dot, o_gemv

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _at(t, off):
    buf = torch.full((t.numel() + off + 9,), float("nan"), dtype=t.dtype, device=DEV)
    buf[off:off + t.numel()] = t.reshape(-1).to(DEV)
    return buf[off:off + t.numel()], buf


def _gemv(m, n, lda, storage, g, off, beta):
    A = W.integers((m, lda), -3, 3, g, storage)
    x, y = W.integers(n, -3, 3, g), W.integers(m, -8, 8, g)
    want, _ = o_gemv(2.0, A, x, beta, y)
    A[:, n:] = float("nan")
    ad, _ = _at(A, off)
    xd, _ = _at(x, 1)
    yd, ybuf = _at(y if beta else torch.full((m,), float("nan")), 2)
    return ("gemv", 2.0, ad.view(m, lda), xd, beta, yd), want, ybuf


def _red(kind, n, storage, g, ox, oy):
    x, y = W.integers(n, -4, 4, g, storage), W.integers(n, -3, 3, g, storage)
    xd, yd = _at(x, ox)[0], _at(y, oy)[0]
    return (("dot", xd, yd), o_dot(x, y)[0]) if kind == "dot" else (("asum", xd), o_asum(x))


def _run_and_check(problems, wants, bufs, acc, runs=2):
    b = L.Batch(problems, acc=acc)
    ys = [p[5].clone() if p[0] == "gemv" else None for p in problems]
    for _ in range(runs):
        for p, y in zip(problems, ys):
            if y is not None:
                p[5].copy_(y)
        for r in b.results:
            if r is not None:
                r.fill_(float("nan"))
        b.run()
        torch.cuda.synchronize()
        for i, (p, want) in enumerate(zip(problems, wants)):
            if p[0] == "gemv":
                assert (p[5].cpu().double().numpy() == want).all(), (i, p[2].shape)
                buf, m = bufs[i], p[5].numel()
                assert torch.isnan(buf[:2]).all() and torch.isnan(buf[2 + m:]).all(), i
            else:
                assert b.results[i].item() == want, (i, p[0], p[1].numel())
    b.close()


@pytest.mark.parametrize("storage", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("acc", ["f32", "comp", "f64combine"])
def test_every_row_and_length_class(gpu_device, storage, acc):
    E = 4 if storage == "f32" else 8
    g = W.gen(90)
    problems, wants, bufs = [], [], []
    edges = [8, 16, 32, 64, 128, 192, 256, 320, 384, 448, 512, 768, 1024, 1100]
    columns = [0, 1, 2, E - 1, E, E + 1] + [v for k in edges for v in (k * E - 1, k * E, k * E + 1, k * E + E // 2 + 1)]
    banner("batch wave classes", storage, acc)
    for j, n in enumerate(columns):
        for m, pad in ((1, 0), (5, 1)) + (((67, 0),) if j % 3 == 0 else ()):
            p, want, buf = _gemv(m, n, max(n + pad, 1), storage, g, j % 3, 0.0 if j % 4 == 0 else 0.5)
            problems.append(p)
            wants.append(want)
            bufs.append(buf)
    step = 64 * E
    for j, n in enumerate([0, 1, E - 1, E, E + 1, step - 1, step, step + 1, 4 * step, 8 * step + 3, 16384 // (16 // E),
                           40_003, 130_001, 262_144 + 7]):
        for kind in ("asum", "dot"):
            p, want = _red(kind, n, storage, g, j % 4, (3 * j) % 5)
            problems.append(p)
            wants.append(want)
            bufs.append(None)
    _run_and_check(problems, wants, bufs, acc)


@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_more_tiles_than_wavefronts(gpu_device, storage):
    """Thousands of short problems and one long one: tiles are drawn."""
    g = W.gen(91)
    problems, wants, bufs = [], [], []
    x = W.integers(9000 * 64, -4, 4, g, storage).to(DEV)
    for i in range(9000):
        n = 1 + (i * 37) % 64
        v = x[i * 64:i * 64 + n]
        problems.append(("asum", v))
    sums = x.view(9000, 64).double().abs().cumsum(1).cpu()
    wants = [sums[i, (i * 37) % 64].item() for i in range(9000)]
    bufs = [None] * 9000
    p, want = _red("dot", 3_000_001, storage, g, 0, 1)
    problems.append(p), wants.append(want), bufs.append(None)
    p, want, buf = _gemv(3001, 333, 333, storage, g, 1, 0.5)
    problems.append(p), wants.append(want), bufs.append(buf)
    banner("batch wave drawn", storage)
    _run_and_check(problems, wants, bufs, "f32", runs=4)


@pytest.mark.parametrize("above", [0, 1])
def test_both_sides_of_the_size_line(gpu_device, above):
    """One tile per wavefront at 64 KiB each (one launch) and work-group tiles
    just above (a bigger batch has the finer reduction split); sums of a sparse
    0/1 vector stay below 2^24, so they are exact in any order."""
    g = W.gen(92)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n = 65536 // 4 * 4 * 4 * cus          # binary32, if four work-groups fit a compute unit
    x = torch.zeros(n, dtype=torch.float32)
    x[::11] = 1.0
    problems, wants = [("asum", x.to(DEV))], [float(-(-n // 11))]
    for i in range(3 * above):
        p, want = _red("dot", 1000 + i, "f32", g, i % 5, 1)
        problems.append(p), wants.append(want)
    banner("batch size line", above)
    _run_and_check(problems, wants, [None] * len(problems), "f32")
