"""GPU parity of MD (Fig. 7): forces from neighbour lists, Lennard-Jones.

The oracle decides updateF's test "distance < t" exactly (binary64 on the
stored positions); the kernel decides r^2 < binary32(t^2) on a binary32
r^2.  The two can differ only for pairs whose squared distance lies within
the kernel's rounding of t^2 (R2_BAND below), so every such pair is found in
binary64 and its term is allowed either way; every other pair must be
decided alike.  Forces are held to 1e-5 of the magnitude of their terms,
per particle and component (sum over the interacting neighbours of
|repulsive| + |attractive| times |d|: the sum of the forces cancels, so a
plain relative error is unbounded).
"""
import itertools

import numpy as np
import pytest
import torch

import paper_1502_02389_amd as L
import workloads as W
from tests.gpu_util import banner

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BAR = 1e-5
# The kernel's r^2 = (dx dx + dy dy) + dz dz in binary32 from rounded
# differences is within (1 + u)^5 - 1 ~ 5u of the exact r^2 (u = 2^-24: one
# rounding per difference, squared, one per square, two additions), and
# binary32(t^2) within u of t^2; 8u leaves room for second-order terms.
R2_BAND = 8 * 2.0 ** -24


def borderline_pairs(pos, nbr, cutoff):
    """Listed (particle, neighbour) pairs whose binary64 squared distance lies
    within R2_BAND * t^2 of t^2: the only pairs the kernel may decide
    differently from the exact test."""
    p = pos[:, :3].astype(np.float64)
    n, k = nbr.shape
    t2 = float(cutoff) ** 2
    found = {}
    step = max(1, (1 << 22) // max(k, 1))
    for lo in range(0, n if k else 0, step):
        idx = nbr[lo:lo + step]
        valid = (idx >= 0) & (idx < n)
        d = p[lo:lo + len(idx), None, :] - p[np.where(valid, idx, 0)]
        r2 = (d * d).sum(-1)
        for a, b in zip(*np.nonzero(valid & (np.abs(r2 - t2) <= R2_BAND * t2))):
            found.setdefault(lo + int(a), []).append(int(idx[a, b]))
    return found


def pair_term(pos, i, j, params):
    """The oracle's term of neighbour j in particle i's force (decided by the
    oracle's own test), the term itself, and its magnitude."""
    import oracle

    two = np.ascontiguousarray(pos[[i, j]])
    nb = np.array([[1], [-1]], np.int32)
    cutoff, eps, sigma = params
    f, m = oracle.md(two, nb, 1e30, eps, sigma, with_mass=True)
    inside = bool(np.any(oracle.md(two, nb, cutoff, eps, sigma)[0] != 0.0))
    return inside, f[0], m[0]


def check(got, pos, nbr, params):
    import oracle

    pos_np, nbr_np = pos.numpy(), nbr.numpy()
    ref, mass = oracle.md(pos_np, nbr_np, *params, with_mass=True)
    g = got.cpu().numpy().astype(np.float64)
    assert np.all(g[:, 3] == 0.0)
    err = np.abs(g[:, :3] - ref)
    bad = np.nonzero((err > BAR * mass + 1e-30).any(1))[0]
    border = borderline_pairs(pos_np, nbr_np, params[0]) if len(bad) else {}
    for i in bad:
        # only a particle with pairs at the cutoff may differ, and only by
        # some of those pairs' terms, each counted in or out
        assert i in border, (int(i), float((err[i] / np.maximum(mass[i], 1e-30)).max()))
        terms = [pair_term(pos_np, i, j, params) for j in border[i]]
        assert len(terms) <= 8, (int(i), len(terms))
        ok = False
        for flips in itertools.product((False, True), repeat=len(terms)):
            adj, m = ref[i].copy(), mass[i].copy()
            for flip, (inside, f, fm) in zip(flips, terms):
                if flip:
                    adj += -f if inside else f
                    m += fm
            if np.all(np.abs(g[i, :3] - adj) <= BAR * m + 1e-30):
                ok = True
                break
        assert ok, (int(i), border[i])
    return ref


def test_paper_size_system(gpu_device):
    pos, nbr, params = W.md_system()
    banner("md 12288 particles", nbr.shape)
    f = L.md(pos.to(DEV), nbr.to(DEV), *params)
    ref = check(f, pos, nbr, params)
    # the lists are symmetric, so the forces sum to ~0 (Newton's third law)
    tot = f.cpu().double()[:, :3].sum(0)
    assert float(tot.abs().max()) <= 1e-5 * float(np.abs(ref).sum())


KNOBS = [dict(lanes_per_item=l, vec_bytes=v, unroll=u, block=b)
         for l, v, u, b in [(1, 4, 1, 64), (1, 16, 4, 256), (2, 8, 2, 128), (4, 16, 1, 1024), (8, 16, 2, 256),
                            (8, 4, 4, 512), (16, 16, 4, 256), (16, 8, 1, 64), (4, 4, 2, 256)]]


@pytest.mark.parametrize("kn", KNOBS, ids=[str(i) for i in range(len(KNOBS))])
def test_every_knob_point_and_list_shapes(gpu_device, kn):
    pos, nbr, params = W.md_system(box=(9, 7, 11), slots=96, seed=71)
    n = pos.shape[0]
    pd = pos.to(DEV)
    for k in (96, 37, 1, 0):     # 37: odd length (one index per load), 0: no neighbours
        sub = nbr[:, :k].contiguous()
        banner("md knobs", kn, "k", k)
        out = torch.empty((n, 4), device=DEV)
        st = L.lift_md_ex(n, pd.data_ptr(), k, sub.to(DEV).data_ptr() if k else 0, *params, out.data_ptr(),
                          L.knobs(**kn), torch.cuda.current_stream().cuda_stream)
        assert st == L.LIFT_OK
        check(out, pos, sub, params)
    # lists starting 4 bytes past a 16-byte boundary
    buf = torch.empty(n * 96 + 1, dtype=torch.int32, device=DEV)
    view = buf[1:].view(n, 96)
    view.copy_(nbr.to(DEV))
    out = torch.empty((n, 4), device=DEV)
    assert L.lift_md_ex(n, pd.data_ptr(), 96, view.data_ptr(), *params, out.data_ptr(), L.knobs(**kn),
                        torch.cuda.current_stream().cuda_stream) == L.LIFT_OK
    check(out, pos, nbr, params)


def test_empty_slots_and_degenerate_sizes(gpu_device):
    pos, nbr, params = W.md_system(box=(5, 5, 5), slots=64, seed=72)
    n = pos.shape[0]
    junk = nbr.clone()
    junk[:, ::5] = -1
    junk[:, 1::7] = n
    junk[:, 2::11] = 2 ** 31 - 1
    junk[:, 3::13] = -(2 ** 31)
    banner("md empty slots")
    check(L.md(pos.to(DEV), junk.to(DEV), *params), pos, junk, params)
    one = torch.tensor([[0.5, 0.5, 0.5, 0.0]])
    lone = torch.tensor([[-1, 1, 5]], dtype=torch.int32)
    f = L.md(one.to(DEV), lone.to(DEV), *params)
    assert torch.equal(f.cpu(), torch.zeros(1, 4))
    assert L.md(torch.zeros((0, 4), device=DEV), torch.zeros((0, 8), dtype=torch.int32, device=DEV),
                *params).shape == (0, 4)


def test_cutoff_boundary(gpu_device):
    # pairs at exactly t, 1 ulp inside and 1 ulp outside (both within the
    # kernel's band: either decision is allowed, the force must be one of
    # the two), and pairs 64 ulps inside and outside, which the kernel must
    # decide as the exact test does
    t = 1.25
    tf = np.float32(t)
    seps = [tf, np.nextafter(tf, np.float32(0)), np.nextafter(tf, np.float32(2)),
            np.float32(t * (1 - 64 * 2.0 ** -24)), np.float32(t * (1 + 64 * 2.0 ** -24))]
    pos = torch.zeros((2 * len(seps), 4))
    for c, sep in enumerate(seps):
        pos[2 * c, 1] = pos[2 * c + 1, 1] = 3.0 * c
        pos[2 * c + 1, 0] = float(sep)
    nbr = torch.tensor([[i ^ 1] for i in range(2 * len(seps))], dtype=torch.int32)
    banner("md cutoff boundary")
    f = L.md(pos.to(DEV), nbr.to(DEV), t, 1.0, 1.0).cpu()
    assert torch.all(f[0:2] == 0)              # exactly t: r^2 = t^2 in binary32 too
    assert torch.all(f[6:8, 0] != 0)           # 64 ulps inside
    assert torch.all(f[8:10] == 0)             # 64 ulps outside
    check(f, pos, nbr, (t, 1.0, 1.0))


def test_cutoff_pairs_where_binary32_rounding_decides(gpu_device):
    # separations whose exact distance and binary32 r^2 fall on opposite
    # sides of the cutoff: the kernel's result must equal the oracle's with
    # that one term counted in or out
    from tests.test_oracle_md import _near_cutoff_pairs

    t = 2.5
    qs = [q for v in _near_cutoff_pairs(t, count=6, seed=11).values() for q in v]
    pos = torch.zeros((2 * len(qs), 4))
    for c, q in enumerate(qs):
        pos[2 * c, 0] = pos[2 * c + 1, 0] = 8.0 * c
        pos[2 * c + 1, :3] += torch.from_numpy(q)
    nbr = torch.tensor([[i ^ 1] for i in range(2 * len(qs))], dtype=torch.int32)
    banner("md binary32 borderline pairs", len(qs))
    check(L.md(pos.to(DEV), nbr.to(DEV), t, 1.0, 1.0), pos, nbr, (t, 1.0, 1.0))


def test_bitwise_deterministic(gpu_device):
    pos, nbr, params = W.md_system()
    pd, nd = pos.to(DEV), nbr.to(DEV)
    a = L.md(pd, nd, *params)
    for _ in range(5):
        assert torch.equal(L.md(pd, nd, *params), a)


def _md_plain(pos, nbr, params, defaults=False):
    """Forces through the plain entry point (no knobs: the library's tuned
    entry on this device), the call the benchmark times; or, with
    ``defaults``, with explicit all-zero knobs (the built-in defaults)."""
    pd, nd = pos.to(DEV), nbr.to(DEV)
    out = torch.empty((pos.shape[0], 4), dtype=torch.float32, device=DEV)
    s = torch.cuda.current_stream().cuda_stream
    if defaults:
        assert L.lift_md_ex(pos.shape[0], pd.data_ptr(), nbr.shape[1], nd.data_ptr(), *params, out.data_ptr(),
                            L.knobs(), s) == 0
    else:
        assert L.lift_md(pos.shape[0], pd.data_ptr(), nbr.shape[1], nd.data_ptr(), *params, out.data_ptr(),
                         s) == 0
    return out


def test_paper_size_system_library_default_launch(gpu_device):
    pos, nbr, params = W.md_system()
    banner("md 12288 particles, library default launch")
    check(_md_plain(pos, nbr, params), pos, nbr, params)


@pytest.mark.parametrize("launch,shuffle", [("plain entry point", True), ("library defaults", True),
                                            ("plain entry point", False)])
def test_large_system(gpu_device, launch, shuffle):
    pos, nbr, params = W.md_system(W.MD_BOX_LARGE, shuffle=shuffle)
    banner("md 2^20 particles", launch, "random order" if shuffle else "lattice order")
    f = _md_plain(pos, nbr, params, defaults=launch == "library defaults")
    check(f, pos, nbr, params)


# ------------------------------------------------------------------ passes over slices of the positions


def _large_system(n, k, order, seed, device):
    """n particles on a jittered line of unit cells (1024 x 32 lattice planes),
    every particle's k neighbours among the nearest lattice offsets; the
    particle order is the lattice's, random, or random in its first half.
    Built on the GPU (the oracle sees the same bits)."""
    g = torch.Generator(device)
    g.manual_seed(seed)
    i = torch.arange(n, device=device)
    ny, nz = 32, 32
    c = torch.stack([i // (ny * nz), i // nz % ny, i % nz], 1)
    pos = torch.zeros((n, 4), device=device)
    where = c.to(torch.float32) + torch.rand((n, 3), generator=g, device=device) * 0.2 - 0.1
    perm = i.clone()
    if order == "random":
        perm = torch.randperm(n, generator=g, device=device)
    elif order == "mixed":
        perm[: n // 2] = torch.randperm(n // 2, generator=g, device=device)
    old = torch.empty_like(perm)
    old[perm] = i
    pos[:, :3] = where[old]
    co = c[old]
    offs = sorted((a * a + b * b + d * d, a, b, d) for a in range(-2, 3) for b in range(-2, 3) for d in range(-2, 3)
                  if (a, b, d) != (0, 0, 0))
    nbr = torch.full((n, k), -1, dtype=torch.int32, device=device)
    nx = (n + ny * nz - 1) // (ny * nz)
    for j, (_, a, b, d) in enumerate(offs[:k]):
        x, y, z = co[:, 0] + a, co[:, 1] + b, co[:, 2] + d
        at = (x * ny + y) * nz + z
        ok = (x >= 0) & (x < nx) & (y >= 0) & (y < ny) & (z >= 0) & (z < nz) & (at < n)
        nbr[:, j] = torch.where(ok, perm[torch.where(ok, at, 0)], -1).to(torch.int32)
    return pos.contiguous(), nbr


@pytest.mark.parametrize("n,k,order", [(468_753, 24, "random"), (500_001, 20, "mixed"), (700_002, 13, "random"),
                                       (1_100_007, 6, "random"), (600_000, 18, "lattice"), (480_000, 124, "random")])
def test_passes_over_slices(gpu_device, n, k, order):
    """Systems of 2, 3 and 4 slices (and a row length of each index width, rows
    longer than 64 and padding within them): forces as the oracle has them,
    fourth component 0, whatever the output held before, on every run the same bits."""
    pos, nbr = _large_system(n, k, order, n % 1000, DEV)
    params = (W.MD_CUTOFF, W.MD_EPSILON, W.MD_SIGMA)
    banner("md passes", n, k, order)
    out = torch.full((n, 4), float("nan"), device=DEV)
    L.md(pos, nbr, *params, out=out)
    first = out.clone()
    out.fill_(1.0)
    L.md(pos, nbr, *params, out=out)
    assert torch.equal(first.view(torch.int32), out.view(torch.int32))
    check(out, pos.cpu(), nbr.cpu(), params)


def test_passes_in_a_graph_and_under_the_timing_hook(gpu_device):
    n, k = 520_000, 10
    pos, nbr = _large_system(n, k, "random", 5, DEV)
    params = (W.MD_CUTOFF, W.MD_EPSILON, W.MD_SIGMA)
    want = L.md(pos, nbr, *params)
    ev = L.HipEvents(2)
    banner("md passes timed")
    try:
        assert L.lift_time_next_launch(ev.events[0], ev.events[1]) == 0
        got = L.md(pos, nbr, *params)
        torch.cuda.synchronize()
        assert 0.0 < ev.elapsed_ms(0, 1) < 50.0
        assert torch.equal(got, want)
    finally:
        ev.close()
    s = torch.cuda.Stream(device=DEV)
    out = torch.empty((n, 4), device=DEV)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        s.wait_stream(torch.cuda.default_stream())
        with torch.cuda.graph(graph, stream=s):
            L.md(pos, nbr, *params, out=out)
        for _ in range(3):
            out.fill_(float("nan"))
            graph.replay()
            s.synchronize()
            assert torch.equal(out, want)
    graph.reset()


@pytest.mark.parametrize("n,k,order", [(469_001, 140, "random"), (800_003, 21, "random"), (470_000, 64, "mixed")])
def test_passes_with_padding_anywhere(gpu_device, n, k, order):
    """Rows whose padding comes first, rows with holes, empty rows, rows of one
    slice only (sorted either way): every pass reads what it still needs."""
    pos, nbr = _large_system(n, k, order, n % 1000, DEV)
    i = torch.arange(n, device=DEV)[:, None]
    hole = (torch.arange(k, device=DEV)[None, :] * 7 + i) % 5 == 0
    nbr = torch.where((i // 8 % 6 == 1) & hole, -1, nbr)
    nbr = torch.where(i // 8 % 6 == 2, nbr.flip(1), nbr)
    nbr = torch.where(i // 4 % 12 == 6, -1, nbr)
    nbr = torch.where(i // 8 % 6 == 4, nbr.sort(1).values, nbr)
    nbr = torch.where(i // 8 % 6 == 5, nbr.sort(1, descending=True).values, nbr).contiguous()
    params = (W.MD_CUTOFF, W.MD_EPSILON, W.MD_SIGMA)
    banner("md passes padding", n, k, order)
    out = torch.full((n, 4), float("nan"), device=DEV)
    L.md(pos, nbr, *params, out=out)
    first = out.clone()
    L.md(pos, nbr, *params, out=out)
    assert torch.equal(first.view(torch.int32), out.view(torch.int32))
    check(out, pos.cpu(), nbr.cpu(), params)
