"""Performance cases: the calls a program makes of this library, over the sizes it meets.

``listed()`` names the fixed cases, ``draw(rng)`` gives further ones of the same
ranges; ``prepare`` builds a case's inputs on the GPU from a seed, ``run`` makes
one pass through the public entry points, ``work`` counts the bytes and
operations the pass cannot do without, and ``exact`` evaluates the same
results in binary64 with plain torch.

Families (``op``):

* ``dot``   : one eager reduction call, from a few hundred elements (a latency
              a program pays per call) upwards.
* ``graph`` : scal, asum and dot on a handful of vectors, captured into a HIP
              graph and replayed: how a solver's inner loop on small and
              middling vectors is run.
* ``step``  : scal + asum + dot on fp32 vectors, the benchmark's step.
* ``lag``   : asum of a view and the lag-one product dot(x[1:], x[:-1]): odd
              lengths, and operands that never share an alignment.
* ``half``  : asum and dot of 16-bit vectors with a chosen accumulation.
* ``gemv``  : y = alpha A x + beta y, contiguous A of any shape: square, ragged
              (an odd row length), a few very long rows, many short ones.
* ``batch`` : many uneven asum / dot / gemv problems planned once, run at once.
* ``bs``    : BlackScholes over a vector of prices.
* ``md``    : Lennard-Jones forces over neighbour lists, particles in random
              or in lattice order.
"""
import ctypes
import math
import random

import torch

import paper_1502_02389_amd as L

DEV = "cuda:0"
DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
CODE = {"f32": L.LIFT_F32, "bf16": L.LIFT_BF16, "f16": L.LIFT_F16}
BYTES = {"f32": 4, "bf16": 2, "f16": 2}
ALPHA = 2.5
GEMV_ALPHA, GEMV_BETA = 1.0, 0.5
STRIKE, RATE, VOLATILITY, YEARS = 20.0, 0.02, 0.30, 1.0
CUTOFF, EPSILON, SIGMA, RLIST, SLOTS = 2.5, 1.0, 1.0, 2.8, 128
GRAPH_VECTORS = 8


def listed():
    return [
        # the latency of one small eager call (a few thousand elements)
        {"name": "dot_small", "op": "dot", "n": 4097, "dtype": "f32", "acc": "f32"},
        # a solver's inner loop on 4 MiB vectors, replayed from a graph
        {"name": "graph_2p20", "op": "graph", "n": 1 << 20},
        # the benchmark's step: 64 MiB vectors, the paper's 16M-element size
        {"name": "step_2p24", "op": "step", "n": 1 << 24},
        # lag-one statistics of an odd-length series
        {"name": "lag_2p23", "op": "lag", "n": (1 << 23) + 5, "dtype": "f32", "acc": "f32"},
        # long 16-bit vectors, compensated accumulation
        {"name": "half_2p26", "op": "half", "n": 1 << 26, "dtype": "bf16", "acc": "comp"},
        # the paper's small matrix
        {"name": "gemv_4096", "op": "gemv", "m": 4096, "n": 4096, "dtype": "f32", "acc": "f32"},
        # a large 16-bit matrix
        {"name": "gemv_bf16_16384", "op": "gemv", "m": 16384, "n": 16384, "dtype": "bf16", "acc": "f32"},
        # a contiguous 16-bit matrix whose odd row length leaves rows unaligned
        {"name": "gemv_ragged", "op": "gemv", "m": 20000, "n": 4099, "dtype": "bf16", "acc": "f32"},
        # a long vector against a small basis (an orthogonalisation step)
        {"name": "gemv_wide", "op": "gemv", "m": 32, "n": 1 << 20, "dtype": "f32", "acc": "f32"},
        # the benchmark's uneven batch in 16-bit storage
        {"name": "batch_mixed", "op": "batch", "n_red": 4096, "n_gemv": 256, "hi_exp": 20.0, "mn_hi": 4096,
         "dtype": "bf16", "shapes": 4},
        # the paper's option count
        {"name": "bs_2p22", "op": "bs", "n": 1 << 22},
        # a large particle system in the order its generator leaves it (random)
        {"name": "md_2p20", "op": "md", "nx": 128, "ny": 128, "nz": 64, "shuffle": True},
    ]


def _log(rng, lo, hi):
    return int(2.0 ** rng.uniform(math.log2(lo), math.log2(hi + 1)))


def draw(rng):
    op = rng.choice(["dot", "graph", "step", "lag", "half", "gemv", "gemv", "batch", "bs", "md"])
    acc = rng.choice(["f32", "f32", "comp", "f64combine"])
    if op == "dot":
        dtype = rng.choice(["f32", "bf16", "f16"])
        return {"op": op, "n": _log(rng, 200, 1 << 26), "dtype": dtype, "acc": acc}
    if op == "graph":
        return {"op": op, "n": _log(rng, 256, 1 << 22)}
    if op == "step":
        return {"op": op, "n": _log(rng, 1 << 16, 1 << 27)}
    if op == "lag":
        return {"op": op, "n": _log(rng, 1 << 10, 1 << 26), "dtype": rng.choice(["f32", "bf16", "f16"]), "acc": acc}
    if op == "half":
        return {"op": op, "n": _log(rng, 1 << 16, 1 << 28), "dtype": rng.choice(["bf16", "f16"]), "acc": acc}
    if op == "gemv":
        m = _log(rng, 8, 1 << 16)
        n = min(_log(rng, 64, 1 << 20), (1 << 28) // m)
        if rng.random() < 0.5:              # half of the matrices have rows of whole 16-byte vectors
            n = max(64, n // 8 * 8)
        return {"op": op, "m": m, "n": n, "dtype": rng.choice(["f32", "bf16", "f16"]), "acc": acc}
    if op == "batch":
        return {"op": op, "n_red": _log(rng, 16, 2048), "n_gemv": _log(rng, 4, 100), "hi_exp": rng.choice([12.0, 16.0, 20.0]),
                "mn_hi": rng.choice([256, 1024, 4096]), "dtype": rng.choice(["f32", "bf16"]), "shapes": rng.randrange(1 << 20)}
    if op == "bs":
        return {"op": op, "n": _log(rng, 1 << 10, 1 << 25)}
    return {"op": "md", "nx": rng.randint(8, 128), "ny": rng.randint(8, 128), "nz": rng.randint(8, 64),
            "shuffle": rng.random() < 0.5}


# ---------------------------------------------------------------- inputs


def _gen(seed):
    g = torch.Generator(DEV)
    g.manual_seed(seed)
    return g


def _uniform(n, g, dtype="f32"):
    x = torch.rand(n, generator=g, device=DEV).mul_(2).sub_(1)
    return x.to(DTYPE[dtype])


def _normal(shape, g, dtype="f32"):
    return torch.randn(shape, generator=g, device=DEV).to(DTYPE[dtype])


def _batch_shapes(case):
    """(kind, n) of the reductions and (m, n) of the gemv problems: lengths
    log-uniform from 2^8, kinds alternating, m and n uniform from 64."""
    r = random.Random(case["shapes"])
    reds = [("dot" if i % 2 == 0 else "asum", int(2.0 ** r.uniform(8.0, case["hi_exp"]))) for i in range(case["n_red"])]
    gemvs = [(r.randint(64, case["mn_hi"]), r.randint(64, case["mn_hi"])) for _ in range(case["n_gemv"])]
    return reds, gemvs


def _batch_inputs(case, seed):
    """One buffer per kind of operand, every problem's part starting on a
    64-element boundary (as separate allocations would be aligned)."""
    reds, gemvs = _batch_shapes(case)
    up = lambda v: (v + 63) // 64 * 64
    g = _gen(seed)
    red_at, at = [], 0
    for kind, n in reds:
        y = at + up(n)
        red_at.append((at, y))
        at = y + (up(n) if kind == "dot" else 0)
    v = _uniform(max(at, 1), g, case["dtype"])
    a_at, x_at, y_at, a, x, y = [], [], [], 0, 0, 0
    for m, n in gemvs:
        a_at.append(a)
        x_at.append(x)
        y_at.append(y)
        a, x, y = a + up(m * n), x + up(n), y + up(m)
    return {"v": v, "red_at": red_at, "A": _normal(max(a, 1), g, case["dtype"]), "x": _normal(max(x, 1), g),
            "y": _normal(max(y, 1), g), "a_at": a_at, "x_at": x_at, "y_at": y_at}


def _md_inputs(case, seed):
    """Particles on a jittered unit lattice with the neighbours within RLIST,
    nearest first, padded with -1 to SLOTS."""
    g = _gen(seed)
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    n = nx * ny * nz
    i = torch.arange(n, device=DEV)
    c = torch.stack([i // (ny * nz), i // nz % ny, i % nz], 1)
    jitter = torch.rand((n, 3), generator=g, device=DEV).mul_(0.2).sub_(0.1)
    where = c.to(torch.float32) + jitter
    perm = torch.randperm(n, generator=g, device=DEV) if case["shuffle"] else i      # new index of old particle
    r = int(math.ceil(RLIST))
    near = sorted((a * a + b * b + d * d, a, b, d) for a in range(-r, r + 1) for b in range(-r, r + 1)
                  for d in range(-r, r + 1) if 0 < a * a + b * b + d * d <= RLIST * RLIST)[:SLOTS]
    old = torch.empty_like(perm)
    old[perm] = i                                                                     # old index of new particle
    cx, cy, cz = c[old].unbind(1)
    nbr = torch.full((n, SLOTS), -1, dtype=torch.int32, device=DEV)
    for j, (_, a, b, d) in enumerate(near):
        x, y, z = cx + a, cy + b, cz + d
        ok = (x >= 0) & (x < nx) & (y >= 0) & (y < ny) & (z >= 0) & (z < nz)
        at = torch.where(ok, (x * ny + y) * nz + z, 0)
        nbr[:, j] = torch.where(ok, perm[at], -1).to(torch.int32)
    pos = torch.zeros((n, 4), device=DEV)
    pos[:, :3] = where[old]
    return pos, nbr


def _inputs(case, seed):
    op = case["op"]
    g = _gen(seed)
    if op in ("dot", "half"):
        return {"x": _uniform(case["n"], g, case["dtype"]), "y": _uniform(case["n"], g, case["dtype"])}
    if op == "graph":
        return {"x": [_uniform(case["n"], g) for _ in range(GRAPH_VECTORS)], "y": [_uniform(case["n"], g) for _ in range(GRAPH_VECTORS)]}
    if op == "step":
        return {"x": _uniform(case["n"], g), "y": _uniform(case["n"], g)}
    if op == "lag":
        return {"x": _uniform(case["n"], g, case["dtype"])}
    if op == "gemv":
        return {"A": _normal((case["m"], case["n"]), g, case["dtype"]), "x": _normal(case["n"], g), "y": _normal(case["m"], g)}
    if op == "batch":
        return _batch_inputs(case, seed)
    if op == "bs":
        return {"s": torch.rand(case["n"], generator=g, device=DEV).mul_(25).add_(5)}
    pos, nbr = _md_inputs(case, seed)
    return {"pos": pos, "nbr": nbr}


class _Batch:
    """A planned batch on its inputs (the handle goes with it)."""

    def __init__(self, case, d):
        reds, gemvs = _batch_shapes(case)
        eb = BYTES[case["dtype"]]
        self.inputs = d
        self.results = torch.zeros(len(reds), device=DEV)
        probs = (L.lift_problem * (len(reds) + len(gemvs)))()
        v, r = d["v"].data_ptr(), self.results.data_ptr()
        for i, ((kind, n), (x, y)) in enumerate(zip(reds, d["red_at"])):
            p = probs[i]
            p.kind, p.n, p.a, p.out = (L.LIFT_KIND_DOT if kind == "dot" else L.LIFT_KIND_ASUM), n, v + x * eb, r + 4 * i
            if kind == "dot":
                p.b = v + y * eb
        a, x, y = d["A"].data_ptr(), d["x"].data_ptr(), d["y"].data_ptr()
        for i, (m, n) in enumerate(gemvs):
            p = probs[len(reds) + i]
            p.kind, p.m, p.n, p.lda = L.LIFT_KIND_GEMV, m, n, n
            p.a, p.b, p.out = a + d["a_at"][i] * eb, x + d["x_at"][i] * 4, y + d["y_at"][i] * 4
            p.alpha, p.beta = GEMV_ALPHA, GEMV_BETA
        self.handle = ctypes.c_void_p()
        status = L.lift_batch_create(probs, len(probs), CODE[case["dtype"]], L.ACC["f32"], L.LIFT_F32, None, self.handle)
        if status != L.LIFT_OK:
            raise L.LiftError(status, "lift_batch_create")

    def __del__(self):
        if self.handle:
            L.lift_batch_destroy(self.handle)
            self.handle = None


def prepare(case, seed):
    d = _inputs(case, seed)
    op = case["op"]
    state = {"case": case, "in": d}
    if op == "step":
        state["out"] = torch.empty_like(d["x"])
    elif op == "bs":
        state["out"] = torch.empty((case["n"], 2), device=DEV)
    elif op == "md":
        state["out"] = torch.empty_like(d["pos"])
    elif op == "batch":
        state["batch"] = _Batch(case, d)
    elif op == "graph":
        out = [torch.empty_like(x) for x in d["x"]]
        stream = torch.cuda.Stream(device=DEV)
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            L.asum(d["x"][0])               # the stream's workspace exists before the capture
            stream.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                res = []
                for x, y, o in zip(d["x"], d["y"], out):
                    L.scal(ALPHA, x, out=o)
                    res += [L.asum(x), L.dot(x, y)]
        torch.cuda.current_stream().wait_stream(stream)
        state.update(graph=graph, outs={"scal": out, "sums": res})
    return state


def run(state):
    case, d = state["case"], state["in"]
    op = case["op"]
    if op == "dot":
        return L.dot(d["x"], d["y"], acc=case["acc"])
    if op == "graph":
        state["graph"].replay()
        return state["outs"]
    if op == "step":
        L.scal(ALPHA, d["x"], out=state["out"])
        return state["out"], L.asum(d["x"]), L.dot(d["x"], d["y"])
    if op == "lag":
        x = d["x"]
        return L.asum(x[1:], acc=case["acc"]), L.dot(x[1:], x[:-1], acc=case["acc"])
    if op == "half":
        return (L.asum(d["x"], acc=case["acc"], result_dtype=torch.float64),
                L.dot(d["x"], d["y"], acc=case["acc"], result_dtype=torch.float64))
    if op == "gemv":
        return L.gemv(GEMV_ALPHA, d["A"], d["x"], GEMV_BETA, d["y"], acc=case["acc"])
    if op == "batch":
        b = state["batch"]
        status = L.lift_batch_run(b.handle, torch.cuda.current_stream().cuda_stream)
        if status != L.LIFT_OK:
            raise L.LiftError(status, "lift_batch_run")
        return {"results": b.results, "y": d["y"]}
    if op == "bs":
        return L.blackscholes(d["s"], STRIKE, RATE, VOLATILITY, YEARS, out=state["out"])
    return L.md(d["pos"], d["nbr"], CUTOFF, EPSILON, SIGMA, out=state["out"])


# ---------------------------------------------------------------- work and exact results


def work(case):
    op = case["op"]
    if op in ("dot", "half", "lag"):
        n, eb = case["n"], BYTES[case["dtype"]]
        if op == "dot":
            return {"bytes": 2 * n * eb, "flops": 2 * n}
        if op == "half":
            return {"bytes": 2 * n * eb, "flops": 4 * n}     # x read once for both
        return {"bytes": n * eb, "flops": 4 * n}
    if op == "graph":
        return {"bytes": GRAPH_VECTORS * 12 * case["n"], "flops": GRAPH_VECTORS * 5 * case["n"]}
    if op == "step":
        return {"bytes": 12 * case["n"], "flops": 5 * case["n"]}
    if op == "gemv":
        m, n = case["m"], case["n"]
        return {"bytes": m * n * BYTES[case["dtype"]] + 4 * n + 8 * m, "flops": 2 * m * n}
    if op == "batch":
        reds, gemvs = _batch_shapes(case)
        eb = BYTES[case["dtype"]]
        nbytes = sum(n * eb * (2 if k == "dot" else 1) + 4 for k, n in reds) + sum(m * n * eb + 4 * n + 8 * m for m, n in gemvs)
        return {"bytes": nbytes, "flops": 2 * sum(n for _, n in reds) + 2 * sum(m * n for m, n in gemvs)}
    if op == "bs":
        return {"bytes": 12 * case["n"], "flops": 60 * case["n"]}
    n = case["nx"] * case["ny"] * case["nz"]
    return {"bytes": n * (4 * SLOTS + 32), "flops": 20 * n * 90}


def _dot64(x, y):
    """x . y in binary64, a part at a time."""
    return sum((a.double() * b.double()).sum() for a, b in zip(x.split(1 << 26), y.split(1 << 26)))


def _asum64(x):
    return sum(a.double().abs().sum() for a in x.split(1 << 26))


def _gemv64(A, x, y):
    z = torch.cat([(a.double() * x.double()).sum(1) for a in A.split(max(1, (1 << 27) // A.shape[1]))])
    return GEMV_ALPHA * z + GEMV_BETA * y.double()


def _bs64(s):
    s = s.double()
    d1 = (torch.log(s / STRIKE) + (RATE + VOLATILITY * VOLATILITY / 2) * YEARS) / (VOLATILITY * math.sqrt(YEARS))
    d2 = d1 - VOLATILITY * math.sqrt(YEARS)
    cdf = lambda d: torch.erfc(-d / math.sqrt(2.0)) / 2
    k = STRIKE * math.exp(-RATE * YEARS)
    return torch.stack([s * cdf(d1) - k * cdf(d2), k * cdf(-d2) - s * cdf(-d1)], 1)


def _md64(pos, nbr):
    n = pos.shape[0]
    p = pos[:, :3].double()
    force = torch.zeros((n, 4), dtype=torch.float64, device=pos.device)
    for lo in range(0, n, 1 << 16):
        ids = nbr[lo:lo + (1 << 16)].long()
        used = (ids >= 0) & (ids < n)
        d = p[lo:lo + (1 << 16), None, :] - p[torch.where(used, ids, 0)]
        r2 = (d * d).sum(2)
        used &= r2 < CUTOFF * CUTOFF
        r2 = torch.where(used, r2, 1.0)
        s6 = (SIGMA * SIGMA / r2) ** 3
        f = torch.where(used, 24 * EPSILON / r2 * (2 * s6 * s6 - s6), 0.0)
        force[lo:lo + (1 << 16), :3] = (f[:, :, None] * d).sum(1)
    return force


def exact(case, seed):
    d = _inputs(case, seed)
    op = case["op"]
    if op == "dot":
        return _dot64(d["x"], d["y"])
    if op == "graph":
        return {"scal": [ALPHA * x.double() for x in d["x"]],
                "sums": [r for x, y in zip(d["x"], d["y"]) for r in (_asum64(x), _dot64(x, y))]}
    if op == "step":
        return ALPHA * d["x"].double(), _asum64(d["x"]), _dot64(d["x"], d["y"])
    if op == "lag":
        x = d["x"]
        return _asum64(x[1:]), _dot64(x[1:], x[:-1])
    if op == "half":
        return _asum64(d["x"]), _dot64(d["x"], d["y"])
    if op == "gemv":
        return _gemv64(d["A"], d["x"], d["y"])
    if op == "batch":
        reds, gemvs = _batch_shapes(case)
        v = d["v"]
        res = [_dot64(v[x:x + n], v[y:y + n]) if k == "dot" else _asum64(v[x:x + n])
               for (k, n), (x, y) in zip(reds, d["red_at"])]
        out = d["y"].double()               # what lies between two problems' rows stays as it was
        for (m, n), a, x, y in zip(gemvs, d["a_at"], d["x_at"], d["y_at"]):
            out[y:y + m] = _gemv64(d["A"][a:a + m * n].view(m, n), d["x"][x:x + n], d["y"][y:y + m])
        return {"results": torch.stack(res), "y": out}
    if op == "bs":
        return _bs64(d["s"])
    return _md64(d["pos"], d["nbr"])
