"""Build ``liblift.so`` (gfx950) in-tree with hipcc.

``python -m paper_1502_02389_amd.build`` compiles every translation unit under
``csrc/`` in parallel into ``_build/`` and links the shared library next to
this file; that takes hipcc alone.  Where torch, Python's headers and a C++
compiler are there too, the binding's native route (``_tensor_calls.so``) is
built beside it; without it the tensor calls take the binding's own, slower
code.  All device code is compiled with packed-FP32 instructions
disabled and without floating-point contraction (fma is written explicitly
where the arithmetic wants it).

Before compiling, the autotuner's cache (``tuning.json``) is turned into a
C table (``_build/lift_tuned_table.inc``) of knob sets keyed by device
architecture, compute-unit count, op, storage, accumulation and log2 size
bucket; the library uses an entry when a call passes no knobs and runs on a
device of that architecture and CU count.
"""
from __future__ import annotations

import concurrent.futures as cf
import json
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "liblift.so")
TUNING = os.path.join(HERE, "tuning.json")
TUNED_INC = os.path.join(BUILD, "lift_tuned_table.inc")
ARCH = "gfx950"

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CFLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}", f"-I{BUILD}",
]

# op names of the tuning cache -> the library's tuned-op codes (lift_api.cpp)
TUNED_OPS = {"scal": 0, "asum": 1, "dot": 2, "gemv": 3, "batch": 4, "blackscholes": 5, "md": 6}
TUNED_STORAGE = {"f32": 0, "bf16": 1, "f16": 2}
TUNED_ACC = {"f32": 0, "comp": 1, "f64combine": 2}
KNOB_FIELDS = ("block", "vec_bytes", "unroll", "rows_per_wave", "split", "wg_per_cu", "row_split",
               "lanes_per_item", "interleave", "lane_form")


def tuned_table_rows(path: str = TUNING):
    """(arch, cus, op, storage, acc, bucket, row bucket, knob tuple) for every
    cache entry (row bucket -1 = any: every op but gemv), or [] when the cache
    is missing or records no device architecture."""
    try:
        with open(path) as f:
            data = json.load(f)
    except (OSError, ValueError):
        return []
    dev = data.get("device") or {}
    arch, cus = dev.get("arch"), dev.get("cus")
    if not isinstance(arch, str) or not arch.isalnum() or not isinstance(cus, int):
        return []
    rows = []
    for key, ent in sorted(data.get("entries", {}).items()):
        parts = key.split("/")
        op, storage, acc, bucket = parts[:4]
        if (op == "gemv") != (len(parts) == 5) or len(parts) not in (4, 5):
            raise ValueError(f"tuning entry {key}: expected op/storage/acc/bucket (gemv: /row bucket)")
        row_bucket = int(parts[4]) if op == "gemv" else -1
        kn = ent["knobs"]
        unknown = set(kn) - set(KNOB_FIELDS)
        if unknown:
            raise ValueError(f"tuning entry {key}: unknown knobs {sorted(unknown)}")
        rows.append((arch, cus, TUNED_OPS[op], TUNED_STORAGE[storage], TUNED_ACC[acc], int(bucket), row_bucket,
                     tuple(int(kn.get(f, 0)) for f in KNOB_FIELDS)))
    return rows


def write_tuned_table(path: str = TUNING, out: str = TUNED_INC) -> int:
    """Write the C initialisers of the tuned table; returns the entry count."""
    rows = tuned_table_rows(path)
    lines = ["// generated by paper_1502_02389_amd/build.py from tuning.json; do not edit",
             "// {arch, cus, op, storage, acc, log2 bucket, log2 row bucket (-1: any), {block, vec_bytes, unroll,",
             "//  rows_per_wave, split, wg_per_cu, row_split, lanes_per_item, interleave, lane_form}}"]
    for arch, cus, op, st, acc, bucket, row_bucket, k in rows:
        lines.append(f'{{"{arch}", {cus}, {op}, {st}, {acc}, {bucket}, {row_bucket}, '
                     f'{{{k[0]}, {k[1]}, {k[2]}, {k[3]}, {k[4]}LL, {k[5]}, {k[6]}, {k[7]}, {k[8]}, {k[9]}}}}},')
    text = "\n".join(lines) + "\n"
    try:
        with open(out) as f:
            if f.read() == text:
                return len(rows)
    except OSError:
        pass
    with open(out, "w") as f:
        f.write(text)
    return len(rows)


# CPU sanitizer build (``--sanitize``): host code instrumented with
# AddressSanitizer and UndefinedBehaviorSanitizer, device code unchanged;
# a separate library (LIFT_LIB selects it for the binding), run on the CPU
# with the compiler's ASan runtime preloaded (see sanitizer_env()).
SAN_BUILD = os.path.join(HERE, "_build_san")
SAN_LIB = os.path.join(HERE, "liblift_san.so")
SAN_FLAGS = ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
             "-Xarch_host", "-fno-sanitize-recover=undefined", "-Xarch_host", "-fno-omit-frame-pointer", "-g"]


def asan_runtime() -> str:
    """The clang ASan runtime that instrumented host code needs preloaded."""
    r = subprocess.run([HIPCC, "--print-file-name=libclang_rt.asan-x86_64.so"], capture_output=True, text=True)
    path = r.stdout.strip()
    if r.returncode != 0 or not os.path.isabs(path) or not os.path.exists(path):
        raise RuntimeError("clang ASan runtime not found")
    return path


def sanitizer_env(oracle_lib: str | None = None) -> dict:
    """Environment for `pytest -m "not gpu"` against the sanitizer builds."""
    env = {"LD_PRELOAD": asan_runtime(), "LIFT_LIB": SAN_LIB,
           "ASAN_OPTIONS": "detect_leaks=0:halt_on_error=1:abort_on_error=1",
           "UBSAN_OPTIONS": "halt_on_error=1:print_stacktrace=1"}
    if oracle_lib:
        env["ORACLE_LIB"] = oracle_lib
    return env


# The binding's native route: host code only, against the installed torch.
TENSOR_CALLS = os.path.join(HERE, "_tensor_calls.so")
TENSOR_CALLS_SRC = "tensor_calls.cpp"


def sources():
    return sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".cpp")) and f != TENSOR_CALLS_SRC)


def build_tensor_calls() -> str:
    """Compile csrc/tensor_calls.cpp into _tensor_calls.so; returns its path."""
    import sysconfig

    import torch

    base = os.path.dirname(torch.__file__)
    tmp = TENSOR_CALLS + ".tmp"
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-fvisibility=hidden",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           f"-I{sysconfig.get_paths()['include']}", f"-I{base}/include", f"-I{base}/include/torch/csrc/api/include",
           os.path.join(CSRC, TENSOR_CALLS_SRC), "-o", tmp, f"-L{base}/lib", "-ltorch_python", "-ltorch_cpu", "-lc10"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed on {TENSOR_CALLS_SRC}:\n{r.stderr}")
    os.replace(tmp, TENSOR_CALLS)
    return TENSOR_CALLS


def native_route() -> str | None:
    """The native route, or None if it cannot be built here: that is reported,
    and none of an earlier build is left behind."""
    try:
        return build_tensor_calls()
    except Exception as e:   # no torch, no headers, no compiler, or it refuses the source
        if os.path.exists(TENSOR_CALLS):
            os.remove(TENSOR_CALLS)
        print(f"{os.path.basename(TENSOR_CALLS)} is not built, the tensor calls go without it: {e}", file=sys.stderr)
        return None


def _compile(src: str, sanitize: bool = False) -> str:
    obj = os.path.join(SAN_BUILD if sanitize else BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *CFLAGS, *(SAN_FLAGS if sanitize else []), "-c", os.path.join(CSRC, src), "-o", obj]
    if src.endswith(".cpp"):
        cmd[1:1] = ["-x", "hip"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr}")
    return obj


def build(jobs: int | None = None, verbose: bool = False, sanitize: bool = False) -> str:
    """Compile all sources and link liblift.so (with ``sanitize``, the host
    code instrumented, into liblift_san.so); returns the library path."""
    os.makedirs(BUILD, exist_ok=True)
    tuned = write_tuned_table()
    if sanitize:
        os.makedirs(SAN_BUILD, exist_ok=True)
    lib = SAN_LIB if sanitize else LIB
    srcs = sources()
    jobs = jobs or min(len(srcs), max(1, min(os.cpu_count() or 1, 16)))
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        if not sanitize:
            ex.submit(native_route)
        objs = list(ex.map(lambda f: _compile(f, sanitize), srcs))
    tmp = lib + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, lib)
    if verbose:
        print(f"built {lib} from {len(srcs)} sources ({tuned} tuned entries)", file=sys.stderr)
    return lib


def clean():
    for d in (BUILD, SAN_BUILD):
        shutil.rmtree(d, ignore_errors=True)
    for f in (LIB, SAN_LIB, TENSOR_CALLS):
        if os.path.exists(f):
            os.remove(f)


if __name__ == "__main__":
    if "--sanitize" in sys.argv[1:]:
        build(verbose=True, sanitize=True)
        sys.path.insert(0, ROOT)
        import oracle

        env = sanitizer_env(oracle.build(force=True, sanitize=True))
        print(" ".join(f"{k}={v}" for k, v in env.items()) + ' python -m pytest tests -m "not gpu"')
    else:
        build(verbose=True)
