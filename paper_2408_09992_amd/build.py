"""Compile the HIP library (csrc/*.hip and the .hpp parts they include -> libpqtopk.so, in-tree) for gfx950, and the
Python entry points' marshalling (csrc/py_native.cpp, host code against torch's headers -> _pqnative.so).

The translation units are compiled side by side (the scan kernels are large: tens of seconds each) and linked
into one shared library.  `python -m paper_2408_09992_amd.build --library-only` builds that library alone, which needs
neither torch nor Python's headers; `--incremental` compiles only what is older than its sources."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

_HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(_HERE)
CSRC = os.path.join(_HERE, "csrc")
OBJ = os.path.join(_HERE, "_build")                              # object files (not tracked)
SOURCES = sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))
PUBLIC_HEADERS = sorted(os.path.join(ROOT, "include", f) for f in os.listdir(os.path.join(ROOT, "include")) if f.endswith(".h"))
HEADERS = PUBLIC_HEADERS + sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hpp"))
LIB = os.path.join(_HERE, "libpqtopk.so")
NATIVE_SOURCE = os.path.join(CSRC, "py_native.cpp")
NATIVE = os.path.join(_HERE, "_pqnative.so")
NATIVE_TORCH = os.path.join(_HERE, "_build", "native_torch.txt")   # the torch and the Python _pqnative.so was built against

# -packed-fp32-ops switches the packed FP32 instructions (v_pk_add_f32 and friends) off in the DEVICE code.  hipcc hands
# -Xclang options to its host pass as well, where the x86 back end answers with one line per function saying that it does
# not know the feature; those lines (and only those) are dropped from what the compiler prints.
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-ffp-contract=off",                                       # the kernels spell out every fused multiply-add
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # kernel arguments that are plain values arrive in scalar registers instead of being loaded by every wave first
    "-mllvm", "-amdgpu-kernarg-preload-count=14",
    "-Wall", "-Wno-unused-command-line-argument",
]
_HOST_PASS_NOISE = "'-packed-fp32-ops' is not a recognized feature for this target (ignoring feature)"


def _torch_identity() -> str:
    """What _pqnative.so has to match, or "" without torch."""
    try:
        import torch
    except ImportError:
        return ""
    return f"torch {torch.__version__}, python {sys.version_info[0]}.{sys.version_info[1]}\n"


def _native_is_stale() -> bool:
    identity = _torch_identity()
    if not identity:
        return False                                             # (nothing to build it against, and nothing that would load it)
    try:
        with open(NATIVE_TORCH) as f:
            if f.read() != identity:
                return True
        t = os.path.getmtime(NATIVE)
    except OSError:
        return True
    return any(os.path.getmtime(p) > t for p in PUBLIC_HEADERS + [NATIVE_SOURCE])


def _library_is_stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    return any(os.path.getmtime(p) > t for p in SOURCES + HEADERS)


def is_stale() -> bool:
    return _library_is_stale() or _native_is_stale()


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(line for line in r.stdout.splitlines() if _HOST_PASS_NOISE not in line)
    if out.strip():
        print(out, file=sys.stderr, flush=True)
    if r.returncode != 0:
        raise subprocess.CalledProcessError(r.returncode, cmd)


def _build_native(verbose):
    """_pqnative.so; linked after libpqtopk.so, which it finds beside itself."""
    identity = _torch_identity()
    if not identity:
        print("no torch: _pqnative.so, which only serves torch programs, is not built", file=sys.stderr, flush=True)
        return
    import torch
    root = os.path.dirname(os.path.abspath(torch.__file__))
    _run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
          f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I", os.path.join(ROOT, "include"),
          "-isystem", sysconfig.get_paths()["include"], "-isystem", os.path.join(root, "include"),
          "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"), "-isystem", "/opt/rocm/include",
          NATIVE_SOURCE, "-o", NATIVE, "-L", _HERE, "-lpqtopk", "-L", os.path.join(root, "lib"),
          "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_hip", "-ltorch_python", "-Wl,-rpath,$ORIGIN"], verbose)
    with open(NATIVE_TORCH, "w") as f:
        f.write(identity)


def build(force: bool = True, verbose: bool = False, jobs: int = 0, library_only: bool = False) -> str:
    """Run hipcc, then (unless `library_only`) the C++ compiler for the Python entry points.  Cross-compiles on a host without
    a GPU."""
    if force or _library_is_stale():
        _build_library(force, verbose, jobs)
    if not library_only and (force or _native_is_stale()):
        _build_native(verbose)
    return LIB


def _build_library(force: bool, verbose: bool, jobs: int) -> None:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ, exist_ok=True)
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    objs = [os.path.join(OBJ, os.path.basename(s)[:-4] + ".o") for s in SOURCES]
    newest_header = max(os.path.getmtime(h) for h in HEADERS)

    def compile_one(pair):
        src, obj = pair
        if not force and os.path.exists(obj) and os.path.getmtime(obj) > max(os.path.getmtime(src), newest_header):
            return
        _run([hipcc, *HIPCC_FLAGS, *inc, "-c", src, "-o", obj], verbose)

    jobs = jobs or min(len(SOURCES), max(1, min(int(os.environ.get("MAX_JOBS", "8")), os.cpu_count() or 1)))
    with ThreadPoolExecutor(max_workers=jobs) as pool:
        list(pool.map(compile_one, zip(SOURCES, objs)))
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs], verbose)


if __name__ == "__main__":
    print(build(force="--incremental" not in sys.argv, verbose=True, library_only="--library-only" in sys.argv))
