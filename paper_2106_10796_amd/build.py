"""Build libcdsgd.so (HIP kernels + C ABI) for gfx950 with hipcc, and the binding's native calls, in-tree."""
import hashlib
import importlib.util
import os
import re
import shutil
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
SRC = os.path.join(PKG, "csrc", "cdsgd.hip")
SRC_HOST = [os.path.join(PKG, "csrc", "cdsgd_cost_model.cpp")]   # host-only parts of the library
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libcdsgd.so")
SRC_CALLS = os.path.join(PKG, "csrc", "py_calls.cpp")            # host code against Python's and torch's headers
CALLS = os.path.join(PKG, "_calls.so")
CALLS_FLAGS = ["-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", "-DUSE_ROCM=1"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # IEEE as written: no contraction of a*b+c behind our back (the fused
    # multiply-adds of the update rules are spelled out), denormals kept
    "-ffp-contract=off", "-fno-fast-math",
    # no packed-fp32 instructions from the auto-vectoriser
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # a kernel's first 14 words of arguments arrive in registers: one trip to memory less before its first load
    # (layer ranges of a million elements: 10.3 -> 9.9 us a launch)
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wall", "-Wno-unused-command-line-argument",
]


def hipcc_path() -> str:
    p = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(p):
        raise RuntimeError("hipcc not found")
    return p


def source_id(extra_flags=()) -> str:
    """Identity of what the library is made from: its sources, the headers and the flags (16 hex digits).
    It is compiled into the library (cdsgd_build_id) so that a library can be matched to the tree."""
    h = hashlib.sha256()
    headers = sorted(os.path.join(INCLUDE, f) for f in os.listdir(INCLUDE) if f.endswith(".h"))
    csrc = os.path.dirname(SRC)                       # cdsgd.hip includes the kernels' .hpp files beside it
    sources = sorted(os.path.join(csrc, f) for f in os.listdir(csrc) if f.endswith((".hip", ".hpp", ".cpp")))
    sources = [p for p in sources if os.path.basename(p) != os.path.basename(SRC_CALLS)]
    assert SRC in sources and all(p in sources for p in SRC_HOST)
    for path in [*sources, *headers]:
        h.update(os.path.basename(path).encode() + b"\0")
        with open(path, "rb") as fh:
            h.update(fh.read())
        h.update(b"\0")
    h.update(" ".join([*HIPCC_FLAGS, *extra_flags]).encode())
    return h.hexdigest()[:16]


def _torch_dir():
    spec = importlib.util.find_spec("torch")
    if spec is None or not spec.submodule_search_locations:
        raise RuntimeError("torch is not installed")
    return spec.submodule_search_locations[0]


def _torch_version() -> str:
    """torch.__version__, without the import."""
    try:
        with open(os.path.join(_torch_dir(), "version.py")) as fh:
            m = re.search(r"^__version__ = ['\"](.*)['\"]", fh.read(), re.M)
    except (OSError, RuntimeError):
        return ""
    return m.group(1) if m else ""


def calls_for(library: str) -> tuple:
    """What the native calls are built for: a library (its identity), a torch and a Python."""
    return library, _torch_version(), sysconfig.get_config_var("SOABI") or ""


def calls_id(library=None) -> str:
    """Identity of the native calls, which also depend on what they are built for."""
    with open(SRC_CALLS, "rb") as fh:
        parts = [fh.read().decode(), " ".join(CALLS_FLAGS), *calls_for(library or source_id())]
    return hashlib.sha256("\0".join(parts).encode()).hexdigest()[:16]


def built_id(path=LIB):
    """The source identity a built library carries, or None (no library, or one without an identity)."""
    try:
        with open(path, "rb") as fh:
            m = re.search(rb"CDSGD_BUILD_ID=([0-9a-f]{16})", fh.read())
    except OSError:
        return None
    return m.group(1).decode() if m else None


def _compile(cmd, out, tmp, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("%s failed:\n%s" % (os.path.basename(cmd[0]), r.stdout))
    # the host pass does not know the packed-fp32 target feature: harmless
    log = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l and l.strip())
    if verbose and log:
        print(log, flush=True)
    os.replace(tmp, out)
    return out


def build(extra_flags=(), out=LIB, verbose=False) -> str:
    """The library, and beside it (the default place) the native calls where they can be built."""
    library = source_id(extra_flags)
    tmp = out + ".tmp%d" % os.getpid()
    _compile([hipcc_path(), *HIPCC_FLAGS, *extra_flags, '-DCDSGD_BUILD_ID_HEX="%s"' % library,
              "-I", INCLUDE, SRC, *SRC_HOST, "-o", tmp], out, tmp, verbose)
    if out == LIB:
        _build_calls_if_possible(library, verbose)
    return out


def build_calls(verbose=False, library=None) -> str:
    torch_dir = _torch_dir()
    tmp = CALLS + ".tmp%d" % os.getpid()
    made_for = ['-DCDSGD_CALLS_%s="%s"' % kv for kv in zip(("LIBRARY", "TORCH", "SOABI"), calls_for(library or source_id()))]
    return _compile([os.environ.get("CXX", "g++"), *CALLS_FLAGS, '-DCDSGD_BUILD_ID_HEX="%s"' % calls_id(library), *made_for,
                     "-I", INCLUDE, "-isystem", os.path.join(torch_dir, "include"),
                     "-isystem", sysconfig.get_paths()["include"], SRC_CALLS, "-L", os.path.join(torch_dir, "lib"),
                     "-ltorch_python", "-ltorch_cpu", "-lc10", "-o", tmp], CALLS, tmp, verbose)


def _build_calls_if_possible(library=None, verbose=False):
    """The binding does without the native calls (by ctypes, a microsecond or more slower a call), so a machine
    without a C++ compiler or without Python's or torch's headers still has a library it can use."""
    try:
        build_calls(verbose, library)
    except (OSError, RuntimeError) as e:
        print("the binding's native calls were not built, it will use ctypes: %s" % str(e).strip()[:400], file=sys.stderr, flush=True)


def ensure_built() -> str:
    """Build (the library, and the binding's native calls) if none is there or if the one that is there was made from other
    sources, headers or flags than the tree now holds (tests, the smoke check and the benchmark call this;
    the binding itself never builds).  The comparison is by content, not by
    file time, so a tree that was copied elsewhere together with its library is not rebuilt."""
    if not os.path.exists(LIB) or built_id(LIB) != source_id():
        return build()
    if built_id(CALLS) != calls_id():
        _build_calls_if_possible()
    return LIB


if __name__ == "__main__":
    print(build(extra_flags=sys.argv[1:], verbose=True))
