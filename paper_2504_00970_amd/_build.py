"""Builds libsentencekv.so (gfx950) in-tree with hipcc, and the module that calls it from Python with the host compiler."""
from __future__ import annotations

import contextlib
import os
import shutil
import subprocess
import sysconfig
import warnings

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libsentencekv.so")
# profiling build (-DSKV_PHASE_STAMPS): the decode kernels record the wall clock at marked places, see csrc/skv_stamps.h;
# built by `python -m paper_2504_00970_amd._build --stamps`, loaded by `bench.py --phase-stamps`
LIB_STAMPS = os.path.join(HERE, "libsentencekv_stamps.so")
CALLS = os.path.join(HERE, "_calls.so")
SOURCES = ["api.hip", "prefill.hip", "decode.hip", "retain.hip"]
HEADERS = [os.path.join(CSRC, "skv_internal.h"), os.path.join(CSRC, "skv_device.h"), os.path.join(CSRC, "skv_stamps.h"),
           os.path.join(INCLUDE, "sentencekv.h")]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # packed fp32 instructions stay off: the compiler would otherwise form them from scalar float code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wextra", "-Wno-unused-command-line-argument",
]


def stale(lib: str = "") -> bool:
    lib = lib or LIB
    if not os.path.exists(lib):
        return True
    t = os.path.getmtime(lib)
    deps = [os.path.join(CSRC, s) for s in SOURCES] + HEADERS
    return any(os.path.getmtime(d) > t for d in deps)


def _calls_built_for() -> str:
    """What the call module depends on besides its source; the module carries it as a string."""
    import torch
    return f"libsentencekv calls for Python {sysconfig.get_python_version()}, torch {torch.__version__}"


def calls_fit() -> bool:
    """The call module is there and was built for this Python and this torch."""
    if not os.path.exists(CALLS):
        return False
    with open(CALLS, "rb") as f:
        return (_calls_built_for() + "\0").encode() in f.read()


def calls_stale() -> bool:
    if not calls_fit():
        return True
    t = os.path.getmtime(CALLS)
    return any(os.path.getmtime(d) > t for d in (os.path.join(CSRC, "calls.cpp"), os.path.join(INCLUDE, "sentencekv.h")))


def _host_compiler() -> str:
    return next((c for c in map(shutil.which, ("g++", "c++", "clang++", "amdclang++")) if c), "/opt/rocm/bin/amdclang++")


def _calls_command() -> list:
    import torch
    t = os.path.dirname(torch.__file__)
    return [_host_compiler(), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", f"-I{INCLUDE}", "-isystem", f"{t}/include",
            "-isystem", f"{t}/include/torch/csrc/api/include", "-isystem", sysconfig.get_paths()["include"],
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}", f'-DSKV_BUILT_FOR="{_calls_built_for()}"',
            os.path.join(CSRC, "calls.cpp"), "-o", CALLS + ".tmp", f"-L{t}/lib", "-ltorch_python", "-ltorch_cpu", "-lc10",
            f"-Wl,-rpath,{t}/lib"]


def _start(cmd: list, verbose: bool):
    if verbose:
        print(" ".join(cmd), flush=True)
    return subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)


def _finish_calls(proc) -> bool:
    """Puts the module that `proc` compiles in place.  Where it cannot be built (no host compiler, no Python headers) there is none, and the
    binding calls through ctypes."""
    out = str(proc) if isinstance(proc, OSError) else proc.communicate()[0]
    if isinstance(proc, OSError) or proc.returncode != 0:
        with contextlib.suppress(OSError):
            os.remove(CALLS)                          # one of an older source
        warnings.warn("the module for calls from Python was not built, they go through ctypes:\n" + out)
        return False
    os.replace(CALLS + ".tmp", CALLS)
    return True


def build_calls(verbose: bool = False) -> bool:
    """Compile the call module alone; False (and a warning) where that is not possible."""
    try:
        proc = _start(_calls_command(), verbose)
    except OSError as e:
        proc = e
    return _finish_calls(proc)


def build(force: bool = True, verbose: bool = False, stamps: bool = False) -> str:
    """Compile the library and the call module: one compiler process per source file, side by side, then one link.  With
    force=False up-to-date ones are kept.  stamps=True builds the profiling variant of the library (LIB_STAMPS) instead."""
    lib = LIB_STAMPS if stamps else LIB
    calls = None
    if not stamps and (force or calls_stale()):
        try:
            calls = _start(_calls_command(), verbose)
        except OSError as e:
            calls = e
    try:
        if force or stale(lib):
            _build_lib(lib, verbose, stamps)
    finally:
        if calls is not None:
            _finish_calls(calls)
    return lib


def _build_lib(lib: str, verbose: bool, stamps: bool) -> None:
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    objdir = os.path.join(HERE, "_build", "stamps" if stamps else "lib")
    os.makedirs(objdir, exist_ok=True)
    compile_flags = [f for f in HIPCC_FLAGS if f != "-shared"] + (["-DSKV_PHASE_STAMPS"] if stamps else [])
    jobs = []
    for src in SOURCES:
        obj = os.path.join(objdir, src + ".o")
        jobs.append((src, obj, _start([hipcc, *compile_flags, f"-I{INCLUDE}", f"-I{CSRC}", "-c", os.path.join(CSRC, src), "-o", obj], verbose)))
    failed = []
    for src, _, proc in jobs:
        out, _ = proc.communicate()
        if proc.returncode != 0:
            failed.append(f"{src}:\n{out}")
    if failed:
        raise RuntimeError("compilation failed:\n" + "\n".join(failed))
    proc = _start([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *[obj for _, obj, _ in jobs], "-o", lib + ".tmp"], verbose)
    out, _ = proc.communicate()
    if proc.returncode != 0:
        raise RuntimeError("link failed:\n" + out)
    os.replace(lib + ".tmp", lib)


if __name__ == "__main__":
    import sys
    print(build(force=True, verbose=True, stamps="--stamps" in sys.argv[1:]))
