"""Build libkvl.so (HIP, gfx950) in-tree with hipcc.  Run as a module or call build()."""
from __future__ import annotations

import hashlib
import os
import subprocess
import sys
import sysconfig
import warnings

_HERE = os.path.dirname(os.path.abspath(__file__))
_ROOT = os.path.dirname(_HERE)
CSRC = os.path.join(_HERE, "csrc")
LIB = os.path.join(_HERE, "libkvl.so")
# for this interpreter alone: the module is laid out by its headers
NATIVE = os.path.join(_HERE, "_native" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))
NATIVE_SOURCES = [os.path.join(_ROOT, "include", "kvl.h"), os.path.join(CSRC, "kvl_python.cpp")]
SOURCES = ["kvl_plan.hip", "kvl_kernels.hip", "kvl_h2d.hip", "kvl_stream.hip", "kvl_noalloc.hip", "kvl_sched.cpp"]


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    return "hipcc"


def native_key() -> str:
    """What the binding's module is built from (its marker is in the built file)."""
    digest = hashlib.sha256()
    for path in NATIVE_SOURCES:
        with open(path, "rb") as f:
            digest.update(f.read())
    return "kvl-native-" + digest.hexdigest()[:24]


def native_is_current() -> bool:
    """Whether the binding's module is there and was built from the present sources (found without loading it)."""
    if not os.path.exists(NATIVE):
        return False
    if not all(os.path.exists(path) for path in NATIVE_SOURCES):
        return True             # nothing to compare it with
    with open(NATIVE, "rb") as f:
        return native_key().encode() in f.read()


def build_native(verbose: bool = False) -> str:
    """Compile the module with the per-layer calls of the binding (host code only; always rebuilds)."""
    tmp = NATIVE + f".tmp{os.getpid()}"
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra",
           "-Wno-missing-field-initializers", f'-DKVL_NATIVE_KEY="{native_key()}"', "-I" + os.path.join(_ROOT, "include"),
           "-I" + sysconfig.get_paths()["include"], os.path.join(CSRC, "kvl_python.cpp"), "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        if os.path.exists(tmp):
            os.unlink(tmp)
        raise RuntimeError("the binding's module does not compile:\n" + res.stderr)
    os.replace(tmp, NATIVE)
    return NATIVE


def build(verbose: bool = False) -> str:
    """Compile every source for gfx950 and link the shared library (always rebuilds)."""
    cmd = [hipcc(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-mllvm", "-amdgpu-kernarg-preload-count=14",       # scalar arguments of kernels in registers (see kvl_pack_quick_tile_kernel)
           "-Wall", "-Wextra", "-Wno-unused-command-line-argument",
           "-I" + os.path.join(_ROOT, "include"), "-I" + CSRC]
    cmd += [os.path.join(CSRC, s) for s in SOURCES]
    tmp = LIB + f".tmp{os.getpid()}"
    cmd += ["-o", tmp, "-Wl,-rpath,/opt/rocm/lib", "-Wl,--no-undefined"]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass does not know the packed-fp32 feature switch and says so; that is harmless
    noise = ("packed-fp32-ops' is not a recognized feature", "'-packed-fp32-ops' is not")
    err = "\n".join(l for l in res.stderr.splitlines() if not any(n in l for n in noise))
    if res.returncode != 0:
        if os.path.exists(tmp):
            os.unlink(tmp)
        raise RuntimeError("hipcc failed:\n" + err)
    if verbose and err.strip():
        print(err, file=sys.stderr)
    os.replace(tmp, LIB)
    # without a host compiler or Python's headers the binding marshals by ctypes alone
    try:
        build_native(verbose)
    except (OSError, RuntimeError) as e:
        warnings.warn(f"built without the module of the per-layer calls, which take twice as long on the host so: {e}", RuntimeWarning)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
