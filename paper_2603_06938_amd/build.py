"""Builds libswimba.so (HIP, gfx950 only) and the host-side module _native.so in-tree."""
from __future__ import annotations

import importlib.util
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libswimba.so")
NATIVE = os.path.join(HERE, "_native.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def _run(cmd, what, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("%s failed:\n%s\n%s" % (what, r.stdout, r.stderr))


def _compile_native(verbose):
    """Object file of csrc/native.cpp: host code against CPython and libtorch, no kernels."""
    from torch.utils import cpp_extension
    obj = os.path.join(OBJ, "native.o")
    inc = ["-I" + d for d in cpp_extension.include_paths(device_type="cuda")]
    _run(["g++", "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
          *inc, "-I" + sysconfig.get_paths()["include"], "-I", os.path.join(ROOT, "include"),
          "-c", os.path.join(CSRC, "native.cpp"), "-o", obj], "g++ native.cpp", verbose)
    return obj


def _link_native(obj, verbose):
    from torch.utils import cpp_extension
    tmp = NATIVE + ".tmp%d" % os.getpid()
    _run(["g++", "-shared", "-o", tmp, obj, *("-L" + d for d in cpp_extension.library_paths(device_type="cuda")),
          "-L" + HERE, "-l:libswimba.so", "-ltorch_python", "-ltorch", "-ltorch_cpu", "-ltorch_hip", "-lc10", "-lc10_hip",
          "-Wl,-rpath,$ORIGIN"], "linking _native.so", verbose)
    os.replace(tmp, NATIVE)


def build(verbose: bool = False) -> str:
    """Compile every .hip under csrc/ and link the shared library; then the host-side module on top of it.

    The C library needs nothing from torch: it is in place before the module is waited for, and where torch is not
    installed it is all there is to build."""
    os.makedirs(OBJ, exist_ok=True)
    srcs = sources()

    def cc(src):
        obj = os.path.join(OBJ, os.path.basename(src)[:-4] + ".o")
        cmd = [HIPCC, *FLAGS, "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed on %s:\n%s\n%s" % (src, r.stdout, r.stderr))
        msgs = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
        if verbose and msgs.strip():
            print(msgs, flush=True)
        return obj

    with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        native = ex.submit(_compile_native, verbose) if importlib.util.find_spec("torch") else None
        objs = list(ex.map(cc, srcs))
    tmp = LIB + ".tmp%d" % os.getpid()
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (r.stdout, r.stderr))
    os.replace(tmp, LIB)
    if native is None:
        print("torch is not installed: no Python module, libswimba.so only", file=sys.stderr)
    else:
        _link_native(native.result(), verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
