"""Builds libhif8.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree.

Every .hip / .cpp file under csrc/ is one translation unit; they are compiled in parallel
into _build/ and linked into one shared library.  binding/native_call.cpp, the marshalling of Python arguments,
becomes an extension module of its own (g++, Python's and torch's headers), _native_call-*.so; the library does not need it.
"""
import glob
import hashlib
import os
import re
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJDIR = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libhif8.so")
NATIVE_SRC = os.path.join(PKG, "binding", "native_call.cpp")
NATIVE_INPUTS = [NATIVE_SRC, os.path.join(ROOT, "include", "hif8.h")]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.cpp")))


def headers():
    return sorted(glob.glob(os.path.join(CSRC, "*.hpp")) + glob.glob(os.path.join(ROOT, "include", "*.h")))


HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-fno-fast-math", "-ffp-contract=off", "-fhip-fp32-correctly-rounded-divide-sqrt",
    "-fno-gpu-flush-denormals-to-zero",
    # keep packed-FP32 instructions out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def native_path() -> str:
    """Where the extension module is for this torch and this Python, whose C++ and C interfaces it is compiled against, and for these sources; a module
    for others is not found, and so not loaded."""
    import torch
    digest = hashlib.sha256()
    for f in NATIVE_INPUTS:
        with open(f, "rb") as src:
            digest.update(src.read())
    kind = re.sub(r"[^\w.]", "_", "%s-%s" % (torch.__version__, sysconfig.get_config_var("SOABI")))
    return os.path.join(PKG, "_native_call-%s-%s.so" % (kind, digest.hexdigest()[:12]))


def build_native(force: bool = True, verbose: bool = False) -> str:
    """The extension module that hif8.py calls the library through."""
    path = native_path()
    if not force and os.path.exists(path):
        return path
    import torch
    from torch.utils import cpp_extension
    dirs = [os.path.join(ROOT, "include"), sysconfig.get_paths()["include"]] + cpp_extension.include_paths()
    tmp = path + ".tmp.%d" % os.getpid()
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI]
    for d in dirs:
        cmd += ["-isystem", d]
    cmd += [NATIVE_SRC, "-o", tmp]
    for d in cpp_extension.library_paths():
        cmd += ["-L", d]
    cmd += ["-ltorch_python", "-ltorch_cpu", "-lc10", "-ldl"]  # found by their names in a process that has imported torch
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed on %s:\n%s" % (NATIVE_SRC, r.stdout))
    os.replace(tmp, path)
    for old in glob.glob(glob.escape(path[:-len("-0123456789ab.so")]) + "-*.so"):  # of other sources
        if old != path:
            os.remove(old)
    return path


def is_stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    return any(os.path.getmtime(f) > t for f in sources() + headers())


def build(force: bool = True, verbose: bool = False, jobs: int = 8, native: bool = True) -> str:
    """The library and, if `native`, the extension module."""
    if not force and not is_stale():
        if native:
            build_native(False, verbose)
        return LIB
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJDIR, exist_ok=True)
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    hdr_time = max(os.path.getmtime(h) for h in headers())

    def compile_one(src):
        obj = os.path.join(OBJDIR, os.path.basename(src) + ".o")
        if (not force and os.path.exists(obj)
                and os.path.getmtime(obj) >= max(os.path.getmtime(src), hdr_time)):
            return obj
        lang = ["-x", "hip"] if src.endswith(".hip") else []
        cmd = [hipcc] + HIPCC_FLAGS + inc + ["-c"] + lang + [src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed on %s:\n%s" % (src, r.stdout))
        return obj

    with ThreadPoolExecutor(max_workers=jobs) as pool:
        extension = pool.submit(build_native, force, verbose) if native else None
        objs = list(pool.map(compile_one, sources()))
        if extension:
            extension.result()
    tmp = LIB + ".tmp.%d" % os.getpid()
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    import sys
    print(build(force="--incremental" not in sys.argv, verbose=True))
