"""Build the C-ABI library ``libss_scan.so`` from ``csrc/`` with hipcc for gfx950, and then ``_marshal.so``, through which
the binding makes its hot calls, with the host compiler.  The library needs hipcc alone and is complete before the module is
begun, which is left out, with a note, where torch, the Python headers or g++ are missing.

The library is built in-tree (next to this file) so that it travels with the source
tree; nothing is compiled at import time.  ``build_microbench`` builds the stand-alone
ceilings program of ``microbench/`` the same way.
"""
import glob
import os
import shutil
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor

from . import isa_check

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libss_scan.so")
MARSHAL_SRC = os.path.join(CSRC, "ss_marshal.cpp")
MARSHAL = os.path.join(PKG, "_marshal.so")
BUILD_DIR = os.path.join(PKG, "_build")
MICROBENCH_SRC = os.path.join(PKG, "microbench", "ss_ceilings.hip")
MICROBENCH = os.path.join(PKG, "microbench", "ss_ceilings")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-munsafe-fp-atomics",                     # hardware float atomics, no CAS loops
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",  # no packed-FP32 VALU ops
    "-Wno-unused-command-line-argument",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _hipcc():
    return shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


def _run(cmd, cwd, verbose):
    res = subprocess.run(cmd, cwd=cwd, capture_output=True, text=True)
    if verbose or res.returncode != 0:
        print(res.stdout)
        print("\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l))
    if res.returncode != 0:
        raise RuntimeError("compiler failed: " + " ".join(cmd))


def device_assembly(directory=BUILD_DIR):
    """The device assembly that the compiler left there."""
    return sorted(glob.glob(os.path.join(directory, "*gfx950*.s")))


def _check_device_code(directory):
    """The device code must not contain what isa_check looks for."""
    for asm in device_assembly(directory):
        with open(asm) as f:
            found = isa_check.check(f.read())
        if found:
            raise RuntimeError("%s: %d findings, the first: %s" % (asm, len(found), found[0]))


def build_library(verbose=False, jobs=None):
    """Compile every .hip source (in parallel) and link libss_scan.so, then _marshal.so; returns the library's path."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    objs = []

    def compile_one(src):
        obj = os.path.join(BUILD_DIR, os.path.basename(src)[:-4] + ".o")
        _run([_hipcc()] + HIPCC_FLAGS + inc + ["-save-temps=obj", "-c", "-o", obj, src], BUILD_DIR, verbose)
        return obj

    with ThreadPoolExecutor(max_workers=jobs or min(8, os.cpu_count() or 1)) as pool:
        objs = list(pool.map(compile_one, sources()))
    _check_device_code(BUILD_DIR)
    out = os.path.join(BUILD_DIR, "libss_scan.so")
    _run([_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", out] + objs, BUILD_DIR, verbose)
    shutil.copy2(out, LIB)
    missing = build_marshal(verbose)
    if missing:
        print("%s is built; %s is not, for want of %s: the binding marshals all calls in Python" % (LIB, MARSHAL, missing))
    return LIB


def build_marshal(verbose=False):
    """Compile _marshal.so against the built library.  Returns what is missing for it, or None."""
    if os.path.exists(MARSHAL):
        os.remove(MARSHAL)   # one that is left behind must not call another library than it was built for
    try:
        from torch.utils import cpp_extension
    except ImportError:
        return "torch"
    python_inc = sysconfig.get_paths()["include"]
    if not os.path.exists(os.path.join(python_inc, "Python.h")):
        return "the Python headers"
    if not shutil.which("g++"):
        return "g++"
    obj, out = os.path.join(BUILD_DIR, "ss_marshal.o"), os.path.join(BUILD_DIR, "_marshal.so")
    inc = [a for d in cpp_extension.include_paths() + [python_inc, os.path.join(ROOT, "include")] for a in ("-isystem", d)]
    _run(["g++", "-O2", "-std=c++17", "-fPIC", "-c", "-o", obj, MARSHAL_SRC] + inc, BUILD_DIR, verbose)
    dirs = [a for d in cpp_extension.library_paths() for a in ("-L", d)]
    _run(["g++", "-shared", "-o", out, obj, "-L", os.path.dirname(LIB), "-lss_scan"] + dirs +
         ["-ltorch_python", "-ltorch_cpu", "-lc10", "-Wl,-rpath,$ORIGIN"], BUILD_DIR, verbose)
    shutil.copy2(out, MARSHAL)
    return None


def build_microbench(verbose=False):
    """Compile the stand-alone ceilings program (microbench/ss_ceilings); returns its path."""
    bdir = os.path.join(BUILD_DIR, "microbench")
    os.makedirs(bdir, exist_ok=True)
    out = os.path.join(bdir, "ss_ceilings")
    flags = [f for f in HIPCC_FLAGS if f != "-fPIC"]
    _run([_hipcc()] + flags + ["-save-temps=obj", "-o", out, MICROBENCH_SRC], bdir, verbose)
    _check_device_code(bdir)
    shutil.copy2(out, MICROBENCH)
    return MICROBENCH


if __name__ == "__main__":
    print(build_library(verbose=True))
    print(build_microbench(verbose=True))
