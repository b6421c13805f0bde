"""Compiles pieces of the kernel templates' shared prologue (csrc/templates/common.hip) for the host, so that a test calls the code the kernels
run and not a copy of it."""
import ctypes
import os
import re
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "clang++")
STUBS = """#define __device__
#define __host__
#define __forceinline__ inline
static struct { int x, y, z; } blockIdx;
static inline int min(int a, int b) { return a < b ? a : b; }
"""


def compile_common(defines, functions):
    """defines: the text of opevo_kernel_defines (or -D options alone); functions: C++ with extern "C" functions over what common.hip
    declares.  Returns the loaded library."""
    options = defines.split(":", 1)[-1].split()
    macros = "".join("#define %s %s\n" % m.groups() for m in (re.match(r"-D(\w+)=(\S+)$", o) for o in options) if m)
    common = open(os.path.join(ROOT, "paper_2006_05664_amd", "csrc", "templates", "common.hip")).read()
    with tempfile.TemporaryDirectory() as d:
        src, lib = os.path.join(d, "t.cpp"), os.path.join(d, "t.so")
        with open(src, "w") as fh:
            fh.write(STUBS + macros + common + functions)
        subprocess.run([CLANG, "-std=c++17", "-O1", "-w", "-shared", "-fPIC", src, "-o", lib], check=True)
        return ctypes.CDLL(lib)
