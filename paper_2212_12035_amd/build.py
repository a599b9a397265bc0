"""Builds libharris.so for gfx950 with hipcc (cross-compiles without a GPU), and the native marshalling of the Python
binding (cbinding/harris_call.cpp, host code against torch's headers) with the host compiler.

Every source file is compiled to an object of its own, all at once, and the objects are linked
into paper_2212_12035_amd/libharris.so; the objects live in a build folder beside it.  The library needs hipcc
alone.  The binding's module is optional: without torch or a host compiler, or if it does not compile, a
warning says so, no module is left that belongs to another build, and the binding's Python code does its work.
"""
from __future__ import annotations

import glob
import os
import subprocess
import sysconfig
import warnings

_PKG = os.path.dirname(os.path.abspath(__file__))
_ROOT = os.path.dirname(_PKG)
CSRC = os.path.join(_PKG, "csrc")
LIB = os.path.join(_PKG, "libharris.so")
BUILD_DIR = os.path.join(_PKG, "_build")
NATIVE = os.path.join(_PKG, "_harris_call" + sysconfig.get_config_var("EXT_SUFFIX"))      # for this Python alone

SOURCES = ("harris_tiles_f32.hip", "harris_tiles_u8.hip", "harris_tiles_f32_words.hip", "harris_tiles_u8_words.hip",
           "harris_patches.hip", "harris_bands.hip", "harris_grouped.hip", "harris_copy.hip", "harris_launch.cpp", "harris_api.cpp")
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # the compiler must not form packed-FP32 instructions on its own
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I" + os.path.join(_ROOT, "include"), "-I" + CSRC,
]


class _NativeBuild:
    """The compilation of the binding's native marshalling, beside the library's."""

    def __init__(self):
        self.tmp, self.process, self.error = NATIVE + ".tmp.%d" % os.getpid(), None, None
        try:
            import torch
            base = os.path.dirname(os.path.abspath(torch.__file__))
            cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
                   '-DHARRIS_TORCH_VERSION="%s"' % torch.__version__,
                   "-I" + os.path.join(base, "include"), "-I" + os.path.join(base, "include", "torch", "csrc", "api", "include"),
                   "-I" + sysconfig.get_paths()["include"], "-I" + os.path.join(_ROOT, "include"), os.path.join(_PKG, "cbinding", "harris_call.cpp"),
                   "-L" + os.path.join(base, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-o", self.tmp]
            self.process = subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        except (ImportError, AttributeError, OSError) as e:
            self.error = str(e)

    def finish(self):
        """Waits, and puts the module where the binding finds it, instead of all others; or warns, and leaves none."""
        if self.process is not None:
            out, _ = self.process.communicate()
            if self.process.returncode != 0:
                self.error = out
        for old in glob.glob(os.path.join(os.path.dirname(NATIVE), "_harris_call*.so")):
            os.remove(old)
        if self.error is None:
            os.replace(self.tmp, NATIVE)
            return
        if os.path.exists(self.tmp):
            os.remove(self.tmp)
        warnings.warn("the binding's native marshalling is not built, its calls go through Python: " + self.error)


def build_library() -> str:
    """Compile and link the library, and the binding's native part where that can be; returns the library's path.
    Raises RuntimeError with the compiler's output if the library fails."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(BUILD_DIR, exist_ok=True)
    native = _NativeBuild()
    try:
        jobs = []
        for name in SOURCES:
            obj = os.path.join(BUILD_DIR, os.path.splitext(name)[0] + ".o")
            cmd = [hipcc, *HIPCC_FLAGS, "-c", os.path.join(CSRC, name), "-o", obj]
            jobs.append((name, obj, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        failed = []
        for name, obj, proc in jobs:
            out, _ = proc.communicate()
            if proc.returncode != 0:
                failed.append("%s:\n%s" % (name, out))
        if failed:
            raise RuntimeError("hipcc failed building libharris.so\n" + "\n".join(failed))
        tmp = LIB + ".tmp.%d" % os.getpid()
        link = subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *[obj for _, obj, _ in jobs], "-o", tmp],
                              capture_output=True, text=True)
        if link.returncode != 0:
            raise RuntimeError("hipcc failed linking libharris.so\n" + link.stdout + link.stderr)
        os.replace(tmp, LIB)
    finally:
        native.finish()
    return LIB


if __name__ == "__main__":
    print("built", build_library())
    sys.exit(0)
