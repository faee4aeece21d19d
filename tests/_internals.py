"""Values of a list that no entry point returns, read through the library's own header."""
import ctypes
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = """
#include "internal.h"
extern "C" long list_est_items(const nb_list *l) { return l->est_items; }
"""


def load(folder):
    """The reader, compiled into `folder` (host code only)."""
    src, so = os.path.join(folder, "internals.cpp"), os.path.join(folder, "internals.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(rocm, "include"),
                    "-I" + os.path.join(ROOT, "paper_1306_1737_amd", "csrc"), src, "-o", so], check=True)
    lib = ctypes.CDLL(so)
    lib.list_est_items.argtypes, lib.list_est_items.restype = [ctypes.c_void_p], ctypes.c_long
    return lib
