"""Builds the library's host-only headers (csrc/score_plan.h, csrc/stage1_plan.h) behind C functions for ctypes."""
import ctypes
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@functools.lru_cache(None)
def host_library(source):
    with tempfile.TemporaryDirectory() as tmp:
        src, so = os.path.join(tmp, "plan.cpp"), os.path.join(tmp, "plan.so")
        with open(src, "w") as f:
            f.write(source)
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I" + os.path.join(ROOT, "include"),
                        "-I" + os.path.join(ROOT, "paper_2506_02850_amd", "csrc"), src, "-o", so], check=True)
        return ctypes.CDLL(so)
