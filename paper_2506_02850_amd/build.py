"""Builds libmetok.so (HIP, gfx950) with hipcc and _host.so (the native part of binding.py) with g++, in-tree.  Run as `python -m paper_2506_02850_amd.build`."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmetok.so")
HOST = os.path.join(HERE, "_host.so")
SOURCES = ["core.hip", "stage1.hip", "stage2.hip", "stage3.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument"]


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found; the METok library can only be built with ROCm")
    return exe


def host_command(obj: str) -> list:
    """Compiles host.cpp against this interpreter and its torch."""
    import sysconfig

    import torch
    from torch.utils.cpp_extension import include_paths

    inc = ["-I" + p for p in (os.path.join(ROOT, "include"), sysconfig.get_paths()["include"])]
    inc += [x for p in include_paths() for x in ("-isystem", p)]
    abi = "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI)
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", abi, *inc, "-c", os.path.join(CSRC, "host.cpp"), "-o", obj]


def build(verbose: bool = True) -> str:
    from torch.utils.cpp_extension import library_paths

    objs = []
    build_dir = os.path.join(HERE, "_build")
    os.makedirs(build_dir, exist_ok=True)
    procs = []
    for src in SOURCES:
        obj = os.path.join(build_dir, src.replace(".hip", ".o"))
        cmd = [hipcc(), *FLAGS, "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-c", os.path.join(CSRC, src), "-o", obj]
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    host_obj = os.path.join(build_dir, "host.o")
    procs.append(("host.cpp", subprocess.Popen(host_command(host_obj), stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l and l.strip())
        if p.returncode != 0:
            raise RuntimeError(f"the compiler failed on {src}:\n{out}")
        if verbose and out:
            print(out)
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    subprocess.run(cmd, check=True)
    torch_lib = library_paths()[0]
    subprocess.run(["g++", "-shared", "-fPIC", "-o", HOST, host_obj, "-L" + HERE, "-l:libmetok.so", "-Wl,-rpath,$ORIGIN", "-L" + torch_lib,
                    "-ltorch_python", "-ltorch_cpu", "-lc10"], check=True)
    if verbose:
        print("built", LIB, "and", os.path.basename(HOST))
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
