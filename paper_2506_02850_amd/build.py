"""Builds libmetok.so (HIP, gfx950) with hipcc and the module _host (the native part of binding.py, for this interpreter and torch)
with g++, in-tree.  Run as `python -m paper_2506_02850_amd.build`."""
from __future__ import annotations

import glob
import os
import shutil
import subprocess
import sys
import sysconfig
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmetok.so")
HOST = os.path.join(HERE, "_host" + sysconfig.get_config_var("EXT_SUFFIX"))
SOURCES = ["core.hip", "stage1.hip", "stage2.hip", "stage3.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument"]


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found; the METok library can only be built with ROCm")
    return exe


def host_commands(obj: str, target: str) -> list:
    """Compiles host.cpp against this interpreter and its torch, and links it against libmetok.so beside it."""
    import torch
    from torch.utils.cpp_extension import include_paths, library_paths

    inc = ["-I" + p for p in (os.path.join(ROOT, "include"), sysconfig.get_paths()["include"])]
    inc += [x for p in include_paths() for x in ("-isystem", p)]
    defines = ["-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), '-DMETOK_TORCH_VERSION="%s"' % torch.__version__]
    return [["g++", "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", *defines, *inc, "-c", os.path.join(CSRC, "host.cpp"), "-o", obj],
            ["g++", "-shared", "-fPIC", "-o", target, obj, "-L" + HERE, "-l:libmetok.so", "-Wl,-rpath,$ORIGIN", "-L" + library_paths()[0],
             "-ltorch_python", "-ltorch_cpu", "-lc10"]]


def build_host(target: str = HOST) -> str:
    """Builds the native part of binding.py.  The library and binding.py work without it (each call then spends more host time
    in Python), so that a machine without g++ or torch's headers gets a message instead of no build.  Returns that message, or ""."""
    try:
        with tempfile.TemporaryDirectory() as tmp:
            for cmd in host_commands(os.path.join(tmp, "host.o"), target):
                p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
                if p.returncode != 0:
                    return p.stdout or f"{cmd[0]} failed"
    except (ImportError, OSError) as e:
        return str(e)
    return ""


def build(verbose: bool = True) -> str:
    objs = []
    build_dir = os.path.join(HERE, "_build")
    os.makedirs(build_dir, exist_ok=True)
    procs = []
    for src in SOURCES:
        obj = os.path.join(build_dir, src.replace(".hip", ".o"))
        cmd = [hipcc(), *FLAGS, "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-c", os.path.join(CSRC, src), "-o", obj]
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l and l.strip())
        if p.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{out}")
        if verbose and out:
            print(out)
    for old in glob.glob(os.path.join(HERE, "_host*.so")):          # linked against the library of before
        os.remove(old)
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    subprocess.run(cmd, check=True)
    failed = build_host()
    if failed:
        print(f"{os.path.basename(HOST)} was not built, calls go through ctypes:\n{failed}", file=sys.stderr)
    if verbose:
        print("built", LIB, "" if failed else "and " + os.path.basename(HOST))
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
