"""Build the C-ABI library ``libvecinfer.so`` for gfx950 with hipcc (in-tree)."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libvecinfer.so")
# the hot calls' argument checks, see csrc/fastcall.cpp; named after the interpreter it is built for, so that no other loads it
FASTCALL = os.path.join(HERE, "_fastcall" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))
SOURCES = ["api.hip", "merge.hip", "encode.hip", "calibrate.hip", "probe.hip", "decode_lut.hip", "decode_roles.hip"]
# the matrix-core attention kernels, compiled once for the calls without a residual window and once for those with one
MFMA_SOURCES = ["decode_mfma.hip", "decode_mfma_wide.hip", "decode_mfma_wide64.hip", "decode_mfma_tiled.hip"]

# Packed-fp32 VALU forms are switched off for the device pass: hipcc otherwise forms them
# from plain float code.
#
# Kernel-argument preloading: the leading scalar arguments of a kernel (up to 14 dwords) are placed
# in scalar registers by the command processor before a wavefront starts, so the attention and
# merge kernels issue their first memory requests without a trip to the argument buffer (1.4 us
# per kernel when that buffer is cold).  Code built this way still runs where the firmware does
# not preload: the kernel then enters through a short compatibility prologue that loads the same
# registers itself.
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-mllvm", "-amdgpu-kernarg-preload-count=16"]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    raise RuntimeError("hipcc not found")


def fastcall_command() -> list | None:
    """The host compiler's line for the Python module; None without Python's headers (the calls then go through ctypes)."""
    python = sysconfig.get_paths()["include"]
    if not os.path.exists(os.path.join(python, "Python.h")):
        return None
    import torch

    root = os.path.dirname(torch.__file__)
    return ["g++", "-O2", "-std=c++17", "-Wall", "-shared", "-fPIC", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}",
            "-isystem", os.path.join(root, "include"), "-isystem", os.path.join(root, "include/torch/csrc/api/include"), "-I", python,
            os.path.join(CSRC, "fastcall.cpp"), "-o", FASTCALL, "-L", os.path.join(root, "lib"), "-ltorch_python", "-ltorch",
            "-ltorch_cpu", "-lc10"]


def build_fastcall() -> None:
    """Compile the Python module.  The library does without it: where its compiler or torch's headers are missing or do not
    fit, a message says so and the calls go through ctypes."""
    for old in {FASTCALL, os.path.join(HERE, "_fastcall.so")}:       # (what earlier builds made, any interpreter loads the latter)
        if os.path.exists(old):
            os.remove(old)
    why = "no Python headers"
    try:
        cmd = fastcall_command()
        if cmd:
            r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
            if r.returncode == 0:
                return
            why = r.stdout
    except (ImportError, OSError) as e:        # no torch, no compiler
        why = str(e)
    print(f"{os.path.basename(FASTCALL)} is not built, calls go through ctypes: {why}", file=sys.stderr, flush=True)


def build(verbose: bool = False, extra_flags=()) -> str:
    """Compile every kernel source and link the shared library, then the Python module.  Always recompiles."""
    objs = []
    procs = []
    units = [(src, src, []) for src in SOURCES]
    for src in MFMA_SOURCES:
        units += [(src, src, ["-DVECINFER_WINDOW=0"]), (src, src.replace("decode_mfma", "decode_mfma_window"), ["-DVECINFER_WINDOW=1"])]
    for src, name, defines in units:
        obj = os.path.join(CSRC, name.replace(".hip", ".o"))
        cmd = [hipcc(), *FLAGS, *defines, *extra_flags, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    for src, pr in procs:
        out, _ = pr.communicate()
        # the host pass warns that it does not know the packed-fp32 feature: harmless
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l and l.strip())
        if pr.returncode != 0:
            raise RuntimeError(f"compiling {src} failed:\n{out}")
        if verbose and out:
            print(out, flush=True)
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    subprocess.run(cmd, check=True)
    build_fastcall()
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
