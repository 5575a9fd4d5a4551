"""Build the HIP library for gfx950 in-tree (``libfaser_verify.so`` next to this file)."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libfaser_verify.so")
SOURCES = ["attend_items.hip", "controller.hip", "greedy_accept.hip", "hbm_probe.hip", "kv_append.hip", "library.hip", "prune_compact.hip", "rank_check.hip", "spec_accept.hip", "verify_attention.hip"]
# packed fp32 ops are switched off on purpose (the compiler would otherwise form v_pk_*_f32)
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
         "-packed-fp32-ops", "-Wno-unused-command-line-argument"]


MARSHAL = os.path.join(HERE, "_marshal.so")


def marshal_command() -> list:
    """g++ line of the binding's host-only helper (no device code, no symbols of the HIP library)."""
    import torch

    root = os.path.dirname(torch.__file__)
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",  # what torch's headers and HIP's want to be told
            "-I", sysconfig.get_paths()["include"], "-isystem", "/opt/rocm/include", "-isystem", os.path.join(root, "include"),
            os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL, "-L", os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-ltorch_hip", "-lc10_hip", "-lc10",
            "-Wl,-rpath," + os.path.join(root, "lib")]


def build(verbose: bool = False) -> str:
    """Compile every source with hipcc and link the shared library, and the binding's helper.  Always recompiles."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs = []
    objs = []
    for src in SOURCES:
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        objs.append(obj)
        cmd = [hipcc] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    cmd = marshal_command()
    if verbose:
        print(" ".join(cmd), flush=True)
    procs.append(("marshal.cpp", subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for src, pr in procs:
        out, _ = pr.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l and l.strip())
        if pr.returncode != 0:
            raise RuntimeError(f"compiling {src} failed:\n{out}")
        if verbose and out:
            print(out)
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    subprocess.check_call(cmd)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
