"""Builds liblookat.so (HIP, gfx950; hipcc) and _marshal.so (the binding's native marshalling; g++ against torch's headers)
in-tree.  `python -m paper_2601_10155_amd.build`."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "liblookat.so")
MARSHAL = os.path.join(PKG, "_marshal.so")
OBJ_DIR = os.path.join(PKG, "_build")

# -packed-fp32-ops off: keeps the compiler from forming packed fp32 instructions.
COMMON = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          # leading kernel arguments arrive in scalar registers at wave launch (no load round trip)
          "-mllvm", "-amdgpu-kernarg-preload-count=16",
          "-I", os.path.join(ROOT, "include"), "-I", CSRC]
# per-file extras: the encoder's distance must not be contracted into fused multiply-adds
EXTRA = {"encode.hip": ["-ffp-contract=off"], "encode_filter.hip": ["-ffp-contract=off"]}


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found; the LOOKAT library needs ROCm to build")
    return exe


def sources() -> list[str]:
    return sorted(f for f in os.listdir(CSRC) if f.endswith(".hip"))


def marshal_command() -> list[str]:
    import sysconfig

    import torch
    from torch.utils.cpp_extension import include_paths, library_paths
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I", os.path.join(ROOT, "include"), "-I", sysconfig.get_path("include")]
    for d in include_paths():
        cmd += ["-isystem", d]
    cmd += [os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL]
    for d in library_paths():
        cmd += ["-L", d]
    return cmd + ["-lc10", "-ltorch_cpu", "-ltorch_python"]


def build(verbose: bool = True, force: bool = True) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    cc = hipcc()
    objs = []
    procs = []
    failed = None
    for src in sources():
        obj = os.path.join(OBJ_DIR, src.replace(".hip", ".o"))
        objs.append(obj)
        path = os.path.join(CSRC, src)
        deps = [path] + [os.path.join(CSRC, h) for h in os.listdir(CSRC) if h.endswith(".h")] + \
               [os.path.join(ROOT, "include", "lookat.h")]
        if not force and os.path.exists(obj) and all(os.path.getmtime(obj) >= os.path.getmtime(d) for d in deps):
            continue
        cmd = [cc, *COMMON, *EXTRA.get(src, []), "-c", path, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    deps = [os.path.join(CSRC, "marshal.cpp"), os.path.join(ROOT, "include", "lookat.h")]
    if force or not (os.path.exists(MARSHAL) and all(os.path.getmtime(MARSHAL) >= os.path.getmtime(d) for d in deps)):
        cmd = marshal_command()
        if verbose:
            print(" ".join(cmd), flush=True)
        if os.path.exists(MARSHAL):
            os.remove(MARSHAL)
        try:
            procs.append(("marshal.cpp", subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        except OSError as e:
            failed = str(e)
    for src, p in procs:
        out, _ = p.communicate()
        # hipcc's host pass does not know the packed-fp32 feature name and says so: harmless
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            if src != "marshal.cpp":
                raise RuntimeError(f"the compiler failed on {src}:\n{out}")
            failed = out        # (the library works without it: linked first)
        if verbose and out.strip():
            print(out, flush=True)
    cmd = [cc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    if failed:
        raise RuntimeError(f"the compiler failed on marshal.cpp (the library is built, and loads without it):\n{failed}")
    return LIB


if __name__ == "__main__":
    build(force="--incremental" not in sys.argv)
    print(LIB)
