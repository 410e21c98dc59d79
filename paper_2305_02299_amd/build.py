"""Builds libsrigl.so (the C-ABI library) in-tree with hipcc for gfx950, and the CPython module in front of it with g++."""
from __future__ import annotations

import os
import subprocess

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libsrigl.so")
FRONT = os.path.join(PKG, "_front.so")
SOURCES = ["condense.hip", "fwd.hip", "fwd_klane_stream.hip", "fwd_rowlane_f32.hip", "fwd_rowlane_bf16.hip", "fwd_rowlane_f32_i16.hip", "fwd_rowlane_bf16_i16.hip", "fwd_rowloop.hip", "fwd_rowloop_f32.hip", "fwd_rowloop_bf16.hip", "fwd_rowloop_f32_i16.hip", "fwd_rowloop_bf16_i16.hip", "fwd_blocked.hip", "structured.hip", "mlp.hip", "update.hip", "csr.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # packed fp32 VALU forms stay off for every kernel of this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # A kernel's first words of arguments (structs passed by value are not among them) arrive in scalar registers with its wavefronts, instead of by a load that
    # everything else waits for.  16 is what is asked for; a wavefront has 16 registers for it and two hold the pointer to the arguments, so that 14 words come, or 13 where a
    # pointer would be split.  0.15 to 0.4 us a launch: 4096 -> 16384 bf16 at one row 5.47 -> 5.25 us, 768 -> 3072 at batch 256 8.41 -> 8.14, its update 42.3 -> 41.7, 3072 -> 768 with 538
    # stored at 16 rows 6.26 -> 6.00 (level on another card)
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wno-unused-command-line-argument",
]


def build(verbose: bool = False, defines=(), out: str = LIB) -> str:
    """Compile every HIP source (one hipcc process each, in parallel) and link paper_2305_02299_amd/libsrigl.so.
    Always recompiles."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    flags = [f for f in HIPCC_FLAGS if f != "-shared"] + ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    flags += ["-D" + d for d in defines]
    objdir = os.path.join(PKG, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs = []
    for s in SOURCES:
        obj = os.path.join(objdir, os.path.splitext(s)[0] + (".%d.o" % os.getpid()))
        cmd = [hipcc] + flags + ["-c", os.path.join(CSRC, s), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((obj, cmd, subprocess.Popen(cmd)))
    if out == LIB:
        procs.append(start_front(objdir, verbose))
    objs = []
    for obj, cmd, pr in procs:
        if pr.wait() != 0:
            raise subprocess.CalledProcessError(pr.returncode, cmd)
        objs.append(obj)
    front = objs.pop() if out == LIB else None
    tmp = out + ".tmp.%d" % os.getpid()
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs)
    os.replace(tmp, out)
    if front:
        link_front(front)
        objs.append(front)
    for o in objs:
        os.remove(o)
    return out


def start_front(objdir: str, verbose: bool = False):
    """Starts the compiler on the CPython module between torch tensors and libsrigl.so (host code only)."""
    import sysconfig

    import torch
    tdir = os.path.dirname(torch.__file__)
    obj = os.path.join(objdir, "front.%d.o" % os.getpid())
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), "-I", os.path.join(ROOT, "include")]
    for inc in (os.path.join(tdir, "include"), os.path.join(tdir, "include", "torch", "csrc", "api", "include"),
                os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), sysconfig.get_paths()["include"]):
        cmd += ["-isystem", inc]
    cmd += ["-c", os.path.join(CSRC, "front.cpp"), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    return obj, cmd, subprocess.Popen(cmd)


def link_front(obj: str) -> None:
    import torch
    tmp = FRONT + ".tmp.%d" % os.getpid()
    subprocess.check_call(["g++", "-shared", "-o", tmp, obj, "-L", PKG, "-l:libsrigl.so", "-L",
                           os.path.join(os.path.dirname(torch.__file__), "lib"), "-ltorch_python", "-ltorch_cpu", "-ltorch_hip", "-lc10", "-lc10_hip",
                           "-Wl,-rpath,$ORIGIN"])
    os.replace(tmp, FRONT)


if __name__ == "__main__":
    print(build(verbose=True))
