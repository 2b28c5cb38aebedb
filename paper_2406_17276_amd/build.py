"""Compile the HIP sources into libopttree.so for gfx950 and the Python binding's native half into _binding.so
(in-tree, next to the sources)."""
from __future__ import annotations

import importlib.util
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libopttree.so")
BINDING = os.path.join(HERE, "_binding.so")
SOURCES = ["api.hip", "row_scan.hip", "tree_build.hip", "build_fused.hip", "tree_select.hip", "tree_expand.hip", "tree_attn.hip", "verify.hip", "yardstick.hip"]

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument", "-Wno-inline-asm",
    # leading scalar kernel arguments arrive in registers at wavefront start (documented LLVM AMDGPU feature for
    # gfx940 and later; the compiler keeps a fallback entry that reads them from memory)
    "-mllvm", "-amdgpu-kernarg-preload-count=12",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
]
# per-file additions, row_scan.hip: without -disable-machine-licm 1 % slower (13B-shaped adaptive build 23.2 -> 23.5 us, builds of
# 128256-token rows 2191 -> 2201 us), at the same number of registers and no spills either way.
# build_fused.hip: without -disable-machine-licm constants of the exponential are kept in registers throughout (79 registers
# instead of 55, and 64 are what two workgroups of 1024 threads leave).
EXTRA_FLAGS = {"row_scan.hip": ["-mllvm", "-disable-machine-licm"],
               "build_fused.hip": ["-mllvm", "-disable-machine-licm"]}


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs = []
    objs = []
    for src in SOURCES:
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        objs.append(obj)
        cmd = [hipcc] + FLAGS + EXTRA_FLAGS.get(src, []) + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    binding_obj = os.path.join(objdir, "binding.o")
    procs.append(("binding.cpp", subprocess.Popen(binding_compile_command(binding_obj), stdout=subprocess.PIPE,
                                                  stderr=subprocess.STDOUT, text=True)))
    failed = False
    for src, pr in procs:
        out, _ = pr.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if pr.returncode != 0:
            failed = True
            sys.stderr.write(f"--- {src} failed ---\n{out}\n")
        elif verbose and out.strip():
            print(out)
    if failed:
        raise RuntimeError("hipcc failed")
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    subprocess.run(cmd, check=True)
    torch_lib = os.path.join(torch_dir(), "lib")
    subprocess.run(["g++", "-shared", "-o", BINDING, binding_obj, "-L" + HERE, "-lopttree", "-Wl,-rpath,$ORIGIN", "-L" + torch_lib,
                    "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip", "-Wl,-rpath," + torch_lib], check=True)
    build_abi_client()
    return LIB


def torch_dir() -> str:
    return os.path.dirname(importlib.util.find_spec("torch").origin)


def binding_compile_command(obj: str):
    """Host code only (tensors in, library calls, tensors out): the host compiler against torch's headers."""
    inc = os.path.join(torch_dir(), "include")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return ["g++", "-std=c++17", "-O2", "-fPIC", "-fvisibility=hidden", "-w", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
            "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-isystem", inc,
            "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"), "-isystem", os.path.join(rocm, "include"),
            "-isystem", sysconfig.get_paths()["include"], "-c", os.path.join(CSRC, "binding.cpp"), "-o", obj]


def build_abi_client() -> str:
    """The plain-C caller of the library that the GPU tests run (tests/abi_client.c): gcc, the public header and
    the HIP runtime only."""
    src = os.path.join(ROOT, "tests", "abi_client.c")
    exe = os.path.join(ROOT, "tests", "abi_client")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    cmd = ["gcc", "-std=c11", "-O2", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROOT, "include"),
           "-I" + os.path.join(rocm, "include"), src, "-o", exe, "-L" + HERE, "-lopttree",
           "-L" + os.path.join(rocm, "lib"), "-lamdhip64", "-Wl,-rpath,$ORIGIN/../paper_2406_17276_amd",
           "-Wl,-rpath," + os.path.join(rocm, "lib")]
    subprocess.run(cmd, check=True)
    return exe


if __name__ == "__main__":
    print(build(verbose=True))
