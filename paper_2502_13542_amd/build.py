"""Builds libactqkv.so (HIP, gfx950) with one hipcc call and the Python extension module that calls
it with one g++ call, both next to this file."""
from __future__ import annotations

import os
import shutil
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libactqkv.so")
NATIVE = os.path.join(HERE, "_native.so")

SOURCES = ["api.hip", "probe.hip", "score.hip", "select.hip", "attn_prefill_f32.hip",
           "attn_prefill_mfma.hip", "attn_decode.hip", "append.hip", "cutoff.hip", "gather.hip",
           "decode_retrieve.hip", "attn_static.hip"]

FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
         # packed fp32 instructions are kept out of the generated code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function"]


def _native_command() -> list:
    import torch
    root = os.path.dirname(torch.__file__)
    flags = ["-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1"]
    include = ["-I" + sysconfig.get_paths()["include"], "-isystem" + os.path.join(root, "include"),
               "-isystem" + os.path.join(root, "include", "torch", "csrc", "api", "include"), "-isystem/opt/rocm/include"]
    libs = ["-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10", "-ldl"]
    return [shutil.which("g++") or "g++"] + flags + include + [os.path.join(CSRC, "py_native.cpp"), "-o", NATIVE] + libs


def build(verbose: bool = False) -> str:
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    commands = [[hipcc] + FLAGS + [os.path.join(CSRC, s) for s in SOURCES] + ["-o", LIB], _native_command()]
    if verbose:
        print("\n".join(" ".join(c) for c in commands))
    running = [subprocess.Popen(c, stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True) for c in commands]
    noise = "is not a recognized feature for this target"
    failed = []
    for c, r in zip(commands, running):
        err = "\n".join(l for l in r.communicate()[1].splitlines() if noise not in l)
        if r.returncode != 0:
            failed.append(os.path.basename(c[0]) + " failed:\n" + err)
        elif verbose and err.strip():
            print(err)
    if failed:
        raise RuntimeError("\n".join(failed))
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
