"""Builds libfastocr.so (hand-written HIP kernels + C ABI) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libfastocr.so")
SOURCES = ["api.hip", "attn.hip", "attn_f32.hip", "score.hip", "score_resident.hip", "focal_fused.hip", "topk.hip", "probe.hip"]

# Packed-FP32 VALU forms are switched off for all device code (they have given silently wrong
# results on these machines); hipcc's host pass does not know the feature and says so.
# The first arguments of a kernel (16 words with the two of their own address, so 14; before the first structure) are in scalar registers when its waves start.
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-mllvm", "-amdgpu-kernarg-preload-count=16",
         "-Wno-unused-command-line-argument", "-I", INCLUDE, "-I", CSRC]


# Host code only under AddressSanitizer and UndefinedBehaviorSanitizer (the device code is built as
# always): a checking build for the CPU-only tests of the argument validation, never the product.
HOST_SANITIZE = ["-g", "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
                 "-Xarch_host", "-fno-sanitize-recover=undefined", "-Xarch_host", "-fno-omit-frame-pointer"]
LIB_HOSTSAN = os.path.join(HERE, "libfastocr_hostsan.so")


# The binding's hot path (csrc/pycall.cpp), a Python extension over torch's own tensor headers; host code only.  The binding does without it
# where it is not there, so the library is built also where it cannot be.
CALL_LIB = os.path.join(HERE, "_fastocr_call.so")
CALL_LIB_HOSTSAN = os.path.join(HERE, "_fastocr_call_hostsan.so")


def _call_command(out: str, hipcc: str, host_sanitize: bool):
    import sysconfig
    import torch
    home = os.path.dirname(torch.__file__)
    inc = os.path.join(home, "include")
    # (the checking build with the compiler whose sanitizer runtime the library's own checking build needs)
    compiler = ["g++", "-O2"]
    if host_sanitize:
        clang = os.path.join(os.path.dirname(os.path.dirname(hipcc)), "lib", "llvm", "bin", "clang++")
        compiler = [clang, "-O1", "-g", "-fsanitize=address", "-fsanitize=undefined", "-fno-sanitize-recover=undefined",
                    "-fno-sanitize=vptr,function", "-fno-omit-frame-pointer", "-shared-libsan"]
    return [*compiler, "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            "-I", INCLUDE, "-I", CSRC, "-isystem", inc, "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"),
            "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "pycall.cpp"), "-o", out,
            "-L", os.path.join(home, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]


def build(verbose: bool = False, host_sanitize: bool = False) -> str:
    """Compile every source and link the shared library; returns its path."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    procs = []
    flags = FLAGS + (HOST_SANITIZE if host_sanitize else [])
    lib = LIB_HOSTSAN if host_sanitize else LIB
    for src in SOURCES:
        obj = os.path.join(CSRC, src.replace(".hip", ".san.o" if host_sanitize else ".o"))
        cmd = [hipcc, *flags, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    call_lib = CALL_LIB_HOSTSAN if host_sanitize else CALL_LIB
    call_tmp = call_lib + f".tmp{os.getpid()}"
    try:
        call = subprocess.Popen(_call_command(call_tmp, hipcc, host_sanitize), stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        call_why = ""
    except Exception as e:                                       # no torch, no compiler
        call, call_why = None, str(e)
    failed = False
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "is not a recognized feature for this target" not in l)
        if p.returncode != 0:
            failed = True
            sys.stderr.write(f"--- {src} failed ---\n{out}\n")
        elif verbose and out.strip():
            print(out)
    if call is not None:
        call_why, _ = call.communicate()
    # the extension belongs to the library of the same sources: an older one goes, whatever came of the new one
    built = call is not None and call.returncode == 0
    if not built or failed:
        for f in (call_tmp,) if failed else (call_tmp, call_lib):
            if os.path.exists(f):
                os.remove(f)
    if failed:
        raise RuntimeError("hipcc failed")
    if not built:
        sys.stderr.write(f"--- pycall.cpp was not built: calls go through ctypes, about 3 us slower ---\n{call_why}\n")
    tmp = lib + f".tmp{os.getpid()}"
    link = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs]
    if host_sanitize:
        link += ["-fsanitize=address", "-fsanitize=undefined", "-shared-libsan"]
    subprocess.check_call(link)
    os.replace(tmp, lib)
    if built:
        os.replace(call_tmp, call_lib)
    return lib


if __name__ == "__main__":
    print(build(verbose=True))
