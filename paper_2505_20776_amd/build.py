"""Build libspecext.so (HIP kernels + C ABI) for gfx950 with hipcc, and the Python side's argument marshalling, in-tree."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_PATH = os.path.join(PKG_DIR, "libspecext.so")
# per-source extra flags: the matrix-core kernels with a softmax are compiled with the matrix-core results in
# architectural VGPRs (the softmax reads them with vector ALU instructions, which cannot read AGPRs);
# the row-split kernels never produce a NaN on their hot path, and saying so spares the max
# reductions one canonicalising instruction per operand
EXTRA_FLAGS = {"prefix_mfma.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
               "prefix_mfma_rows.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form", "-fno-honor-nans"],
               "prefix_f32.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form", "-fno-honor-nans"],
               "prefill_rows.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form", "-fno-honor-nans"]}
SOURCES = ["api.hip", "prefix_generic.hip", "prefix_mfma.hip", "prefix_mfma_rows.hip", "prefix_f32.hip", "tree_merge.hip", "retrieval.hip",
           "accept.hip", "materialized.hip", "prefill_rows.hip", "calibrate.hip"]


def hipcc_path() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (set HIPCC or install ROCm under /opt/rocm)")


STAMPS_LIB_PATH = os.path.join(PKG_DIR, "libspecext_stamps.so")


MARSHAL_PATH = os.path.join(PKG_DIR, "_marshal.so")


def _marshal_command(out: str):
    """(command, reason why there is none).  Host code only: the host compiler, against Python's and torch's headers; torch's
    libraries are those already loaded."""
    import sysconfig

    try:
        import torch
        from torch.utils.cpp_extension import include_paths
    except ImportError as e:
        return None, f"torch: {e}"
    cxx = next((c for c in (os.environ.get("CXX"), shutil.which("g++"), shutil.which("c++"), "/opt/rocm/llvm/bin/clang++")
                if c and (os.path.exists(c) or shutil.which(c))), None)
    if cxx is None:
        return None, "no C++ compiler found (set CXX)"
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(hipcc_path())))
    includes = include_paths() + [sysconfig.get_paths()["include"], os.path.join(rocm, "include"), "/opt/rocm/include"]
    lib_dir = os.path.join(os.path.dirname(torch.__file__), "lib")
    return ([cxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-w", "-D__HIP_PLATFORM_AMD__=1",
             f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"]
            + [a for i in includes if os.path.isdir(i) for a in ("-isystem", i)]
            + [os.path.join(CSRC, "marshal.cpp"), "-o", out, "-L" + lib_dir, "-ltorch_python", "-ltorch_cpu", "-lc10",
               "-lc10_hip"]), None


def compile_command(src: str, stamps: bool = False):
    """hipcc with the flags of one source, without its input and output."""
    return [
        hipcc_path(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
        "-mllvm", "-amdgpu-kernarg-preload-count=14",        # a kernel's first arguments in registers at its start (csrc/common.h)
        "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-Wall", "-Wno-unused-function", "-Wno-inline-asm",
    ] + (["-DSPECEXT_TAIL_STAMPS"] if stamps else []) + EXTRA_FLAGS.get(src, [])


def build_library(verbose: bool = True, stamps: bool = False) -> str:
    """Compile every HIP source for gfx950 and link libspecext.so next to this file.
    stamps=True builds the profiling variant libspecext_stamps.so instead (-DSPECEXT_TAIL_STAMPS: the row-split
    prefix kernel and the fused merge tail leave wall-clock stamps of their phases in the workspace; see
    paper_2505_20776_amd/phase_stamps.py).
    The marshalling beside it needs torch and a host compiler.  Where it cannot be built the library still is; an older
    _marshal.so, which may not fit it, goes."""
    obj_dir = os.path.join(PKG_DIR, "_build_stamps" if stamps else "_build")
    os.makedirs(obj_dir, exist_ok=True)
    lib_path = STAMPS_LIB_PATH if stamps else LIB_PATH
    procs = []
    objs = []
    for src in SOURCES:
        obj = os.path.join(obj_dir, src.replace(".hip", ".o"))
        objs.append(obj)
        procs.append((src, subprocess.Popen(compile_command(src, stamps) + ["-c", os.path.join(CSRC, src), "-o", obj],
                                            stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    marshal_tmp = MARSHAL_PATH + ".tmp"
    marshal_cmd, marshal_error = _marshal_command(marshal_tmp) if not stamps else (None, None)
    marshal = marshal_cmd and subprocess.Popen(marshal_cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    failed = False
    for src, pr in procs:
        out, _ = pr.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if pr.returncode != 0:
            failed = True
            sys.stderr.write(f"[specext build] {src} failed:\n{out}\n")
        elif verbose and out.strip():
            sys.stderr.write(f"[specext build] {src}:\n{out}\n")
    if marshal:
        out, _ = marshal.communicate()
        if marshal.returncode != 0:
            marshal_error = out
    if failed:
        raise RuntimeError("hipcc failed")
    tmp = lib_path + ".tmp"
    subprocess.run([hipcc_path(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs, check=True)
    os.replace(tmp, lib_path)
    if marshal_error is not None:
        sys.stderr.write(f"[specext build] {lib_path} is built, _marshal.so is not:\n{marshal_error}\n")
        if os.path.exists(MARSHAL_PATH):
            os.remove(MARSHAL_PATH)
    elif not stamps:
        os.replace(marshal_tmp, MARSHAL_PATH)
    return lib_path


if __name__ == "__main__":
    print(build_library(stamps="--stamps" in sys.argv[1:]))
