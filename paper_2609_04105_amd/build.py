"""Build libfp4attn.so (the HIP kernels and the C-ABI) in-tree with hipcc for gfx950,
and _binding.so (the native call path of the Python binding) with the host compiler.

Usage: python paper_2609_04105_amd/build.py [--jobs N]   (does not import the package)
"""
import argparse
import importlib.util
import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(HERE, "libfp4attn.so")
BINDING = os.path.join(HERE, "_binding.so")
SOURCES = ["fwd_mxfp4_guard.hip", "fwd_mxfp4_causal.hip", "fwd_mxfp4_ex2.hip", "fwd_mxfp4.hip",
           "fwd_mxfp4_ex2_dense.hip", "fwd_mxfp4_fp8pv.hip", "fwd_bf16.hip", "api.hip", "quantize.hip", "mfma_stream.hip"]
# The attention kernels never rely on NaN ordering in fmax; without this flag the
# compiler canonicalizes every fmax operand with an extra v_max_f32.
EXTRA = {f: ["-fno-honor-nans"] for f in ("fwd_mxfp4.hip", "fwd_mxfp4_ex2.hip", "fwd_mxfp4_ex2_dense.hip",
                                          "fwd_mxfp4_guard.hip", "fwd_mxfp4_causal.hip", "fwd_mxfp4_fp8pv.hip",
                                          "fwd_bf16.hip")}
ARCH = "gfx950"

HIPCC = os.environ.get("HIPCC", shutil.which("hipcc") or "/opt/rocm/bin/hipcc")
FLAGS = [
    f"--offload-arch={ARCH}",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-Wall",
    "-Wno-unused-function",
    # packed fp32 vector instructions stay disabled for every kernel
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def _compile(src):
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, *EXTRA.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _run(what, cmd):
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"{what} failed:\n{res.stderr}")


def _build_binding():
    """csrc/binding.cpp against the installed torch and the library just linked; False,
    and no binding, where torch or its headers are not installed (the library and its
    C-ABI need neither, and the package's calls then go through its Python checks)."""
    spec = importlib.util.find_spec("torch")
    torch_dir = spec.submodule_search_locations[0] if spec is not None else ""
    if not os.path.exists(os.path.join(torch_dir, "include", "ATen", "core", "Tensor.h")):
        if os.path.exists(BINDING):
            os.remove(BINDING)   # of another torch and an older library
        return False
    tmp = BINDING + ".tmp"
    _run("binding build", [
        os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-DUSE_ROCM",
        "-D__HIP_PLATFORM_AMD__", "-D_GLIBCXX_USE_CXX11_ABI=1", "-I" + sysconfig.get_paths()["include"],
        "-isystem", os.path.join(torch_dir, "include"),
        "-isystem", os.path.join(torch_dir, "include", "torch", "csrc", "api", "include"),
        "-isystem", os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"),
        os.path.join(CSRC, "binding.cpp"), "-o", tmp, "-L" + HERE, "-l:libfp4attn.so",
        "-L" + os.path.join(torch_dir, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip",
        "-Wl,-rpath,$ORIGIN"])
    os.replace(tmp, BINDING)
    return True


def build(jobs=8, verbose=True):
    """Compile every HIP source for gfx950, link the shared library and, where torch is
    installed, build the binding (always rebuilds)."""
    os.makedirs(BUILD, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    _run("link", [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp])
    os.replace(tmp, LIB)
    bound = _build_binding()
    if verbose:
        print(f"built {LIB}\n" + (f"built {BINDING}" if bound else "torch or its headers are missing: no _binding.so"))
    return LIB


if __name__ == "__main__":
    ap = argparse.ArgumentParser()
    ap.add_argument("--jobs", type=int, default=8)
    build(ap.parse_args().jobs)
