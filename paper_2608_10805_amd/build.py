"""Build step for libwtconv.so (hipcc, gfx950), in-tree next to this file.

Every HIP source is compiled with packed-FP32 instructions disabled
(``-target-feature -packed-fp32-ops``); the kernels are written for plain
fp32 VALU FMAs. Sources compile to objects in parallel (the forward and
backward instantiations of the fused kernel live in separate translation
units), then link into one shared library.
"""
import os
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "libwtconv.so")
SOURCES = ["wtconv_api.cpp", "wtconv_noalloc.cpp", "wtconv_fwd.hip", "wtconv_mixed.hip", "wtconv_bwd.hip",
           "wtconv_bwd9.hip", "wtconv_phase_fwd.hip", "wtconv_phase_grad.hip", "wtconv_grad.hip",
           "wtconv_kernels.hip", "wtconv_tiny.hip"]
# measurement helper used only by the benchmark (sustained VALU rate)
PROBE_LIB = os.path.join(HERE, "libvalu_probe.so")
PROBE_SOURCES = ["valu_probe.hip"]
# native host path of the autograd wrapper: a Python extension against torch's headers
TORCH_LIB = os.path.join(HERE, "_wtconv_torch.so")
TORCH_SOURCE = "wtconv_torch.cpp"
ARCH = os.environ.get("WTCONV_OFFLOAD_ARCH", "gfx950")


def hipcc():
    return os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")


def hipcc_flags():
    return ["--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC", "-Wall",
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-I", INCLUDE, "-I", CSRC]


def _compile(sources, lib, extra, verbose):
    with tempfile.TemporaryDirectory(prefix="wtconv_build_") as tmp:
        def one(src):
            obj = os.path.join(tmp, src + ".o")
            cmd = [hipcc()] + hipcc_flags() + list(extra or []) + ["-x", "hip", "-c", os.path.join(CSRC, src),
                                                                    "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True)
            return obj

        workers = max(1, min(len(sources), int(os.environ.get("MAX_JOBS", "8"))))
        with ThreadPoolExecutor(max_workers=workers) as pool:
            objs = list(pool.map(one, sources))
        cmd = [hipcc(), "--offload-arch=" + ARCH, "-shared", "-fPIC"] + objs + ["-o", lib + ".tmp"]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
    os.replace(lib + ".tmp", lib)


def _torch_toolchain():
    """(g++, torch's folder), or None where one of them or torch's headers is
    missing: the wrapper then runs from Python alone."""
    import importlib.util
    import shutil

    gxx, spec = shutil.which("g++"), importlib.util.find_spec("torch")
    t = os.path.dirname(spec.origin) if spec and spec.origin else ""
    if not gxx or not os.path.exists(os.path.join(t, "include", "torch", "extension.h")):
        return None
    return gxx, t


def _compile_torch(verbose):
    import sysconfig

    found = _torch_toolchain()
    if found is None:
        print("no g++ or no torch headers: the autograd wrapper's native host path is left out", flush=True)
        if os.path.exists(TORCH_LIB):  # (of other sources, perhaps)
            os.remove(TORCH_LIB)
        return
    import torch
    gxx, t = found
    includes = [os.path.join(t, "include"), os.path.join(t, "include", "torch", "csrc", "api", "include"),
                os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), sysconfig.get_paths()["include"]]
    cmd = [gxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-DTORCH_EXTENSION_NAME=_wtconv_torch",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), "-I", INCLUDE]
    for d in includes:
        cmd += ["-isystem", d]
    cmd += [os.path.join(CSRC, TORCH_SOURCE), "-o", TORCH_LIB + ".tmp", "-L", os.path.join(t, "lib"), "-lc10",
            "-lc10_hip", "-ltorch_cpu", "-ltorch", "-ltorch_python"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(TORCH_LIB + ".tmp", TORCH_LIB)


def build(verbose: bool = False, extra=None) -> str:
    """Compile every HIP source (libwtconv.so and the benchmark's VALU probe) and
    the autograd wrapper's native host path (where g++ and torch's headers are
    there); return the path of libwtconv.so."""
    _compile(SOURCES, LIB, extra, verbose)
    _compile_torch(verbose)
    _compile(PROBE_SOURCES, PROBE_LIB, extra, verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
