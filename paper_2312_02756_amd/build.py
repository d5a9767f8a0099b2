"""Build step of the gfx950 library (hipcc -> paper_2312_02756_amd/libglv.so) and
of the native part of its Python binding (g++ -> paper_2312_02756_amd/_native.so).

Each HIP source is compiled for gfx950 only, then linked into one shared
library exporting the C ABI of include/glv.h.  The library links the HIP
runtime by its soname (libamdhip64.so.7); inside a process that has already
imported torch, the loader binds it to the runtime torch loaded, so one HIP
runtime serves both.

_native.so is host code against torch's headers and libglv.so, found beside it.

Packed FP32 instructions are switched off for device code
(-target-feature -packed-fp32-ops): the scalar forms are used instead.
"""

import concurrent.futures as cf
import importlib.util
import os
import shutil
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
REPO = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(REPO, "include")
BUILD = os.path.join(HERE, "_build")
SOURCES = ["glv_abi.hip", "glv_autotune.hip", "kernels_elementwise.hip", "kernels_jagged.hip",
           "kernels_analysis.hip"]
NATIVE = "bind_native.cpp"
ARCH = "gfx950"


def library_path() -> str:
    return os.path.join(HERE, "libglv.so")


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found (ROCm is required to build the library)")


def compile_flags():
    return ["-std=c++17", "-O3", "-fPIC", f"--offload-arch={ARCH}", "-I", INCLUDE, "-I", CSRC,
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-Wall", "-Wno-unused-variable", "-Wno-unused-but-set-variable"]


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc()] + compile_flags() + ["-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass does not know the device-only feature flag: drop that note
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{out}")
    if verbose and out.strip():
        print(out, flush=True)
    return obj


def native_path() -> str:
    return os.path.join(HERE, "_native.so")


def _run_host(cmd, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed for {NATIVE}:\n{r.stdout}")


def _torch_dir() -> str:
    return list(importlib.util.find_spec("torch").submodule_search_locations)[0]


def _compile_native(verbose: bool) -> str:
    obj = os.path.join(BUILD, "bind_native.o")
    inc = os.path.join(_torch_dir(), "include")
    system = [inc, os.path.join(inc, "torch", "csrc", "api", "include"), "/opt/rocm/include",
              sysconfig.get_paths()["include"]]
    _run_host(["g++", "-std=c++17", "-O2", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", "-I", INCLUDE]
              + [f for d in system for f in ("-isystem", d)] + ["-c", os.path.join(CSRC, NATIVE), "-o", obj], verbose)
    return obj


def _link_native(obj: str, verbose: bool) -> None:
    lib = os.path.join(_torch_dir(), "lib")
    tmp = native_path() + ".tmp"
    _run_host(["g++", "-shared", "-o", tmp, obj, "-L", HERE, "-l:libglv.so", "-Wl,-rpath,$ORIGIN", "-L", lib,
               "-ltorch_python", "-ltorch_cpu", "-ltorch", "-lc10", "-lc10_hip"], verbose)
    os.replace(tmp, native_path())


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=len(SOURCES) + 1) as ex:
        native = ex.submit(_compile_native, verbose)
        objs = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
        native_obj = native.result()
    out = library_path()
    tmp = out + ".tmp"
    cmd = [_hipcc(), "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, out)
    _link_native(native_obj, verbose)
    return out


if __name__ == "__main__":
    print(build(verbose=True))
