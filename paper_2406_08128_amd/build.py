"""Build libchela.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree.

    python -m paper_2406_08128_amd.build          # compile everything, link
"""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ_DIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libchela.so")
HOST_MODULE = os.path.join(HERE, "_chela_host.so")
SOURCES = ["chela_api.hip", "chela_kernels_f32.hip", "chela_kernels_bf16.hip", "chela_kernels_conv.hip",
           "chela_kernels_convmx.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# packed-fp32 VALU forms are switched off for every device compile (they have given wrong results on this chip now and then)
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # keep MFMA accumulators in architectural VGPRs: every accumulator here is read back by the vector ALU
         # (rounding to bf16) once per chunk, and AGPR<->VGPR copies would double that work
         "-mllvm", "-amdgpu-mfma-vgpr-form",
         "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option"]


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    msgs = [ln for ln in r.stdout.splitlines() if "packed-fp32-ops" not in ln and ln.strip()]
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, "\n".join(msgs)))
    return obj


def _build_host_module() -> bool:
    """The host path of the plain calls as a Python module (csrc/chela_host.cpp): host code only, against torch's headers.  It is a
    shortcut: where there is no compiler for it or no headers the library is built all the same, and no module of an earlier build
    stays beside it.
    NDEBUG keeps a per-thread counter of pybind11's reference counting out of it: once a library with per-thread data of its
    own that nothing reads has been loaded, this C library looks up the per-thread data of every older library the slow way,
    and each call into torch took a fifth to a third longer for the rest of the process (an attention call's host side 12.0 us,
    without it 10.0)."""
    import sysconfig
    if os.path.exists(HOST_MODULE):
        os.remove(HOST_MODULE)
    try:
        import torch
        tdir = os.path.dirname(os.path.abspath(torch.__file__))
        cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-DNDEBUG", "-D__HIP_PLATFORM_AMD__=1",
               "-DUSE_ROCM=1",
               "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), "-I" + os.path.join(tdir, "include"),
               "-I" + os.path.join(tdir, "include", "torch", "csrc", "api", "include"),
               "-I" + os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), "-I" + sysconfig.get_paths()["include"],
               os.path.join(CSRC, "chela_host.cpp"), "-o", HOST_MODULE, "-L" + os.path.join(tdir, "lib"),
               "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        failed = r.stdout if r.returncode != 0 else None
    except (ImportError, OSError) as e:
        failed = str(e)
    if failed is not None:
        print("host module not built, calls take the slower host path:\n" + failed, file=sys.stderr)
    return failed is None


def build(verbose: bool = True) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(4, len(SOURCES) + 1)) as ex:
        host = ex.submit(_build_host_module)
        objs = list(ex.map(_compile, SOURCES))
        host.result()
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout)
    if verbose:
        print("built", LIB)
    return LIB


def build_host_ubsan(verbose: bool = False) -> str:
    """libchela with the HOST half of the API file (argument checks, planner, scratch bookkeeping) compiled under
    UndefinedBehaviorSanitizer in trap mode: undefined behaviour stops the process, and no sanitizer runtime has to be
    loaded.  The kernels' objects are the ordinary ones (built first if they are missing).  For the CPU test tier only:
    the result lives in the build folder and is never what the binding loads by default."""
    objs = [os.path.join(OBJ_DIR, os.path.splitext(src)[0] + ".o") for src in SOURCES]
    if not all(os.path.exists(o) for o in objs):
        build(verbose=False)
    api_obj = os.path.join(OBJ_DIR, "chela_api_ubsan.o")
    san = ["-Xarch_host", "-fsanitize=undefined", "-Xarch_host", "-fsanitize-trap=undefined",
           "-Xarch_host", "-fno-sanitize-recover=undefined"]
    cmd = [HIPCC, *[f for f in FLAGS if f != "-O3"], "-O1", *san, "-c", os.path.join(CSRC, "chela_api.hip"), "-o", api_obj]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc (host UBSan) failed:\n" + r.stdout)
    lib = os.path.join(OBJ_DIR, "libchela_ubsan.so")
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", lib, api_obj, *objs[1:]]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout)
    if verbose:
        print("built", lib)
    return lib


if __name__ == "__main__":
    build()
    sys.exit(0)
