"""Build liblesjet.so in-tree with hipcc for gfx950.

    python -m paper_2301_00817_amd.build          # compile everything

Objects go to paper_2301_00817_amd/_build/, the library to
paper_2301_00817_amd/_lib/liblesjet.so.  Compilation is parallel over the
source files and always redone (the build is the 'does it compile' check).
"""
import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
BUILD = os.path.join(PKG, "_build")
LIBDIR = os.path.join(PKG, "_lib")
LIB = os.path.join(LIBDIR, "liblesjet.so")
ARCH = os.environ.get("LESJET_ARCH", "gfx950")

SOURCES = ["api.cpp", "geometry.hip", "ghost.hip", "residual_ref.hip", "residual_fused.hip",
           "residual_fused_wide.hip", "residual_fused32.hip",
           "residual_fused32_wide.hip", "rk.hip", "diag.hip", "adjoint.hip", "dynamic.hip"]

CFLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    # packed FP32 instructions are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


# Per-source flags.  The FP64 stage kernel (bound by latency) is scheduled for
# instruction-level parallelism: 0.7 % less time per launch on MI355X than the
# default scheduling.  The FP32 stage kernel (residual_fused32*.hip) keeps the
# default, under which its residuals and stages 1-4 fit four waves per SIMD
# without spilling (3 % faster than with the ILP scheduling, which spills).
_MAX_ILP = ["-mllvm", "-amdgpu-sched-strategy=max-ilp"]
SOURCE_FLAGS = {"residual_fused.hip": _MAX_ILP, "residual_fused_wide.hip": _MAX_ILP}

# Host-side ranges around the API calls and RK stages for rocprofv3
# --marker-trace (ROCTx; inert when no tool is attached).
LIBS = ["-L/opt/rocm/lib", "-lrocprofiler-sdk-roctx"]


def _hipcc():
    for c in ("/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found")


def _compile(src, build_dir=BUILD):
    obj = os.path.join(build_dir, os.path.basename(src) + ".o")
    cmd = [_hipcc(), *CFLAGS, *SOURCE_FLAGS.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    if src.endswith(".cpp"):
        cmd.insert(1, "-x")
        cmd.insert(2, "hip")
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr[-6000:]}")
    return obj, r.stderr


CHECKS_SRC = os.path.join(ROOT, "tests", "host_checks.hip")
CHECKS_LIB = os.path.join(LIBDIR, "liblesjet_checks.so")


def build_checks():
    """Host-compiled check library of the device functions (test helper)."""
    os.makedirs(LIBDIR, exist_ok=True)
    tmp = CHECKS_LIB + ".tmp"
    cmd = [_hipcc(), *CFLAGS, "-shared", "-x", "hip", CHECKS_SRC, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on host_checks.hip:\n{r.stderr[-6000:]}")
    os.replace(tmp, CHECKS_LIB)
    return CHECKS_LIB


DEVCHECKS_SRC = os.path.join(ROOT, "tests", "device_checks.hip")
DEVCHECKS_LIB = os.path.join(LIBDIR, "liblesjet_devchecks.so")


def build_device_checks():
    """Device check library of the kernels' fast arithmetic (GPU test helper)."""
    os.makedirs(LIBDIR, exist_ok=True)
    tmp = DEVCHECKS_LIB + ".tmp"
    cmd = [_hipcc(), *CFLAGS, "-shared", DEVCHECKS_SRC, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on device_checks.hip:\n{r.stderr[-6000:]}")
    os.replace(tmp, DEVCHECKS_LIB)
    return DEVCHECKS_LIB


CCLIENT_SRC = os.path.join(ROOT, "tests", "c_client.c")
CCLIENT_EXE = os.path.join(LIBDIR, "c_client")


def build_c_client():
    """Plain C client of the library (GPU test helper): C99, no C++, linked
    against liblesjet.so and the HIP runtime."""
    cc = shutil.which("gcc") or shutil.which("cc")
    if cc is None:
        return None
    tmp = CCLIENT_EXE + ".tmp"
    cmd = [cc, "-std=c99", "-O2", "-Wall", "-Wextra", "-Werror", "-D__HIP_PLATFORM_AMD__",
           "-I", os.path.join(ROOT, "include"), "-I", "/opt/rocm/include", CCLIENT_SRC, "-o", tmp,
           "-L", LIBDIR, "-llesjet", f"-Wl,-rpath,{LIBDIR}", "-L/opt/rocm/lib", "-lamdhip64",
           "-Wl,-rpath,/opt/rocm/lib"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"C client build failed:\n{r.stderr[-6000:]}")
    os.replace(tmp, CCLIENT_EXE)
    return CCLIENT_EXE


def build(verbose=False):
    """Compile all sources, link the library and the test check libraries."""
    os.makedirs(BUILD, exist_ok=True)
    os.makedirs(LIBDIR, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        results = list(ex.map(_compile, SOURCES))
    objs = [o for o, _ in results]
    if verbose:
        for _, err in results:
            if err.strip():
                print(err, file=sys.stderr)
    tmp = LIB + ".tmp"
    cmd = [_hipcc(), "-shared", f"--offload-arch={ARCH}", "-fPIC", "-Wl,--no-undefined", "-o", tmp,
           *objs, *LIBS]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr[-6000:]}")
    os.replace(tmp, LIB)
    if os.path.exists(CHECKS_SRC):
        build_checks()
    if os.path.exists(DEVCHECKS_SRC):
        build_device_checks()
    if os.path.exists(CCLIENT_SRC):
        build_c_client()
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
