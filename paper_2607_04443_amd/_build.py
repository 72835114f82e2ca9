"""Build of the native libraries, in-tree.

  libws.so       the product: HIP kernels for gfx950 (kernels.hip; peaks.hip holds
                 the calibration probes) + the C ABI (hipcc); block.cpp links
                 hipBLASLt for the projections around the attention
  libws_host.so  host-only page-table entry points for CPU tests (g++)
"""
import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB_PATH = os.path.join(PKG, "libws.so")
HOST_LIB_PATH = os.path.join(PKG, "libws_host.so")

HIP_SOURCES = ["kernels.hip", "peaks.hip", "ws_api.cpp", "pagetable.cpp", "block.cpp"]
# hipBLASLt runs the two projections of ws_block_step (plain GEMMs)
LINK_FLAGS = ["-L/opt/rocm/lib", "-Wl,-rpath,/opt/rocm/lib", "-lhipblaslt"]
# Packed fp32 ops are kept out of the generated code on purpose.  The kernels
# never form NaNs from finite inputs (masked logits are -inf, and no -inf - -inf
# is evaluated; a row of zeros normed with eps = 0 aside, whose norm has no
# value), so NaN-quieting canonicalisations are not needed.
# The MFMA builtins are to write vector registers: next to the video kernel's
# accumulation-register O (inline asm) the compiler would otherwise put its S
# tiles there too and copy every logit out before its exponential.
HIP_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
             "-fno-honor-nans",
             "-Wall", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-mllvm", "-amdgpu-mfma-vgpr-form", "-I", INCLUDE, "-I", CSRC]


def _hipcc():
    return shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"build step failed: {' '.join(cmd)}")


def build(verbose=False):
    obj_dir = os.path.join(PKG, "_build")
    os.makedirs(obj_dir, exist_ok=True)
    hipcc = _hipcc()
    jobs = []
    objs = []
    for src in HIP_SOURCES:
        obj = os.path.join(obj_dir, src + ".o")
        lang = ["-x", "hip"] if src.endswith(".hip") else []
        jobs.append([hipcc] + HIP_FLAGS + lang + ["-c", os.path.join(CSRC, src), "-o", obj])
        objs.append(obj)
    host_tmp = HOST_LIB_PATH + ".tmp"
    host_cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall",
                "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", CSRC, os.path.join(CSRC, "pagetable.cpp"),
                os.path.join(CSRC, "pagetable_capi.cpp"), "-o", host_tmp]
    jobs.append(host_cmd)
    with ThreadPoolExecutor(max_workers=4) as ex:
        list(ex.map(lambda c: _run(c, verbose), jobs))
    tmp = LIB_PATH + ".tmp"
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs + LINK_FLAGS, verbose)
    os.replace(tmp, LIB_PATH)
    os.replace(host_tmp, HOST_LIB_PATH)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
