"""Builds libqtamd.so (HIP for gfx950) in-tree with hipcc.

Usage: python -m paper_2504_21440_amd.build   (or build() from Python).
Every HIP source is compiled for gfx950 only.  Packed-FP32 instruction selection is disabled
(``-Xclang -target-feature -Xclang -packed-fp32-ops``); the host pass may warn that it does not
know that feature, which is harmless.
"""
import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libqtamd.so")
SOURCES = ["kernels_csr.hip", "kernels_csr_td.hip", "kernels_assembly.hip", "kernels_dense.hip", "kernels_res.hip", "kernels_op.hip", "kernels_mc.hip", "kernels_mc_reg.hip",
           "kernels_sde.hip", "kernels_sde_reg.hip", "qtamd_sde.cpp", "qtamd_noalloc.hip", "kernels_util.hip",
           "qtamd_runtime.cpp", "qtamd_me.cpp", "qtamd_mc.cpp", "qtamd_server.cpp", "qtamd_tune.cpp"]
ARCH = "gfx950"
# kernels_res.hip: the step loop fills the register file; hoisting the FP64 constants of its logarithm and
# exponential out of the loop took 45 registers per lane (127 against 82 for one element per thread).
EXTRA = {k: ["-mllvm", "-disable-machine-licm"] for k in ("kernels_res.hip", "kernels_mc.hip", "kernels_mc_reg.hip",
                                                           "kernels_sde_reg.hip")}


def _hipcc():
    h = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(h):
        raise RuntimeError("hipcc not found; the HIP library cannot be built")
    return h


def _flags():
    return ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-Xclang", "-target-feature", "-Xclang",
            "-packed-fp32-ops", "-Wno-unused-command-line-argument", "-I", os.path.join(HERE, "..", "include")]


def _compile(src):
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    cmd = [_hipcc()] + _flags() + EXTRA.get(src, []) + ["-c", os.path.join(CSRC, src), "-o", obj]
    if src.endswith(".hip"):
        cmd[1:1] = ["-x", "hip"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr[-6000:]}")
    return obj


def build(verbose=False):
    os.makedirs(OBJ, exist_ok=True)
    srcs = [s for s in SOURCES if os.path.exists(os.path.join(CSRC, s))]
    with cf.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB + ".tmp"
    cmd = [_hipcc(), "-shared", f"--offload-arch={ARCH}", "-fPIC", "-o", tmp] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr[-6000:]}")
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
