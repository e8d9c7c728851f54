"""Build libstriped_attn.so for gfx950 with hipcc (cross-compiles without a GPU).

    python -m paper_2311_09431_amd.build

Objects go to _build/ at the repository root, the library and the binding's _marshal (host code on torch's headers, by
g++) next to this file.
"""
import glob
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

from . import asm_check

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libstriped_attn.so")
OBJ_DIR = os.path.join(ROOT, "_build")

SOURCES = ["api.hip", "permute.hip", "elementwise.hip", "f32_step.hip", "fwd_mfma.hip",
           "bwd_mfma.hip", "bwd_ring.hip", "split_mfma.hip", "f32x3_step.hip", "f32x3_split.hip", "f32_route.hip",
           "rows_step.hip"]

# Flags of single sources.  f32x3_step: score tiles are read by vector instructions right after
# their products, so MFMA results stay out of the accumulation registers (forward 2.20 -> 2.10 ms,
# backward 6.7 -> 6.1 ms for 16 heads, d 128, 4 x 2048 tokens).
SOURCE_FLAGS = {"f32x3_step.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
                "f32x3_split.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]}

# Sources with matrix instructions in asm statements, and their kernels whose accumulators are registers by
# number: the assembly of these is looked over (asm_check.py).
ASM_CHECKED = {"bwd_mfma.hip": ["bwd_dkdv_wide_kernel"], "bwd_ring.hip": ["bwd_dkdv_ring_kernel", "bwd_both_ring_kernel"], "split_mfma.hip": []}

# packed fp32 VALU forms are switched off on purpose for the test machines
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-fno-gpu-rdc",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def _hipcc():
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    raise RuntimeError("hipcc not found")


def _compile(src, extra):
    obj = os.path.join(OBJ_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc(), *FLAGS, *SOURCE_FLAGS.get(src, []), *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    if src in ASM_CHECKED:
        cmd.append("-save-temps=obj")       # the assembly that is assembled; the code is the same
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode:
        raise RuntimeError("hipcc failed on %s:\n%s\n%s" % (src, r.stdout, r.stderr))
    noise = ("packed-fp32-ops", "is not a recognized feature")
    warn = "\n".join(l for l in r.stderr.splitlines() if not any(n in l for n in noise)).strip()
    if warn:
        sys.stderr.write(warn + "\n")
    if src in ASM_CHECKED:
        _check_asm(src, obj)
    return obj


def _check_asm(src, obj):
    stem = obj[:-2]
    with open(stem + "-hip-amdgcn-amd-amdhsa-gfx950.s") as f:
        findings = asm_check.check(f.read(), ASM_CHECKED[src])
    for left in glob.glob(stem + "-h*") + glob.glob(stem + ".hip-*"):
        os.remove(left)
    if findings:
        os.remove(obj)
        raise RuntimeError("%s: the compiled code breaks what its asm statements rest on:\n%s" % (src, "\n".join(findings)))


def build_marshal():
    """The binding's extension module, against the torch that is installed."""
    import sysconfig
    import torch
    at = os.path.dirname(torch.__file__)
    out = os.path.join(HERE, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, "-I" + os.path.join(at, "include"),
           "-I" + os.path.join(at, "include", "torch", "csrc", "api", "include"),
           "-I" + sysconfig.get_paths()["include"], os.path.join(CSRC, "marshal.cpp"), "-o", out,
           "-L" + os.path.join(at, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-Wl,-rpath," + os.path.join(at, "lib")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode:
        raise RuntimeError("g++ failed on marshal.cpp:\n%s\n%s" % (r.stdout, r.stderr))
    return out


def build_library(extra_flags=(), jobs=8):
    """Compile every source and link the shared library; the binding's extension too.  Always recompiles."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        marshal = ex.submit(build_marshal)
        objs = list(ex.map(lambda s: _compile(s, list(extra_flags)), SOURCES))
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-fno-gpu-rdc", *objs, "-o", LIB]
    marshal.result()
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode:
        raise RuntimeError("link failed:\n%s\n%s" % (r.stdout, r.stderr))
    return LIB


if __name__ == "__main__":
    print(build_library(sys.argv[1:]))
