"""Compile librocs.so in-tree for gfx950 (MI355X) with hipcc.

Every .hip source under csrc/ is compiled to an object in _build/ (parallel),
then linked into paper_2607_27744_amd/librocs.so, replaced atomically. The
native call path of ops.py (csrc/binding.cpp, host code only) becomes the
extension module _binding.so beside it, linked against librocs.so and torch.
"""

import concurrent.futures
import os
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
BUILD_DIR = os.path.join(PKG, "_build")
LIB_PATH = os.path.join(PKG, "librocs.so")
BINDING_PATH = os.path.join(PKG, "_binding.so")
SOURCES = ["api.hip", "linear.hip", "attention.hip", "interaction.hip", "lcb.hip", "mlp.hip",
           "fmlinear.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CXX = os.environ.get("CXX", "g++")
ARCH = "gfx950"

# Packed fp32 VALU instructions are switched off for all device code.
FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"),
    "-Wno-unused-command-line-argument",
]


def _run(cmd):
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # The host pass does not know the packed-fp32 feature; that note is noise.
    text = "\n".join(ln for ln in res.stdout.splitlines() if "not a recognized feature" not in ln)
    if res.returncode != 0:
        raise RuntimeError(f"command failed ({res.returncode}): {' '.join(cmd)}\n{text}")
    return text


def _binding_command(obj):
    import torch
    from torch.utils.cpp_extension import include_paths
    inc = [sysconfig.get_paths()["include"], *include_paths()]
    return [CXX, "-O2", "-std=c++17", "-fPIC", "-c", os.path.join(CSRC, "binding.cpp"), "-o", obj,
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            *(f"-I{p}" for p in inc)]


def _link_binding(obj):
    from torch.utils.cpp_extension import library_paths
    tmp = BINDING_PATH + ".tmp"
    _run([CXX, "-shared", "-o", tmp, obj, f"-L{PKG}", "-lrocs", *(f"-L{p}" for p in library_paths()),
          "-lc10", "-ltorch_cpu", "-ltorch_python", "-Wl,-rpath,$ORIGIN"])
    os.replace(tmp, BINDING_PATH)


def build(verbose=False, jobs=None):
    """Compile and link; returns the path of librocs.so."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    objs = [os.path.join(BUILD_DIR, s.replace(".hip", ".o")) for s in SOURCES]
    cmds = [[HIPCC, *FLAGS, "-c", os.path.join(CSRC, s), "-o", o] for s, o in zip(SOURCES, objs)]
    binding = os.path.join(BUILD_DIR, "binding.o")
    cmds.append(_binding_command(binding))
    with concurrent.futures.ThreadPoolExecutor(max_workers=jobs or min(8, len(cmds))) as ex:
        for out in ex.map(_run, cmds):
            if verbose and out.strip():
                print(out)
    tmp = LIB_PATH + ".tmp"
    _run([HIPCC, f"--offload-arch={ARCH}", "-shared", "-o", tmp, *objs])
    os.replace(tmp, LIB_PATH)
    _link_binding(binding)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
