"""Build libfwa.so (hipcc, gfx950) and the torch marshalling module _fwa_torch.so (g++) in-tree:
``python -m paper_2501_06480_amd.build``."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libfwa.so")
TORCH_OUT = os.path.join(HERE, "_fwa_torch.so")
OBJ_DIR = os.path.join(HERE, "_build")
SOURCES = ["fwa_api.hip", "fwa_forward.hip", "fwa_forward_staged.hip", "fwa_forward_wide.hip", "fwa_f32_tile.hip", "fwa_f32_rows.hip", "fwa_backward.hip",
           "fwa_backward_coop.hip", "fwa_backward_large.hip", "fwa_backward_fused.hip", "fwa_backward_wide.hip", "fwa_bias.hip"]
# packed fp32 VALU ops are switched off on purpose: the compiler must not form them
# and matrix-core results go to ordinary VGPRs (no accumulator-register copies).
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wextra",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
               "-mllvm", "-amdgpu-mfma-vgpr-form"]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    return "hipcc"


def build_torch_binding(verbose: bool = True) -> str:
    """Host code only: argument marshalling between torch tensors and the C ABI."""
    import sysconfig
    import torch
    from torch.utils import cpp_extension
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(_hipcc()))) if os.path.sep in _hipcc() else "/opt/rocm"
    includes = [*cpp_extension.include_paths(), os.path.join(rocm, "include"), "/opt/rocm/include", sysconfig.get_paths()["include"]]
    libs = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           *(x for i in includes for x in ("-isystem", i)), os.path.join(CSRC, "torch_binding.cpp"), "-o", TORCH_OUT,
           "-L" + libs, "-ltorch", "-ltorch_cpu", "-ltorch_python", "-lc10", "-lc10_hip",
           "-L" + HERE, "-l:libfwa.so", "-Wl,-rpath,$ORIGIN"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return TORCH_OUT


def build(verbose: bool = True, jobs: int = 6) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    hipcc = _hipcc()

    def compile_one(src):
        obj = os.path.join(OBJ_DIR, src.replace(".hip", ".o"))
        cmd = [hipcc, *HIPCC_FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l and "--hip-link" not in l)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}")
        if verbose and out.strip():
            print(out, flush=True)
        return obj

    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", OUT, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    build_torch_binding(verbose)
    return OUT


if __name__ == "__main__":
    build()
    sys.exit(0)
