"""Build librtopk.so (HIP, gfx950) and the CPython module _rtopk_torch.so in-tree.  Run as `python -m paper_2409_00822_amd.build`."""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ_DIR = os.path.join(HERE, "_build")
LIB_PATH = os.path.join(HERE, "librtopk.so")
BINDING_PATH = os.path.join(HERE, "_rtopk_torch.so")

SOURCES = ["rtopk_api.hip", "rtopk_inst_g4_exact.hip", "rtopk_inst_g4_early.hip", "rtopk_inst_g4_eps.hip",
           "rtopk_inst_small_exact.hip", "rtopk_inst_small_early.hip", "rtopk_inst_small_eps.hip",
           "rtopk_inst_h16_exact.hip", "rtopk_inst_h16_early.hip", "rtopk_inst_dense.hip", "rtopk_inst_block.hip",
           "rtopk_inst_block_var.hip",
           "rtopk_inst_block_dense.hip", "rtopk_inst_block_h16.hip", "rtopk_inst_backward.hip", "rtopk_inst_stream.hip",
           "rtopk_inst_split.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-ffp-contract=off",          # the fp32 midpoint must round exactly like a scalar CPU evaluation
    "-fno-gpu-flush-denormals-to-zero",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
]


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, os.path.splitext(src)[0] + ".o")
    cmd = ["hipcc", *HIPCC_FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    subprocess.check_call(cmd)
    return obj


def _compile_binding() -> str:
    """The CPython module between the Python entry points and the library: host code, torch's headers."""
    import sysconfig

    import torch

    inc = os.path.join(os.path.dirname(torch.__file__), "include")
    obj = os.path.join(OBJ_DIR, "rtopk_torch.o")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
                           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
                           "-isystem", inc, "-isystem", os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"),
                           "-isystem", sysconfig.get_paths()["include"], "-I" + os.path.join(ROOT, "include"),
                           "-c", os.path.join(CSRC, "rtopk_torch.cpp"), "-o", obj])
    return obj


def _link_binding(obj: str) -> None:
    import torch

    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    subprocess.check_call(["g++", "-shared", obj, "-o", BINDING_PATH, "-L" + lib, "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_hip",
                           "-ltorch_python", "-L" + HERE, "-lrtopk", "-Wl,-rpath,$ORIGIN"])


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    # regenerate the inline-assembly search loops (a no-op when the committed file is current)
    subprocess.check_call([sys.executable, os.path.join(CSRC, "gen_search_loops.py")], stdout=subprocess.DEVNULL)
    with concurrent.futures.ThreadPoolExecutor(max_workers=8) as ex:
        binding = ex.submit(_compile_binding)
        objs = list(ex.map(_compile, SOURCES))
        binding_obj = binding.result()
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB_PATH])
    _link_binding(binding_obj)
    if verbose:
        print("built", LIB_PATH)
    return LIB_PATH


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
