"""Build in-tree: the HIP library paper_2207_10702_amd/libroast_hip.so (gfx950 only) and the Python layer's _roast_call.so."""
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libroast_hip.so")
CALL = os.path.join(HERE, "_roast_call.so")    # host code: the launching calls of binding.py
SOURCES = ["roast_api.hip", "roast_mm_generic.hip", "roast_mm_mfma.hip", "roast_mm_wide.hip", "roast_mm_direct.hip", "roast_mm_ring.hip", "roast_mm_window.hip", "roast_reduce.hip", "roast_embed.hip", "roast_optim.hip"]
FLAGS = ["-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
         "-packed-fp32-ops", "-fno-gpu-rdc", "-Wall", "-Wno-unused-function",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.sep not in c or os.path.exists(c)):
            return c
    return "hipcc"


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    subprocess.run([_hipcc(), *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj], check=True)
    return obj


def _compile_call(_=None) -> None:
    import torch
    root = torch.__path__[0]
    inc, lib = os.path.join(root, "include"), os.path.join(root, "lib")
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}",
                    "-I" + os.path.join(ROOT, "include"), "-isystem", inc, "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"),
                    "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "roast_call.cpp"), "-o", CALL,
                    "-L" + lib, "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10"], check=True)


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES) + 1)) as ex:
        call = ex.submit(_compile_call)
        objs = list(ex.map(_compile, SOURCES))
        call.result()
    subprocess.run([_hipcc(), "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB, *objs], check=True)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
