"""Build in-tree: the HIP library paper_2207_10702_amd/libroast_hip.so (gfx950 only) and the Python layer's _roast_call.so."""
import hashlib
import os
import subprocess
import sys
import sysconfig
import tempfile
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


def call_stamp() -> str:
    """What a build of roast_call.cpp is for: its source, this Python and this torch, whose structures it reads."""
    import torch
    h = hashlib.sha256(f"{sys.version} {torch.__version__}".encode())
    for path in (os.path.join(CSRC, "roast_call.cpp"), os.path.join(ROOT, "include", "roast.h")):
        with open(path, "rb") as f:
            h.update(f.read())
    return "roast_call for " + h.hexdigest()[:32]


def call_is_current(path: str) -> bool:
    if not os.path.exists(path):
        return False
    if not os.path.exists(os.path.join(CSRC, "roast_call.cpp")):
        return True                            # (nothing to compare with)
    with open(path, "rb") as f:
        return call_stamp().encode() in f.read()


def compile_call(path: str = CALL) -> None:
    """Written beside its place and then moved there: another process finds a whole file or none.  NDEBUG: torch's headers bring a thread-local counter
    without it, and while a library with thread-local data of which a thread has used none is loaded, glibc before 2.39 looks up every other
    thread-local variable of that thread the long way (t.is_cuda, t.stride and the like took a third longer)."""
    import torch
    root = torch.__path__[0]
    inc, lib = os.path.join(root, "include"), os.path.join(root, "lib")
    fd, part = tempfile.mkstemp(prefix="_roast_call.", suffix=".so", dir=os.path.dirname(path))
    os.close(fd)
    try:
        subprocess.run(["g++", "-O2", "-DNDEBUG", "-std=c++17", "-fPIC", "-shared", "-Wall", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}",
                        f'-DROAST_CALL_STAMP="{call_stamp()}"', "-I" + os.path.join(ROOT, "include"), "-isystem", inc, "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"),
                        "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "roast_call.cpp"), "-o", part,
                        "-L" + lib, "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10"], check=True)
        os.chmod(part, 0o755)
        os.replace(part, path)
    except BaseException:
        os.unlink(part)
        raise


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES) + 1)) as ex:
        call = ex.submit(compile_call)
        objs = list(ex.map(_compile, SOURCES))
        call.result()
    subprocess.run([_hipcc(), "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB, *objs], check=True)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
