"""Compile csrc/*.hip into paper_2604_15750_amd/libdlm.so for gfx950 and csrc/decisions_py.c into _decisions (in-tree, no torch dependency)."""
import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libdlm.so")
# (tagged with the interpreter it was built for: it reads that one's objects, and another does not load it)
OUT_PY = os.path.join(HERE, "_decisions" + sysconfig.get_config_var("EXT_SUFFIX"))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# amdgpu-kernarg-preload-count: a kernel's first arguments (14 dwords at most, up to the first struct) arrive in scalar registers with the
# launch instead of by a trip to memory, so its first loads go out at once (161 launches of an in-block pass of the 8B model: 2888 -> 2864 us;
# the 13 of the fp32 model's 54.0 -> 53.0).
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-mllvm", "-amdgpu-kernarg-preload-count=14", "-Wno-unused-command-line-argument"] + os.environ.get("DLM_EXTRA_HIPCC_FLAGS", "").split()


def build(verbose=False):
    srcs = sorted(f for f in os.listdir(CSRC) if f.endswith(".hip"))
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)

    def cc(src):
        obj = os.path.join(objdir, src[:-4] + ".o")
        cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{err}")
        if verbose and err.strip():
            print(err, file=sys.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(cc, srcs))
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", OUT, *objs], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    build_extension()
    return OUT


def build_extension():
    """The decisions' calls without ctypes; without gcc or Python's headers there is none, and they go through ctypes."""
    for old in (OUT_PY, os.path.join(os.path.dirname(OUT_PY), "_decisions.so")):  # (the latter: without a tag)
        if os.path.exists(old):
            os.remove(old)
    gcc, include = shutil.which("gcc"), sysconfig.get_paths()["include"]
    if gcc is None or not os.path.exists(os.path.join(include, "Python.h")):
        print("no gcc or no Python.h: block_boundary and select_parallel are called through ctypes", file=sys.stderr)
        return None
    r = subprocess.run([gcc, "-O2", "-shared", "-fPIC", "-I", include, "-o", OUT_PY, os.path.join(CSRC, "decisions_py.c")], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("gcc failed on decisions_py.c:\n" + r.stderr)
    return OUT_PY


if __name__ == "__main__":
    print(build(verbose=True))
