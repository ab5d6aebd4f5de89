"""Compile the HIP/C++ sources under csrc/ into libtensor_tiling.so (gfx950 only) and the binding's extension module.

    python -m paper_1805_04170_amd.build
"""
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libtensor_tiling.so")
CALLS = os.path.join(PKG, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))

# -packed-fp32-ops: keep the compiler from forming packed fp32 instructions (hipcc's host pass warns that it does
# not know the feature; harmless)
COMMON = ["-O3", "-std=c++17", "-fPIC", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC] + os.environ.get("TT_EXTRA_CXXFLAGS", "").split()
HIPFLAGS = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def sources():
    return sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".cpp")))


def _compile(src):
    out = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    cmd = ["hipcc"] + COMMON + (HIPFLAGS if src.endswith(".hip") else []) + ["-c", os.path.join(CSRC, src), "-o", out]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    log = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("compile failed: %s\n%s" % (" ".join(cmd), log))
    if log.strip():
        sys.stderr.write(log + "\n")
    return out


def build_calls():
    """the binding's extension module (host code; the library's functions reach it by address)"""
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-I" + os.path.join(ROOT, "include"), "-I" + sysconfig.get_paths()["include"],
           os.path.join(CSRC, "python", "calls.cpp"), "-o", CALLS]
    subprocess.check_call(cmd)
    return CALLS


def build(jobs=8):
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, sources()))
    cmd = ["hipcc", "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB] + objs
    subprocess.check_call(cmd)
    build_calls()       # last: it needs Python's headers, the library does not
    return LIB


if __name__ == "__main__":
    print(build())
