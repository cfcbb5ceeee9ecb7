"""Build the HIP library (gfx950 only) in-tree, paper_2411_04965_amd/lib/libbitlinear.so, and the host-only module beside it that
marshals arguments for the Python binding, bitlinear_marshal.<torch>.<python>.so."""
import glob
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB_DIR = os.path.join(HERE, "lib")
LIB = os.path.join(LIB_DIR, "libbitlinear.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def _compile(src):
    obj = os.path.join(OBJ, os.path.basename(src)[:-4] + ".o")
    cmd = [HIPCC] + FLAGS + ["-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    return src, obj, r


def _build_marshal():
    import sysconfig

    import torch
    from torch.utils import cpp_extension

    from .binding import MARSHAL_PATH

    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL_PATH]
    for d in cpp_extension.include_paths() + [sysconfig.get_paths()["include"]]:
        cmd += ["-isystem", d]
    for d in cpp_extension.library_paths():
        cmd += ["-L" + d]
    cmd += ["-ltorch_python", "-ltorch_cpu", "-lc10"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("building bitlinear_marshal failed:\n" + r.stderr)


def _build_library(verbose, jobs):
    os.makedirs(OBJ, exist_ok=True)
    os.makedirs(LIB_DIR, exist_ok=True)
    objs = []
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        for src, obj, r in ex.map(_compile, sources()):
            errs = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
            if r.returncode != 0:
                raise RuntimeError("hipcc failed on %s:\n%s" % (src, r.stderr))
            if verbose and errs.strip():
                print(errs, file=sys.stderr)
            objs.append(obj)
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs,
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)


def build(verbose=True, jobs=4):
    _build_library(verbose, jobs)
    for old in glob.glob(os.path.join(glob.escape(LIB_DIR), "bitlinear_marshal*.so")):
        os.remove(old)
    try:
        _build_marshal()
    except Exception as e:                       # (no C++ compiler, no headers: the library needs neither, and the binding has ctypes)
        print("bitlinear_marshal not built, the binding goes through ctypes: %s" % e, file=sys.stderr)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build()
