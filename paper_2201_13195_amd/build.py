"""Builds librmm.so (HIP, gfx950 only) in-tree with hipcc, and the package's host module.

    python -m paper_2201_13195_amd.build

Every .hip file under csrc/ is compiled to an object and the objects are linked
into paper_2201_13195_amd/librmm.so, which needs hipcc alone; csrc/torch_host.cpp (no
device code) becomes paper_2201_13195_amd/_rmm_host.so next to it, which the Python package
needs and which takes the headers of the installed torch and of Python.
Nothing is cached between calls.

    python -m paper_2201_13195_amd.build --library     librmm.so only (a C or C++ program's build;
                                                       works without torch: run this file itself)
"""
import importlib.util
import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ_DIR = os.path.join(HERE, "_build")
LIB_PATH = os.path.join(HERE, "librmm.so")
HOST_PATH = os.path.join(HERE, "_rmm_host.so")

# Packed-fp32 instructions are switched off on purpose (device flag, hipcc only).
HIPCC_FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950", "-fno-gpu-rdc",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def _hipcc():
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found")
    return exe


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def _compile(src):
    obj = os.path.join(OBJ_DIR, os.path.basename(src)[:-4] + ".o")
    cmd = [_hipcc(), *HIPCC_FLAGS, "-c", src, "-o", obj]
    p = subprocess.run(cmd, capture_output=True, text=True)
    if p.returncode != 0:
        raise RuntimeError("hipcc failed on %s:\n%s\n%s" % (src, p.stdout, p.stderr))
    return obj


def _torch_dir():
    spec = importlib.util.find_spec("torch")
    if spec is None:
        raise RuntimeError("the host module needs an installed torch (build(host=False): librmm.so only)")
    return os.path.dirname(spec.origin)


def _compile_host():
    """csrc/torch_host.cpp -> object, against the headers of the installed torch."""
    obj, inc = os.path.join(OBJ_DIR, "torch_host.o"), os.path.join(_torch_dir(), "include")
    system = [inc, os.path.join(inc, "torch", "csrc", "api", "include"), "/opt/rocm/include", sysconfig.get_paths()["include"]]
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-Wall", "-Wextra", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           *[a for d in system for a in ("-isystem", d)], "-c", os.path.join(CSRC, "torch_host.cpp"), "-o", obj]
    p = subprocess.run(cmd, capture_output=True, text=True)
    if p.returncode != 0:
        raise RuntimeError("g++ failed on torch_host.cpp:\n%s\n%s" % (p.stdout, p.stderr))
    sys.stderr.write(p.stderr)
    return obj


def _link_host(obj):
    lib, tmp = os.path.join(_torch_dir(), "lib"), HOST_PATH + ".tmp"
    cmd = ["g++", "-shared", obj, "-o", tmp, "-L" + lib, "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_hip", "-ltorch_python",
           "-L" + HERE, "-lrmm", "-Wl,-rpath,$ORIGIN"]
    p = subprocess.run(cmd, capture_output=True, text=True)
    if p.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (p.stdout, p.stderr))
    os.replace(tmp, HOST_PATH)


def build_library():
    """librmm.so from the .hip sources."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(_compile, sources()))
    tmp = LIB_PATH + ".tmp"
    cmd = [_hipcc(), "-shared", "-fPIC", "--offload-arch=gfx950", "-fno-gpu-rdc", *objs, "-o", tmp]
    p = subprocess.run(cmd, capture_output=True, text=True)
    if p.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (p.stdout, p.stderr))
    os.replace(tmp, LIB_PATH)


def build(verbose=False, host=True):
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=2) as ex:
        obj = ex.submit(_compile_host) if host else None
        build_library()
    if host:
        _link_host(obj.result())
    if verbose:
        print("built", LIB_PATH, *([HOST_PATH] if host else []))
    return LIB_PATH


if __name__ == "__main__":
    build(verbose=True, host="--library" not in sys.argv[1:])
    sys.exit(0)
