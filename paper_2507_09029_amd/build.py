"""Builds libsdp_hip.so (gfx950) from csrc/*.hip with hipcc and the Python call module from csrc/sdp_native.cpp, in-tree."""
import glob
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libsdp_hip.so")
NATIVE = os.path.join(HERE, "_sdp_native.so")
NATIVE_FOR = os.path.join(OBJ, "_sdp_native.torch")  # version of the torch it was built against
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc", "-ffp-contract=off",
    # packed fp32 VALU ops are kept off for every device function in this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def _stale(target, deps):
    if not os.path.exists(target):
        return True
    t = os.path.getmtime(target)
    return any(os.path.getmtime(d) > t for d in deps)


def _native_stale(deps, torch_version):
    """The call module uses torch's C++ interface: it is as old as its sources or built against another torch."""
    if _stale(NATIVE, deps) or not os.path.exists(NATIVE_FOR):
        return True
    with open(NATIVE_FOR) as f:
        return f.read() != torch_version


def build_library(force=False, verbose=False):
    os.makedirs(OBJ, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    hdrs = glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(ROOT, "include", "*.h"))
    jobs = []
    objs = []
    for src in srcs:
        obj = os.path.join(OBJ, os.path.basename(src)[:-4] + ".o")
        objs.append(obj)
        if force or _stale(obj, [src] + hdrs):
            jobs.append([HIPCC, *FLAGS, "-c", src, "-o", obj])

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        return cmd, r.returncode, r.stdout

    with ThreadPoolExecutor(max_workers=min(8, max(1, len(jobs)))) as ex:
        for cmd, rc, out in ex.map(run, jobs):
            noise = ("-packed-fp32-ops' is not a recognized feature", "is not a recognized feature for this target")
            text = "\n".join(l for l in out.splitlines() if not any(n in l for n in noise))
            if rc != 0:
                raise RuntimeError(f"hipcc failed: {' '.join(cmd)}\n{text}")
            if verbose and text.strip():
                print(text)
    if force or jobs or _stale(LIB, objs):
        cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
        _, rc, out = run(cmd)
        if rc != 0:
            raise RuntimeError(f"link failed:\n{out}")
    src = os.path.join(CSRC, "sdp_native.cpp")
    import torch

    if force or _native_stale([src] + hdrs, torch.__version__):
        T = os.path.dirname(torch.__file__)
        cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC",
               f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DSDP_TORCH_VERSION="{torch.__version__}"', "-I", os.path.join(ROOT, "include"),
               "-I", os.path.join(T, "include"), "-I", os.path.join(T, "include", "torch", "csrc", "api", "include"),
               "-I", sysconfig.get_paths()["include"], src, "-o", NATIVE, "-L", HERE, "-l:libsdp_hip.so",
               "-L", os.path.join(T, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-Wl,-rpath,$ORIGIN"]
        _, rc, out = run(cmd)
        if rc != 0:
            raise RuntimeError(f"building {NATIVE} failed:\n{out}")
        with open(NATIVE_FOR, "w") as f:
            f.write(torch.__version__)
    return LIB


if __name__ == "__main__":
    print(build_library(force="--force" in sys.argv, verbose=True))
