"""Builds libsymi.so (gfx950) with hipcc and _marshal.so with g++, in-tree.  `python -m paper_2504_19925_amd.build`."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsymi.so")
# microbenchmarks of the part's ceilings (bench.py --ceiling): a library of their own, so that
# nothing of them is part of the product's ABI
CEILINGS_LIB = os.path.join(HERE, "libsymi_ceilings.so")
# the binding's argument marshalling (host code against torch's headers)
MARSHAL_LIB = os.path.join(HERE, "_marshal.so")
SOURCES = ["api.hip", "route.hip", "place.hip", "dispatch.hip", "gemm.hip", "adam.hip", "comm_plan.hip", "router.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def marshal_command():
    import sysconfig

    import torch
    t = os.path.dirname(torch.__file__)
    inc = [os.path.join(t, "include"), os.path.join(t, "include", "torch", "csrc", "api", "include"),
           "/opt/rocm/include", sysconfig.get_paths()["include"]]
    lib = os.path.join(t, "lib")
    return ([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
             f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"]
            + [x for i in inc for x in ("-isystem", i)] + ["-I", os.path.join(ROOT, "include"),
             os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL_LIB, "-L" + lib, "-ltorch_python", "-ltorch",
             "-ltorch_cpu", "-lc10", "-lc10_hip", "-Wl,-rpath," + lib])


def build(verbose: bool = True) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc] + FLAGS + [os.path.join(CSRC, s) for s in SOURCES] + ["-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    cmd = [hipcc] + FLAGS + [os.path.join(CSRC, "ceilings.hip"), "-o", CEILINGS_LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    build_marshal(verbose)
    return LIB


def build_marshal(verbose: bool = True) -> bool:
    """Builds _marshal.so if the host compiler and the headers of Python and torch are there.  Without it
    the binding calls the library through ctypes; an older one does not stay beside a new libsymi.so."""
    if os.path.exists(MARSHAL_LIB):
        os.remove(MARSHAL_LIB)
    cmd = marshal_command()
    if verbose:
        print(" ".join(cmd), flush=True)
    try:
        subprocess.run(cmd, check=True)
    except (OSError, subprocess.CalledProcessError) as e:
        print(f"_marshal.so was not built, device calls will go through ctypes: {e}", file=sys.stderr, flush=True)
        return False
    return True


if __name__ == "__main__":
    build()
    sys.exit(0)
