"""Compiles csrc/*.hip into libver.so (gfx950) and csrc/marshal.cpp into _marshal.so (host) next to this file."""
import glob
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(HERE, "libver.so")
MARSHAL = os.path.join(HERE, "_marshal.so")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument"]


def _marshal_command() -> list:
    import torch
    t = os.path.dirname(os.path.abspath(torch.__file__))
    return ["g++", "-O2", "-std=c++17", "-shared", "-fPIC", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            f"-isystem{t}/include", f"-isystem{t}/include/torch/csrc/api/include", f"-I{sysconfig.get_paths()['include']}",
            os.path.join(HERE, "csrc", "marshal.cpp"), "-o", MARSHAL, f"-L{t}/lib", "-ltorch_python", "-ltorch_cpu", "-lc10", f"-Wl,-rpath,{t}/lib"]


def build(verbose: bool = True) -> str:
    srcs = sorted(glob.glob(os.path.join(HERE, "csrc", "*.hip")))
    objs = []
    procs = []
    os.makedirs(os.path.join(HERE, "_build"), exist_ok=True)
    for s in srcs:
        o = os.path.join(HERE, "_build", os.path.basename(s)[:-4] + ".o")
        objs.append(o)
        procs.append((s, subprocess.Popen(["hipcc", *FLAGS, "-c", s, "-o", o],
                                          stderr=subprocess.PIPE, text=True)))
    procs.append(("marshal.cpp", subprocess.Popen(_marshal_command(), stderr=subprocess.PIPE, text=True)))
    for s, p in procs:
        _, err = p.communicate()
        err = "\n".join(l for l in err.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError(f"compilation of {s} failed:\n{err}")
        if verbose and err.strip():
            print(err, file=sys.stderr)
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    return LIB


if __name__ == "__main__":
    print(build())
