"""Compile the HIP sources into paper_2106_05609_amd/libgas.so for gfx950, and the binding's marshalling into _marshal.so."""
import glob
import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libgas.so")
MARSHAL, MARSHAL_SOURCE = os.path.join(HERE, "_marshal.so"), os.path.join(HERE, "csrc", "marshal.cpp")
SOURCES = sorted(glob.glob(os.path.join(HERE, "csrc", "*.hip")))
HEADERS = sorted(glob.glob(os.path.join(HERE, "csrc", "*.h"))) + [os.path.join(ROOT, "include", "gas.h")]

FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument", "-I" + os.path.join(ROOT, "include")]


def stale() -> bool:
    if not os.path.exists(LIB) or not os.path.exists(MARSHAL):
        return True
    t = os.path.getmtime(LIB)
    return any(os.path.getmtime(f) > t for f in SOURCES + HEADERS) or _marshal_stale()


def built_for() -> str:
    """What _marshal.so is compiled against, beside its sources: it reads torch's tensors by their layout in memory."""
    import torch
    return f"torch {torch.__version__}, C++ ABI {int(torch._C._GLIBCXX_USE_CXX11_ABI)}, {sysconfig.get_config_var('SOABI')}"


def _marshal_stale() -> bool:
    if not os.path.exists(MARSHAL) or any(os.path.getmtime(f) > os.path.getmtime(MARSHAL)
                                          for f in (MARSHAL_SOURCE, os.path.join(ROOT, "include", "gas.h"))):
        return True
    with open(MARSHAL, "rb") as f:
        return built_for().encode() + b"\0" not in f.read()          # the module's own string, without importing it


def _marshal_commands(obj):
    """Host code that reads torch's tensors: compiled against the torch that is imported, linked to libgas.so beside it."""
    import torch
    from torch.utils import cpp_extension
    compile_ = ["g++", "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
                f'-DGAS_BUILT_FOR="{built_for()}"',
                "-I" + os.path.join(ROOT, "include"), "-I" + sysconfig.get_paths()["include"]]
    for d in cpp_extension.include_paths():
        compile_ += ["-isystem", d]
    link = ["g++", "-shared", "-o", MARSHAL, obj, "-L" + HERE, "-l:" + os.path.basename(LIB), "-Wl,-rpath,$ORIGIN"]
    link += ["-L" + d for d in cpp_extension.library_paths()] + ["-ltorch_python", "-ltorch_cpu", "-lc10"]
    return compile_ + ["-c", MARSHAL_SOURCE, "-o", obj], link


def build(force: bool = True, verbose: bool = False) -> str:
    if force or stale():
        objs = []
        build_dir = os.path.join(HERE, "_build")
        os.makedirs(build_dir, exist_ok=True)
        procs = []
        marshal, link_marshal = force or _marshal_stale(), None
        if marshal:
            cmd, link_marshal = _marshal_commands(os.path.join(build_dir, "marshal.cpp.o"))
            if verbose:
                print(" ".join(cmd))
            procs.append((MARSHAL_SOURCE, subprocess.Popen(cmd)))
        for src in SOURCES:
            obj = os.path.join(build_dir, os.path.basename(src) + ".o")
            objs.append(obj)
            if (not force and os.path.exists(obj)
                    and os.path.getmtime(obj) > max(os.path.getmtime(f) for f in [src] + HEADERS)):
                continue
            cmd = ["hipcc"] + [f for f in FLAGS if f != "-shared"] + ["-c", src, "-o", obj]
            if verbose:
                print(" ".join(cmd))
            procs.append((src, subprocess.Popen(cmd)))
        for src, p in procs:
            if p.wait() != 0:
                raise RuntimeError(f"the compiler failed on {src}")
        subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-pthread", "-o", LIB] + objs)
        if link_marshal:
            subprocess.check_call(link_marshal)
    return LIB


if __name__ == "__main__":
    import sys
    print(build(force="--incremental" not in sys.argv, verbose=True))
