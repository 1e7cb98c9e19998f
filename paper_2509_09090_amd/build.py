"""Builds libsqap.so (the gfx950 HIP library) and _calls.so (the binding's argument marshalling) in-tree."""
import glob
import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libsqap.so")
CALLS = os.path.join(HERE, "_calls.so")
CALLS_SOURCE = os.path.join(HERE, "csrc", "calls.cpp")
SOURCES = sorted(glob.glob(os.path.join(HERE, "csrc", "*.hip")))
HEADERS = sorted(glob.glob(os.path.join(HERE, "csrc", "*.h"))) + [os.path.join(ROOT, "include", "sqap.h")]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CXX = os.environ.get("CXX", "/opt/rocm/bin/amdclang++")       # comes with hipcc
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off", "-fhip-fp32-correctly-rounded-divide-sqrt",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result",
    "-I", os.path.join(ROOT, "include"),
]


def _older(built, sources):
    return not os.path.exists(built) or any(os.path.getmtime(f) > os.path.getmtime(built) for f in sources)


def is_stale():
    return _older(LIB, SOURCES + HEADERS) or _older(CALLS, [CALLS_SOURCE] + HEADERS) or not _built_for_this_torch()


def _torch_mark():
    import torch
    return "sqap: built for torch " + torch.__version__


def _built_for_this_torch():
    """_calls.so holds torch's internal layouts, of the version that its mark names."""
    with open(CALLS, "rb") as f:
        return _torch_mark().encode() + b"\0" in f.read()


def _calls_command():
    """Host code only: Python's and torch's headers, no kernels."""
    import torch
    at = os.path.dirname(torch.__file__)
    include = [os.path.join(at, "include"), os.path.join(at, "include", "torch", "csrc", "api", "include"), "/opt/rocm/include"]
    return ([CXX, "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
             "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), '-DSQAP_TORCH_MARK="%s"' % _torch_mark()]
            + [f for i in include for f in ("-isystem", i)]
            + ["-I", sysconfig.get_paths()["include"], "-I", os.path.join(ROOT, "include"), CALLS_SOURCE, "-o", CALLS,
               "-L" + os.path.join(at, "lib"), "-lc10", "-lc10_hip", "-ltorch_python", "-ltorch_cpu"])


def build(force=True, verbose=False):
    """Compile every kernel for gfx950.  Returns the library path."""
    if not force and not is_stale():
        return LIB
    procs = [(CALLS_SOURCE, subprocess.Popen(_calls_command()))]
    objs = []
    for src in SOURCES:
        obj = src[:-4] + ".o"
        cmd = [HIPCC] + [f for f in FLAGS if f != "-shared"] + ["-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd))
        procs.append((src, subprocess.Popen(cmd)))
        objs.append(obj)
    failed = [src for src, pr in procs if pr.wait() != 0]          # (all of them are waited for)
    if failed:
        raise RuntimeError("the compiler failed on " + ", ".join(failed))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    subprocess.run(cmd, check=True)
    for o in objs:
        os.remove(o)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
