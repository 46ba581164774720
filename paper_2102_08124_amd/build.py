"""Builds libtmask.so (the HIP kernels + C ABI) in-tree for gfx950 with hipcc, and _calls.so (the native half of binding.py).

Usage: python -m paper_2102_08124_amd.build [--force]
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtmask.so")
CALLS = os.path.join(HERE, "_calls.so")
CALLS_SOURCE = os.path.join(CSRC, "tmask_calls.cpp")
ABI = os.path.join(HERE, "..", "include", "tmask.h")
SOURCES = ["tmask_kernels.hip", "tmask_colwise.hip", "tmask_spmm.hip", "tmask_extras.hip"]
HEADERS = ["tmask_device.hpp", "tmask_solvers.hpp", "tmask_pack.hpp", "tmask_approx4.hpp", "tmask_networks.hpp", "tmask_pruned.hpp", "tmask_approx_sel.hpp", "tmask_pack4.hpp", "tmask_pack8.hpp", "tmask_exact_balance.hpp", "tmask_exact_spread.hpp", "tmask_column.hpp", "tmask_approx_spread.hpp", "tmask_fused4.hpp", "tmask_spmm_choice.hpp", "tmask_sum_choice.hpp", "tmask_host.hpp", os.path.join("..", "..", "include", "tmask.h")]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
         # packed fp32 VALU ops are kept off on the test machines
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function"]


def _stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    return any(os.path.getmtime(os.path.join(CSRC, f)) > t for f in SOURCES + HEADERS)


def calls_stamp() -> str:
    """What _calls.so is built for: it uses the layout of this torch's tensors and of this Python's objects."""
    import torch
    return "torch %s hip %s python %d.%d" % ((torch.__version__, torch.version.hip) + sys.version_info[:2])


def calls_stale() -> bool:
    """Whether _calls.so is missing, older than its source or the C ABI, or built for another torch or Python."""
    if not os.path.exists(CALLS):
        return True
    if any(os.path.getmtime(f) > os.path.getmtime(CALLS) for f in (CALLS_SOURCE, ABI)):
        return True
    with open(CALLS, "rb") as f:
        return calls_stamp().encode() + b"\0" not in f.read()


def build_calls(force: bool = False, verbose: bool = False) -> str:
    """The extension module that turns tensors into arguments; links against the torch that will load it."""
    if not force and not calls_stale():
        return CALLS
    import torch
    root = os.path.dirname(torch.__file__)
    tmp = CALLS + ".tmp%d" % os.getpid()
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), '-DTMASK_BUILT_FOR="%s"' % calls_stamp(),
           "-I" + os.path.join(root, "include"), "-I" + os.path.join(root, "include", "torch", "csrc", "api", "include"),
           "-I" + sysconfig.get_paths()["include"], "-I/opt/rocm/include", "-L" + os.path.join(root, "lib"), "-o", tmp, CALLS_SOURCE,
           "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("g++ failed compiling tmask_calls.cpp")
    os.replace(tmp, CALLS)
    return CALLS


def build(force: bool = False, verbose: bool = False) -> str:
    """Compile what is older than its sources (or everything with force=True).  The translation units are compiled side by
    side into _build/ (not tracked), then linked.  Without a g++ or torch's headers there is no _calls.so, and binding.py goes
    through ctypes."""
    try:
        build_calls(force, verbose)
    except (ImportError, OSError, RuntimeError) as e:
        if os.path.exists(CALLS):
            os.remove(CALLS)                      # not one of other sources
        sys.stderr.write("no _calls.so (%s): calls will go through ctypes\n" % e)
    if not (force or _stale()):
        return LIB
    from concurrent.futures import ThreadPoolExecutor
    obj_dir = os.path.join(HERE, "_build")
    os.makedirs(obj_dir, exist_ok=True)
    compile_flags = [f for f in FLAGS if f != "-shared"]

    def compile_one(src: str) -> str:
        obj = os.path.join(obj_dir, "%s.%d.o" % (os.path.splitext(src)[0], os.getpid()))
        cmd = [HIPCC] + compile_flags + ["-c", "-o", obj, os.path.join(CSRC, src)]
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            sys.stderr.write(res.stdout + res.stderr)
            raise RuntimeError("hipcc failed compiling %s" % src)
        return obj

    with ThreadPoolExecutor(max_workers=len(SOURCES)) as pool:
        objs = list(pool.map(compile_one, SOURCES))
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    for o in objs:
        os.remove(o)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("hipcc failed linking libtmask.so")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv, verbose=True))
