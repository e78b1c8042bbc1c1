"""Compile the rlcs HIP library in-tree for gfx950.

    python -m paper_2608_17641_amd.build

produces ``paper_2608_17641_amd/librlcs.so`` from the translation units ``csrc/rlcs_*.hip``
(one per group of entry points, compiled in parallel; kernels in ``csrc/rlcs_*.h``) against
the public header ``include/rlcs.h``, and ``paper_2608_17641_amd/libprobe.so`` from
``csrc/probe_stream.hip``: reference kernels that bench.py times beside the library (a streaming
copy with GAE's byte split, an empty launch), not part of the library; and
``paper_2608_17641_amd/_binding.<python>-torch<version>.so`` from ``csrc/binding.cpp``, the native
side of the Python binding (host code only, g++ against PyTorch's headers, so built once for each
Python and PyTorch it is to run with).
"""
from __future__ import annotations

import glob
import os
import shutil
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "librlcs.so")
PROBE_LIB = os.path.join(PKG, "libprobe.so")
PROBE_SOURCE = os.path.join(CSRC, "probe_stream.hip")
BINDING_SOURCE = os.path.join(CSRC, "binding.cpp")
SOURCES = sorted(glob.glob(os.path.join(CSRC, "rlcs_*.hip")))
HEADERS = sorted(glob.glob(os.path.join(CSRC, "rlcs_*.h"))) + [os.path.join(INCLUDE, "rlcs.h")]

ARCH = "gfx950"


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (ROCm is required to build the rlcs library)")


FLAGS = [
    "-O3", f"--offload-arch={ARCH}", "-std=c++17", "-fPIC",
    # packed fp32 instructions are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # no sinking of the stores that end two branches into one store through a selected address:
    # where the element-wise and vector load paths of a chunk last wrote different arrays (the
    # truncation continuation of its last step in one, its bootstrap in the other), that store
    # kept both arrays in private memory, 12 bytes per lane written through to HBM (masked GAE
    # 4096 x 256: 25 % more bytes written, 6.08 -> 5.20 us without; discounted returns on rows
    # of 255 steps 5.85 -> 4.92 us)
    "-mllvm", "-simplifycfg-sink-common=false",
    "-Wall", "-Wno-unused-function",
]


def compile_command(src: str, obj: str):
    return [hipcc(), *FLAGS, f"-I{INCLUDE}", f"-I{CSRC}", "-c", "-o", obj, src]


def link_command(objs, out: str = LIB):
    return [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", out, *objs]


def binding_lib() -> str:
    """The native binding of the running Python and PyTorch, built or not."""
    import torch
    return os.path.join(PKG, f"_binding.{sys.implementation.cache_tag}-torch{torch.__version__}.so")


def binding_command(out: str):
    import sysconfig

    import torch
    root = os.path.dirname(torch.__file__)
    inc = os.path.join(root, "include")
    # NDEBUG also takes out a thread-local counter of pybind11's headers: glibc before 2.39 looks up the
    # thread-local variables of every library loaded earlier the slow way, on each access, once a
    # library with any is loaded and its own are not accessed (torch.empty 1.45 -> 1.72 us)
    return ["g++", "-O2", "-DNDEBUG", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wno-unknown-pragmas",
            "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            f"-I{INCLUDE}", f"-I{inc}", f"-I{os.path.join(inc, 'torch', 'csrc', 'api', 'include')}",
            f"-I{sysconfig.get_paths()['include']}", "-isystem", "/opt/rocm/include",
            "-o", out, BINDING_SOURCE, f"-L{os.path.join(root, 'lib')}",
            "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]


_NOISE = ("is not a recognized feature for this target", "(ignoring feature)")


def _run(cmd):
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in res.stderr.splitlines() if not any(n in l for n in _NOISE))
    return res.returncode, err


def build(force: bool = True, verbose: bool = False) -> str:
    """Compile librlcs.so, libprobe.so and the native binding: all of them when force, else those
    that do not exist yet (a binding for another Python or PyTorch does not count)."""
    binding = binding_lib()
    jobs = {}  # output -> (objects to link, sources to compile into them)
    with tempfile.TemporaryDirectory(prefix="rlcs_build_") as tmpdir:
        for out, sources in ((LIB, SOURCES), (PROBE_LIB, [PROBE_SOURCE])):
            if force or not os.path.exists(out):
                jobs[out] = [(src, os.path.join(tmpdir, os.path.basename(src) + ".o")) for src in sources]
        want_binding = force or not os.path.exists(binding)
        binding_tmp = binding + f".tmp{os.getpid()}"
        with ThreadPoolExecutor(max_workers=max(1, min(8, os.cpu_count() or 1)) + 1) as pool:
            pending = pool.submit(_run, binding_command(binding_tmp)) if want_binding else None
            compiles = [so for pairs in jobs.values() for so in pairs]
            results = list(pool.map(lambda so: (so[0], _run(compile_command(*so))), compiles))
            if pending:
                results.append((BINDING_SOURCE, pending.result()))
        for src, (rc, err) in results:
            if rc != 0:
                raise RuntimeError(f"compiling {src} failed ({rc}):\n{err}")
            if verbose and err.strip():
                print(err, file=sys.stderr)
        for out, pairs in jobs.items():
            tmp = out + f".tmp{os.getpid()}"
            rc, err = _run(link_command([obj for _, obj in pairs], tmp))
            if rc != 0:
                if os.path.exists(tmp):
                    os.remove(tmp)
                raise RuntimeError(f"link of {os.path.basename(out)} failed ({rc}):\n{err}")
            os.replace(tmp, out)
        if want_binding:
            os.replace(binding_tmp, binding)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose=True))
