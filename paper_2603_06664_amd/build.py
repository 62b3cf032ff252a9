"""Build libcrope.so (HIP, gfx950) in-tree with hipcc.  No torch extension machinery: the
library is a plain C-ABI shared object loaded with ctypes; only _fastcall.so, which hands torch tensors
to it, is compiled against torch's headers."""
from __future__ import annotations

import os
import subprocess
import sys
import warnings

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libcrope.so")
SOURCES = ["crope_api.hip", "rope.hip", "attention.hip", "project.hip"]
# measurement aids of bench.py (an MFMA-only loop and a plain copy): a library of their own,
# so that nothing in libcrope.so exists only for the benchmark
CEILINGS_LIB = os.path.join(HERE, "libcrope_ceilings.so")
CEILINGS_SOURCE = "ceilings.hip"
# issue-level microbenchmark (a standalone executable): the instruction-rate figures quoted for the
# attention kernel's design come from it
ISSUE_BENCH = os.path.join(HERE, "issue_bench")
ISSUE_BENCH_SOURCE = "issue_bench.hip"
# argument marshalling of the per-chunk calls (a Python extension module; host code only)
FASTCALL = os.path.join(HERE, "_fastcall.so")
FASTCALL_SOURCE = "fastcall.cpp"
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument"]
# attention.hip: score accumulators in vector registers, where the softmax reads them; without the
# option the compiler gives every MFMA of a kernel with more than 256 registers accumulation
# registers and copies each score out
SOURCE_FLAGS = {"attention.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}


def _stale() -> bool:
    built = (LIB, CEILINGS_LIB, FASTCALL)
    if not all(os.path.exists(f) for f in built) or not fastcall_current():
        return True
    t = min(os.path.getmtime(f) for f in built)
    deps = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".hip", ".h", ".cpp"))] + \
           [os.path.join(HERE, "..", "include", "crope.h"), os.path.abspath(__file__)]   # the flags are in here
    return any(os.path.getmtime(d) > t for d in deps)


def fastcall_tag() -> str:
    """What the extension is compiled for: torch's C++ classes are not the same from version to version."""
    import torch
    return "torch %s, Python %d.%d" % (torch.__version__, *sys.version_info[:2])


def fastcall_current() -> bool:
    if not os.path.exists(FASTCALL):
        return False
    with open(FASTCALL, "rb") as f:
        return fastcall_tag().encode() in f.read()


def _fastcall_command() -> list:
    import sysconfig
    import torch
    from torch.utils import cpp_extension
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
            "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, '-DCROPE_FASTCALL_FOR="%s"' % fastcall_tag(),
            *[f for d in cpp_extension.include_paths() for f in ("-isystem", d)],
            "-I" + sysconfig.get_paths()["include"], os.path.join(CSRC, FASTCALL_SOURCE), "-o", FASTCALL + ".tmp",
            *["-L" + d for d in cpp_extension.library_paths()], "-ltorch_python", "-ltorch_cpu", "-lc10"]


def build_fastcall() -> bool:
    """Compile the extension.  It needs g++ and the headers of torch and Python, which the library does not: where that
    fails the binding does without, so it is a warning, and no extension of older sources stays behind."""
    try:
        cmd = _fastcall_command()
        p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        why = None if p.returncode == 0 else "%s failed: %s\n%s" % (cmd[0], " ".join(cmd), p.stdout)
    except Exception as e:   # no compiler, or a torch without its headers
        why = "%s: %s" % (type(e).__name__, e)
    if why is None:
        os.replace(FASTCALL + ".tmp", FASTCALL)
        return True
    if os.path.exists(FASTCALL):
        os.remove(FASTCALL)
    warnings.warn("%s was not built: %s" % (os.path.basename(FASTCALL), why))
    return False


def build(force: bool = False, verbose: bool = False) -> str:
    if not force and not _stale():
        return LIB
    objs = []
    procs = []
    cmd = ["hipcc", *FLAGS, "-shared", os.path.join(CSRC, CEILINGS_SOURCE), "-o", CEILINGS_LIB + ".tmp"]
    procs.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    cmd = ["hipcc", *[f for f in FLAGS if f not in ("-fPIC", "-fvisibility=hidden")],
           os.path.join(CSRC, ISSUE_BENCH_SOURCE), "-o", ISSUE_BENCH]
    procs.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for src in SOURCES:
        obj = os.path.join(CSRC, src.replace(".hip", ".o"))
        cmd = ["hipcc", *FLAGS, *SOURCE_FLAGS.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
        procs.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    build_fastcall()   # while hipcc runs
    for cmd, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError("%s failed: %s\n%s" % (cmd[0], " ".join(cmd), out))
        if verbose and out.strip():
            print(out)
    # link against libamdhip64 by soname only (no rpath): inside a torch process the
    # already-loaded runtime is used.
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB + ".tmp"]
    subprocess.run(cmd, check=True)
    os.replace(LIB + ".tmp", LIB)
    os.replace(CEILINGS_LIB + ".tmp", CEILINGS_LIB)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose=True))
