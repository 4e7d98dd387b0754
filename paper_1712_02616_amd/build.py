"""Compile libiabn.so (the HIP kernels and the C ABI) for gfx950 with hipcc.

Each translation unit of ``csrc/`` compiles to an object file in parallel,
then one link makes the shared library.  ``build_probe`` compiles the
benchmark's bandwidth probes (``bench_probe.hip``) into a library of their
own, ``libiabn_probe.so``; libiabn does not contain or use them.  The tests'
``libiabn_abandon.so`` is libiabn with the fp16 and fp32 slice-resident
kernels built to abandon every other slice (``csrc/tile.h``).
"""

from __future__ import annotations

import glob
import os
import shutil
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
SOURCES = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
HEADERS = sorted(glob.glob(os.path.join(CSRC, "*.h"))) + [os.path.join(ROOT, "include", "iabn.h")]
LIB = os.path.join(HERE, "libiabn.so")
ABANDON_LIB = os.path.join(HERE, "libiabn_abandon.so")
ABANDON_SOURCES = ("slice_fwd_f16.hip", "slice_bwd_f16.hip", "slice_fwd_f32.hip", "slice_bwd_f32.hip")
ABANDON_FLAG = "-DIABN_TEST_ABANDON"
BINDING_SRC = os.path.join(HERE, "binding.cpp")
PROBE_SRC = os.path.join(HERE, "bench_probe.hip")
PROBE_LIB = os.path.join(HERE, "libiabn_probe.so")
ARCH = "gfx950"

FLAGS = ["--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         # Packed fp32 VALU instructions stay off on this target.
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found; it is needed to build libiabn.so")


def _run(cmd):
    return subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True)


def build(verbose: bool = False, abandon: bool = False) -> str:
    """Always recompiles; writes libiabn.so next to this file atomically.
    abandon: the tests' libiabn_abandon.so too."""
    cc = hipcc()
    with tempfile.TemporaryDirectory(prefix="iabn_build_") as tmp:
        objs, abandon_objs, procs = [], [], []

        def compile_(src, obj, extra=()):
            cmd = [cc] + FLAGS + list(extra) + ["-c", "-o", obj, src]
            procs.append((cmd, _run(cmd)))
            return obj

        # The largest units first.
        for src in sorted(SOURCES, key=lambda s: "slice" not in s):
            name = os.path.basename(src)
            objs.append(compile_(src, os.path.join(tmp, name + ".o")))
            abandon_objs.append(compile_(src, os.path.join(tmp, name + ".abandon.o"), [ABANDON_FLAG])
                                if abandon and name in ABANDON_SOURCES else objs[-1])
        errors = []
        for cmd, p in procs:
            out, err = p.communicate()
            if p.returncode != 0:
                errors.append("%s\n%s" % (" ".join(cmd), err))
            elif verbose and err:
                print(err)
        if errors:
            raise RuntimeError("hipcc failed:\n" + "\n".join(errors))
        for lib, parts in [(LIB, objs)] + ([(ABANDON_LIB, abandon_objs)] if abandon else []):
            out = lib + ".tmp%d" % os.getpid()
            cmd = [cc, "--offload-arch=" + ARCH, "-shared", "-fPIC", "-o", out] + parts
            res = subprocess.run(cmd, capture_output=True, text=True)
            if res.returncode != 0:
                raise RuntimeError("link failed (%d):\n%s\n%s"
                                   % (res.returncode, " ".join(cmd), res.stderr))
            os.replace(out, lib)
    return LIB


def binding_lib() -> str:
    """The Python binding's fast path for this torch and this Python, whose
    C++ and C interfaces it is compiled against."""
    import sysconfig

    import torch

    return os.path.join(HERE, "_binding.torch-%s.%s.so" % (torch.__version__,
                                                           sysconfig.get_config_var("SOABI")))


def build_binding() -> str:
    """Always recompiles the Python binding's fast path (host code against
    torch's and Python's headers)."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension

    rocm = os.path.dirname(os.path.dirname(os.path.realpath(hipcc())))
    incs = [os.path.join(ROOT, "include"), os.path.join(rocm, "include"),
            sysconfig.get_paths()["include"]] + cpp_extension.include_paths()
    lib = binding_lib()
    out = lib + ".tmp%d" % os.getpid()
    libs = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = (["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
            "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, "-o", out, BINDING_SRC] +
           [a for i in incs for a in ("-isystem", i)] +
           ["-L", libs, "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip",
            "-Wl,-rpath," + libs])
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("building the binding failed (%d):\n%s\n%s"
                           % (res.returncode, " ".join(cmd), res.stderr))
    os.replace(out, lib)
    return lib


def build_probe() -> str:
    """Always recompiles libiabn_probe.so (the benchmark's bandwidth probes)."""
    out = PROBE_LIB + ".tmp%d" % os.getpid()
    cmd = [hipcc()] + FLAGS + ["-shared", "-o", out, PROBE_SRC]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed (%d):\n%s\n%s" % (res.returncode, " ".join(cmd), res.stderr))
    os.replace(out, PROBE_LIB)
    return PROBE_LIB


def is_built() -> bool:
    return os.path.exists(LIB)


if __name__ == "__main__":
    print(build(verbose=True))
    print(build_binding())
    print(build_probe())
