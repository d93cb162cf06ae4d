"""Compile the HIP sources under ``csrc/`` (in-tree, gfx950 only) into two shared libraries, and the Python binding:

* ``libssd_hip.so``      the product: every source directly under ``csrc/``;
* ``libssd_measure.so``  the same objects plus ``csrc/measure/`` (per-kernel timing of a prefill, peak
  probes): calls that create events and wait, kept out of the product library;
* ``_ssd_binding.so``    the native marshalling of ``ssd.py`` (``csrc/binding/``, host code, against torch's C++ headers).
                       Without it -- no headers, no g++ of torch's ABI -- everything works, with some 5 us more host time
                       a call: ``build`` then only warns.

``hipcc`` cross-compiles without a GPU.  Every source is compiled to an object once and the objects are
linked twice.  Packed-fp32 instruction selection is disabled (``-Xclang -target-feature -Xclang
-packed-fp32-ops``) for every device translation unit.
"""
from __future__ import annotations

import glob
import importlib.metadata
import os
import shutil
import subprocess
import sys
import sysconfig
import tempfile
import warnings
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libssd_hip.so")
MEASURE_LIB = os.path.join(HERE, "libssd_measure.so")
BINDING = os.path.join(HERE, "_ssd_binding.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unknown-warning-option",
]

# Per source: matrix instructions on architectural registers.  In a kernel with one wave per SIMD the compiler otherwise
# keeps accumulators in accumulation registers and moves them, 8 cycles each, wherever the vector unit works on them.
EXTRA_FLAGS = {"ssd_prefill_mfma.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]}


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def measure_sources():
    return sorted(glob.glob(os.path.join(CSRC, "measure", "*.hip")))


def binding_sources():
    return sorted(glob.glob(os.path.join(CSRC, "binding", "*.cpp")))


def torch_version() -> str:
    return importlib.metadata.version("torch")


def build_binding(verbose: bool = False) -> None:
    import torch
    home = os.path.dirname(torch.__file__)
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"))))
    includes = [INCLUDE, os.path.join(home, "include"), os.path.join(home, "include", "torch", "csrc", "api", "include"),
                os.path.join(rocm, "include"), "/opt/rocm/include", sysconfig.get_path("include")]
    tmp = BINDING + ".tmp%d" % os.getpid()
    lib = os.path.join(home, "lib")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1",
           "-DUSE_ROCM=1", "-DSSD_TORCH_VERSION=\"%s\"" % torch_version(), "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI)]
    cmd += [a for i in includes for a in ("-isystem", i)] + binding_sources() + ["-o", tmp, "-L" + lib]
    cmd += ["-ltorch_python", "-ltorch_cpu", "-ltorch", "-lc10_hip", "-lc10", "-Wl,-rpath," + lib]
    if verbose:
        print(" ".join(cmd), file=sys.stderr)
    subprocess.run(cmd, check=True)
    os.replace(tmp, BINDING)


def needs_build() -> bool:
    if not all(os.path.exists(f) for f in (LIB, MEASURE_LIB, BINDING)):
        return True
    with open(BINDING, "rb") as f:
        if ("built for torch %s;" % torch_version()).encode() not in f.read():
            return True
    t = min(os.path.getmtime(f) for f in (LIB, MEASURE_LIB, BINDING))
    deps = sources() + measure_sources() + glob.glob(os.path.join(CSRC, "*.hpp")) + \
        glob.glob(os.path.join(INCLUDE, "*.h")) + binding_sources()
    return any(os.path.getmtime(f) > t for f in deps)


def build(force: bool = True, verbose: bool = False) -> str:
    """Run hipcc.  With ``force=False`` up-to-date libraries are kept.  Returns the product library's path."""
    if not force and not needs_build():
        return LIB
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmpdir = tempfile.mkdtemp(prefix="ssd_build_")
    try:
        def compile_one(src):
            obj = os.path.join(tmpdir, os.path.basename(src) + ".o")
            cmd = [hipcc] + HIPCC_FLAGS + EXTRA_FLAGS.get(os.path.basename(src), [])
            cmd += ["-I", INCLUDE, "-I", CSRC, "-c", src, "-o", obj]
            if verbose:
                print(" ".join(cmd), file=sys.stderr)
            subprocess.run(cmd, check=True)
            return obj

        with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as pool:
            binding = pool.submit(build_binding, verbose)
            objs = list(pool.map(compile_one, sources() + measure_sources()))
            try:
                binding.result()
            except (subprocess.CalledProcessError, OSError, ImportError) as e:
                warnings.warn("the native marshalling was not built, calls go through Python: %s" % e)
        n = len(sources())
        for lib, members in ((LIB, objs[:n]), (MEASURE_LIB, objs)):
            tmp = lib + ".tmp%d" % os.getpid()
            cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + members
            if verbose:
                print(" ".join(cmd), file=sys.stderr)
            subprocess.run(cmd, check=True)
            os.replace(tmp, lib)
    finally:
        shutil.rmtree(tmpdir, ignore_errors=True)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose=True))
