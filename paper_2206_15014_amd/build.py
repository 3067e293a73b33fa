"""Build libnm.so in-tree with hipcc for gfx950 (cross-compiles without a GPU)."""
from __future__ import annotations

import hashlib
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libnm.so")
# Argument marshalling of the binding's hot calls, for this interpreter alone: any other has its own suffix and does not find it.
PYTHON_MODULE = os.path.join(HERE, "_nm_python" + sysconfig.get_config_var("EXT_SUFFIX"))
# (source, extra flags, object name).  The LDS-direct GEMM kernels are one source compiled once per
# set of N:M patterns, so that their many instantiations build in parallel.
DMA_SETS = 11
SOURCES = [("nm_gemm_dma.hip", ["-DNM_DMA_SET=%d" % k], "nm_gemm_dma_%d.o" % k) for k in range(DMA_SETS)] + \
          [(s, [], s.replace(".hip", ".o")) for s in ["nm_api.hip", "nm_compress.hip", "nm_gemm.hip", "nm_gemm_any.hip", "nm_project.hip", "nm_quantize_act.hip", "nm_scale_search.hip"]]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def source_digest() -> str:
    """Of everything the library is made from; the library carries the one it was built with (nm_test_source_digest), so
    one that was linked from older objects, or built before a change, is told from one of this tree."""
    h = hashlib.sha256()
    for folder in (os.path.join(ROOT, "include"), CSRC):
        for name in sorted(n for n in os.listdir(folder) if n.endswith((".h", ".hip", ".c"))):
            with open(os.path.join(folder, name), "rb") as f:
                data = f.read()
            h.update(b"%s %d\n" % (name.encode(), len(data)) + data)
    with open(os.path.join(HERE, "build.py"), "rb") as f:
        h.update(f.read())
    return h.hexdigest()


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    noise = ("packed-fp32-ops", "1 warning generated", "warnings generated")
    out = "\n".join(l for l in res.stdout.splitlines() if not any(n in l for n in noise))
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out)


def remove_python_modules(folder: str) -> None:
    for name in os.listdir(folder):
        if name.startswith("_nm_python.") and name.endswith(".so"):
            os.unlink(os.path.join(folder, name))


def build_python_module(include: str, target: str, hipcc: str, verbose: bool = False) -> bool:
    """False where the interpreter's headers are not there: the binding then goes through ctypes alone."""
    if not os.path.exists(os.path.join(include, "Python.h")):
        return False
    tmp = target + ".tmp.%d" % os.getpid()
    try:
        _run([hipcc, "-x", "c", "-O2", "-fPIC", "-shared", "-Wall", "-I", os.path.join(ROOT, "include"), "-I", include,
              os.path.join(CSRC, "nm_python.c"), "-o", tmp], verbose)
        os.replace(tmp, target)
    finally:
        if os.path.exists(tmp):
            os.unlink(tmp)
    return True


def build(verbose: bool = False) -> str:
    """Compile every source to an object (in parallel, one hipcc each) and link them into libnm.so.
    Objects live in a temporary directory, so the tree only ever holds sources and the library."""
    import concurrent.futures
    import shutil
    import tempfile
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    compile_flags = [f for f in HIPCC_FLAGS if f != "-shared"] + ["-DNM_SOURCE_DIGEST=" + source_digest()]
    tmpdir = tempfile.mkdtemp(prefix="libnm_build_")
    tmp = LIB + ".tmp.%d" % os.getpid()
    try:
        objs = [os.path.join(tmpdir, o) for _, _, o in SOURCES]
        jobs = [[hipcc, *compile_flags, *extra, "-c", "-o", o, os.path.join(CSRC, s)] for (s, extra, _), o in zip(SOURCES, objs)]
        workers = max(1, min(len(jobs), (os.cpu_count() or 2), 8))
        with concurrent.futures.ThreadPoolExecutor(max_workers=workers) as pool:
            list(pool.map(lambda c: _run(c, verbose), jobs))
        _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs], verbose)
        remove_python_modules(HERE)            # (they call the library that goes now)
        os.replace(tmp, LIB)
        build_python_module(sysconfig.get_paths()["include"], PYTHON_MODULE, hipcc, verbose)
    finally:
        shutil.rmtree(tmpdir, ignore_errors=True)
        if os.path.exists(tmp):
            os.unlink(tmp)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
