"""Every source of the library is accepted by the compiler as it stands in the tree, whatever built library lies beside it, and
the library that is loaded was built from these sources."""
import ctypes
import os
import shutil
import subprocess

import pytest

from paper_2206_15014_amd import binding, build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no compiler")
@pytest.mark.parametrize("source", sorted({s for s, _, _ in build.SOURCES}))
def test_front_end(source):
    extra = next(e for s, e, _ in build.SOURCES if s == source)
    flags = [f for f in build.HIPCC_FLAGS if f != "-shared"]
    res = subprocess.run([HIPCC, *flags, *extra, "-fsyntax-only", os.path.join(build.CSRC, source)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout


def test_library_is_of_these_sources():
    hook = getattr(binding.raw(), "nm_test_source_digest", None)
    assert hook is not None, "a library from before the sources it is tested with"
    hook.restype = ctypes.c_char_p
    assert hook().decode() == build.source_digest(), "the library was not built from the sources beside it: build again"
