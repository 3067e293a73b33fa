"""Every source of the library is accepted by the compiler as it stands in the tree, whatever built library lies beside it."""
import os
import shutil
import subprocess

import pytest

from paper_2206_15014_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="no compiler")
@pytest.mark.parametrize("source", sorted({s for s, _, _ in build.SOURCES}))
def test_front_end(source):
    extra = next(e for s, e, _ in build.SOURCES if s == source)
    flags = [f for f in build.HIPCC_FLAGS if f != "-shared"]
    res = subprocess.run([HIPCC, *flags, *extra, "-fsyntax-only", os.path.join(build.CSRC, source)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout
