"""The C marshalling of nm_gemm against the ctypes one: both hand the library the same arguments (CPU, a recorder in the
library's place), and what the C side does not take it leaves to ctypes."""
import ctypes
import os
import sysconfig

import numpy as np
import pytest
import torch

from paper_2206_15014_amd import binding, build

T, K, O = 5, 32, 12


@pytest.fixture()
def recorder():
    lib = binding._load()
    if not os.path.exists(os.path.join(sysconfig.get_paths()["include"], "Python.h")):
        pytest.skip("no Python.h, so no marshalling module: the binding goes through ctypes alone")
    assert binding._native is not None, "the marshalling module is not built"
    seen = []
    proto = ctypes.CFUNCTYPE(ctypes.c_int, *lib.nm_gemm.argtypes)

    @proto
    def record(*args):
        seen.append(args)
        return 7

    class Lib:
        nm_gemm = record

    binding._native.bind(ctypes.cast(record, ctypes.c_void_p).value)
    yield Lib, seen
    binding._native.bind(ctypes.cast(lib.nm_gemm, ctypes.c_void_p).value)


def _tensors():
    wide = torch.zeros(T, 2 * K, dtype=torch.int8)
    return {"X": torch.zeros(T, K, dtype=torch.int8), "Xwide": wide[:, :K], "vals": torch.zeros(64, dtype=torch.uint8),
            "meta": torch.zeros(64, dtype=torch.uint8), "scales": torch.zeros(O), "bias": torch.zeros(O),
            "acc": torch.zeros(T, O, dtype=torch.int32), "out": torch.zeros(T, O + 4)[:, :O], "dev": torch.ones(1)}


# X, act_scale, bias, acc, out, ldo, stream, act_scale_dev
CALLS = [("X", 0.25, "bias", None, "out", None, 0, None), ("Xwide", 3, None, "acc", None, None, 5, "dev"), ("X", 1e300, None, None, None, None, 0, None),
         ("X", float("nan"), "bias", "acc", "out", 99, 2 ** 63 + 8, None), ("X", True, 4096, "acc", 8192, None, 0, None), ("X", -0.0, None, None, "out", -3, 0, None)]


@pytest.mark.parametrize("call", CALLS)
def test_same_arguments(recorder, call):
    lib, seen = recorder
    t = _tensors()
    X, act, bias, acc, out, ldo, stream, dev = (t.get(a, a) if isinstance(a, str) else a for a in call)
    args = (X, act, t["vals"], t["meta"], t["scales"], O, 2, 4, 8, bias, acc, out, 2, ldo, stream, 1, dev)
    assert binding._native.gemm(*args) == 7
    assert binding._gemm_ctypes(lib, *args) == 7
    assert len(seen) == 2
    for a, b in zip(*seen):
        assert a == b or (a != a and b != b)


@pytest.mark.parametrize("place, value", [(5, 12.0), (6, np.int64(2)), (1, np.float32(1.0)), (1, "1"), (13, 1.5), (14, None)])
def test_left_to_ctypes(recorder, place, value):
    _, seen = recorder
    t = _tensors()
    args = [t["X"], 0.5, t["vals"], t["meta"], t["scales"], O, 2, 4, 8, None, None, t["out"], 2, None, 0, 1, None]
    args[place] = value
    assert binding._native.gemm(*args) is None and not seen


def test_exceptions_pass_through(recorder):
    t = _tensors()
    args = [t["X"], 0.5, t["vals"], t["meta"], object(), O, 2, 4, 8, None, None, t["out"], 2, None, 0, 1, None]
    with pytest.raises(AttributeError):
        binding._native.gemm(*args)
    args[4], args[0] = t["scales"], t["X"].reshape(-1)
    assert binding._native.gemm(*args) is None     # not two dimensions: ctypes' path raises as it did


def test_module_is_of_this_interpreter():
    """Compiled against one interpreter's own structures, so named for it alone: plain `.so` every interpreter would load."""
    suffix = sysconfig.get_config_var("EXT_SUFFIX")
    assert suffix != ".so" and build.PYTHON_MODULE == os.path.join(build.HERE, "_nm_python" + suffix)
    assert [n for n in os.listdir(build.HERE) if n.startswith("_nm_python.") and n.endswith(".so")] in ([], [os.path.basename(build.PYTHON_MODULE)])


def test_no_module_outlives_its_library(tmp_path):
    """A build that makes none leaves none: an older module would call the new library's function with the old arguments."""
    for name in ("_nm_python.so", "_nm_python" + sysconfig.get_config_var("EXT_SUFFIX"), "_nm_python.cpython-38-x86_64-linux-gnu.so", "_nm_other.so"):
        (tmp_path / name).write_bytes(b"")
    build.remove_python_modules(str(tmp_path))
    assert os.listdir(tmp_path) == ["_nm_other.so"]
    assert build.build_python_module(str(tmp_path), str(tmp_path / "made.so"), "no compiler is asked") is False
    assert os.listdir(tmp_path) == ["_nm_other.so"]


@pytest.mark.parametrize("native", [False, True])
@pytest.mark.parametrize("status", [0, -2])
def test_entry_point_on_either_side(monkeypatch, status, native):
    """nm_gemm itself, without the module (as where it is not built) and with one that leaves the call to ctypes."""
    seen = []

    class Lib:
        @staticmethod
        def nm_gemm(*args):
            seen.append(args)
            return status

        @staticmethod
        def nm_status_string(code):
            return b"refused"

    class LeavesIt:
        @staticmethod
        def gemm(*args):
            return None

    monkeypatch.setattr(binding, "_lib", Lib)
    monkeypatch.setattr(binding, "_native", LeavesIt if native else None)
    t = _tensors()
    call = lambda: binding.nm_gemm(t["Xwide"], 0.25, t["vals"], t["meta"], t["scales"], O, 2, 4, 8, bias=t["bias"], out=t["out"], out_dtype=2, stream=16, layout=1)
    if status:
        with pytest.raises(binding.NMError) as e:
            call()
        assert e.value.code == status
    else:
        acc, out = call()
        assert acc is None and out is t["out"]
    assert seen[0] == (t["Xwide"].data_ptr(), T, K, 2 * K, 0.25, None, t["vals"].data_ptr(), t["meta"].data_ptr(), t["scales"].data_ptr(), O, 2, 4, 8, 1,
                       t["bias"].data_ptr(), None, t["out"].data_ptr(), 2, O + 4, 16)
