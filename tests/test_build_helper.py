"""The binding's C helper is not needed to build: where the interpreter's
headers or a C++ compiler are missing there is none, and gate lists are
converted in Python.  It carries the ABI of the interpreter it is built for in
its name."""

import os
import sysconfig

import numpy as np
import pytest

import circuits as C
import paper_1805_00988_amd as sv
from paper_1805_00988_amd import _lib
from paper_1805_00988_amd import build as B


@pytest.mark.parametrize("missing", ["headers", "compiler"])
def test_builds_without(missing, monkeypatch, tmp_path):
    out = tmp_path / "helper.so"
    out.write_bytes(b"of other sources")
    monkeypatch.setattr(B, "PY_OUT", str(out))
    if missing == "headers":
        monkeypatch.setattr(B.sysconfig, "get_paths", lambda *a, **k: {"include": str(tmp_path)})
    else:
        monkeypatch.setenv("CXX", str(tmp_path / "no-such-compiler"))
    assert B.build_py() == ""
    assert not out.exists()  # no helper of other sources is left to be loaded


def test_gate_lists_without_the_helper(monkeypatch, tmp_path):
    gates = C.random_circuit(9, 3, 1, "X").gates
    want = sv.ops_from_gates(gates).tobytes()
    monkeypatch.setattr(_lib, "_fill", None)
    monkeypatch.setattr(_lib, "PY_LIB_PATH", str(tmp_path / "none.so"))
    assert _lib.fill_ops(gates, np.zeros(len(gates), sv.SV_OP_DTYPE).ctypes.data, len(gates)) == -1
    assert sv.ops_from_gates(gates).tobytes() == want


def test_name_holds_the_abi():
    assert B.PY_OUT == _lib.PY_LIB_PATH
    assert os.path.basename(B.PY_OUT) == "libsvpy" + sysconfig.get_config_var("EXT_SUFFIX")
