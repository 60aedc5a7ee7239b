"""Gate lists to sv_op records: the C helper against the general conversion
over the forms a gate's fields may take, and the same errors where the
general conversion raises."""

import numpy as np
import pytest

import circuits as C
import paper_1805_00988_amd as sv
from paper_1805_00988_amd import _lib

G = C.Gate


class Loose:
    def __init__(self, **kw):
        self.__dict__.update({"name": "H", "targets": (0,), "controls": (), "theta": 0.0, "param": -1, "matrix": None})
        self.__dict__.update(kw)


def general(gates, monkeypatch):
    with monkeypatch.context() as m:
        m.setattr(_lib, "fill_ops", lambda *a: -1)
        return sv.ops_from_gates(gates)


FORMS = {
    "random": lambda: C.random_circuit(9, 4, 1, "X").gates,
    "tuple": lambda: tuple(C.qft_circuit(7).gates),
    "params": lambda: C.hea_circuit(5, 2, 3).gates,
    "controls": lambda: [G("X", (0,), tuple(range(1, 12))), G("Z", (3,), (63,)), G("Z", (3,), (5, 5))],
    "lists": lambda: [Loose(targets=[2], controls=[0, 1]), Loose(name="U1", theta=1)],
    "numpy": lambda: [Loose(targets=(np.int64(4),), controls=[np.int32(2)], theta=np.float64(0.5), param=np.int64(3))],
    "float32": lambda: [Loose(name="RX", theta=np.float32(0.3))],
    "array": lambda: [Loose(targets=np.array([5]), controls=np.array([1, 2]))],
    "range": lambda: [Loose(controls=range(2, 4))],
    "bool": lambda: [Loose(targets=(True,), param=False)],
    "integral_float": lambda: [Loose(targets=(2.0,))],
    "matrices": lambda: [G("H", (0,)), G("U", (1,), (), 0.0, -1, C.random_unitary(2, np.random.default_rng(1))),
                         G("U", (2, 0), (3,), 0.0, -1, C.random_unitary(4, np.random.default_rng(2)))],
    "negative": lambda: [Loose(targets=(-1,))],
    "three_targets": lambda: [Loose(targets=(1, 2, 3))],
    "no_angle": lambda: [Loose(theta=None)],
    "queued": lambda: [sv._Op("U1", [np.int64(1)], (2,), 0.25), sv._Op("H", (0,))],
}


@pytest.mark.parametrize("form", sorted(FORMS))
def test_equal_to_the_general_conversion(form, monkeypatch):
    gates = FORMS[form]()
    assert sv.ops_from_gates(gates).tobytes() == general(gates, monkeypatch).tobytes()


def test_plain_lists_take_the_helper():
    gates = C.random_circuit(9, 4, 1, "X").gates
    arr = np.zeros(len(gates), sv.SV_OP_DTYPE)
    assert _lib.fill_ops(gates, arr.ctypes.data, len(gates)) == 0
    assert _lib.fill_ops([Loose(controls=range(2))], arr.ctypes.data, 1) == -1


@pytest.mark.parametrize("bad", [
    [Loose(name="CNOT")], [Loose(targets=())], [Loose(targets=(1 << 40,))], [Loose(controls=(-1,))],
    [Loose(controls=(64,))], [Loose(controls=(63, 63))], [Loose(theta="x")], [Loose(param=None)],
    [Loose(), object()], [Loose(name="U", matrix=np.eye(8))]])
def test_same_errors(bad, monkeypatch):
    with pytest.raises(Exception) as want:
        general(bad, monkeypatch)
    with pytest.raises(type(want.value)):
        sv.ops_from_gates(bad)
