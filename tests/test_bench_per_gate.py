"""bench.py's rates of the streamed gate kernels are taken on a dense register
(the kernels leave zeros as they are, so a basis state would count bytes that
are not moved), and the register is left in the circuits' final state.  On the
CPU: a stand-in for the library that applies the gates with the oracle."""

import types

import numpy as np
import pytest

import bench
import circuits as C
import oracle as O
import paper_1805_00988_amd as sv
from paper_1805_00988_amd import _lib

torch = pytest.importorskip("torch")
O.build(force=False)


def test_rates_are_taken_on_a_dense_register(monkeypatch):
    n = 8
    qft, rnd = C.config1(n, 0)
    amps = torch.zeros(1 << n, dtype=torch.complex128)
    gates = {}
    zeros = []

    class Lib:
        def sv_set_basis(self, h, x):
            amps.copy_(torch.from_numpy(O.basis_state(n, x)))
            return 0

        def sv_timing(self, h, on):
            return 0

        def sv_run(self, h, ops, count, params, n_params, mode):
            if mode == sv.SV_RUN_PER_GATE:
                zeros.append(int((amps == 0).sum()))
            else:
                amps.copy_(torch.from_numpy(O.run_gates(n, list(gates[count]), amps.numpy().copy())))
            return 0

    gates[len(qft.gates)], gates[len(rnd.gates)] = qft.gates, rnd.gates
    assert len(gates) == 2
    monkeypatch.setattr(bench, "read_stats", lambda lib, h: {"gate1_stream": (1, 1.0, 1.0, 0.0)})
    reg = {"n": n, "dtype": "c128", "state": types.SimpleNamespace(handle=None, amps=amps), "qft": qft, "rnd": rnd,
           "ops_qft": sv.ops_from_gates(qft.gates), "ops_rnd": sv.ops_from_gates(rnd.gates)}
    out = bench.per_gate_breakdown([reg], Lib(), sv, _lib)
    assert out[f"{n}q_c128"]["gate1_stream"]["all"]["launches"] == len(qft.gates) + len(rnd.gates)
    assert len(zeros) == len(qft.gates) + len(rnd.gates) and max(zeros) == 0
    want = O.run_gates(n, list(qft.gates) + list(rnd.gates), O.basis_state(n, qft.basis))
    np.testing.assert_allclose(amps.numpy(), want, atol=1e-12, rtol=0)
