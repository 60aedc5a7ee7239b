"""Registers that hold mostly zeros: tiles and waves of zeros are left as
they are, which must not show.  Basis states at the ends of the register and
of a tile, gates that move few qubits, buffers written after the basis state
was set (dense, and with a single amplitude in a tile's last wave), and
batches whose circuits leave qubits untouched."""

import numpy as np
import pytest

import circuits as C
import oracle as O
from helpers import C128_ATOL, c64_bound, random_state

pytestmark = pytest.mark.gpu

DTYPES = ["c64", "c128"]


def _tol(dtype, gates):
    return C128_ATOL if dtype == "c128" else c64_bound(len(gates))


def _gates(n, which):
    top = C.Gate("H", (n - 1,))
    u = C.random_unitary(2, np.random.default_rng(5))
    v = C.random_unitary(4, np.random.default_rng(6))
    return {
        "diagonal": [C.Gate("T", (0,)), C.Gate("U1", (n - 1,), (3,), 0.7), C.Gate("RZ", (n - 2,), (), 0.4)],
        "exchange": [C.Gate("X", (n - 1,)), C.Gate("X", (0,), (n - 1,)), C.Gate("X", (n - 2,), (1,))],
        "few": [top, C.Gate("X", (0,), (n - 1,)), C.Gate("U", (2,), (), 0.0, -1, u),
                C.Gate("U", (1, n - 2), (), 0.0, -1, v), C.Gate("RY", (n - 1,), (0,), 0.3)],
        "random": list(C.random_circuit(n, 4, seed=11, entangler="X").gates),
        "qft": list(C.qft_circuit(n).gates),
    }[which]


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("which", ["diagonal", "exchange", "few", "random", "qft"])
@pytest.mark.parametrize("tiled", [True, False])
def test_from_basis_states(dtype, which, tiled):
    import paper_1805_00988_amd as sv
    n = 16
    gates = _gates(n, which)
    st = sv.State(n, dtype)
    for x in (0, 1, (1 << 12) - 1, 1 << 12, (1 << n) - 1, 0b1010011000101101):
        st.set_basis(x).run(gates, mode=sv.SV_RUN_TILED if tiled else sv.SV_RUN_PER_GATE)
        ref = O.run_gates(n, gates, O.basis_state(n, x))
        assert np.max(np.abs(st.numpy() - ref)) <= _tol(dtype, gates), x
    st.close()


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("k", [4, 5])
def test_fused_from_basis_states(dtype, k):
    import paper_1805_00988_amd as sv
    n = 16
    gates = list(C.random_circuit(n, 4, seed=12, entangler="Z").gates)
    st = sv.State(n, dtype)
    for x in (0, (1 << n) - 1):
        st.set_basis(x).run_fused(gates, k, sv.SV_PREC_NATIVE)
        ref = O.run_gates(n, gates, O.basis_state(n, x))
        # a block of 2^k terms per output at worst for every gate
        tol = C128_ATOL if dtype == "c128" else 2.0 ** k * 4.0 * 2.0 ** -24 * len(gates)
        assert np.max(np.abs(st.numpy() - ref)) <= tol, x
    st.close()


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("tiled", [True, False])
def test_buffer_written_after_the_basis_state(dtype, tiled):
    import torch
    import paper_1805_00988_amd as sv
    n = 15
    gates = _gates(n, "random")
    np_dt = np.complex64 if dtype == "c64" else np.complex128
    single = np.zeros(1 << n, np_dt)
    single[(1 << n) - 1 - 63] = -1.0j
    for psi in (random_state(n, 3).astype(np_dt), single):
        st = sv.State(n, dtype)
        st.set_basis(5)
        st.amps.copy_(torch.from_numpy(psi))
        st.run(gates, mode=sv.SV_RUN_TILED if tiled else sv.SV_RUN_PER_GATE)
        ref = O.run_gates(n, gates, psi.astype(np.complex128))
        assert np.max(np.abs(st.numpy() - ref)) <= _tol(dtype, gates)
        st.close()


@pytest.mark.parametrize("dtype", DTYPES)
def test_batch_with_untouched_qubits(dtype):
    import paper_1805_00988_amd as sv
    n = 16
    circs = [C.Circuit(n, _gates(n, w), 0, None, w) for w in ("diagonal", "exchange", "few", "random", "qft")]
    circs.append(C.Circuit(n, [C.Gate("X", (n - 1,))], 0, None, "top"))
    circs.append(C.Circuit(n, _gates(n, "random")[:9], 0, None, "part"))
    zmask = (1 << (n - 1)) | 1
    for keep in (True, False):
        b = sv.Batch(circs, dtype, z_mask=zmask, keep_states=keep)
        z = b.run().results()
        np.testing.assert_array_equal(b.run().results(), z)
        for i, c in enumerate(circs):
            ref = O.run(c)
            tol = _tol(dtype, c.gates)
            assert abs(z[i] - O.expectation_z(ref, n, [zmask], [1.0])) <= 2 * tol, c.name
            if keep:
                assert np.max(np.abs(b.state(i) - ref)) <= tol, c.name
        b.close()
