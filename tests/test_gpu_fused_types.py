"""Fused blocks of a complex128 register are FP64 whatever arithmetic the call
names: every call forms the same passes and blocks, so its amplitudes are the
same bit for bit, and within 1e-12 of the oracle's."""

import numpy as np
import pytest

import circuits as C
import oracle as O
from helpers import C128_ATOL

pytestmark = pytest.mark.gpu


def _deep_on_few_qubits(n, k):
    """Gates enough on k qubits for a block to be cheaper than plain sweeps."""
    rng = np.random.default_rng(4)
    qs = [0, 3, n // 2, n - 3, n - 1][:k]
    return [C.Gate("U", (qs[i % k],), (), 0.0, -1, C.random_unitary(2, rng)) for i in range(32)]


CIRCUITS = {
    "few": _deep_on_few_qubits,
    "random_x": lambda n, k: list(C.random_circuit(n, 24, seed=3, entangler="X").gates),
    "random_z": lambda n, k: list(C.random_circuit(n, 24, seed=3, entangler="Z").gates),
}


@pytest.mark.parametrize("which", sorted(CIRCUITS))
@pytest.mark.parametrize("k", [4, 5])
def test_complex128_blocks_do_not_depend_on_the_precision(which, k):
    import paper_1805_00988_amd as sv
    n = 16
    gates = CIRCUITS[which](n, k)
    st = sv.State(n, "c128")
    blocks, amps = [], []
    for prec in (sv.SV_PREC_NATIVE, sv.SV_PREC_FP32, sv.SV_PREC_SPLIT_BF16):
        blocks.append(st.set_basis(5).run_fused(gates, k, prec))
        amps.append(st.numpy())
    st.close()
    assert blocks[0] == blocks[1] == blocks[2]
    assert which != "few" or blocks[0] > 0
    np.testing.assert_array_equal(amps[1], amps[0])
    np.testing.assert_array_equal(amps[2], amps[0])
    assert np.max(np.abs(amps[0] - O.run_gates(n, gates, O.basis_state(n, 5)))) <= C128_ATOL
