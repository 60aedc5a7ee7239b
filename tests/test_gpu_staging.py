"""Runs whose passes need more staging memory than the handle's arena has:
it is enlarged between the passes of one call, while earlier ones are in
flight, and again by the call's end.  The same call repeated then finds it
large enough, and gives the same amplitudes bit for bit.

Tolerances, with eps the state's precision: 4 sqrt(2) eps per gate, as for
plain passes, plus 2^k * 4 eps per block, of which there is at most one per
gate."""

import math

import numpy as np
import pytest

import circuits as C
import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("k", [4, 5])
def test_arena_grows_within_a_fused_run(dtype, k):
    import paper_1805_00988_amd as sv
    n = 15
    gates = list(C.random_circuit(n, 500, seed=9, entangler="Z").gates)  # more than 1 MiB of records
    st = sv.State(n, dtype)  # a new handle, whose arena is still empty
    runs = []
    for _ in range(3):
        st.set_basis(5).run_fused(gates, k, sv.SV_PREC_NATIVE)
        runs.append(st.numpy())
    st.close()
    np.testing.assert_array_equal(runs[0], runs[1])
    np.testing.assert_array_equal(runs[0], runs[2])
    ref = O.run_gates(n, gates, O.basis_state(n, 5))
    eps = 2.0 ** (-24 if dtype == "c64" else -53)
    assert np.max(np.abs(runs[0] - ref)) <= len(gates) * eps * (4.0 * math.sqrt(2.0) + 2**k * 4.0)
