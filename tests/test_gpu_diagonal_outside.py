"""Uncontrolled diagonal gates whose target lies outside the tile are applied
as a factor per tile, d0 and d1 / d0: gates whose d0 is zero or far smaller than
d1 (projectors, damping) need their target in the tile.  Against the gate's
definition; the oracle's rounding bound for the gates, scaled by the largest
entry."""

import numpy as np
import pytest

import circuits as C
import oracle as O
from helpers import C128_ATOL, c64_bound

pytestmark = pytest.mark.gpu

ENTRIES = {"projector_1": (0.0, 1.0), "projector_0": (1.0, 0.0), "zero": (0.0, 0.0), "scaled_1": (0.0, 0.5j),
           "tiny": (1e-300, 0.7), "tiny_f32": (1e-42, 0.7), "small": (1e-9, 1.0), "damping": (0.6, 0.8)}


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("which", sorted(ENTRIES))
def test_any_diagonal_gate(dtype, which):
    import paper_1805_00988_amd as sv
    n = 17
    u = np.diag(np.array(ENTRIES[which], np.complex128))
    gates = [C.Gate("H", (q,)) for q in range(n)]
    gates += [C.Gate("U", (n - 1,), (), 0.0, -1, u), C.Gate("RX", (0,), (), 0.4), C.Gate("U", (n - 2,), (), 0.0, -1, u),
              C.Gate("RY", (1,), (), 0.3), C.Gate("U", (3,), (), 0.0, -1, u), C.Gate("RX", (n - 1,), (), 0.2)]
    st = sv.State(n, dtype)
    st.set_basis(3).run(gates[:n]).run(gates[n:])
    got = st.numpy()
    st.close()
    want = O.run_gates(n, gates, O.basis_state(n, 3))
    tol = C128_ATOL if dtype == "c128" else c64_bound(len(gates))
    assert np.max(np.abs(got - want)) <= tol
