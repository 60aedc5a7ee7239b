"""Complex64 gates that round differently for different states keep the entries
that are exact: the norm correction of a pass, which scales its last one-qubit
gate, takes back only what the rounding does to every state alike.  Each
circuit takes one amplitude through powers of 0.5 or of 1 only, so its value is
exact in complex64 (no tolerance); the gate's other entries round."""

import numpy as np
import pytest

import circuits as C

pytestmark = pytest.mark.gpu

# gate, target's value, what the amplitude is multiplied by
GATES = {
    "diagonal": (np.diag([0.5, 0.7]), 0, 0.5),
    "real": (np.array([[0.5, 0.7], [0.0, 0.3]]), 0, 0.5),
    "complex": (np.array([[0.5, 0.7j], [0.0, 0.3 + 0.7j]]), 0, 0.5),
    "unitary": (np.diag([np.exp(0.3j), 1.0]), 1, 1.0),
}


@pytest.mark.parametrize("which", sorted(GATES))
@pytest.mark.parametrize("n,q", [(3, 1), (8, 7), (15, 14)])
def test_exact_entries_stay_exact(which, n, q):
    import paper_1805_00988_amd as sv
    u, bit, factor = GATES[which]
    gates = [C.Gate("U", (q,), (), 0.0, -1, u.astype(np.complex128))] * 100
    st = sv.State(n, "c64")
    st.set_basis(bit << q).run(gates)
    got = st.numpy()
    st.close()
    want = np.zeros(1 << n, np.complex64)
    want[bit << q] = factor ** 100
    np.testing.assert_array_equal(got, want)
