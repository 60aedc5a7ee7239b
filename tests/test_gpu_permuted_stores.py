"""Tile passes whose X and controlled X gates are applied by permuted stores:
passes of such gates alone (one sweep that reads and writes the state),
between sweeps and at a pass's end, with controls in and outside the tile,
controls of both kinds at once and several controls (which stay records),
from the narrowest register whose sweeps can permute."""

import numpy as np
import pytest

import circuits as C
import oracle as O
from helpers import assert_state_close, random_state

pytestmark = pytest.mark.gpu

NP_DT = {"c64": np.complex64, "c128": np.complex128}


def _gates(n, kind, seed):
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(6 * n):
        q = [int(x) for x in rng.choice(n, 3, replace=False)]
        r = rng.random()
        if kind == "only" or r < 0.6:
            k = int(rng.choice([0, 1, 1, 1, 1, 2]))
            out.append(C.Gate("X", (q[0],), tuple(q[1:1 + k])))
        elif r < 0.7:
            out.append(C.Gate("U1", (q[0],), (q[1],), float(rng.uniform(0, 6))))
        elif r < 0.75 and kind == "pairs":
            out.append(C.Gate("U", (q[0], q[1]), (), 0.0, -1, C.random_unitary(4, rng)))
        else:
            name = ["H", "RY", "RX", "RZ", "T", "Y"][int(rng.integers(6))]
            out.append(C.Gate(name, (q[0],), (q[1],) if rng.random() < 0.2 else (), float(rng.uniform(0, 6))))
    return out


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("kind", ["only", "mixed", "pairs"])
@pytest.mark.parametrize("n", [8, 9, 10, 12, 13, 15, 17])
def test_circuits_of_x_gates(dtype, kind, n):
    import torch
    import paper_1805_00988_amd as sv
    psi = random_state(n, 70 + n).astype(NP_DT[dtype])
    for seed in (n, 100 + n):
        gates = _gates(n, kind, seed)
        st = sv.State(n, dtype)
        st.amps.copy_(torch.from_numpy(psi))
        st.run(gates)
        ref = O.run_gates(n, gates, psi.astype(np.complex128))
        if kind == "only":  # a permutation changes no amplitude
            np.testing.assert_array_equal(st.numpy(), ref.astype(NP_DT[dtype]))
        assert_state_close(st.numpy(), ref, dtype, len(gates))
        st.close()


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("entangler", ["ladder", "ring"])
def test_chains(dtype, entangler):
    import paper_1805_00988_amd as sv
    n = 16
    c = C.hea_circuit(n, 3, seed=2, entangler=entangler).bound()
    st = sv.State(n, dtype)
    st.set_basis(9).run(c.gates, c.params)
    assert_state_close(st.numpy(), O.run_gates(n, c.gates, O.basis_state(n, 9)), dtype, len(c))
    st.close()
