"""Sampling over blocks and runs of blocks: one block, one run, several runs,
more runs than a wave searches at once, mass only at the edges of runs; and
collapses whose measured qubits lie inside a vector, a wave and above."""

import numpy as np
import pytest

import oracle as O
from helpers import EPS32, EPS64, random_state

pytestmark = pytest.mark.gpu

NP_DT = {"c64": np.complex64, "c128": np.complex128}


def _state(n, dtype, psi):
    import torch
    import paper_1805_00988_amd as sv
    st = sv.State(n, dtype)
    st.amps.copy_(torch.from_numpy(psi.astype(NP_DT[dtype])))
    return st


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n", [8, 11, 12, 13, 18, 20])
def test_mass_at_the_edges_of_runs(dtype, n):
    rng = np.random.default_rng(n)
    block = 1 << max(min(n, 8), n - 16)
    n_blocks = (1 << n) // block
    # the first and last amplitude of the first, second and last blocks of runs of 16
    at = sorted({b * block + e for b in range(n_blocks) if b % 16 in (0, 1, 15) for e in (0, block - 1)})
    psi = np.zeros(1 << n, np.complex128)
    psi[at] = rng.standard_normal(len(at)) + 1j * rng.standard_normal(len(at))
    psi[at[len(at) // 2]] = 0.0
    psi = (psi / np.linalg.norm(psi)).astype(NP_DT[dtype]).astype(np.complex128)
    # targets inside every outcome's interval, away from its ends by more than rounding
    p = np.abs(psi) ** 2
    hit = np.flatnonzero(p)
    c = np.cumsum(p)
    hit = hit[:: max(1, len(hit) // 4000)]
    u = (c[hit] - 0.5 * p[hit]) / c[-1]
    keep = p[hit] > 1e4 * len(p) * EPS64 * c[-1]
    u, hit = np.concatenate([u[keep], [0.0, 1.0 - EPS64]]), hit[keep]
    st = _state(n, dtype, psi)
    got = st.sample(u)
    np.testing.assert_array_equal(got[:-2], hit)
    np.testing.assert_array_equal(got[:-2], O.sample(psi, n, u)[:-2])
    assert got[-2] == np.flatnonzero(p)[0] and got[-1] == np.flatnonzero(p)[-1]
    st.close()


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n,mask", [(1, 1), (6, 0b1), (6, 0b100001), (13, 0b1000000000011), (14, 0b10000010000000)])
def test_collapse_leaves_only_the_outcome(dtype, n, mask):
    psi = random_state(n, 40 + n).astype(NP_DT[dtype]).astype(np.complex128)
    for value in (0, mask, mask & -mask):
        st = _state(n, dtype, psi)
        ref = psi.copy()
        p = st.collapse(mask, value)
        p_ref = O.collapse(ref, n, mask, value)
        assert abs(p - p_ref) <= 2.0 ** n * EPS64
        got = st.numpy()
        out = (np.arange(1 << n) & mask) != value
        assert not np.any(got[out])
        # one rounding of the factor, one of the product
        eps = EPS64 * 2.0 ** n if dtype == "c128" else 4 * EPS32
        assert np.max(np.abs(got - ref)) <= eps * np.max(np.abs(ref))
        st.close()
