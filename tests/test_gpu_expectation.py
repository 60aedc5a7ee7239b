"""Z-string expectations at the sizes where the reduction's index splits
change: fewer amplitudes than one round of a workgroup, exactly one, several,
masks on every part of the index, one register mask shared by all terms, the
term limit, and amplitudes or coefficients that are not finite."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _reference(p, masks, coeffs):
    x = np.arange(len(p), dtype=np.uint64)
    h = np.zeros(len(p))
    for m, c in zip(masks, coeffs):
        par = np.zeros(len(p), np.uint64)
        for b in range(64):
            if (m >> b) & 1:
                par ^= (x >> np.uint64(b)) & np.uint64(1)
        h += np.where(par == 1, -c, c)
    return float(np.sum(p * h))


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n", [1, 2, 8, 9, 11, 12, 13, 17, 21])
def test_terms_over_every_index_part(dtype, n):
    import torch
    import paper_1805_00988_amd as sv
    rng = np.random.default_rng(n)
    psi = rng.standard_normal(1 << n) + 1j * rng.standard_normal(1 << n)
    psi /= np.linalg.norm(psi)
    st = sv.State(n, dtype)
    st.amps.copy_(torch.from_numpy(psi).to(st.amps.dtype))
    a = st.amps.cpu().numpy().astype(np.complex128)
    p = a.real ** 2 + a.imag ** 2
    ring = [(1 << i) | (1 << ((i + 1) % n)) for i in range(n)]
    sets = [([0], [1.0]), ([(1 << n) - 1], [-2.5]), (ring, list(rng.standard_normal(len(ring))))]
    sets += [([1 << q], [1.0]) for q in range(n)]
    sets.append(([int(m) for m in rng.integers(0, 1 << n, 64)], list(rng.standard_normal(64))))
    for masks, coeffs in sets:
        # FP64 sums over at most 16 rounds, a 16-point transform, 64 terms and
        # a tree: under 256 roundings of quantities bounded by sum |c|; numpy's
        # pairwise sum adds fewer
        tol = 256 * 2.0 ** -53 * sum(abs(c) for c in coeffs)
        got = st.expectation(masks, coeffs)
        assert abs(got - _reference(p, masks, coeffs)) <= tol, (n, masks)
    st.close()


@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_values_that_are_not_finite(dtype):
    import paper_1805_00988_amd as sv
    n = 13
    st = sv.State(n, dtype)
    masks = [1 << q for q in range(n)]
    st.amps[5] = complex(float("inf"), 0.0)
    coeffs = [2.0 ** -(q + 1) for q in range(n)]  # h(x) is nowhere 0
    assert st.expectation(masks, coeffs) == -np.inf  # h(5) < 0
    assert st.expectation([0], [3.0]) == np.inf
    st.amps[5] = complex(float("nan"), 0.0)
    assert np.isnan(st.expectation(masks, coeffs))
    st.set_basis(0)
    assert st.expectation([1, 2], [np.inf, 1.0]) != st.expectation([1, 2], [1.0, 1.0])
    st.close()
