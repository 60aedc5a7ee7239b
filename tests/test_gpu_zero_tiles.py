"""Tile passes that test their tiles for zeros, which they do from 128 MiB on
while a qubit outside the tile has not been moved since the register was set
to a basis state.  That a tile is left as it is must not show: every run is
compared with the same run on a register whose qubits have all been moved,
whose passes do not look for zeros, bit for bit (zeros of either sign), and the
states of circuits with the oracle.  Starts: basis states, buffers written
after the basis state was set (dense, and with one amplitude at the end of a
lane, a wave, a tile or the register)."""

import math

import numpy as np
import pytest

import circuits as C
import oracle as O
from helpers import C128_ATOL, c64_bound

pytestmark = pytest.mark.gpu

N = {"c64": 24, "c128": 23}  # the smallest that look for zeros
NP = {"c64": np.complex64, "c128": np.complex128}


def _unitaries(qs, count, seed):
    rng = np.random.default_rng(seed)
    return [C.Gate("U", (qs[i % len(qs)],), (), 0.0, -1, C.random_unitary(2, rng)) for i in range(count)]


def _circuit(n, which):
    v = C.random_unitary(4, np.random.default_rng(6))
    return {
        # one pass: a single sweep; one whose stores permute; several sweeps
        "sweep": [C.Gate("H", (n - 1,)), C.Gate("RX", (n - 2,), (), 0.3), C.Gate("T", (1,))],
        "permuted": [C.Gate("H", (n - 1,)), C.Gate("RY", (2,), (), 0.7), C.Gate("X", (0,), (n - 1,)),
                     C.Gate("X", (n - 2,), (n - 3,)), C.Gate("X", (4,))],
        "sweeps": [C.Gate("RX", (q,), (), 0.2 + q) for q in range(9)] + [C.Gate("X", (q + 1,), (q,)) for q in range(8)],
        "two_qubit": [C.Gate("U", (1, n - 2), (), 0.0, -1, v), C.Gate("U", (3, 2), (n - 1,), 0.0, -1, v),
                      C.Gate("RY", (n - 1,), (0,), 0.3)],
        "phases": [C.Gate("H", (0,))] + [C.Gate("U1", (0,), (q,), 0.1 * q) for q in range(1, n)] + [C.Gate("H", (1,))],
        "layers": list(C.random_circuit(n, 2, seed=11, entangler="X").gates),
    }[which]


CIRCUITS = ["sweep", "permuted", "sweeps", "two_qubit", "phases", "layers"]


def _starts(dtype):
    """(name, index of a basis state or the buffer to write) of the register."""
    import torch
    n = N[dtype]
    td = torch.complex64 if dtype == "c64" else torch.complex128
    gen = torch.Generator("cuda").manual_seed(3)
    out = [("0", 0), ("last", (1 << n) - 1)]
    dense = torch.empty(1 << n, dtype=td, device="cuda")
    torch.view_as_real(dense).normal_(generator=gen)
    out.append(("dense", dense.mul_(2.0 ** (-(n + 1) / 2))))
    for x in (1, 63, 1 << 12, (1 << 20) - 1, (1 << n) - 64, (1 << n) - 1):
        one = torch.zeros(1 << n, dtype=td, device="cuda")
        one[x] = -1.0j
        out.append((f"one at {x}", one))
    return out


def _prepare(st, start, all_moved):
    import torch
    st.set_basis(start if isinstance(start, int) else 5)
    if all_moved:
        keep = st.amps.clone()
        st.run([C.Gate("H", (q,)) for q in range(st.n)])
        st.amps.copy_(keep)
    if isinstance(start, torch.Tensor):
        st.amps.copy_(start)


def _both(st, start, run):
    """The state after run() with passes that look for zeros, and what it
    returned; the other passes' state has to be the same."""
    import torch
    _prepare(st, start, True)
    run(st)
    want = torch.view_as_real(st.amps).clone()
    _prepare(st, start, False)
    ret = run(st)
    got = torch.view_as_real(st.amps)
    same = (got == want) | (got.isnan() & want.isnan())
    assert bool(same.all())
    return ret


def _reference(n, start, gates):
    psi = O.basis_state(n, start) if isinstance(start, int) else start.cpu().numpy().astype(np.complex128)
    return O.run_gates(n, gates, psi)


@pytest.mark.parametrize("dtype", sorted(N))
@pytest.mark.parametrize("which", CIRCUITS)
def test_tile_passes(dtype, which):
    import paper_1805_00988_amd as sv
    n = N[dtype]
    gates = _circuit(n, which)
    st = sv.State(n, dtype)
    for name, start in _starts(dtype):
        _both(st, start, lambda s: s.run(gates))
        if name in ("last", "dense", "one at 63"):
            tol = C128_ATOL if dtype == "c128" else c64_bound(len(gates))
            assert np.max(np.abs(st.numpy() - _reference(n, start, gates))) <= tol, name
    st.close()


PRECS = [("c64", "fp32"), ("c64", "bf16"), ("c128", "native")]


@pytest.mark.parametrize("dtype,prec", PRECS)
@pytest.mark.parametrize("k", [4, 5])
def test_dense_blocks(dtype, prec, k):
    """Two blocks of k qubits in one pass, on the matrix cores."""
    import paper_1805_00988_amd as sv
    n = N[dtype]
    code = {"fp32": sv.SV_PREC_FP32, "bf16": sv.SV_PREC_SPLIT_BF16, "native": sv.SV_PREC_NATIVE}[prec]
    # deep enough on each block's qubits to be cheaper than plain sweeps
    sets = [[0, 2, n - 1, n - 2, 4][:k], [1, 3, n - 3, n - 4, n - 5][:k]]
    gates = _unitaries(sets[0], 60, 4) + _unitaries(sets[1], 60, 5)
    st = sv.State(n, dtype)
    for name, start in _starts(dtype):
        blocks = _both(st, start, lambda s: s.run_fused(gates, k, code))
        assert blocks >= 2
        if name in ("last", "dense"):
            eps = 2.0 ** -24
            tol = C128_ATOL
            if dtype == "c64":  # as in the tests of the blocks: per block, and per gate
                tol = blocks * 2.0 ** k * (4.0 * eps if prec == "fp32" else 2.0 ** -15) + len(gates) * 4.0 * math.sqrt(2.0) * eps
            assert np.max(np.abs(st.numpy() - _reference(n, start, gates))) <= tol, name
    st.close()


@pytest.mark.parametrize("dtype,huge", [("c64", 1e200), ("c128", None)])
@pytest.mark.parametrize("fused", [False, True])
def test_entries_beyond_the_precision(dtype, huge, fused):
    """An entry that is infinite in the state's precision makes zeros NaN: then
    every tile runs.  (So large that products with a block's other entries are
    too.)  Complex128 entries are finite or refused."""
    import paper_1805_00988_amd as sv
    n = N[dtype]
    st = sv.State(n, dtype)
    if huge is None:
        bad = C.Gate("U", (1,), (), 0.0, -1, np.array([[1.0, 0.0], [0.0, np.inf]], complex))
        for f in (lambda: st.run([bad, bad]), lambda: st.run_fused([bad, bad], 4)):
            with pytest.raises(sv.SVError):
                f()
        st.close()
        return
    gates = [C.Gate("H", (0,)), C.Gate("U", (1,), (), 0.0, -1, np.array([[huge, 0.0], [1.0, 0.5]], complex)),
             C.Gate("H", (2,))] + (_unitaries([3, 4, n - 1, n - 2], 60, 4) if fused else [])
    run = (lambda s: s.run_fused(gates, 4, sv.SV_PREC_FP32)) if fused else (lambda s: s.run(gates))
    _both(st, 0, run)
    assert np.isnan(st.numpy()[-1 - 2])  # qubit 1 clear: huge times 0
    st.close()
