"""The passes that sv_run's tiled mode forms (sv_schedule with tile_qubits 0):
its own tiles, of 14 qubits in complex64 and 13 in complex128.  On the host,
as for tiles of 12 qubits: the gates replayed pass by pass give the in-order
oracle run, gates that share a qubit keep their order, every tile holds the low
block, at most its number of qubits and the targets of its gates.  On the GPU:
sv_run launches exactly these passes."""

import ctypes

import numpy as np
import pytest

import circuits as C
import oracle as O
import paper_1805_00988_amd as sv
from test_schedule_host import KINDS, LOW, circuit, mask, tile_exempt

O.build(force=False)

TILE = {"c64": 14, "c128": 13}


def _check(circ, n, dtype, gp, tiles, most):
    params = circ.params
    assert gp.min() == 0 and sorted(set(gp.tolist())) == list(range(len(tiles)))
    low = mask(range(min(n, LOW[dtype])))
    for p, S in enumerate(tiles):
        members = [i for i in range(len(circ.gates)) if gp[i] == p]
        if S == 0:
            assert len(members) == 1
            continue
        assert bin(S).count("1") <= most and S & low == low and S < (1 << n)
        for i in members:
            if not tile_exempt(circ.gates[i], params):
                assert mask(circ.gates[i].targets) & ~S == 0, (p, i)
    last = {}
    for i, g in enumerate(circ.gates):
        for q in g.qubits:
            assert gp[last.get(q, i)] <= gp[i]
            last[q] = i


@pytest.mark.parametrize("level", [0, 1, 2])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [15, 16])
def test_passes_preserve_the_circuit(kind, n, dtype, level):
    circ = circuit(kind, n, seed=n + level)
    gp, tiles = sv.sv_schedule(n, dtype, circ.gates, level, params=circ.params, tile_qubits=0)
    _check(circ, n, dtype, gp, tiles, TILE[dtype])
    own = sv.sv_schedule(n, dtype, circ.gates, level, params=circ.params, tile_qubits=TILE[dtype])
    assert own[1] == tiles and np.array_equal(own[0], gp)
    order = sorted(range(len(circ.gates)), key=lambda i: (gp[i], i))
    got = O.run_gates(n, [circ.gates[i] for i in order], O.basis_state(n, circ.basis))
    np.testing.assert_allclose(got, O.run(circ), atol=1e-12, rtol=0)


def test_a_register_of_one_tile_is_one_pass():
    for dtype, n in (("c64", 14), ("c128", 13)):
        circ = C.random_circuit(n, 8, 3, "X", n // 2)
        gp, tiles = sv.sv_schedule(n, dtype, circ.gates, tile_qubits=0)
        assert tiles == [(1 << n) - 1] and set(gp.tolist()) == {0}


@pytest.mark.parametrize("n,dtype,most", [(32, "c64", (48, 39, 33)), (30, "c128", (36, 31, 28))])
def test_larger_tiles_take_no_more_passes(n, dtype, most):
    """The benchmark's circuits: no more passes than on tiles of 12 qubits (the
    numbers at levels 0, 1, 2), and no more at a higher level."""
    qft, rnd = C.config1(n, 0)
    got = []
    for lv in (0, 1, 2):
        gp, tiles = sv.sv_schedule(n, dtype, rnd.gates, lv, tile_qubits=0)
        _check(rnd, n, dtype, gp, tiles, TILE[dtype])
        got.append(len(tiles))
    assert all(g <= m for g, m in zip(got, most)) and got == sorted(got, reverse=True)
    assert all(len(sv.sv_schedule(n, dtype, qft.gates, lv, tile_qubits=0)[1]) <= 5 for lv in (0, 1, 2))


@pytest.mark.parametrize("dtype,bad", [("c64", 6), ("c64", 15), ("c128", 5), ("c128", 14), ("c64", -1)])
def test_tiles_outside_the_range_are_refused(dtype, bad):
    with pytest.raises(sv.SVError):
        sv.sv_schedule(16, dtype, C.random_circuit(16, 2, 0, "X", 8).gates, 0, tile_qubits=bad)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [13, 17, 24])
def test_sv_run_launches_these_passes(kind, n, dtype):
    import torch  # noqa: F401  (its HIP runtime first)
    from paper_1805_00988_amd import _lib
    lib = _lib.load()
    circ = circuit(kind, n, seed=n)
    tiles = sv.sv_schedule(n, dtype, circ.gates, params=circ.params, tile_qubits=0)[1]
    st = sv.State(n, dtype)
    _lib.check(lib.sv_timing(st.handle, 1))
    st.run(circ.gates, circ.params)
    stats, count = (_lib.sv_kernel_stat * 16)(), ctypes.c_int()
    _lib.check(lib.sv_timing_read(st.handle, stats, 16, ctypes.byref(count)))
    launches = {stats[i].name.decode(): stats[i].launches for i in range(count.value)}
    st.close()
    assert launches.pop("tile_pass", 0) == sum(1 for S in tiles if S)
    assert sum(launches.values()) == sum(1 for S in tiles if not S)
