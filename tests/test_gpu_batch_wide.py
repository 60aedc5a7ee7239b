"""Batches around the line between LDS-resident circuits and circuits that
advance pass by pass over HBM states: batches of one kind only and of both,
widths on either side of the tile, circuits with different numbers of passes
(a wide one may have a single pass), every tile size of the tuner's range."""

import numpy as np
import pytest

import circuits as C
import oracle as O
from helpers import C128_ATOL, c64_bound

pytestmark = pytest.mark.gpu


def _circuits(which, tile):
    wide = [C.hea_circuit(tile + 1, 2, seed=3, entangler="ladder").bound(),
            C.random_circuit(tile + 3, 1, seed=4, entangler="X"),
            C.random_circuit(tile + 2, 5, seed=5, entangler="Z"),
            C.Circuit(tile + 2, [C.Gate("H", (0,)), C.Gate("RY", (1,), (0,), 0.9)], 0, None, "one_pass"),
            C.random_circuit(tile + 1, 3, seed=6, entangler="X")]
    small = [C.random_circuit(tile, 2, seed=7, entangler="X"), C.random_circuit(tile - 1, 4, seed=8, entangler="Z"),
             C.hea_circuit(5, 3, seed=9, entangler="ladder").bound()]
    mixed = [x for pair in zip(wide, small + small) for x in pair]
    return {"wide": wide, "one_wide": wide[1:2], "small": small, "mixed": mixed}[which]


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("which", ["wide", "one_wide", "small", "mixed"])
@pytest.mark.parametrize("below", [0, 2])
def test_wide_and_resident_circuits(dtype, which, below):
    import paper_1805_00988_amd as sv
    tile = (13 if dtype == "c64" else 12) - below
    circs = _circuits(which, tile)
    zmask = 0b10011
    for keep in (True, False):
        b = sv.Batch(circs, dtype, z_mask=zmask, keep_states=keep)
        b.config(tile, 4 if dtype == "c64" else 3, 64)
        z = b.run().results()
        np.testing.assert_array_equal(b.run().results(), z)
        for i, c in enumerate(circs):
            ref = O.run(c)
            tol = C128_ATOL if dtype == "c128" else c64_bound(max(1, len(c)))
            assert abs(z[i] - O.expectation_z(ref, c.n, [zmask], [1.0])) <= 2 * tol, (i, c.n)
            if keep:
                assert np.max(np.abs(b.state(i) - ref)) <= tol, (i, c.n)
        b.close()
