"""Registers of the tile pass's kernels at full size, from the resource report
the build writes: two workgroups share a compute unit, so complex128 (512
threads, two waves per SIMD each) may use 128 vector registers and complex64
(1024 threads, four waves per SIMD each) 64."""

import json
import os

import pytest

from conftest import ROOT

REPORT = os.path.join(ROOT, "paper_1805_00988_amd", "_build", "kernel_resources.json")


@pytest.mark.parametrize("kernel,instances,most,waves", [("_ZN2sv6k_tileIfLi4E", 8, 64, 8),
                                                          ("_ZN2sv6k_tileIdLi4E", 4, 128, 4)])
def test_two_workgroups_of_the_tile_pass_share_a_compute_unit(kernel, instances, most, waves):
    if not os.path.exists(REPORT):
        pytest.skip("library not built in this tree")
    res = {k: v for k, v in json.load(open(REPORT)).items() if k.startswith(kernel)}
    assert len(res) == instances
    for name, v in res.items():
        assert v["VGPRs"] + v.get("AGPRs", 0) <= most, (name, v)
        assert v["Occupancy"] >= waves and not v.get("ScratchSize", 0), (name, v)
