"""Staging memory that runs out, on the CPU: libsv.so on a stand-in for the HIP
runtime (fake_hip.cpp) that runs no kernel, counts launches and refuses
allocations.  A call that fails for lack of memory has launched nothing, so the
state is unchanged; one that has launched passes always finishes, reusing the
arena and splitting a pass that does not fit it."""

import json
import os
import shutil
import subprocess
import sys

import pytest

from conftest import ROOT

SCRIPT = r"""
import ctypes, json, sys
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)  # before libsv.so, which then calls it
fake.fake_limit.argtypes = [ctypes.c_size_t]
fake.fake_launches.argtypes = [ctypes.c_char_p]
fake.fake_launches.restype = ctypes.c_long
fake.fake_live.restype = ctypes.c_long
import numpy as np
import circuits as C
import paper_1805_00988_amd as sv
from paper_1805_00988_amd import _lib
lib = _lib.load()
out = {}
ANY = (1 << 64) - 1

def alloc(n, dtype):
    h = ctypes.c_void_p()
    _lib.check(lib.sv_alloc(n, _lib.SV_C64 if dtype == "c64" else _lib.SV_C128, None, None, ctypes.byref(h)))
    return h

def plain(h, gates):
    ops = sv.ops_from_gates(gates)
    return lib.sv_run(h, sv._opptr(ops), len(gates), None, 0, sv.SV_RUN_TILED)

def fused(h, gates, k, prec, blocks=None):
    ops, nb = sv.ops_from_gates(gates), ctypes.c_int()
    rc = lib.sv_run_fused(h, sv._opptr(ops), len(gates), None, 0, k, prec, ctypes.byref(nb))
    return rc, nb.value

def counted(f):
    fake.fake_reset()
    rc = f()
    return {"rc": rc, "tile": fake.fake_launches(b"k_tile"), "dense": fake.fake_launches(b"k_dense")}

def units(qs, count, seed):
    rng = np.random.default_rng(seed)
    return [C.Gate("U", (qs[i % len(qs)],), (), 0.0, -1, C.random_unitary(2, rng)) for i in range(count)]

few = [C.Gate("H", (0,)), C.Gate("RX", (1,), (), 0.3), C.Gate("X", (2,), (1,))]
one_pass = units(list(range(7)), 20000, 1)                   # more than 1 MiB of records in one pass
layers = list(C.random_circuit(25, 3, 3, "X").gates)         # the same behind other passes
large_last = layers + [C.Gate("H", (24,))] + [C.Gate("X", (q,), (24,)) for q in range(7)] + one_pass
many = list(C.random_circuit(25, 300, 3, "X").gates)         # more than 1 MiB in many passes
many_20 = list(C.random_circuit(20, 1500, 3, "X").gates)
wide = list(C.random_circuit(13, 2000, 3, "Z").gates)         # one fused pass, cheaper as plain sweeps
dense = []                                                   # blocks of 5, some with variants, more than 1 MiB of operands
for i in range(90):
    qs = [(3 * i + j) % 12 for j in range(5)]
    dense += units(qs, 40, 10 + i) + [C.Gate("Z", (qs[j],), (20 + j,)) for j in range(4)]
    dense += [C.Gate("X", (qs[j + 1],), (qs[j],)) for j in range(4)]

cases = {
    "plain_one_pass": (25, "c64", lambda h: plain(h, one_pass)),
    "plain_large_last": (25, "c64", lambda h: plain(h, large_last)),
    "plain_many": (25, "c64", lambda h: plain(h, many)),
    "plain_one_pass_c128": (24, "c128", lambda h: plain(h, one_pass)),
    "fused_plain": (13, "c64", lambda h: fused(h, wide, 4, sv.SV_PREC_FP32)),
    "fused_blocks": (26, "c64", lambda h: fused(h, dense, 5, sv.SV_PREC_FP32)),
    "fused_blocks_bf16": (26, "c64", lambda h: fused(h, dense, 5, sv.SV_PREC_SPLIT_BF16)),
    "fused_blocks_c128": (25, "c128", lambda h: fused(h, dense, 5, sv.SV_PREC_NATIVE)),
}
for name, (n, dtype, call) in cases.items():
    r = {}
    h = alloc(n, dtype)
    fake.fake_limit(0)
    r["none"] = counted(lambda: call(h))             # no arena, and none to be had
    fake.fake_limit(ANY)
    lib.sv_free(h)
    h = alloc(n, dtype)
    fused(h, few, 4, sv.SV_PREC_NATIVE)              # an arena of 1 MiB
    fake.fake_limit(0)
    r["small"] = counted(lambda: call(h))            # and no larger one
    fake.fake_limit(ANY)
    r["free"] = counted(lambda: call(h))
    r["again"] = counted(lambda: call(h))
    lib.sv_free(h)
    r["live"] = fake.fake_live()
    out[name] = r
# room for an arena just large enough, not for one four times the old one
h = alloc(25, "c64")
fused(h, few, 4, sv.SV_PREC_NATIVE)
fake.fake_limit(4 << 20)
out["just_enough"] = counted(lambda: plain(h, one_pass))
fake.fake_limit(ANY)
lib.sv_free(h)
# states below 256 MiB stage all passes before the first launch
h = alloc(20, "c64")
fused(h, few, 4, sv.SV_PREC_NATIVE)
fake.fake_limit(0)
out["staged_together"] = counted(lambda: plain(h, many_20))
fake.fake_limit(ANY)
lib.sv_free(h)
out["live"] = fake.fake_live()
print(json.dumps(out))
"""


@pytest.fixture(scope="module")
def results(tmp_path_factory):
    cxx = shutil.which(os.environ.get("CXX") or "g++")
    if not cxx:
        pytest.skip("no C++ compiler")
    fake = tmp_path_factory.mktemp("fake") / "fake_hip.so"
    subprocess.run([cxx, "-O1", "-shared", "-fPIC", os.path.join(ROOT, "tests", "fake_hip.cpp"), "-o", str(fake)],
                   check=True)
    r = subprocess.run([sys.executable, "-c", SCRIPT, str(fake)], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    return json.loads(r.stdout.splitlines()[-1])


CASES = ["plain_one_pass", "plain_large_last", "plain_many", "plain_one_pass_c128", "fused_plain", "fused_blocks",
         "fused_blocks_bf16", "fused_blocks_c128"]


def _rc(x):
    return x["rc"][0] if isinstance(x["rc"], list) else x["rc"]


@pytest.mark.parametrize("name", CASES)
def test_without_any_arena_nothing_is_launched(results, name):
    r = results[name]["none"]
    assert _rc(r) < 0 and r["tile"] == 0 and r["dense"] == 0


@pytest.mark.parametrize("name", CASES)
def test_a_call_goes_on_in_the_arena_it_has(results, name):
    r = results[name]
    small, free = r["small"], r["free"]
    assert _rc(free) == 0 and _rc(small) == 0
    assert small["rc"] == free["rc"]  # as many blocks
    if name != "plain_many":  # its passes fit one by one; these do not
        assert small["tile"] + small["dense"] > free["tile"] + free["dense"]
    assert (small["dense"] > 0) == (free["dense"] > 0) == name.startswith("fused_blocks")
    assert r["again"] == free


@pytest.mark.parametrize("name", CASES)
def test_every_allocation_is_given_back(results, name):
    assert results[name]["live"] == 0 and results["live"] == 0


def test_an_arena_just_large_enough(results):
    assert _rc(results["just_enough"]) == 0 and results["just_enough"]["tile"] == 1


def test_passes_staged_together_are_all_or_none(results):
    r = results["staged_together"]
    assert _rc(r) < 0 and r["tile"] == 0
