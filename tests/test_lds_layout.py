"""The LDS layout of the sweeps' exchanges (lds_layout.hpp, plain C++) at every
tile size of its kernels.  The compiler evaluates it for every bit of a tile,
as a constant: a table shorter than the largest tile's bits is a read past its
end, which is not one.  The layout has to be a permutation of the tile that
keeps each index in its row of banks, linear over XOR."""

import os
import shutil
import subprocess

import pytest

from conftest import ROOT

PROGRAM = r"""
#include "lds_layout.hpp"
#include <cstdio>
#include <tuple>
#include <vector>
using namespace sv;
constexpr uint32_t columns(int bytes, int m) {
    uint32_t x = 0;
    for (int b = 0; b < m; ++b) x ^= sweep_swizzle(1u << b, bytes);
    return x;
}
template <uint32_t> struct Constant {};
template <int D> using Evaluated = std::tuple<
    Constant<columns(D == SV_C64 ? 4 : 8, tile_max_qubits(D))>,
    Constant<columns(D == SV_C64 ? 4 : 8, adjoint_tile_qubits(D))>,
    Constant<columns(D == SV_C64 ? 8 : 16, batch_tile_qubits(D))>>;
template class std::vector<Evaluated<SV_C64>>;
template class std::vector<Evaluated<SV_C128>>;
// linear, within the row, one to one; printed with the tile's size
static void check(const char *what, int bytes, int m) {
    const uint32_t n = 1u << m, row = 1u << swizzle_row_bits(bytes);
    std::vector<char> hit(n, 0);
    bool ok = true;
    for (uint32_t l = 0; l < n; ++l) {
        const uint32_t p = sweep_swizzle(l, bytes);
        uint32_t q = 0;
        for (int b = 0; b < m; ++b)
            if ((l >> b) & 1u) q ^= sweep_swizzle(1u << b, bytes);
        ok = ok && p < n && p == q && p / row == l / row && !hit[p];
        if (p < n) hit[p] = 1;
    }
    std::printf("%s %d %d %s\n", what, bytes, m, ok ? "ok" : "wrong");
}
int main() {
    for (int d : {SV_C64, SV_C128}) {
        const int comp = d == SV_C64 ? 4 : 8;
        for (int m = 1; m <= tile_max_qubits(d); ++m) check("tile", comp, m);
        for (int m = 1; m <= adjoint_tile_qubits(d); ++m) check("adjoint", comp, m);
        for (int m = 1; m <= batch_tile_qubits(d); ++m) check("batch", 2 * comp, m);
    }
}
"""


def test_layout_of_every_tile_size(tmp_path):
    cxx = os.environ.get("CXX") or shutil.which("g++")
    if not cxx:
        pytest.skip("no C++ compiler")
    src, exe = tmp_path / "layout.cpp", tmp_path / "layout"
    src.write_text(PROGRAM)
    r = subprocess.run([cxx, "-std=c++17", "-O1", "-I" + os.path.join(ROOT, "paper_1805_00988_amd", "csrc"), str(src),
                        "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lines = r.stdout.split("\n")[:-1]
    assert len(lines) == 14 + 12 + 13 + 13 + 11 + 12
    assert not [x for x in lines if not x.endswith(" ok")]
