// Tile sizes of the sweep kernels and the LDS layout of their exchanges:
// plain C++ shared by the host code and the launchers.
#pragma once

#include <cstddef>
#include <cstdint>

#include "../../include/sv.h"

namespace sv {

// Largest tile, in qubits, of the gate tile pass (k_gate.hip), the batch
// kernels (k_batch.hip) and the adjoint's reverse sweep (k_adjoint.hip).
constexpr int tile_max_qubits(int dtype) { return dtype == SV_C64 ? 14 : 13; }
constexpr int batch_tile_qubits(int dtype) { return dtype == SV_C64 ? 13 : 12; }
constexpr int adjoint_tile_qubits(int dtype) { return dtype == SV_C64 ? 12 : 11; }

// LDS layout of the sweeps' exchanges: the index bits within one row of the
// 64 banks (64, 32 or 16 entries of 4, 8 or 16 bytes) are XOR-ed with a fixed
// linear function of the higher bits, one constant per bit.  The constants
// are the best of a random search over all sets of 4 (16 bytes: 3) register
// positions in a 12-bit tile, by the cycles that lanes 0 to 31 (16 bytes: 15)
// take in a model of the banks: 1.03, 1.25 and 1.14 on average, 2 at worst.
// Lanes in the order of the tile never differ in bits 9 and up; the last
// constant for 4 bytes, of bit 13, which only permuted stores see, is the best
// for one controlled X on top, over all sets in a 14-bit tile (1.15 cycles;
// other values up to 1.18).  In the tiles in use, of 14 and 13 bits, the
// accesses in order take 1.02 and 1.24 cycles.
// The columns are the host's, so any linear function costs the same; folds by
// shifts of the index, which the kernels could compute, gave 1.6 for 8 bytes
// (conflict cycles 14 % of a complex128 pass's busy cycles before, 3 % now).
inline constexpr uint8_t kSwizzle4[] = {0x3e, 0x39, 0x0d, 0x0e, 0x1c, 0x22, 0x12, 0x00};
inline constexpr uint8_t kSwizzle8[] = {0x1d, 0x0b, 0x1a, 0x0e, 0x1a, 0x10, 0x19, 0x0d};
inline constexpr uint8_t kSwizzle16[] = {0x0f, 0x0a, 0x0d, 0x05, 0x00, 0x02, 0x0d, 0x0a, 0x09};
constexpr int swizzle_row_bits(int bytes) { return bytes == 4 ? 6 : bytes == 8 ? 5 : 4; }

constexpr uint32_t sweep_swizzle(uint32_t l, int bytes) {
    const uint8_t *k = bytes == 4 ? kSwizzle4 : bytes == 8 ? kSwizzle8 : kSwizzle16;
    const int row = swizzle_row_bits(bytes);
    uint32_t r = l;
    for (int i = 0; l >> (row + i); ++i)
        if ((l >> (row + i)) & 1u) r ^= k[i];
    return r;
}

// A constant for every bit above the row of the largest tile that is
// exchanged in entries of that size, none of which leaves the row: component
// by component in the tile pass and the reverse sweep, whole amplitudes in
// the batch kernels.
template <size_t N>
constexpr bool swizzle_covers(const uint8_t (&k)[N], int bytes, int tile_qubits) {
    const int row = swizzle_row_bits(bytes);
    for (size_t i = 0; i < N; ++i)
        if (k[i] >> row) return false;
    return tile_qubits <= row + (int)N;
}
static_assert(swizzle_covers(kSwizzle4, 4, tile_max_qubits(SV_C64)), "complex64 tile pass");
static_assert(swizzle_covers(kSwizzle8, 8, tile_max_qubits(SV_C128)), "complex128 tile pass");
static_assert(swizzle_covers(kSwizzle8, 8, batch_tile_qubits(SV_C64)), "complex64 batches");
static_assert(swizzle_covers(kSwizzle16, 16, batch_tile_qubits(SV_C128)), "complex128 batches");
static_assert(swizzle_covers(kSwizzle4, 4, adjoint_tile_qubits(SV_C64)), "complex64 reverse sweep");
static_assert(swizzle_covers(kSwizzle8, 8, adjoint_tile_qubits(SV_C128)), "complex128 reverse sweep");

} // namespace sv
