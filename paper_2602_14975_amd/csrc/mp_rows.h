// Byte offsets of the neighbour rows that the matrix-core message kernels
// (mp_mx.hip) gather, plain arithmetic for host and device.
#pragma once
#include <cstdint>

namespace nnp {

constexpr uint32_t kRowFeatures = 128;

// Feature offset fo (bytes, less than a row of F floats) of row j, rows of F
// and of 3F floats: 32 bits, two shift-adds per edge (64 bits would take a
// vector register more for each row in flight and twice the additions).
constexpr uint32_t row_offset(uint32_t j, uint32_t fo) { return (j << 9) + fo; }
constexpr uint32_t row3_offset(uint32_t j, uint32_t fo) { return (j << 10) + row_offset(j, fo); }

// The atoms whose rows these offsets reach, 2,796,203.  Larger systems take the
// vector message kernels, whose offsets have 64 bits.
constexpr int64_t kRowOffsetAtoms = ((int64_t(1) << 32) - 4 * kRowFeatures) / (12 * kRowFeatures) + 1;

}  // namespace nnp
