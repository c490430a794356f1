// Byte offsets of the per-atom blocks' buffer loads (atom_block.hip), plain
// arithmetic for host and device.
//
// A buffer load adds a lane offset and a uniform one to its descriptor's base.
// Which part the descriptor's bound covers is not the same everywhere: the
// compiler documents the lane offset alone, the hardware compares it with the
// size less the uniform offset, which is below zero, and then bounds nothing,
// once the uniform offset is past the end.  So no load relies on the bound for
// its uniform part: weights are addressed inside their matrix by every lane,
// and of rows only what is the same in all of them (column, feature slice) is
// uniform, while the row, which may be absent, is in the lane offset.
#pragma once
#include <cstdint>

namespace nnp {
namespace atom_block {

constexpr int kFeatures = 128;
constexpr int kWaves = 8;                        // wavefronts of a block
constexpr int kSliceFeatures = kFeatures / kWaves;  // features of a wavefront's slice

// ------------------------------------------------------- packed weights --
// A matrix [N][32 KS] as launch_pack_frags lays it out: per piece slices of 16
// rows of slice_bytes each.
constexpr uint32_t slice_bytes(int KS) { return 64u * kSliceFeatures * uint32_t(KS); }
constexpr uint32_t piece_bytes(int N, int KS) { return uint32_t(N) * uint32_t(KS) * 64u; }
// A lane's unit within a step: quarter q = lane / 16 of the fragment, row a =
// lane % 16 of the slice (`apart`: see put_slice).
constexpr uint32_t unit_offset(int q, int a, bool apart) {
    return uint32_t((apart ? 4 * (q >> 1) + 2 * (q & 1) : 2 * (q & 1) + (q >> 1)) * 16 + a) * 16u;
}
// Step f of a product over NT slices and KN steps of 32 k.  The loads run ahead
// of the products: past the last step they read the last one again, whose
// data is not used.
constexpr uint32_t step_offset(int f, int NT, int KN, bool apart) {
    const int ks = f / NT < KN ? f / NT : KN - 1;
    return uint32_t(apart ? (ks >> 1) * 2048 + (ks & 1) * 256 : ks * 1024);
}
// The slice of wavefront w in a matrix of N rows: of one with fewer slices than
// wavefronts the wavefronts past them, which use nothing of it, take the last.
constexpr int slice_within(int w, int N) {
    const int last = N / kSliceFeatures - 1;
    return w < last ? w : last;
}

// ----------------------------------------------------------- rows of atoms --
// Rows [atom][C][ld] of float32 from the tile's first atom.  Lane part: row
// a + 16 g, piece h of the slice; uniform part: the slice at column c0 of c.
template <int C, int ld>
constexpr uint32_t row_lane_offset(int a, int g, int h) {
    return uint32_t((a + 16 * g) * (C * ld * 4) + 16 * h);
}
template <int C, int ld>
constexpr uint32_t row_uniform_offset(int c, int c0, int w) {
    return uint32_t((c * ld + c0 + kSliceFeatures * w) * 4);
}

}  // namespace atom_block
}  // namespace nnp
