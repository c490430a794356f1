"""Byte offsets of the per-atom blocks' buffer loads (csrc/atom_block_addr.h),
every lane, step and wavefront of every product and of a last tile of every
size: inside the matrix, or inside the rows that exist, whether a descriptor's
bound covers the lane offset alone or is compared with the size less the
uniform offset (which bounds nothing once that is past the end)."""

import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_14975_amd", "csrc")

PROGRAM = r"""
#include "atom_block_addr.h"
#include <cstdio>
#include <initializer_list>
using namespace nnp::atom_block;

static int bad = 0;
static void check(bool ok, const char* what, int a, int b, int c, int d) {
    if (!ok && bad++ < 10) std::printf("%s: %d %d %d %d\n", what, a, b, c, d);
}

// A matrix of N rows read by all wavefronts: NT slices w, w + step ..., KN of
// KS steps; the loads run up to 16 steps ahead.
static void weights(int N, int NT, int step, int KN, int KS) {
    for (int np : {1, 3})
        for (int apart = 0; apart < 2; ++apart)
            for (int w = 0; w < kWaves; ++w) {
                const uint32_t first = uint32_t(slice_within(w, N)) * slice_bytes(KS);
                for (int f = 0; f < KN * NT + 16; ++f)
                    for (int p = 0; p < np; ++p)
                        for (int lane = 0; lane < 64; ++lane) {
                            const uint32_t in_slice = step_offset(f, NT, KN, apart) + unit_offset(lane / 16, lane % 16, apart);
                            const uint32_t at = first + uint32_t(f % NT * step) * slice_bytes(KS) + uint32_t(p) * piece_bytes(N, KS) + in_slice;
                            check(in_slice + 16 <= slice_bytes(KS) && at + 16 <= np * piece_bytes(N, KS), "weights", N, w, f, lane);
                            if (f < KN * NT && w * kSliceFeatures < N) check(slice_within(w, N) == w, "slice", N, w, f, lane);
                        }
            }
}

template <int C, int ld>
static void rows(int TA) {
    for (int present = 1; present <= TA; ++present) {
        const uint32_t size = uint32_t(present) * C * ld * 4;
        for (int w = 0; w < kWaves; ++w)
            for (int c = 0; c < C; ++c)
                for (int c0 = 0; c0 < ld; c0 += kFeatures)
                    for (int g = 0; g < TA / 16; ++g)
                        for (int lane = 0; lane < 64; ++lane) {
                            const int row = lane % 16 + 16 * g;
                            const uint32_t v = row_lane_offset<C, ld>(lane % 16, g, lane / 16), u = row_uniform_offset<C, ld>(c, c0, w);
                            const bool lane_bound = v < size, hardware_bound = v < size - u;
                            if (row < present) {
                                check(lane_bound && hardware_bound && v + u + 16 <= size, "present row", present, row, w, lane);
                                check(v + u == uint32_t(((row * C + c) * ld + c0 + kSliceFeatures * w + 4 * (lane / 16)) * 4), "element", present, row, w, lane);
                            } else {
                                check(!lane_bound && !hardware_bound, "absent row", present, row, w, lane);
                            }
                        }
    }
}

int main() {
    weights(256, 2, 8, 4, 4);   // U V; M1 transposed
    weights(128, 1, 1, 8, 8);   // M1
    weights(384, 3, 8, 4, 4);   // M2, W2
    weights(384, 2, 8, 4, 4);   // M2, last layer
    weights(128, 1, 1, 4, 4);   // square ones, T_0, T_2
    weights(128, 1, 1, 12, 12); // M2, W2 transposed
    weights(128, 1, 1, 8, 12);  // M2 transposed, last layer
    for (int pp = 32; pp <= 128; pp += 16) weights(pp, 1, 1, 4, 4);  // T_0, T_2 transposed, one to six species
    for (int TA : {16, 32}) {
        rows<1, 128>(TA);
        rows<3, 128>(TA);
        rows<1, 384>(TA);
    }
    return bad != 0;
}
"""


def test_every_load_is_inside_its_array(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    src = tmp_path / "addresses.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "addresses"
    subprocess.run([cxx, "-std=c++17", "-O2", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
