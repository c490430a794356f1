"""Row offsets of the matrix-core message kernels (csrc/mp_rows.h): exact up to
the number of atoms they are chosen for, wrapped past it, and the choice of
kernels on both sides of it."""

import ctypes as C
import os
import shutil
import subprocess

import pytest

from paper_2602_14975_amd import nnp

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_14975_amd", "csrc")
ATOMS = 2796203  # (2^32 - 512) / 1536, rounded down, + 1

PROGRAM = r"""
#include "mp_rows.h"
#include <cstdio>
using namespace nnp;
int main() {
    const uint64_t last = uint64_t(kRowOffsetAtoms) - 1;
    for (uint64_t fo = 0; fo < 4 * kRowFeatures; fo += 4)
        for (uint64_t back = 0; back < 1000; ++back) {
            const uint64_t j = last - back, k = back;
            if (row3_offset(uint32_t(j), uint32_t(fo)) != 1536 * j + fo || row_offset(uint32_t(j), uint32_t(fo)) != 512 * j + fo) return 1;
            if (row3_offset(uint32_t(k), uint32_t(fo)) != 1536 * k + fo) return 1;
        }
    // one atom more: the last feature's offset wraps
    if (row3_offset(uint32_t(last + 1), 508) == 1536 * (last + 1) + 508) return 2;
    std::printf("%lld\n", (long long)kRowOffsetAtoms);
}
"""


def test_offsets_reach_the_atoms_they_serve(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    src = tmp_path / "rows.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "rows"
    subprocess.run([cxx, "-std=c++17", "-O2", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and int(r.stdout) == ATOMS


class Route(C.Structure):
    _fields_ = [("matrix_cores", C.c_bool), ("species_sum", C.c_bool)]


@pytest.mark.parametrize("n,mx", [(1, True), (89373, True), (ATOMS, True), (ATOMS + 1, False), (2**31 - 1, False)])
def test_larger_systems_take_the_vector_kernels(n, mx):
    f = getattr(nnp.lib(), "_ZN3nnp13message_routeEiiil")  # nnp::message_route(F, K, cut, n)
    f.restype, f.argtypes = Route, [C.c_int, C.c_int, C.c_int, C.c_int64]
    r = f(128, 16, 0, n)
    assert (r.matrix_cores, r.species_sum) == (mx, mx)
