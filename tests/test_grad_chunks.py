"""Rows per partial sum of the weight adjoints (csrc/grad_chunk.h): chunks of
256 rows up to the most blocks that a launch's y and z dimensions have, longer
ones beyond, for every number of atoms a system may have."""

import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_14975_amd", "csrc")

PROGRAM = r"""
#include "grad_chunk.h"
#include <cstdio>
using nnp::grad_chunk;
static int64_t chunks(int64_t rows) { return (rows + grad_chunk(rows) - 1) / grad_chunk(rows); }
int main() {
    const int64_t edge = int64_t(65535) * 256;
    if (grad_chunk(1) != 256 || grad_chunk(3 * 24576) != 256 || grad_chunk(edge) != 256 || grad_chunk(edge + 1) != 512) return 1;
    for (int64_t n = 1; n < (int64_t(1) << 31); n += n / 1000 + 1)
        if (chunks(3 * n) > 65535 || grad_chunk(3 * n) % 256) return 2;
    if (chunks(3 * ((int64_t(1) << 31) - 1)) > 65535) return 3;
}
"""


def test_chunks_fit_a_launch(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    src = tmp_path / "chunks.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "chunks"
    subprocess.run([cxx, "-std=c++17", "-O2", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], timeout=60).returncode == 0
