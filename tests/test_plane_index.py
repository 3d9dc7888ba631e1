"""Addresses of the walls' planes in grids of 2^29 walls and more, on the CPU.

The kernels that walk a cell's walls hold the wall's index in 32 bits; a call
may have up to 2^31 - 2 walls, whose planes are four values each.  The address
they form (plane_at) is checked at the indices where 32 bits would not do.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "em_internal.h"
#include <cstdio>
int main()
{
    for (int32_t j : {0, 1, (1 << 29) - 1, 1 << 29, (1 << 29) + 1, 1 << 30, 0x7ffffffd}) {
        const int64_t at = em::plane_at(j);
        if (at < 0 || at / 4 != j || at % 4 != 0) return std::printf("wall %d at %lld\n", j, (long long)at), 1;
    }
    return 0;
}
"""


def test_plane_addresses(tmp_path):
    cxx = next((c for c in ("/opt/rocm/llvm/bin/clang++", shutil.which("g++")) if c and os.path.exists(c)), None)
    if cxx is None:
        pytest.skip("no C++ compiler")
    src, exe = tmp_path / "plane.cpp", str(tmp_path / "plane")
    src.write_text(PROGRAM)
    inc = ["-I" + os.path.join(ROOT, "tests", "serve_host"),
           "-I" + os.path.join(ROOT, "paper_2404_17084_amd", "csrc"), "-I" + os.path.join(ROOT, "include")]
    subprocess.check_call([cxx, "-std=c++17", "-O1"] + inc + [str(src), "-o", exe])
    assert subprocess.run([exe]).returncode == 0
