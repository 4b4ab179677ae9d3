"""Launch shapes of the attention kernels (csrc/attn_plan.hpp, host arithmetic
only), compiled for the CPU."""
import ctypes as C
import os
import subprocess

import pytest

from paper_2606_10944_amd import build as hip_build

CSRC = os.path.join(hip_build.HERE, "csrc")

SHIM = r"""
#include "attn_plan.hpp"
extern "C" {
void grid_rows(int64_t blocks, int64_t threads, int64_t multiple, int64_t* out) {
  const thin::GridRows g = thin::grid_rows(blocks, threads, multiple);
  out[0] = g.x;
  out[1] = g.rows;
}
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "shim.cpp").write_text(SHIM)
    so = d / "shim.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                    str(d / "shim.cpp"), "-o", str(so)], check=True)
    return C.CDLL(str(so))


# The most float queries a call takes (2^30) in blocks of 64, and one block more
# and less than fits a row; prefill tiles of 128 points, 65535 slices.
@pytest.mark.parametrize("blocks,threads,multiple", [
    (1, 256, 1), (4097, 256, 1), ((1 << 24) - 1, 256, 1), (1 << 24, 256, 1),
    ((1 << 24) + 1, 256, 1), (8, 512, 8), ((1 << 23) - 8, 512, 8), (1 << 23, 512, 8),
    (65535 * 2048 + 7 & ~7, 512, 8),
])
def test_grid_rows_fit_the_runtime_and_cover_the_blocks(plan, blocks, threads, multiple):
    out = (C.c_int64 * 2)()
    plan.grid_rows(C.c_int64(blocks), C.c_int64(threads), C.c_int64(multiple), out)
    x, rows = out
    assert x * threads < 1 << 32 and x % multiple == 0
    assert blocks <= x * rows
    assert rows == 1 or x * (rows - 1) < blocks, "a row with nothing to do"
    if blocks * threads < 1 << 32:
        assert (x, rows) == (blocks, 1)


@pytest.mark.parametrize("work", [1, 7, 8, 9, 100, 1003])
def test_prefill_tiles_are_each_taken_once_over_several_grid_rows(plan, work):
    """The prefill kernel's workgroup -> tile mapping (XCD x takes the tiles
    x per .. (x + 1) per - 1) where a row holds few workgroups."""
    out = (C.c_int64 * 2)()
    plan.grid_rows(C.c_int64((work + 7) // 8 * 8), C.c_int64(1 << 27), C.c_int64(8), out)
    x, rows = out
    assert x <= 24 and (work <= 24 or rows > 1)
    per, seen = (work + 7) >> 3, []
    for by in range(rows):
        for bx in range(x):
            at = (bx & 7) * per + (bx >> 3) + (x >> 3) * by
            if at < min(work, ((bx & 7) + 1) * per):
                seen.append(at)
    assert sorted(seen) == list(range(work))
