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
void tile_plan(int64_t S, int64_t n_q, int64_t slots, int64_t* out) {
  const thin::TilePlan p = thin::attn_tile_plan(S, n_q, slots);
  out[0] = p.tiles;
  out[1] = p.split.parts;
  out[2] = p.split.run;
}
int64_t split_blocks(int64_t S, int64_t blocks, int64_t slots) {
  return thin::split_blocks(S, blocks, slots);
}
void share_of(uint32_t id, uint32_t S, uint32_t parts, uint32_t extra, uint32_t* out) {
  const thin::Share s = thin::share_of(id, S, parts, extra);
  out[0] = s.slice;
  out[1] = s.part;
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
    lib = C.CDLL(str(so))
    lib.split_blocks.restype = C.c_int64
    return lib


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


def _ceil(a, b):
    return -(-a // b)


def _tile_cost(S, n_q, tiles, parts):
    """Rounds of the device's 256 workgroups times a workgroup's time, in steps
    of one tile (a step of two takes 1.75, staging the coreset 2)."""
    steps = _ceil(n_q, 128 * tiles)
    run = _ceil(steps, parts)
    return _ceil(S * _ceil(steps, run), 256) * (2.0 + run * (1.0, 1.75)[tiles - 1])


SLICES = [1, 2, 3, 4, 8, 12, 16, 20, 24, 32, 40, 48, 64, 96, 128, 200, 255, 256, 257, 300, 513, 4000]


@pytest.mark.parametrize("S", SLICES)
def test_attention_tile_plan_is_no_worse_than_a_fixed_workgroup_count(plan, S):
    """129-256 keys, d = 128: 256 workgroups of two query tiles, or 512 of one,
    rounded up to whole workgroups per slice, leave a nearly empty last round
    wherever the slices do not divide them."""
    out = (C.c_int64 * 3)()
    for n_q in (1, 33, 128, 129, 256, 257, 1000, 1024, 4096, 8191, 16384, 65536, 1 << 20, 1 << 30):
        plan.tile_plan(C.c_int64(S), C.c_int64(n_q), C.c_int64(256), out)
        tiles, parts, run = out
        step = 128 * tiles
        assert tiles in (1, 2) and parts >= 1 and run >= 1
        assert parts * run * step >= n_q > (parts - 1) * run * step, "every part has queries"
        cost = _tile_cost(S, n_q, tiles, parts)
        for t, want in ((1, 512), (2, 256)):
            fixed = min(_ceil(want, S), _ceil(n_q, 128 * t))
            assert cost <= _tile_cost(S, n_q, t, fixed) + 1e-9, (S, n_q, tiles, parts, t)


@pytest.mark.parametrize("S,n_q,want", [
    (64, 16384, (2, 4, 16)), (32, 65536, (2, 8, 32)),  # the long workloads fill the device
    (8, 4096, (1, 32, 1)), (1, 1024, (1, 8, 1)),       # too few queries for two tiles
    (24, 65536, (2, 10, 26)),                          # 240 workgroups, not 264
])
def test_attention_tile_plan_of_known_sizes(plan, S, n_q, want):
    out = (C.c_int64 * 3)()
    plan.tile_plan(C.c_int64(S), C.c_int64(n_q), C.c_int64(256), out)
    assert tuple(out) == want


@pytest.mark.parametrize("S", [1, 7, 64, 100, 512, 513, 600, 1000, 1023, 1024, 1025, 2000, 65535])
@pytest.mark.parametrize("slots", [512, 1024, 1280])
def test_blocks_of_one_chunk_of_keys_fill_the_device(plan, S, slots):
    for blocks in (1, 2, 4, 5, 16, 65, 257, 1 << 24):
        parts = plan.split_blocks(C.c_int64(S), C.c_int64(blocks), C.c_int64(slots))
        assert 1 <= parts <= blocks
        # no device half empty, where the queries would fill it
        if blocks >= 16:
            assert S * parts > slots // 2 or parts == blocks
            rounds = _ceil(S * parts, slots)
            assert rounds == 1 or S * parts / (rounds * slots) > 0.6, (blocks, parts)


@pytest.mark.parametrize("S,blocks,slots,want", [
    (16, 65, 1024, 64), (64, 65, 1024, 16),  # as many as fit together
    (1, 17, 1024, 17), (600, 4, 1024, 1), (520, 16, 1280, 7), (2000, 8, 512, 1),
])
def test_blocks_of_one_chunk_of_keys_of_known_sizes(plan, S, blocks, slots, want):
    assert plan.split_blocks(C.c_int64(S), C.c_int64(blocks), C.c_int64(slots)) == want


@pytest.mark.parametrize("S,n_q,slots", [(20, 4097, 1024), (20, 4097, 1280), (40, 2049, 1280),
                                         (50, 1500, 1024), (100, 1000, 1280), (3, 300 * 64 + 1, 512),
                                         (40, 33 * 64, 1024), (1, 4097 * 64, 1024)])
def test_shares_of_one_chunk_of_keys_are_dealt_evenly(plan, S, n_q, slots):
    """Every part of every slice once, and no CU (workgroups in turn) with more
    than one longer share beyond the others'."""
    blocks = _ceil(n_q, 64)
    parts = plan.split_blocks(C.c_int64(S), C.c_int64(blocks), C.c_int64(slots))
    extra = blocks % parts
    assert extra > 0
    out = (C.c_uint32 * 2)()
    seen, longer = set(), [0] * 256
    for i in range(S * parts):
        plan.share_of(C.c_uint32(i), C.c_uint32(S), C.c_uint32(parts), C.c_uint32(extra), out)
        seen.add((out[0], out[1]))
        longer[i % 256] += out[1] < extra
    assert seen == {(s, p) for s in range(S) for p in range(parts)}
    assert max(longer) - min(longer) <= 1
