"""Launch rules of the Halve rounds (csrc/score_plan.hpp, host arithmetic only),
compiled for the CPU."""
import ctypes as C
import os
import subprocess

import pytest

from paper_2606_10944_amd import build as hip_build

CSRC = os.path.join(hip_build.HERE, "csrc")

SHIM = r"""
#include "score_plan.hpp"
extern "C" int64_t unit_launch_max(int64_t d, int64_t N, int64_t nbk, int first) {
  return thin::unit_launch_max(d, N, nbk, first != 0);
}
extern "C" int local_staged(int64_t nbk, int64_t lds, int64_t by_registers) {
  return thin::local_staged(nbk, lds, by_registers);
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
    lib.unit_launch_max.restype = C.c_int64
    return lib


def _units(N):
    NC, nb = -(-N // 32), -(-N // 64)
    return 2 * (nb * NC - nb * (nb - 1))


# Launches measured in both forms (whole calls, float rows), and which was faster.
@pytest.mark.parametrize("d,N,buckets,first,units", [
    (64, 1024, 24, True, True), (64, 512, 64, True, True), (64, 512, 100, True, False),
    (64, 800, 48, True, False), (64, 512, 64, False, False), (64, 320, 64, False, True),
    (64, 2048, 6, True, True), (32, 5600, 1, True, True), (32, 512, 128, True, False),
    (128, 256, 33, True, True), (128, 256, 100, True, False), (128, 512, 64, True, False),
    (128, 800, 32, True, False), (128, 1024, 16, True, False), (128, 1024, 8, True, True),
    (128, 2048, 6, True, False), (128, 4096, 1, True, True), (128, 512, 100, False, False),
    (128, 200, 300, True, False), (128, 512, 16, True, True),
    (128, 800, 17, False, True), (128, 800, 16, False, False), (128, 400, 40, True, True),
    (128, 4096, 2, True, True), (128, 2048, 3, True, True), (64, 4096, 2, False, True),
    (64, 1024, 28, False, False), (32, 1024, 25, True, True),
])
def test_float_rounds_take_units_where_those_are_faster(plan, d, N, buckets, first, units):
    most = plan.unit_launch_max(C.c_int64(d), C.c_int64(N), C.c_int64(buckets), int(first))
    assert (_units(N) * buckets <= most) == units, (_units(N) * buckets, most)


@pytest.mark.parametrize("buckets,lds,by_registers,staged", [
    (1, 160 << 10, 2, True), (256, 160 << 10, 2, True), (257, 160 << 10, 2, False),
    (512, 80 << 10, 2, True), (100000, 80 << 10, 2, True),   # as many as the registers allow
    (512, 80 << 10, 3, True), (600, 64 << 10, 3, False),     # two where three fit
    (100000, 53 << 10, 3, True), (1, (160 << 10) + 256, 2, False),
])
def test_local_launches_stage_all_rows_where_it_costs_no_workgroup(plan, buckets, lds,
                                                                  by_registers, staged):
    assert bool(plan.local_staged(C.c_int64(buckets), C.c_int64(lds),
                                  C.c_int64(by_registers))) == staged
