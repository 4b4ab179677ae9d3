"""Properties of the device code that only its gfx950 assembly shows (compiled
here, nothing runs)."""
import os
import re
import subprocess

import pytest

from paper_2606_10944_amd import build as hip_build

CSRC = os.path.join(hip_build.HERE, "csrc")

# Two copies by the compiler's own instruction to one LDS address with a
# copy16_to_lds to another between them: the address is m0, so the second copy
# needs it set again.
M0_PROBE = r"""
#include "common.hpp"
namespace thin {
__global__ void probe(const uint4* a, const uint4* b, uint4* out) {
  typedef const __attribute__((address_space(1))) void* global_t;
  __shared__ __align__(16) uint4 x[192];
  const int l = threadIdx.x & 63;
  auto* lds = (__attribute__((address_space(3))) void*)x;
  __builtin_amdgcn_global_load_lds((global_t)(a + l), lds, 16, 0, 0);
  copy16_to_lds(b + l, lds_offset(x + 64));
  __builtin_amdgcn_global_load_lds((global_t)(a + 64 + l), lds, 16, 0, 0);
  wait_vmcnt<0>();
  __syncthreads();
  out[l] = x[l];
  out[64 + l] = x[64 + l];
}
}  // namespace thin
"""


def _assembly(tmp_path, source: str) -> str:
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(source)
    flags = [f for f in hip_build.FLAGS if f != "-shared"]
    r = subprocess.run([hip_build.hipcc(), *flags, "-I", CSRC, "--cuda-device-only", "-S",
                        str(src), "-o", str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return out.read_text()


def test_copy_to_lds_tells_the_compiler_that_it_changes_m0(tmp_path):
    try:
        hip_build.hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    text = _assembly(tmp_path, M0_PROBE)
    ops = re.findall(r"^\s*(s_mov_b32 m0|global_load_lds_dwordx4)", text, re.M)
    assert ops == ["s_mov_b32 m0", "global_load_lds_dwordx4"] * 3, ops


def test_decision_pass_loads_do_not_wait_for_those_in_flight(tmp_path):
    """The decision pass keeps several blocks' loads in flight.  A load address
    that the compiler forms in a branch ends in a wait for all of them, right
    before the next load."""
    try:
        hip_build.hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")
    with open(os.path.join(CSRC, "compress.hip")) as f:
        text = _assembly(tmp_path, f.read())
    kernels = re.findall(r"^_Z\S*halve_pass_kernel\S*:[^\n]*\n(.*?)^\.Lfunc_end", text, re.M | re.S)
    assert len(kernels) == 5
    for k in kernels:
        ops = [x.split(";")[0].strip() for x in k.split("\n")]
        ops = [x for x in ops if x and not x.startswith(".") and not x.endswith(":")]
        for i, op in enumerate(ops):
            if op.startswith("global_load_dwordx4"):
                before = ops[max(0, i - 8): i]
                assert not any("vmcnt(0)" in x for x in before), before
