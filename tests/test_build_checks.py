"""What the build refuses (CPU only): loads to LDS whose address a vector instruction writes too shortly before, on any path."""
import os
import subprocess

import pytest

from paper_2509_19836_amd import build

KERNEL = """
#include "mfma16.hpp"
using namespace burst;
__global__ void loads(const char* const* p, const char* q, float* out) {
  extern __shared__ char smem[];
  const uint32_t lds = (uint32_t)(uintptr_t)(lds_bytes)smem, off = 16 * threadIdx.x;
  const uint64_t a = reinterpret_cast<uint64_t>(p[threadIdx.x]);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a), hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  const char* from_a_lane = reinterpret_cast<const char*>((uint64_t)hi << 32 | lo);
  const char* argument = q;
  %s(%s, off, lds);
  wait_global_loads();
  out[threadIdx.x] = reinterpret_cast<float*>(smem)[threadIdx.x];
}
"""


def _assembly(tmp_path, load, base):
    src, out = tmp_path / "loads.hip", tmp_path / "loads.s"
    src.write_text(KERNEL % (load, base))
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, *build.FLAGS, "-I", build.CSRC, "--offload-device-only", "-S", str(src), "-o", str(out)], check=True,
                   stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    return out.read_text()


@pytest.mark.parametrize("load", ["load_to_lds", "load_dword_to_lds"])
def test_an_address_read_from_a_lane_is_refused_and_one_from_scalar_arithmetic_is_not(tmp_path, load):
    assert build.check_load_addresses(_assembly(tmp_path, load, "argument"), "loads.hip") == 1
    with pytest.raises(RuntimeError, match="vector instruction"):
        build.check_load_addresses(_assembly(tmp_path, load, "from_a_lane"), "loads.hip")


LOAD = "s_mov_b32 m0, s9\ns_nop 0\nglobal_load_lds_dwordx4 v1, s[2:3] offset:16\n"


@pytest.mark.parametrize("early, text", [
    (True, "v_readlane_b32 s3, v40, 7\ns_add_u32 s4, s4, s5\n" + LOAD),                                  # a spilled register comes back
    (True, "v_readlane_b32 s3, v40, 7\ns_nop 1\n" + LOAD),                                              # four states
    (False, "v_readlane_b32 s3, v40, 7\ns_nop 2\n" + LOAD),                                             # five
    (False, "v_readlane_b32 s4, v40, 7\n" + LOAD),                                                      # another register
    (False, "v_readlane_b32 s4, v40, 7\ns_add_u32 s2, s4, s5\ns_addc_u32 s3, s6, 0\n" + LOAD),          # scalar arithmetic between
    (True, "v_readlane_b32 s3, v40, 7\ns_cmp_eq_u32 s3, 0\n" + LOAD),                                   # (compares write nothing)
    (True, "v_add_co_u32 v1, s[2:3], v1, v2\n" + LOAD),
    (True, "v_cmp_gt_u32 s[2:3], v1, v2\n" + LOAD),
    (True, "s_mov_b32 m0, s9\nglobal_load_lds_dword v1, s[2:3]\n"),
    (True, "v_readfirstlane_b32 s2, v5\ns_cbranch_scc1 .LBB0_3\ns_endpgm\n.LBB0_3:\n" + LOAD),          # by a branch
    (True, "v_readfirstlane_b32 s2, v5\n.LBB0_3: ; %x\n" + LOAD),                                      # past a label
    (False, "v_readfirstlane_b32 s2, v5\ns_branch .LBB0_4\n.LBB0_3:\n" + LOAD + ".LBB0_4:\ns_endpgm\n"),  # not on the path
    (True, ".LBB0_3:\n" + LOAD + "v_readfirstlane_b32 s2, v5\ns_branch .LBB0_3\n"),                     # from the end of a loop
])
def test_distances_on_every_path(early, text):
    if early:
        with pytest.raises(RuntimeError):
            build.check_load_addresses(text, "x.hip")
    else:
        assert build.check_load_addresses(text, "x.hip") == 1
