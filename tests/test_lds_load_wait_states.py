"""The loads that go from global memory straight to LDS are written as assembly, where the compiler inserts no wait states:
the code built here is looked through for the ones the gfx9 hazard rules ask for."""
import os
import re
import subprocess

from paper_2506_16640_amd import build

SOURCE = """
#include "qside.hip.h"
using namespace entmax;
__global__ void k(const char* src, const int* where, uint4* out) {
  extern __shared__ char smem[];
  const uint32_t lds = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem + (threadIdx.x & ~63u) * 16u);
  const char* s = src + __builtin_amdgcn_readfirstlane(where[threadIdx.x >> 6]);
  load_to_lds(s, threadIdx.x * 16u, lds);
  load_to_lds(s + 4096, threadIdx.x * 16u, lds + 4096u);
  lds_loads_wait<0>();
  __syncthreads();
  out[threadIdx.x] = reinterpret_cast<uint4*>(smem)[threadIdx.x ^ 1];
}
"""


def _wait_states(line):
    m = re.match(r"s_nop (\d+)", line)
    return int(m.group(1)) + 1 if m else 1


def _registers(operand):
    m = re.match(r"s\[(\d+):(\d+)\]", operand)
    return {"s%d" % r for r in range(int(m.group(1)), int(m.group(2)) + 1)}


def test_loads_to_lds_keep_the_hazard_rules(tmp_path):
    src, asm = tmp_path / "k.hip", tmp_path / "k.s"
    src.write_text(SOURCE)
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + build.HIPCC_FLAGS + [
        "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC, "--cuda-device-only", "-S", str(src), "-o", str(asm)]
    subprocess.run(cmd, check=True, capture_output=True)
    lines = [re.sub(r";.*", "", l).strip() for l in asm.read_text().splitlines()]
    lines = [l for l in lines if l and not l.startswith(".") and not l.endswith(":")]
    loads = [n for n, l in enumerate(lines) if l.startswith("global_load_lds_dwordx4")]
    assert len(loads) == 2
    for n in loads:
        address = _registers(lines[n].split(",")[1].strip())
        states, m0_seen = 0, False
        for l in reversed(lines[:n]):
            op, _, args = l.partition(" ")
            dst = args.split(",")[0].strip()
            if dst == "m0" and not m0_seen:
                m0_seen = True
                assert states >= 1, "no wait state between the write of m0 and the load that reads it"
            if op.startswith("v_readfirstlane") and dst in address:
                assert states >= 5, "fewer than five wait states between a vector write of the address and the load"
            if states >= 5 and m0_seen:
                break
            states += _wait_states(l)
        assert m0_seen
