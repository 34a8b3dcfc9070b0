"""The inline-assembly copies into LDS wait out their own register hazards: the compiler's hazard pass does not look
into inline assembly, so the instructions it emits around them must not matter.  Compiled to assembly, no device."""
import re
import subprocess

from paper_2607_14695_amd import build as B

# the base register pair comes straight out of vector instructions (v_readfirstlane), as a spilled one would
SRC = """
#include "common.h"
__global__ void copy(const uint32_t* table, float4* out) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[1024];
  const uint32_t lo = __builtin_amdgcn_readfirstlane(table[2 * threadIdx.x]);
  const uint32_t hi = __builtin_amdgcn_readfirstlane(table[2 * threadIdx.x + 1]);
  reflex::lds_dma16(reinterpret_cast<const void*>(((uint64_t)hi << 32) | lo), threadIdx.x * 16u, smem);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  out[threadIdx.x] = reinterpret_cast<const float4*>(smem)[threadIdx.x];
}
"""


def wait_states(ins):
    """Wait states an instruction gives: s_nop n counts n + 1, every other one."""
    m = re.match(r"s_nop\s+(\w+)", ins)
    return int(m.group(1), 0) + 1 if m else 1


def test_copy_with_a_base_from_vector_instructions(tmp_path):
    src = tmp_path / "copy.hip"
    src.write_text(SRC)
    asm = tmp_path / "copy.s"
    subprocess.run([B.HIPCC, *B.DEVICE_FLAGS, "--offload-device-only", "-S", str(src), "-o", str(asm)], check=True,
                   capture_output=True, timeout=110)
    text = asm.read_text()
    body = text[text.index("copy"):].split("s_endpgm")[0]
    ins = [l.split(";")[0].strip() for l in body.splitlines()]
    ins = [l for l in ins if l and not l.startswith(".") and not l.endswith(":")]
    at = [i for i, l in enumerate(ins) if l.startswith("global_load_lds_dwordx4")]
    assert len(at) == 1, ins
    lo, hi = map(int, re.search(r"s\[(\d+):(\d+)\]", ins[at[0]]).groups())
    writes = [i for i, l in enumerate(ins[:at[0]]) if re.match(rf"v_\w+\s+s({lo}|{hi})\b", l)]
    assert writes, ins
    # a vector write of a scalar register, then a vector-memory read of it: 5 wait states (CDNA ISA)
    for i in writes:
        assert sum(wait_states(l) for l in ins[i + 1:at[0]]) >= 5, ins[i:at[0] + 1]
    # M0 written by a scalar instruction, then a copy into LDS: 1
    m0 = max(i for i, l in enumerate(ins[:at[0]]) if re.match(r"s_mov_b32\s+m0", l))
    assert sum(wait_states(l) for l in ins[m0 + 1:at[0]]) >= 1, ins[m0:at[0] + 1]
