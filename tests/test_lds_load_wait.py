"""The assembly of the direct-to-LDS load keeps its own wait states.

A vector-memory instruction may read a scalar register that a vector
instruction wrote only five wait states later; the hardware does not wait and
the compiler does not look into assembly.  So the helper has to supply all
five itself, whatever precedes it: here the descriptor words are read out of
vector lanes right before the load, as spilled scalars are."""

import os
import re
import subprocess

import pytest

from paper_2608_15211_amd import build

SOURCE = """
#include "terra_common.h"
__global__ void k(const int* desc, const int* off, int* out, int base) {
  __shared__ __align__(16) char tile[4096];
  const int d = desc[threadIdx.x];
  const int o = off[threadIdx.x];
  terra::i32x4 rs;
#pragma unroll
  for (int c = 0; c < 4; ++c) rs[c] = __builtin_amdgcn_readlane(d, c);
  LOAD;
  terra::wait_vm<0>();
  terra::lds_barrier();
  out[threadIdx.x] = reinterpret_cast<const int*>(tile)[base ^ threadIdx.x];
}
"""


FORMS = {"one": ("terra::buffer_load_lds16(rs, tile, o)", 1),
         "four": ("const int v[4] = {o, o + 1, o + 2, o + 3}; terra::buffer_load_lds16x4<1024>(rs, tile, v)", 4)}


def _scalars(operand):
    m = re.match(r"s\[(\d+):(\d+)\]$", operand)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.match(r"s(\d+)$", operand)
    return {int(m[1])} if m else set()


@pytest.mark.parametrize("form", FORMS)
def test_descriptor_written_by_vector_instructions(form, tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    src, asm = tmp_path / "k.hip", tmp_path / "k.s"
    src.write_text(SOURCE.replace("LOAD", FORMS[form][0]))
    build._run([build.HIPCC] + build.FLAGS + ["-I" + build.CSRC, "--cuda-device-only", "-S", str(src), "-o", str(asm)])
    states, writes, loads = 0, {}, 0          # writes: scalar register -> wait states at its last vector write
    for line in asm.read_text().splitlines():
        text = line.split(";")[0].strip()
        if not re.match(r"[a-z]\w+(\s|$)", text) or text.endswith(":"):
            continue
        op, _, rest = text.partition(" ")
        args = [a.strip() for a in rest.replace("\t", " ").split(",")]
        if op == "buffer_load_dwordx4" and text.endswith("lds"):
            loads += 1
            for reg in _scalars(args[1]):
                assert reg in writes, "the test's descriptor did not come from vector lanes"
                assert states - writes[reg] - 1 >= 5, "s%d read %d wait states after its write" % (
                    reg, states - writes[reg] - 1)
        if op.startswith("v_read"):
            for reg in _scalars(args[0]):
                writes[reg] = states
        states += 1 + (int(args[0], 0) if op == "s_nop" else 0)
    assert loads == FORMS[form][1]
