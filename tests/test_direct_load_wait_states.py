"""The direct loads to LDS are inline assembly, for which the compiler inserts no wait states.  gfx950 asks for five
between a vector instruction that writes a scalar register and a memory instruction that reads it, so the helpers must
not read the caller's scalar base with the load itself.  Checked on the assembly of a kernel that hands them a base
fresh from v_readfirstlane (no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2508_18182_amd import build as B

SOURCE = r"""
#include "common.h"
using namespace adloco;
extern "C" __global__ void fresh_base(const char* const* tab, unsigned long long mask) {
  extern __shared__ char lds[];
  const unsigned at = lds_address(lds);
  const char* p = tab[threadIdx.x >> 6];
  CALL
}
"""
CALLS = [("direct_load_lds16_s(threadIdx.x * 16u, uniform_ptr(p), at);", 1),
         ("direct_load_lds16_masked2(uniform_ptr(p), threadIdx.x * 16u, at, threadIdx.x * 16u + 1024, at + 1024, mask);", 2)]


def scalars(text):
    out = set()
    for m in re.finditer(r"\bs(\d+)\b|\bs\[(\d+):(\d+)\]", text):
        out |= {int(m[1])} if m[1] else set(range(int(m[2]), int(m[3]) + 1))
    return out


@pytest.mark.parametrize("call,count", CALLS, ids=["plain", "masked"])
def test_base_fresh_from_the_vector_unit(call, count, tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not shutil.which(hipcc):
        pytest.skip("no hipcc")
    src = tmp_path / "k.hip"
    src.write_text(SOURCE.replace("CALL", call))
    asm = tmp_path / "k.s"
    subprocess.run([hipcc, *B.HIPCC_FLAGS, "-I", os.path.join(B.ROOT, "include"), "-I", B.CSRC, "-S",
                    "--offload-device-only", str(src), "-o", str(asm)], check=True, capture_output=True)
    since = {}            # scalar register -> wait states since a vector instruction wrote it
    fresh = loads = 0
    for line in asm.read_text().split("fresh_base:", 1)[1].split(".Lfunc_end")[0].splitlines():
        op, _, rest = line.split(";")[0].strip().partition(" ")
        if not op or op.startswith(".") or op.endswith(":"):
            continue
        if op.startswith("global_load_lds"):
            loads += 1
            close = {r: since[r] for r in scalars(rest) if since.get(r, 9) < 5}
            assert not close, f"{line.strip()}: wait states since a vector write: {close}"
        states = int(rest) + 1 if op == "s_nop" else 1
        since = {r: n + states for r, n in since.items()}
        dst = scalars(rest.split(",")[0])
        if op.startswith("v_readfirstlane"):
            fresh += 1
            since.update({r: 0 for r in dst})
        elif op.startswith("s_"):
            for r in dst:
                since.pop(r, None)
    assert loads == count and fresh >= 2
