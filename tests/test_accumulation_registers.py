"""A kernel that keeps its products in accumulation registers by number, behind the compiler's back, must not share them
with the compiler: outside of inline assembly nothing may touch them, and nothing may be spilled (checked on the
assembly; no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2508_18182_amd import build as B


@pytest.mark.parametrize("source,kernel,count", [("gram_kernels.hip", "gram_region_kernel", 2)])
def test_only_the_assembly_touches_them(source, kernel, count, tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not shutil.which(hipcc):
        pytest.skip("no hipcc")
    asm = tmp_path / "k.s"
    subprocess.run([hipcc, *B.HIPCC_FLAGS, "-I", os.path.join(B.ROOT, "include"), "-I", B.CSRC, "-S", "--offload-device-only",
                    os.path.join(B.CSRC, source), "-o", str(asm)], check=True, capture_output=True)
    text = asm.read_text()
    bodies = re.findall(r"^(_Z\S*%s\S*):.*?\n(.*?)^\.Lfunc_end" % kernel, text, re.M | re.S)
    assert len(bodies) == count
    for name, body in bodies:
        inside, used = False, 0
        for line in body.splitlines():
            if "#ASMSTART" in line or "#ASMEND" in line:
                inside = "#ASMSTART" in line
                continue
            code = line.split(";")[0]
            touches = re.search(r"^\s+[a-z].*[\s,]a(\d+\b|\[)", code)
            used += bool(touches and inside)
            assert inside or not touches, f"{name}: {line.strip()}"
            assert "scratch_" not in code, f"{name}: {line.strip()}"
        assert used > 500
        kd = re.search(r"\.amdhsa_kernel %s\n(.*?)\.end_amdhsa_kernel" % re.escape(name), text, re.S)[1]
        free, offset = (int(re.search(r"\.amdhsa_%s (\d+)" % f, kd)[1]) for f in ("next_free_vgpr", "accum_offset"))
        assert free - offset == 256          # all of them are the kernel's
