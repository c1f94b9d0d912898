"""The norm test's kernels read the accumulator themselves only where it is memory of the context's own device; one that
lies on another device, in managed or in host memory is copied.  The predicate alone, on the CPU."""
import os
import shutil
import subprocess

import pytest

from paper_2508_18182_amd import build as B

SOURCE = r"""
#include <cstdio>
#include "common.h"
int main() {
  hipPointerAttribute_t a{};
  for (auto type : {hipMemoryTypeDevice, hipMemoryTypeHost, hipMemoryTypeManaged})
    for (int device : {0, 1}) {
      a.type = type;
      a.device = device;
      std::printf("%d", int(adloco::is_memory_of(a, 1)));
    }
  return 0;
}
"""


def test_only_memory_of_the_contexts_device(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not shutil.which(hipcc):
        pytest.skip("no hipcc")
    (tmp_path / "t.hip").write_text(SOURCE)
    exe = str(tmp_path / "t")
    subprocess.run([hipcc, *B.HIPCC_FLAGS, "-I", os.path.join(B.ROOT, "include"), "-I", B.CSRC, str(tmp_path / "t.hip"),
                    "-o", exe], check=True, capture_output=True)
    assert subprocess.run([exe], check=True, capture_output=True, text=True).stdout == "010000"
