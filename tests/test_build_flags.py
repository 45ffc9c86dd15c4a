"""The flags every HIP source is compiled with."""
import os
import subprocess

import pytest

from paper_2608_12703_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# Kernels reuse LDS through another type (16-bit keys, then float partials).  A compiler that
# takes the two types for distinct objects answers the last load with the first store's value.
SOURCE = """
#include <hip/hip_runtime.h>
extern "C" __global__ void two_views(float* out, float* p, unsigned short* q) {
  *p = 1.0f;
  *q = 0;
  *out = *p;
}
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_accesses_of_different_types_stay_ordered(tmp_path):
    src, asm = tmp_path / "two_views.hip", tmp_path / "two_views.s"
    src.write_text(SOURCE)
    flags = [f for f in build.HIP_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([HIPCC, *flags, "-S", "--cuda-device-only", str(src), "-o", str(asm)], check=True,
                   capture_output=True)
    body = asm.read_text().split("two_views:", 1)[1].split("s_endpgm", 1)[0]
    assert "global_load_dword" in body      # *p is read again after the 16-bit store
