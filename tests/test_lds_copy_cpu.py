"""CPU: a kernel that copies into LDS (csrc/lds_copy.h) compiles for gfx950 without a warning: the compiler knows which value the
copy needs in M0, a register that an asm statement may not overwrite by itself."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2412_18379_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

KERNEL = r"""
#include "lds_copy.h"
__global__ void k(const float4* from, float4* to)
{
    __shared__ float4 s[2][256];
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    for (int i = 0; i < 2; ++i) cnnsns::lds_copy16(from + 256 * i + threadIdx.x, &s[i][64 * wave]);
    cnnsns::lds_copies_arrived();
    __syncthreads();
    to[threadIdx.x] = s[lane & 1][255 - threadIdx.x];
}
"""


def test_copies_compile_without_a_warning(tmp_path):
    if not os.path.exists(HIPCC) and shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    src = tmp_path / "copy.hip"
    src.write_text(KERNEL)
    r = subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-device-only", "-O3", "-std=c++17", "-Wall", "-I", CSRC,
                        "-S", str(src), "-o", str(tmp_path / "copy.s")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    assert "lds_copy.h" not in r.stderr, r.stderr[-2000:]
    assert (tmp_path / "copy.s").read_text().count("global_load_lds_dwordx4") == 2
