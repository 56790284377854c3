"""CPU: the walks' order of blocks (csrc/xcd_order.h) takes every block of points exactly once, each XCD's in chunks of
consecutive ones, and its grid stays below a launch's 2^32 threads wherever the blocks themselves do."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2412_18379_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include "xcd_order.h"
#include <cstdint>
#include <cstdio>
#include <vector>
using namespace cnnsns;

static int check(unsigned n, unsigned longest)
{
    const XcdOrder o(n, longest);
    if (!o.chunk) return o.grid() == n ? 0 : (printf("n=%u: grid %u\n", n, o.grid()), 1);
    if (o.chunk > longest) return printf("n=%u: chunk %u\n", n, o.chunk), 1;
    if ((uint64_t)n * 256 < (uint64_t)1 << 32 && (uint64_t)o.grid() * 256 >= (uint64_t)1 << 32)
        return printf("n=%u: grid %u\n", n, o.grid()), 1;
    if (n > 100000) return 0;
    std::vector<char> seen(n, 0);
    for (unsigned id = 0; id < o.grid(); ++id) {
        const unsigned b = o.block(id);
        if (b >= n) continue;
        if (seen[b]++) return printf("n=%u: block %u twice\n", n, b), 1;
        if (id >= 8 && b % o.chunk && b != o.block(id - 8) + 1) return printf("n=%u: chunk broken at %u\n", n, b), 1;
    }
    for (char s : seen)
        if (!s) return printf("n=%u: a block is missing\n", n), 1;
    return 0;
}

int main()
{
    for (unsigned longest : { 32u, 128u, 192u }) {
        for (unsigned n = 0; n <= 5000; ++n)
            if (check(n, longest)) return 1;
        for (unsigned n : { 8191u, 31285u, 62571u, 99999u, 1000003u, 16776000u, 16777000u, 16777215u })
            if (check(n, longest)) return 1;
    }
    printf("ok\n");
    return 0;
}
"""


def test_every_block_once_and_no_grid_too_large(tmp_path):
    if not os.path.exists(HIPCC) and shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    src, exe = tmp_path / "xcd_order.cpp", tmp_path / "xcd_order"
    src.write_text(PROGRAM)
    r = subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-I", CSRC,
                        str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout[-1000:] + r.stderr[-1000:]
