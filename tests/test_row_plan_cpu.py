"""CPU: the row segments of the row-streaming FP32 pass (csrc/cnn_rows.h) cover every row of every
strip exactly once, in at most one block per compute unit where the strips allow it."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2412_18379_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include "cnn_rows.h"
#include <cstdio>
#include <vector>
using namespace cnnsns::rows;

static int check(int G, int cus)
{
    const RowPlan p = row_plan(G, cus);
    const int n = p.blocks();
    if (p.strips != (G + SW - 1) / SW) return printf("G=%d: %d strips\n", G, p.strips), 1;
    if (n > cus && n > p.strips) return printf("G=%d cus=%d: %d blocks\n", G, cus, n), 1;
    std::vector<int> end(p.strips, 0);
    for (int s = 0; s < n; ++s) {
        int strip, r0, r1;
        p.at(s, G, strip, r0, r1);
        if (strip < 0 || strip >= p.strips || r0 != end[strip] || r1 <= r0 || r1 > G)
            return printf("G=%d cus=%d: block %d is strip %d rows [%d, %d)\n", G, cus, s, strip, r0, r1), 1;
        end[strip] = r1;
    }
    for (int e : end)
        if (e != G) return printf("G=%d cus=%d: a strip ends at row %d\n", G, cus, e), 1;
    return 0;
}

int main()
{
    std::vector<int> sides;
    for (int G = 1; G <= 1300; ++G) sides.push_back(G);
    for (int G : { 2047, 2048, 2049, 4095, 4096, 4097, 9999, 65535, 65536 }) sides.push_back(G);
    for (int G : sides)
        for (int cus : { 1, 7, 104, 256, 304 })
            if (check(G, cus)) return 1;
    printf("ok\n");
    return 0;
}
"""


def test_row_segments_cover_every_row_once(tmp_path):
    if not os.path.exists(HIPCC) and shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    src = tmp_path / "row_plan.cpp"
    src.write_text(PROGRAM)
    obj, exe = tmp_path / "row_plan.o", tmp_path / "row_plan"
    r = subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-I", CSRC,
                        "-c", str(src), "-o", str(obj)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    # the header's kernels are not launched: their device image and error helpers are stood in for
    stub = tmp_path / "stub.cpp"
    nm = subprocess.run(["nm", "-u", str(obj)], capture_output=True, text=True, check=True).stdout
    fat = [line.split()[-1] for line in nm.splitlines() if "__hip_fatbin" in line]
    stub.write_text("".join(f'extern "C" const char {n}[16] = {{0}};\n' for n in fat))
    r = subprocess.run([HIPCC, str(obj), str(stub), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout[-1000:] + r.stderr[-1000:]
