"""The arithmetic of the unpack's launch (csrc/akv_unpack_plan.h) on the CPU: every size a device can hold fits one launch (fewer than
2^32 threads), and each block of K and V is covered."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <cstdio>
#include "akv_unpack_plan.h"
using namespace akv;
int main()
{
    // 64 KB of K and V planes and as much output per block: 288 GB are about 2.2 million blocks with one output
    const size_t sizes[] = {1, 2, 160, 161, 192, 193, 511, 1023, 1024, 1025, 4096, 493447, 493448, 986894, 986895, 986896, 1100000, 2200000, 8388607};
    for (size_t blocks : sizes)
        for (int kv = 1; kv < 4; ++kv) {
            const bool k = kv & 1, v = kv & 2;
            const UnpackPlan p = unpack_plan(blocks, k, v);
            const bool parts = p.k_parts == int(k) && (!v ? p.v_parts == 0 : (k ? (p.v_parts == 1 || p.v_parts == 16) : (p.v_parts == 2 || p.v_parts == 4 || p.v_parts == 8)));
            if (!parts) return printf("%zu blocks, outputs %d: %d + %d parts have no kernel\n", blocks, kv, p.k_parts, p.v_parts), 1;
            if (p.workgroups != blocks * (p.k_parts + p.v_parts)) return printf("%zu blocks, outputs %d: %zu workgroups\n", blocks, kv, p.workgroups), 1;
            if (p.workgroups * 256 >= 1ull << 32) return printf("%zu blocks, outputs %d: %zu workgroups do not fit a launch\n", blocks, kv, p.workgroups), 1;
        }
    if (unpack_plan(986895, true, true).v_parts != 16 || unpack_plan(1024, true, true).v_parts != 16 || unpack_plan(1023, true, true).v_parts != 1)
        return puts("the line between one and sixteen workgroups per block of V moved"), 1;
    if (unpack_plan(1, false, true).v_parts != 8 || unpack_plan(160, false, true).v_parts != 8 || unpack_plan(161, false, true).v_parts != 4 || unpack_plan(192, false, true).v_parts != 4 || unpack_plan(193, false, true).v_parts != 2)
        return puts("the lines between eight, four and two workgroups per block of V alone moved"), 1;
    if (unpack_plan(size_t(1) << 24, true, true).workgroups != 0) return puts("a launch too large is not refused"), 1;
    puts("clean");
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_every_unpack_fits_one_launch(tmp_path):
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(DRIVER)
    b = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2409_16546_amd", "csrc"),
                        str(src), "-o", str(exe)], capture_output=True, text=True)
    assert b.returncode == 0, b.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "clean" in r.stdout, r.stdout
