"""The arithmetic of the block append (csrc/akv_append_plan.h) on the CPU: the blocks of a launch cover the new tokens once, its
workgroups every part of a block once, and the length of a sequence cannot move while any workgroup of the launch has still to read it."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <cstdio>
#include <initializer_list>
#include <vector>
#include "akv_append_plan.h"
using namespace akv;
template <int S> bool each_once(int blocks, unsigned head)
{
    std::vector<int> seen(2 * S * blocks);
    for (int x = 0; x < 2 * S * blocks; ++x) {
        const AppendPart p = append_part<S>(unsigned(x), unsigned(2 * S * blocks), head);
        if (p.i < 0 || p.i >= blocks || p.v < 0 || p.v > 1 || p.sub < 0 || p.sub >= S) return false;
        ++seen[(p.i * 2 + p.v) * S + p.sub];
    }
    for (int n : seen)
        if (n != 1) return false;
    return true;
}
int main()
{
    long would_stray = 0;
    const int ns[] = {1, 15, 16, 17, 129, 200, 255, 256, 257, 258, 777, 1000, 1024};
    for (int n : ns)
        for (int cnt : {n, n - 1, n / 2 + 1})
            for (int len = 0; len < 520; ++len) {
                if (cnt < 1) continue;
                const int blocks = append_grid_blocks(n);
                int at = len;
                for (int i = 0; i < blocks; ++i) {   // the tokens, each once and in order
                    const AppendBlock x = append_block(len, cnt, i);
                    if (x.t_lo >= x.t_hi) continue;
                    if (x.t_lo != at || x.t_lo / 256 != x.blk || (x.t_hi - 1) / 256 != x.blk) return printf("n %d len %d block %d\n", n, len, i), 1;
                    at = x.t_hi;
                }
                if (at != len + cnt) return printf("n %d len %d: %d of %d tokens\n", n, len, at - len, cnt), 1;
                // Any one workgroup of the launch (block i, K or V, part, head h) is held back until all others have read the length
                // and drawn: the draws so far must not be enough to move it.
                for (int Hkv : {1, 8})
                    for (int parts : {1, 2}) {
                        const int others = 2 * parts * blocks * Hkv - 1;   // the grid's x and y extents, less one
                        if (others >= append_tickets(blocks, Hkv, parts)) return printf("n %d len %d Hkv %d parts %d: the length moves before the last read\n", n, len, Hkv, parts), 1;
                        if (others + 1 != append_tickets(blocks, Hkv, parts)) return printf("n %d len %d Hkv %d parts %d: the length never moves\n", n, len, Hkv, parts), 1;
                    }
                // why those without tokens count: with the moved length some of them would find tokens
                for (int i = 0; i < blocks; ++i) {
                    const AppendBlock x = append_block(len, cnt, i), late = append_block(len + cnt, cnt, i);
                    would_stray += x.t_lo >= x.t_hi && late.t_lo < late.t_hi;
                }
            }
    // the workgroups of a head are every part of both sides of every block, once, wherever the head begins
    for (int blocks = 1; blocks <= 40; ++blocks)
        for (unsigned head = 0; head < 200; ++head)
            if (!each_once<1>(blocks, head) || !each_once<2>(blocks, head)) return printf("blocks %d head %u\n", blocks, head), 1;
    if (!would_stray) return puts("no length shows the hazard"), 1;
    puts("clean");
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_lengths_move_behind_the_last_read(tmp_path):
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(DRIVER)
    b = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2409_16546_amd", "csrc"),
                        str(src), "-o", str(exe)], capture_output=True, text=True)
    assert b.returncode == 0, b.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "clean" in r.stdout, r.stdout
