"""Which scoring launches reduce the window themselves (csrc/window_plan.h): bounds on what that costs a workgroup, compiled for the CPU.  No GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include "window_plan.h"
#include <cstdio>

static int log2_up(long n) { int l = 0; while ((1l << l) < n) ++l; return l; }
// The longest chain of additions behind an element of the window query that has a launch of its own: 128 slices, `run` of them in a row, their sums in
// four rows that are added up in pairs.
static int own_launch_chain(long pairs, int vec) {
    const long run = vec == 8 ? 8 : 4, groups = (pairs + run - 1) / run;
    return (int)((pairs < run ? pairs : run) - 1 + (groups + 3) / 4 - 1) + log2_up(groups < 4 ? groups : 4);
}

int main() {
    int bad = 0, inside = 0, n = 0;
    const int heads[][3] = {{32, 8, 128}, {28, 4, 128}, {32, 1, 128}, {8, 1, 64}, {4, 2, 64}, {16, 16, 64}, {64, 1, 8}, {9, 9, 128}, {6, 2, 32}, {64, 8, 128}};
    for (auto& h : heads)
        for (int vec = 4; vec <= 8; vec += 4)
            for (int w = 1; w <= 128; w = w < 10 ? w + 1 : w * 2)
                for (int nb = 1; nb <= 16384; nb = nb * 3 / 2 + 1)
                    for (int waves = 1; waves <= 16; ++waves)
                        for (int unit = 0; unit <= 64; unit = unit ? unit * 8 : 1) {       // rows of a wave's unit; 0: stored unit keys
                            const int elems = h[1] * h[2], group = h[0] / h[1], bytes = vec == 8 ? 2 : 4;
                            const long long keys = (long long)unit * waves * elems * bytes, window = (long long)w * h[0] * h[2] * bytes;
                            const auto p = slim::window_plan(elems, vec, w, group, nb, waves, keys);
                            ++n;
                            if (!p.slices) { bad += p.threads != 64 * waves; continue; }
                            ++inside;
                            const long pairs = (long)w * group, each = (pairs + p.slices - 1) / p.slices, rounds = (each + 3) / 4;
                            const int chain = log2_up(each < 4 ? each : 4) + (int)rounds - 1 + log2_up(p.slices);
                            bool ok = p.threads >= 64 * waves && p.threads <= 1024 && p.threads % 64 == 0 && (p.slices & (p.slices - 1)) == 0;
                            ok = ok && (long)p.slices * (elems / vec) <= p.threads;                        // one thread per chunk and slice
                            ok = ok && rounds <= 2 && chain <= own_launch_chain(pairs, vec);
                            ok = ok && (p.slices + 1) * elems * 4 + 64 <= 65536;                           // LDS without a raised limit
                            // the windows read: few in a launch that runs at once, or hidden under the workgroup's own keys
                            const bool at_once = nb * (p.threads / 64) <= 4096 && nb * window <= 16 << 20;
                            ok = ok && (at_once || (2 * window <= keys && p.threads == 64 * waves));
                            if (!ok && bad++ < 5)
                                printf("%d/%d x %d, vec %d, window %d, %d blocks of %d waves, unit %d: %d slices, %d threads, %ld rounds, chain %d of %d\n", h[0], h[1],
                                       h[2], vec, w, nb, waves, unit, p.slices, p.threads, rounds, chain, own_launch_chain(pairs, vec));
                        }
    printf("%d calls, %d reduce the window themselves, %d out of bounds\n", n, inside, bad);
    return bad || !inside ? 1 : 0;
}
"""


def test_reducing_the_window_in_the_scoring_launch_is_bounded(tmp_path):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(HARNESS)
    subprocess.run([gxx, "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2508_06447_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    got = subprocess.run([str(exe)], capture_output=True, text=True)
    print(got.stdout)
    assert got.returncode == 0, got.stdout
