"""Which sweeps the marching kernel takes and how it cuts their columns, from the
library's own host code: no wave with many idle lanes, and enough waves that one on
a jump does not end long after the others."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

HARNESS = r'''
#include <hip/hip_runtime.h>
#include <stdio.h>
#include <stdlib.h>
#include "teno_host.hpp"
int main(int argc, char** argv) {
    teno_grid g;
    memset(&g, 0, sizeof(g));
    for (int k = 0; k < 3; ++k) g.n[k] = atoi(argv[1 + k]);
    g.ndim = g.n[2] > 1 ? 3 : 2;
    const bool stage = atoi(argv[4]) != 0;
    printf("%d %d", (int)teno::march_grid(&g, 1, stage),
           g.ndim == 3 ? (int)teno::march_grid(&g, 2, stage) : 0);
    const int groups = (int)((teno::march_cols(&g, 1) + 63) / 64);
    const int n = g.n[1];
    if (n >= 24) {
        const teno::MarchCut cut = teno::march_cut(groups, n, g.ndim == 2);
        printf(" %d %d %d", groups, cut.nseg, cut.period);
        for (int s = 0; s <= cut.nseg; ++s) printf(" %d", teno::march_row(cut, n, s));
    }
    printf("\n");
    return 0;
}
'''


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("rule")
    (d / "rule.cpp").write_text(HARNESS)
    subprocess.run(["g++", "-O1", "-std=c++17", "-mfma", "-ffp-contract=off", "-Wno-attributes",
                    "-pthread", "-I", os.path.join(HERE, "harness", "hip_emu"), "-I",
                    os.path.join(ROOT, "paper_2003_09145_amd", "csrc"), "-o", str(d / "rule"),
                    str(d / "rule.cpp")], check=True)

    def ask(*n, stage=True):
        n = list(n) + [1] * (3 - len(n)) + [int(stage)]
        out = subprocess.run([str(d / "rule"), *map(str, n)], capture_output=True, text=True, check=True)
        return [int(x) for x in out.stdout.split()]
    return ask


@pytest.mark.parametrize("n,want", [
    ((3, 60005), [0, 0]), ((33, 60011), [0, 0]), ((96, 100000), [0, 0]), ((200, 64000), [0, 0]),
    ((65, 200000), [0, 0]), ((60, 200000), [1, 0]), ((59, 200000), [0, 0]), ((128, 100000), [1, 0]),
    ((2048, 2048), [1, 0]), ((2560, 2560), [1, 0]), ((1024, 1024), [0, 0]), ((160000, 30), [1, 0]),
    ((256, 256, 256), [1, 1]), ((128, 128, 128), [0, 0]), ((5, 160003, 5), [0, 0]),
    ((12, 160003, 5), [1, 0]), ((12, 5, 160003), [0, 1]), ((6, 5, 160001), [0, 0]),
    ((5, 400, 5120), [1, 1]), ((65, 23, 160000), [0, 1])])
def test_march_takes_full_waves(rule, n, want):
    assert rule(*n)[:2] == want


@pytest.mark.parametrize("n,step,rhs", [
    ((2048, 2048), 1, 0), ((1792, 2048), 0, 0), ((2560, 2560), 1, 1), ((2304, 2304), 1, 1),
    ((2240, 2240), 1, 0)])
def test_march_takes_right_hand_sides_later(rule, n, step, rhs):
    assert [rule(*n)[0], rule(*n, stage=False)[0]] == [step, rhs]


@pytest.mark.parametrize("n", [
    (2048, 2048), (1024, 4096), (60, 60005), (61, 100003), (2432, 2400), (2896, 2896), (1530, 24003),
    (160000, 30), (2500000, 24), (1000000, 25), (131072, 40), (98304, 96), (98368, 95), (524288, 100),
    (256, 256, 256), (220, 220, 220), (320, 320, 320), (400, 400, 400), (5, 400, 5120),
    (1024, 63, 200), (4096, 24, 320), (4096, 25, 1000), (64, 160000, 3), (250, 36, 300)])
def test_march_cut(rule, n):
    _, _, groups, nseg, period, *rows = rule(*n)
    size = [b - a for a, b in zip(rows, rows[1:])]
    assert len(size) == nseg and rows[0] == 0 and rows[-1] == n[1]
    # what the kernel's staging needs, and what the rule means to keep
    assert min(size) >= 6
    assert nseg % period == 0 and (period == 1 or n[1] >= 12 * nseg)
    # at least two rounds of 2048 waves where the rows allow it
    assert groups * nseg > 2048 or nseg + (8 if len(n) == 2 else 1) > n[1] // 12
    # in 2D each XCD takes an eighth of the segments: the same rows each, the long ones last
    if len(n) == 2 and period > 1:
        assert nseg == 8 * period
        eighth = [rows[(k + 1) * period] - rows[k * period] for k in range(8)]
        assert max(eighth) - min(eighth) <= 1
    half = period // 2
    for k in range(0, nseg, period):
        short, long = size[k:k + half], size[k + half:k + period]
        if short:
            assert max(short) < min(long) and 2 * max(short) + 2 >= max(long)
