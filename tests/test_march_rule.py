"""Which sweeps the marching kernel takes and how it cuts their columns, from the
library's own host code: no wave with many idle lanes."""
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
    printf("%d %d\n", (int)teno::march_grid(&g, 1), g.ndim == 3 ? (int)teno::march_grid(&g, 2) : 0);
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

    def ask(*n):
        n = list(n) + [1] * (3 - len(n))
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
    assert rule(*n) == want
