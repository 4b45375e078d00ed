"""The stencil decisions' fast path on the CPU, through the HIP host emulation
of tests/harness/hip_emu: the cutoff mask that teno5_rec_fast chooses against
the literal formula of the same header, over every epsilon that a grid accepts
(subnormal and near the largest double included) and stencils whose smoothness
indicators lie around it."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2003_09145_amd", "csrc")

HARNESS = r'''
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdio.h>
#include <random>
#include "teno_device.hpp"
#include "teno_host.hpp"
using namespace teno;

template <bool A5>
static long differ(const teno_grid& g, unsigned seed) {
    const SchemeParams S = scheme_of(&g);
    const DecisionConsts K = decision_consts(&g, false);
    std::mt19937_64 rng(seed);
    std::uniform_real_distribution<double> step(-1.0, 1.0), level(-1.0, 3.0);
    long bad = 0;
    for (int i = 0; i < 200000; ++i) {
        // differences around sqrt(eps), with a base of the same order
        const double s = sqrt(g.eps) * exp2(level(rng));
        double v[5], at = s * step(rng);
        for (double& x : v) x = (at += s * step(rng) * (i % 3 ? 1.0 : 0x1p-6));
        uint32_t code;
        (void)teno5_rec_fast<A5>(S, K, &kOmega[0][0], v[0], v[1], v[2], v[3], v[4], &code);
        const uint32_t lit = teno5_decide_literal<A5>(S, v[0], v[1], v[2], v[3], v[4]);
        bad += (code >> 5) != (lit >> 5);
    }
    return bad;
}

int main() {
    long total = 0;
    for (double eps : {0x1p-1074, 0x1p-1071, 1e-320, 1e-310, 1e-300, 1e-280, 1e-40, 1e-6, 1.0,
                       1e280, 1e300, 0x1.fp1022, 0x1.fp1023})
        for (int scheme : {0, 1, 3}) {
            teno_grid g;
            memset(&g, 0, sizeof(g));
            g.ndim = 1;
            g.n[0] = 8;
            g.n[1] = g.n[2] = 1;
            g.dx[0] = g.dx[1] = g.dx[2] = 1.0;
            g.scheme = scheme;
            g.gamma = 1.4;
            g.ct_fixed = 1e-5;
            g.H = 10.0;
            g.Bl = 4;
            g.Bu = 10;
            g.eps = eps;
            g.a1 = 10.5;
            g.a2 = 3.5;
            g.cr = 0.25;
            g.xi = 1e-3;
            if (validate(&g) != TENO_OK) return 2;
            const long n = scheme == 3 ? differ<true>(g, 1) : differ<false>(g, 2);
            if (n) printf("eps %.3g scheme %d: %ld of 200000 masks differ\n", eps, scheme, n);
            total += n;
        }
    printf("differ %ld\n", total);
    return total != 0;
}
'''


def test_fast_decisions_equal_literal_over_epsilon(tmp_path):
    src, exe = tmp_path / "decisions.cpp", tmp_path / "decisions"
    src.write_text(HARNESS)
    subprocess.run(["g++", "-O2", "-std=c++17", "-mfma", "-ffp-contract=off", "-Wno-attributes",
                    "-pthread", "-I", os.path.join(HERE, "harness", "hip_emu"), "-I", CSRC,
                    "-I", os.path.join(ROOT, "include"), "-o", str(exe), str(src)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr
