// Host-side helpers shared by the HIP translation units of libteno.so:
// argument validation and the per-launch scheme / decision constants.
#pragma once

#include <cmath>

#include <math.h>
#include <stdint.h>
#include <string.h>

#include "../../include/teno.h"
#include "teno_device.hpp"
#include "teno_divmagic.hpp"

namespace teno {

inline int validate(const teno_grid* g) {
    if (g == nullptr) return TENO_ERR_ARG;
    if (g->ndim < 1 || g->ndim > 3) return TENO_ERR_ARG;
    for (int k = 0; k < 3; ++k) {
        if (k < g->ndim) {
            if (g->n[k] < 3) return TENO_ERR_ARG;
            if (!(g->dx[k] > 0.0)) return TENO_ERR_ARG;
            if (g->bc[k] < 0 || g->bc[k] > 2) return TENO_ERR_ARG;
        } else if (g->n[k] != 1) {
            return TENO_ERR_ARG;
        }
    }
    if (!(g->gamma > 1.0)) return TENO_ERR_ARG;
    if (g->scheme < 0 || g->scheme > 3) return TENO_ERR_ARG;
    if (g->scheme == 0) {
        if (g->Bl < 0 || g->Bu > 20 || g->Bl > g->Bu || !(g->H > 0.0)) return TENO_ERR_ARG;
    }
    if (g->scheme == 3) {
        // floor(beta) of eq 2.16 stays in [floor(a1 - a2), floor(a1)] within the ladder
        if (!(g->a2 >= 0.0) || !(g->a1 - g->a2 >= 0.0) || !(g->a1 <= 20.0)) return TENO_ERR_ARG;
        if (!(g->cr > 0.0) || !(0.9 * g->cr < 1.0) || !(g->xi >= 0.0) || !std::isfinite(g->xi))
            return TENO_ERR_ARG;
    }
    if (!(g->eps > 0.0)) return TENO_ERR_ARG;
    if (g->flags & ~(TENO_FLAG_LITERAL_DECISIONS | TENO_FLAG_MASK_DIGEST)) return TENO_ERR_ARG;
    if (g->theta != TENO_THETA_PRINTED && g->theta != TENO_THETA_CUT) return TENO_ERR_ARG;
    return TENO_OK;
}

inline SchemeParams scheme_of(const teno_grid* g) {
    SchemeParams s;
    s.gamma = g->gamma;
    s.ct_fixed = g->ct_fixed;
    s.H = g->H;
    s.eps = g->eps;
    s.scheme = g->scheme;
    s.Bl = g->Bl;
    s.Bu = g->Bu;
    s.bu_bl = (double)(g->Bu - g->Bl);
    s.a1 = g->a1;
    s.a2 = g->a2;
    s.cr = g->cr;
    s.kA_nan = 0;
    s.theta_cut = (g->scheme == TENO_SCHEME_LAD && g->theta == TENO_THETA_CUT) ? 1 : 0;
    s.epsA = 0.0;
    if (g->scheme == 3) {
        s.kA_nan = (int)std::floor(g->a1 - g->a2);
        s.epsA = ((0.9 * g->cr) / (1.0 - 0.9 * g->cr)) * (g->xi * g->xi);  // eq 2.18
    }
    return s;
}

// The cutoff ladder of eq 3.3 on the host: kLadderHost[k] = 10^-k.
inline const double kLadderHost[21] = {1e0,   1e-1,  1e-2,  1e-3,  1e-4,  1e-5,  1e-6,
                                       1e-7,  1e-8,  1e-9,  1e-10, 1e-11, 1e-12, 1e-13,
                                       1e-14, 1e-15, 1e-16, 1e-17, 1e-18, 1e-19, 1e-20};

// Largest T with 1 / (1 + 2 (1 + T)^6) >= ct (1 + 2^-30), shrunk by 2^-30:
// stencils whose chi~_k are all <= T keep every candidate for any cutoff up
// to ct (the rounding of the literal evaluation is far inside both
// margins).  -1 when ct leaves no such T.
inline double smooth_bound(double ct) {
    if (!(ct > 0.0)) return -1.0;
    const double g = (1.0 / (ct * (1.0 + 0x1p-30)) - 1.0) / 2.0;  // bound on (1 + T)^6
    if (!(g > 1.0)) return -1.0;
    const double T = (std::pow(g, 1.0 / 6.0) - 1.0) * (1.0 - 0x1p-30);
    return T > 0.0 ? T : -1.0;
}

inline DecisionConsts decision_consts_base(const teno_grid* g, bool need_m);

// Decision constants with the host-side margin products filled in.
inline DecisionConsts decision_consts(const teno_grid* g, bool need_m) {
    DecisionConsts K = decision_consts_base(g, need_m);
    K.hi_fac = K.ct_hi * (1.0 + kDecisionMargin);
    K.lo_fac = K.ct_lo * (1.0 - kDecisionMargin);
    K.ymarg = kDecisionMargin * K.nthr_d;
    if (K.literal || K.need_m) K.smooth_t = -1.0;
    K.eps4 = 4.0 * g->eps;
    K.smooth_te = K.smooth_t * K.eps4;
    return K;
}

inline DecisionConsts decision_consts_base(const teno_grid* g, bool need_m) {
    DecisionConsts K;
    memset(&K, 0, sizeof(K));
    // With an epsilon near the ends of the double range the indicators that
    // matter are subnormal or overflow, and four times an indicator does not
    // round as the indicator does (at 2^-1074 a mask in 100000 differed).
    const bool plain_eps = g->eps >= 0x1p-900 && g->eps <= 0x1p900;
    K.literal = (g->flags & TENO_FLAG_LITERAL_DECISIONS) || !plain_eps ? 1 : 0;
    K.need_m = need_m ? 1 : 0;
    K.smooth_t = -1.0;
    K.h_hi = K.h_lo = NAN;
    if (g->scheme == TENO_SCHEME_FIXED_CT) {
        K.ct_hi = K.ct_lo = g->ct_fixed;
        K.smooth_t = smooth_bound(K.ct_hi);
        return K;
    }
    if (g->scheme == TENO_SCHEME_TENO5A) {
        // the cutoff is evaluated per reconstruction; its largest value bounds
        // the smooth-stencil shortcut
        const int khi = (int)std::floor(g->a1 - g->a2);
        K.ct_hi = kLadderHost[khi];
        K.ct_lo = kLadderHost[20];
        K.smooth_t = smooth_bound(K.ct_hi);
        return K;
    }
    if (g->scheme != TENO_SCHEME_LAD) return K;
    K.ct_hi = kLadderHost[g->Bl];
    K.ct_lo = kLadderHost[g->Bu];
    K.smooth_t = smooth_bound(K.ct_hi);
    K.nthr = g->Bu - g->Bl;
    K.nthr_d = (double)K.nthr;
    K.inv_h = 1.0 / g->H;
    if (g->theta == TENO_THETA_CUT) {
        // the approximate max chi~ is within a few ulp of the literal one
        K.h_hi = g->H * (1.0 + kDecisionMargin);
        K.h_lo = g->H * (1.0 - kDecisionMargin);
    }
    return K;
}

// Columns of the marching sweep along `dir` (y or z).
inline int64_t march_cols(const teno_grid* g, int dir) {
    return dir == 1 ? (int64_t)g->n[0] * g->n[2] : (int64_t)g->n[0] * g->n[1];
}

// Whether the marching sweep (teno_march.hip) takes a grid's sweeps along `dir`
// (with or without the stage update), but for those with decision bytes or
// digests.  It pays once its waves (64 columns each) have enough rows to fill the
// chip at two waves per SIMD; below that the face-stream sweep spreads the same
// faces over more waves.  A stencil that is not smooth costs the march more (a
// decision pass stops all 64 columns), so the lines lie where flows full of jumps
// (three planar ones, and the noise behind them) are about even.  Speed against
// the face stream, jump flows (one seed each), then smooth flows:
//  - 2D sweeps with the stage update: step of 1792 x 2048 (57344 rows) 0.94, 1.00,
//    1.03, and 1.03; of 2048^2 (65536) 0.97, 1.01, 1.01, 1.03, 1.06, and 1.07;
//  - without it: right-hand side of 2048^2 0.94, 0.95, 1.00, and 1.03; of 2304^2
//    (82944 rows) 1.00, 1.01, 1.04, and 1.05;
//  - 3D: step of 208^3 (140608 rows) 0.95, 0.98, 1.03, and 1.05; of 220^3 (166540) 0.99,
//    1.04, 1.06, and 1.08; of 256^3 0.99, 1.03, 1.05, and 1.10.
// Idle lanes cost their share, which the face-stream sweep does not pay: a sweep
// of 3 x 60005 cells took 138 us against 13, 33 x 60011 153 / 99, 96 x 100000 481 /
// 421, 200 x 64000 587 / 554, but 128 x 100000 477 / 557; so at most a lane in 16
// may be idle.
inline bool march_grid(const teno_grid* g, int dir, bool stage) {
    if (dir == 0) return false;
    const int64_t cols = march_cols(g, dir), groups = (cols + 63) / 64;
    const int64_t rows = groups * g->n[dir];
    const int64_t least = g->ndim == 3 ? 160000 : stage ? 60000 : 80000;
    if (rows < least || g->n[dir] < 24) return false;
    if (16 * cols < 15 * 64 * groups) return false;
    // 32-bit lane offsets within a wave's columns and block count
    const int64_t plane = (int64_t)g->n[0] * g->n[1];
    return (63 / g->n[0] + 2) * plane < (int64_t(1) << 29) && rows < (int64_t(1) << 31);
}

// Segments of the `n` rows of each of `groups` groups of columns, for waves of which
// the chip holds 2048 at a time.  Waves are dealt out from the last segment to the
// first, to the XCDs in turn or (by_xcd) an eighth of them to each in one stretch;
// the segments dealt out first are twice as long as those dealt out last.  A wave on a
// jump has several times the work of the others, and one that begins late ends
// long after them: with two rounds of equal waves, steps of 256^3 with three
// jumps took 10.89, 9.25 and 8.99 ms (three seeds), uneven 9.91, 8.96 and 8.28; of 2048^2
// 1.40, 1.33 and 1.38 ms, uneven 1.30, 1.28 and 1.32.  Three rounds of equal waves do as
// much for these flows, but stage 5 more rows half as often again: 1% of a smooth
// 256^3 step and 1 to 4% of a 2048^2 one.
// Of the numbers of segments for at least two rounds, with 12 rows each (equal
// ones: three rounds, 8 rows), the one whose rounds take the fewest rows, 1.5 of them
// for the staging ahead of a segment.
inline MarchCut march_cut(int groups, int n, bool by_xcd) {
    int step = by_xcd ? 8 : 1;  // each XCD its own long and short segments
    bool uneven = groups * (int64_t)step <= 12288 && n >= 12 * step;
    if (!uneven) step = 1;
    const int most = n / (uneven ? 12 : 8) / step * step, hi = 12288 / groups;
    int lo = (uneven ? 2048 : 4096) / groups + 1;
    lo = (lo + step - 1) / step * step;
    int nseg = lo < most ? lo : most;
    double best = 1e30;
    for (int k = nseg; k <= hi && k <= most; k += step) {
        const int64_t rounds = ((int64_t)groups * k + 2047) / 2048;
        const double rows = (double)rounds * ((double)((n + k - 1) / k) + 1.5);
        if (rows < best) {
            best = rows;
            nseg = k;
        }
    }
    return {nseg, !uneven ? 1 : by_xcd ? nseg / 8 : nseg};
}

}  // namespace teno
