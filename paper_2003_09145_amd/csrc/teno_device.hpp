// Device-side building blocks of the TENO5-LAD Euler right-hand side
// (Peng et al., arXiv:2003.09145) for gfx950.
//
// Every function here evaluates its formula in one fixed operation order
// (no FMA contraction: the library is built with -ffp-contract=off), so that
// the GPU result is reproducible bit for bit and every cutoff decision is a
// deterministic function of the input state.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "teno_index.hpp"

namespace teno {

// Scheme parameters as the kernels see them (copied from teno_grid).
struct SchemeParams {
    double gamma;
    double ct_fixed;
    double H;
    double eps;
    int32_t scheme;  // 0 LAD, 1 fixed C_T, 2 linear (all stencils kept), 3 TENO5-A
    int32_t Bl, Bu;
    int32_t kA_nan;  // TENO5-A: exponent taken by a non-finite sensor, floor(a1 - a2)
    int32_t theta_cut;  // LAD: 1 sets theta = 0 where max chi~ > H (eq 3.2, cut form)
    double bu_bl;    // LAD: (double)(B_u - B_l) (host-converted)
    double a1, a2;   // TENO5-A: alpha_1, alpha_2 of eq 2.16
    double cr;       // TENO5-A: C_r of eq 2.17
    double epsA;     // TENO5-A: 0.9 C_r / (1 - 0.9 C_r) xi^2 of eq 2.18 (host-evaluated)
};

// Ladder array of Sec. 3 eq 3.3 as decimal literals: kLadder[k] = 10^-k, so
// C_T = Lad(m) = kLadder[m] (eq 3.4).
__constant__ const double kLadder[21] = {
    1e0,  1e-1,  1e-2,  1e-3,  1e-4,  1e-5,  1e-6,  1e-7,  1e-8,  1e-9, 1e-10,
    1e-11, 1e-12, 1e-13, 1e-14, 1e-15, 1e-16, 1e-17, 1e-18, 1e-19, 1e-20};

// Coefficients of Sec. 2: the FP64 quotients of the printed integer ratios.
constexpr double kB13_12 = 13.0 / 12.0;  // eq 2.9-2.11
constexpr double kB1_4 = 0.25;
constexpr double kC1_3 = 1.0 / 3.0;      // eq 2.4-2.6
constexpr double kC7_6 = 7.0 / 6.0;
constexpr double kC11_6 = 11.0 / 6.0;
constexpr double kC1_6 = 1.0 / 6.0;
constexpr double kC5_6 = 5.0 / 6.0;
constexpr double kLin0 = 0.1, kLin1 = 0.6, kLin2 = 0.3;  // linear weights

// ---------------------------------------------------------------------------
// Correctly rounded FP64 division and square root.
//
// The compiler's FP64 a / b sequence on gfx950 is faithful but not always
// correctly rounded (for instance 0.3499999999999998 / 0.12499999999999993
// returns 2.8 instead of 2.8000000000000003), and the method's cutoff
// decisions must match an IEEE-754 evaluation bit for bit.  Both wrappers take
// the hardware result q (within one ulp), form the remainder with one FMA --
// exact, because the remainder of a faithful quotient (a - q b) or root
// (x - s^2) is representable -- and move q to its neighbour when the exact
// value lies beyond the midpoint (ties to even for the quotient; a square
// root of a double is never a midpoint).  Operands are restricted to
// [2^-900, 2^900] in magnitude for the correction (no under/overflow in the
// remainder); outside it the hardware value is returned.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double step_toward(double q, bool up) {
    const long long bits = __double_as_longlong(q);
    return __longlong_as_double(bits + (((q > 0.0) == up) ? 1ll : -1ll));
}

__device__ __forceinline__ bool in_safe_range(double v) {
    const double av = fabs(v);
    return av >= 0x1p-900 && av <= 0x1p900;
}

// b in [2^-400, 2^400): one unsigned compare of the high word, which also
// turns away negative values, zeros, infinities and NaN.
__device__ __forceinline__ bool in_mid_range(double b) {
    return (uint32_t)(__double_as_longlong(b) >> 32) - 0x26f00000u < 0x58f00000u - 0x26f00000u;
}

// Sufficient test that q = RN(a / b) given r = RN(a - q b): |a/b - q| <
// ulp(q)/2 with both neighbours of q one ulp away makes q the nearest
// double.  q = mq 2^eq with |mq| in (1/2, 1) excludes zero, powers of two,
// infinities and NaN; ulp(q)/2 |b| = |b| 2^(eq - 54) is computed exactly when
// it is a normal number (checked; for a subnormal q the bound is smaller than
// the true half-ulp, which only makes the test stricter); and rounding is
// monotone, so |r| below the bound implies the exact remainder is below it,
// whether or not r itself is exact.  Signed zeros and operands outside the
// normal range therefore never pass and take the exact path.
__device__ __forceinline__ bool quotient_is_nearest(double q, double b, double r) {
    int eq;
    const double mq = frexp(q, &eq);
    const double hb = ldexp(fabs(b), eq - 54);
    return fabs(r) < hb && hb >= 0x1p-1000 && fabs(mq) > 0.5;
}

__device__ __forceinline__ double cr_div(double a, double b) {
    const double q = a / b;
    const double r = __builtin_fma(-q, b, a);  // a - q b, exact in the safe range
    if (quotient_is_nearest(q, b, r)) return q;
    if (!(in_safe_range(a) && in_safe_range(b) && in_safe_range(q))) return q;
    if (r == 0.0) return q;
    const bool up = (r > 0.0) == (b > 0.0);     // true quotient above q
    const double qn = step_toward(q, up);
    const double h = 0.5 * ((qn - q) * b);      // remainder at the midpoint, exact
    const double ar = fabs(r), ah = fabs(h);
    if (ar > ah) return qn;
    if (ar == ah) return (__double_as_longlong(q) & 1ll) ? qn : q;
    return q;
}

__device__ __forceinline__ double cr_sqrt_exact(double x) {
    const double s = sqrt(x);
    if (!(x >= 0x1p-900 && x <= 0x1p900)) return s;
    const double r = __builtin_fma(-s, s, x);  // x - s^2, exact
    if (r == 0.0) return s;
    const bool up = r > 0.0;
    const double sn = step_toward(s, up);
    const double sg = s * (sn - s);             // exact: the gap is a power of two
    if (up) return (r > sg) ? sn : s;
    return (r <= sg) ? sn : s;
}

// sqrt(x) correctly rounded.  For x in [2^-400, 2^400) the root comes from the
// hardware reciprocal square root refined by one Goldschmidt and two Newton
// steps (no scaling is needed there).  A root that the test below does not
// certify takes the exact neighbour test on the compiler's root.
// Fast phase: *s is the refined root (for x outside the safe range, any
// value); true when it is certified.  The exact phase is cr_sqrt_exact.
//
// The certificate is a rounding test: with r = x - s^2 (exact) and h = (1 / 2s)
// (1 + d), |d| < 2^-44 (the hardware's reciprocal root has a relative error
// below 2^-23, and one Goldschmidt step squares it), the distance of the root
// from s is r h to a relative 2^-43, so s + r h (1 + 2^-40) rounding to s puts
// the root nearer to s than to any other double (the spacing below a power of
// two included).
__device__ __forceinline__ bool sqrt_fast(double x, double* sout) {
    const double y = __builtin_amdgcn_rsq(x);
    double s = x * y;
    double h = 0.5 * y;
    const double e = __builtin_fma(-h, s, 0.5);
    s = __builtin_fma(s, e, s);
    h = __builtin_fma(h, e, h);
    double d = __builtin_fma(-s, s, x);
    s = __builtin_fma(d, h, s);
    d = __builtin_fma(-s, s, x);
    s = __builtin_fma(d, h, s);
    const double r = __builtin_fma(-s, s, x);
    *sout = s;
    return in_mid_range(x) && __builtin_fma(r * (1.0 + 0x1p-40), h, s) == s;
}
__device__ __forceinline__ double cr_sqrt(double x) {
    double s;
    if (sqrt_fast(x, &s)) return s;
    return cr_sqrt_exact(x);
}

// Reciprocal to within a few ulp: hardware estimate plus two Newton steps.
__device__ __forceinline__ double rcp_nr(double b) {
    double r = __builtin_amdgcn_rcp(b);
    double e = __builtin_fma(-b, r, 1.0);
    r = __builtin_fma(r, e, r);
    e = __builtin_fma(-b, r, 1.0);
    return __builtin_fma(r, e, r);
}

// Correctly rounded reciprocal and quotients without a test per quotient (P.
// Markstein, "Computation of elementary functions on the IBM RISC System/6000
// processor", IBM J. Res. Dev. 34, 1990):
//  - a Newton step y + y (1 - b y) from a y within one ulp of 1 / b rounds to
//    RN(1 / b) unless every mantissa bit of b is set (rcp_nr is within 0.6 ulp:
//    the hardware estimate's 2^-23, squared twice, plus one rounding);
//  - with y = RN(1 / b) and q within one ulp of a / b, q - (q b - a) y rounds
//    to RN(a / b) (the remainder is exact).
// rcp_exact reports whether y is certified: b in [2^-400, 2^400] and its low
// mantissa word not all ones.  quot takes a certified y and an a that is zero
// or within [2^-600, 2^600] in magnitude (quot_ok, and the caller's bound), so
// that no remainder under- or overflows; the negated remainder keeps a zero's
// sign.  Everything else takes cr_div.  Against the test of every quotient's
// remainder with half the spacing of doubles this took 3 of 11 instructions
// off a quotient, 6 of 16 off a reciprocal, and it does not fail for zero
// dividends and powers of two (128 x 512 Rayleigh-Taylor: -6% per step; with
// the 4 beta form below: -6% per 256^3 step, 1326 -> 1180 VALU instructions
// per wave of 63 faces).
__device__ __forceinline__ bool rcp_exact(double b, double* y) {
    const double r = rcp_nr(b);
    *y = __builtin_fma(r, __builtin_fma(-b, r, 1.0), r);
    return in_mid_range(b) && (uint32_t)__double_as_longlong(b) != 0xffffffffu;
}
__device__ __forceinline__ double quot(double a, double b, double y) {
    const double q0 = a * y;
    const double q1 = __builtin_fma(-__builtin_fma(q0, b, -a), y, q0);
    return __builtin_fma(-__builtin_fma(q1, b, -a), y, q1);
}
// Lower bound of quot's dividends (the caller bounds them from above).
__device__ __forceinline__ bool quot_ok(double a) { return !(fabs(a) < 0x1p-600) || a == 0.0; }

// q[i] = a[i] / b correctly rounded for N independent dividends, from y =
// RN(1 / b) (yok: certified, see rcp_exact): one correction branch for all.
template <int N>
__device__ __forceinline__ void cr_div_n(const double (&a)[N], double b, double y, bool yok,
                                         double (&q)[N]) {
    bool ok = yok;
    double big = 0.0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        q[i] = quot(a[i], b, y);
        ok = ok && quot_ok(a[i]);
        big = (i == 0) ? fabs(a[i]) : big + fabs(a[i]);
    }
    if (!(ok && big < 0x1p600)) {
#pragma unroll
        for (int i = 0; i < N; ++i) q[i] = cr_div(a[i], b);
    }
}

// a / b and 1 / b correctly rounded for positive b.
__device__ __forceinline__ double cr_div_p(double a, double b) {
    double y;
    if (rcp_exact(b, &y) && quot_ok(a) && fabs(a) < 0x1p600) return quot(a, b, y);
    return cr_div(a, b);
}
__device__ __forceinline__ double cr_rcp(double b) {
    double y;
    if (rcp_exact(b, &y)) return y;
    return cr_div(1.0, b);
}

// TENO weights of eq 2.15 for each cutoff mask, omega_k = delta_k c_k / D with
// D = (delta_0 c_0 + delta_1 c_1) + delta_2 c_2, folded at compile time in
// IEEE round-to-nearest (the same operations and order as the runtime form).
constexpr double omega_of(int mask, int k) {
    const double d0 = (double)(mask & 1), d1 = (double)((mask >> 1) & 1),
                 d2 = (double)((mask >> 2) & 1);
    const double D = (d0 * 0.1 + d1 * 0.6) + d2 * 0.3;
    const double dk = (k == 0) ? d0 : (k == 1) ? d1 : d2;
    const double ck = (k == 0) ? 0.1 : (k == 1) ? 0.6 : 0.3;
    return mask == 0 ? 0.0 : (dk * ck) / D;
}
__constant__ const double kOmega[8][3] = {
    {omega_of(0, 0), omega_of(0, 1), omega_of(0, 2)},
    {omega_of(1, 0), omega_of(1, 1), omega_of(1, 2)},
    {omega_of(2, 0), omega_of(2, 1), omega_of(2, 2)},
    {omega_of(3, 0), omega_of(3, 1), omega_of(3, 2)},
    {omega_of(4, 0), omega_of(4, 1), omega_of(4, 2)},
    {omega_of(5, 0), omega_of(5, 1), omega_of(5, 2)},
    {omega_of(6, 0), omega_of(6, 1), omega_of(6, 2)},
    {omega_of(7, 0), omega_of(7, 1), omega_of(7, 2)}};

// Decision constants of one launch.  The LAD ladder index m = B_l +
// floor(theta (B_u - B_l)), theta = 1 / (1 + x / H) with x = max_k chi~_k
// (eq 3.1-3.4), is formed from an approximate x and theta and trusted when
// y = theta (B_u - B_l) lies farther than ymarg from an integer: the literal
// chain of correctly rounded operations differs from it by a few ulp.
struct DecisionConsts {
    double inv_h;          // 1 / H
    double nthr_d;         // B_u - B_l
    double ymarg;          // kDecisionMargin (B_u - B_l)
    double ct_hi;          // largest C_T the scheme can use (10^-B_l or C_T)
    double ct_lo;          // smallest C_T (10^-B_u or C_T)
    int32_t nthr;          // B_u - B_l
    int32_t literal;       // 1: evaluate every decision with the literal formula
    int32_t need_m;        // 1: the ladder index is wanted (decision dumps)
                           // (either switches the smooth-stencil bound off)
    int32_t pad_;
    // Smooth-stencil bound: when tau <= smooth_t (min_k beta_k + eps), every
    // chi~_k = tau / (beta_k + eps) is at most smooth_t (to rounding), so each
    // gamma_k of eq 2.8 lies in [1, (1 + smooth_t)^6] and every chi_k is at
    // least 1 / (1 + 2 (1 + smooth_t)^6), which the host chooses above the
    // largest cutoff ct_hi: all three stencils are kept, whatever the ladder
    // index.  Negative: no such bound (never satisfied).
    // (The kernels test 4 tau against 4 min_k beta_k: smooth_te = 4 smooth_t eps.)
    double smooth_t, smooth_te;
    double eps4;           // 4 eps
    // host products of the margins below: ct_hi (1 + margin) and ct_lo (1 -
    // margin) (kept out of the kernels' loops, where the compiler would
    // re-form them for every characteristic field)
    double hi_fac, lo_fac;
    // cut form of theta: max chi~ above h_hi = H (1 + margin) is certainly over
    // H (m = B_l), at or above h_lo = H (1 - margin) it is not trusted; NaN for
    // the printed form, so that neither test holds
    double h_hi, h_lo;
};

// Relative margin inside which an approximate decision value is not trusted
// (the approximate path differs from the literal one by < 200 ulp).
constexpr double kDecisionMargin = 0x1p-40;

// The literal decision of eq 2.8-2.14 / eq 3.1-3.4 (oracle operation order,
// correctly rounded divisions).  Returns m | (mask << 5).
// TENO5-A cutoff of eq 2.16-2.18 on the reconstruction's own values (a..e) =
// (f_{i-2} .. f_{i+2}): sensors eta_j at j = i-1, i, i+1 (eq 2.18, denominator
// df_{j+1/2}^2 + df_{j-1/2}^2), eta_{i+1/2} = their minimum, m = 1 - min(1,
// eta / C_r), g = (1 - m)^4 (1 + 4 m), beta = alpha_1 - alpha_2 (1 - g),
// C_T = 10^-floor(beta).  Operation order of the oracle; returns floor(beta).
template <class SP>
__device__ __forceinline__ int teno5a_cutoff(const SP& S, double a, double b, double c, double d,
                                             double e) {
    const double df0 = b - a, df1 = c - b, df2 = d - c, df3 = e - d;
    // 2 x and 4 x are exact, so the fused forms below round exactly as the
    // oracle's product-then-add
    const double eta0 =
        cr_div(__builtin_fma(2.0, fabs(df1 * df0), S.epsA), (df1 * df1 + df0 * df0) + S.epsA);
    const double eta1 =
        cr_div(__builtin_fma(2.0, fabs(df2 * df1), S.epsA), (df2 * df2 + df1 * df1) + S.epsA);
    const double eta2 =
        cr_div(__builtin_fma(2.0, fabs(df3 * df2), S.epsA), (df3 * df3 + df2 * df2) + S.epsA);
    double eh = eta0;
    if (eta1 < eh) eh = eta1;
    if (eta2 < eh) eh = eta2;
    const double q = cr_div(eh, S.cr);
    const double mA = 1.0 - (q < 1.0 ? q : 1.0);
    const double om = 1.0 - mA;
    const double om2 = om * om;
    const double g = (om2 * om2) * __builtin_fma(4.0, mA, 1.0);
    const double bA = S.a1 - S.a2 * (1.0 - g);
    return (bA >= 0.0) ? (int)floor(bA) : S.kA_nan;
}

// A5: the launch runs TENO5-A (scheme 3); its cutoff code is compiled only
// into the A5 instantiations, so the other schemes' kernels do not carry it.
template <bool A5, class SP>
__device__ __forceinline__ uint32_t teno5_decide_literal(const SP& S, double a,
                                                      double b, double c, double d, double e) {
    const double s01 = __builtin_fma(-2.0, b, a) + c;
    const double s02 = __builtin_fma(3.0, c, __builtin_fma(-4.0, b, a));
    const double s11 = __builtin_fma(-2.0, c, b) + d;
    const double s12 = b - d;
    const double s21 = __builtin_fma(-2.0, d, c) + e;
    const double s22 = __builtin_fma(3.0, c, __builtin_fma(-4.0, d, e));
    const double beta0 = __builtin_fma(kB13_12 * s01, s01, kB1_4 * (s02 * s02));
    const double beta1 = __builtin_fma(kB13_12 * s11, s11, kB1_4 * (s12 * s12));
    const double beta2 = __builtin_fma(kB13_12 * s21, s21, kB1_4 * (s22 * s22));
    const double tau = fabs(beta2 - beta0);
    const double t0 = cr_div(tau, beta0 + S.eps);
    const double t1 = cr_div(tau, beta1 + S.eps);
    const double t2 = cr_div(tau, beta2 + S.eps);
    double y, y2;
    y = 1.0 + t0;
    y2 = y * y;
    const double g0 = (y2 * y2) * y2;
    y = 1.0 + t1;
    y2 = y * y;
    const double g1 = (y2 * y2) * y2;
    y = 1.0 + t2;
    y2 = y * y;
    const double g2 = (y2 * y2) * y2;
    const double sum = (g0 + g1) + g2;
    const double chi0 = cr_div(g0, sum);
    const double chi1 = cr_div(g1, sum);
    const double chi2 = cr_div(g2, sum);
    double ct = 0.0;
    int m = 0;
    if (S.scheme == 0) {
        double x = t0;
        if (t1 > x) x = t1;
        if (t2 > x) x = t2;
        if (S.theta_cut && x > S.H) {
            m = S.Bl;  // theta = 0: the stencil counts as discontinuous
        } else {
            const double theta = cr_div(1.0, 1.0 + cr_div(x, S.H));
            if (theta >= 0.0)
                m = S.Bl + (int)floor(theta * S.bu_bl);
            else
                m = S.Bl;
        }
        ct = kLadder[m];
    } else if (A5) {
        m = teno5a_cutoff(S, a, b, c, d, e);
        ct = kLadder[m];
    } else {
        ct = S.ct_fixed;
    }
    const uint32_t mask = (chi0 < ct ? 0u : 1u) | (chi1 < ct ? 0u : 2u) | (chi2 < ct ? 0u : 4u);
    return (uint32_t)m | (mask << 5);
}

// Decision of a stencil (a..e) = (f_{i-2} .. f_{i+2}) that the smooth-stencil
// bound does not settle: m | (mask << 5).
//
// The cutoff flags and the ladder index are discrete functions of the
// literal formula.  They are first evaluated with approximate reciprocals;
// if any decision value lies within kDecisionMargin of its threshold (or is
// not finite) the lane re-evaluates the literal formula (*certain = false), so
// the decisions equal the literal ones exactly.  b4_k = 4 beta_k; ladder(k) =
// 10^-k.  settled: the caller ignores the result (a lane that only accompanies
// its wave).  WAVE: called by all lanes of a wave, whose branches are then
// taken for the wave as a whole, so that ladder() may exchange values between
// lanes.
template <bool A5, bool WAVE, class SP, class KP, class LAD>
__device__ __forceinline__ uint32_t teno5_decide_fast(const SP& S, const KP& K, const LAD& ladder,
                                                      double b40, double b41, double b42,
                                                      bool settled, double a, double b, double c,
                                                      double d, double e, bool* certain) {
    auto some = [](bool x) { return WAVE ? __ballot(x) != 0 : x; };
    bool sure = K.literal == 0;
    uint32_t m = 0, mask = 7u;
    if (sure) {
        // Approximate gamma_k (eq 2.8) from approximate chi~_k = tau / (beta_k + eps).
        const double tau4 = fabs(b42 - b40);
        const double t0 = tau4 * rcp_nr(b40 + K.eps4);
        const double t1 = tau4 * rcp_nr(b41 + K.eps4);
        const double t2 = tau4 * rcp_nr(b42 + K.eps4);
        double y, y2;
        y = 1.0 + t0;
        y2 = y * y;
        const double g0 = (y2 * y2) * y2;
        y = 1.0 + t1;
        y2 = y * y;
        const double g1 = (y2 * y2) * y2;
        y = 1.0 + t2;
        y2 = y * y;
        const double g2 = (y2 * y2) * y2;
        const double sum = (g0 + g1) + g2;
        // chi_k = g_k / sum against the extreme cutoffs: a flag that is the
        // same for every rung of the ladder needs no ladder index.  TENO5-A
        // evaluates its cutoff exactly and uses it for both bounds.
        double chi_hi = K.ct_hi, chi_lo = K.ct_lo;
        if (A5) {
            m = (uint32_t)teno5a_cutoff(S, a, b, c, d, e);
            chi_hi = chi_lo = ladder((int)m);
        }
        const double hi = (A5 ? chi_hi * (1.0 + kDecisionMargin) : K.hi_fac) * sum;
        const double lo = (A5 ? chi_lo * (1.0 - kDecisionMargin) : K.lo_fac) * sum;
        const bool k0 = g0 >= hi, k1 = g1 >= hi, k2 = g2 >= hi;
        const bool c0 = g0 < lo, c1 = g1 < lo, c2 = g2 < lo;
        sure = settled || (isfinite(sum) && (k0 || c0) && (k1 || c1) && (k2 || c2));
        mask = (k0 ? 1u : 0u) | (k1 ? 2u : 0u) | (k2 ? 4u : 0u);
        if (S.scheme == 0 && (K.need_m || some(!sure))) {
            // ladder index from approximate x and theta.  A NaN t_k makes
            // sum NaN, which already sends the lane to the literal
            // formula; the clamp keeps the table index in range for any x.
            const double x = fmax(fmax(t0, t1), t2);
            const double y = rcp_nr(__builtin_fma(x, K.inv_h, 1.0)) * K.nthr_d;
            const double fl = floor(y);
            const double fr = y - fl;
            bool msure = K.nthr == 0 || (isfinite(x) && fr > K.ymarg && fr < 1.0 - K.ymarg);
            m = (uint32_t)S.Bl + (uint32_t)(int)fmin(fmax(fl, 0.0), K.nthr_d);
            // cut form of theta: x certainly over H gives B_l; x within
            // the margin of H takes the literal formula
            if (x > K.h_hi) {
                m = (uint32_t)S.Bl;
                msure = true;
            } else if (x >= K.h_lo) {
                msure = false;
            }
            if (some(!sure)) {
                const double ct = ladder((int)m);
                const double rs = rcp_nr(sum);
                const double x0 = g0 * rs, x1 = g1 * rs, x2 = g2 * rs;
                const double band = kDecisionMargin * ct;
                const uint32_t lm = (x0 < ct ? 0u : 1u) | (x1 < ct ? 0u : 2u) | (x2 < ct ? 0u : 4u);
                const bool ls = isfinite(sum) && fabs(x0 - ct) > band && fabs(x1 - ct) > band &&
                                fabs(x2 - ct) > band;
                // (with a ladder index that nothing needs, a sure lane stays so)
                if (!sure) {
                    mask = lm;
                    sure = ls && msure;
                } else if (K.need_m) {
                    sure = msure;
                }
            } else {
                sure = sure && msure;
            }
        }
    }
    *certain = sure;
    return m | (mask << 5);
}
template <bool A5>
__device__ __forceinline__ uint32_t teno5_decide(const SchemeParams& S, const DecisionConsts& K,
                                                 double b40, double b41, double b42, double a,
                                                 double b, double c, double d, double e) {
    bool sure;
    const uint32_t cd = teno5_decide_fast<A5, false>(S, K, [](int k) { return kLadder[k]; }, b40, b41,
                                                     b42, false, a, b, c, d, e, &sure);
    if (sure) return cd;
    return teno5_decide_literal<A5>(S, a, b, c, d, e);
}

// One scalar TENO5 reconstruction of the face value from (a..e) =
// (f_{i-2} .. f_{i+2}): smoothness indicators (eq 2.9-2.12), scale
// separation (eq 2.8, 2.13), cutoff (eq 2.14) with C_T from the LAD mapping
// (eq 3.1-3.4), weights (eq 2.15) and combination (eq 2.4-2.7).  The flux is
// the literal combination with the eq 2.15 weights of the mask that the
// decision chose.  *code receives m | (mask << 5).
//
// Four times the smoothness indicators: with b4_k = (13/3 s) s + t t the
// product by 1/4 goes, and the factor 4 is exact.  4 tau < smooth_t (4
// min_k beta_k) + 4 smooth_t eps is one minimum, one fused multiply-add and one
// compare; the strict compare turns an overflow away, a NaN beta_k (it
// needs a NaN stencil value, which makes beta_0 or beta_2 NaN too) a NaN tau.
struct Teno5Beta {
    double b0, b1, b2;  // 4 beta_k
};
__device__ __forceinline__ Teno5Beta teno5_beta4(double a, double b, double c, double d, double e) {
    // sums of products as fused multiply-adds, in the oracle's order; a - 2 b
    // and a - 4 b are single roundings either way (2 b and 4 b are exact for
    // |b| below 2^1021), so they are fused here too
    constexpr double k13_3 = 4.0 * kB13_12;
    const double s01 = __builtin_fma(-2.0, b, a) + c;
    const double s02 = __builtin_fma(3.0, c, __builtin_fma(-4.0, b, a));
    const double s11 = __builtin_fma(-2.0, c, b) + d;
    const double s12 = b - d;
    const double s21 = __builtin_fma(-2.0, d, c) + e;
    const double s22 = __builtin_fma(3.0, c, __builtin_fma(-4.0, d, e));
    Teno5Beta B;
    B.b0 = __builtin_fma(k13_3 * s01, s01, s02 * s02);
    B.b1 = __builtin_fma(k13_3 * s11, s11, s12 * s12);
    B.b2 = __builtin_fma(k13_3 * s21, s21, s22 * s22);
    return B;
}
__device__ __forceinline__ bool teno5_smooth(double smooth_t, double smooth_te, const Teno5Beta& B) {
    return fabs(B.b2 - B.b0) <
           __builtin_fma(smooth_t, __builtin_fmin(__builtin_fmin(B.b0, B.b1), B.b2), smooth_te);
}
// Combination of the candidate fluxes with the weights w (eq 2.4-2.7).
__device__ __forceinline__ double teno5_combine(double w0, double w1, double w2, double a, double b,
                                                double c, double d, double e) {
    const double f0 = __builtin_fma(kC11_6, c, __builtin_fma(kC1_3, a, -kC7_6 * b));
    const double f1 = __builtin_fma(kC1_3, d, __builtin_fma(-kC1_6, b, kC5_6 * c));
    const double f2 = __builtin_fma(-kC1_6, e, __builtin_fma(kC1_3, c, kC5_6 * d));
    return __builtin_fma(w2, f2, __builtin_fma(w0, f0, w1 * f1));
}

template <bool A5>
__device__ __forceinline__ double teno5_rec_fast(const SchemeParams& S, const DecisionConsts& K,
                                                 const double* __restrict__ omega_lds,
                                                 double a, double b, double c, double d,
                                                 double e, uint32_t* code) {
    uint32_t cd = 7u << 5;
    if (S.scheme != 2) {
        const Teno5Beta B = teno5_beta4(a, b, c, d, e);
        if (!teno5_smooth(K.smooth_t, K.smooth_te, B))
            cd = teno5_decide<A5>(S, K, B.b0, B.b1, B.b2, a, b, c, d, e);
    }
    *code = cd;
    const double* w = omega_lds + 3 * (cd >> 5);
    return teno5_combine(w[0], w[1], w[2], a, b, c, d, e);
}

// Local component order of a sweep along DIR: rho, normal momentum, the
// tangential momenta in increasing axis order, E.
template <int ND, int DIR>
struct LocalOrder {
    static constexpr int NC = ND + 2;
    __device__ static constexpr int nat(int q) {
        // q = 0 -> 0; q = 1 -> 1 + DIR; q = 2..ND -> tangential axes; q = NC-1 -> NC-1
        return q == 0 ? 0
               : q == 1 ? 1 + DIR
               : q == NC - 1 ? NC - 1
               : 1 + ((q - 2) < DIR ? (q - 2) : (q - 1));
    }
    // tangential axis index of local tangential slot k = 1 .. ND-1
    __device__ static constexpr int tan_axis(int k) { return (k - 1) < DIR ? (k - 1) : k; }
};

}  // namespace teno
