// Marching sweep along y and z (one axis of L(U), eq 2.2, with the RK stage of
// eq 4.1-4.3 fused on the last axis), for grids that fill the chip with it.
//
// A lane owns one column (all cells along the swept axis at one (x, z) or (x,
// y)) and walks a segment of it face by face, so a wave's 64 columns read and
// write whole 512-byte rows.  The window moves with the lane: f+ of six cells
// stays in registers, f- of five cells and the Roe inputs of three in a ring in
// LDS that only this lane reads and writes (20 KB per wave, two waves per
// SIMD, no barrier).  Against the face-stream sweep, whose waves share the
// cells of one line through LDS,
//  - every cell is staged once per segment (plus 5), with no idle lanes, every
//    index is uniform (scalar): along y of 256^3, per cell, about 1000 vector
//    instructions instead of 1190, about 30 of them integer instead of 200;
//  - the next row's loads are in flight while a face is computed.
// It is bound by instruction issue: two waves per SIMD issue one FP64
// instruction per 5.0 cycles (measured on independent chains; 4.5 with four
// waves), and 250 registers per lane leave no room for a third.
// Measured at 256^3 (turbulence, one box): step with the face stream 8.01 ms, with
// the march 7.27; y 0.75 and z with the stage update 0.83 ms a launch.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include "../../include/teno.h"
#include "teno_device.hpp"
#include "teno_face.hpp"
#include "teno_host.hpp"
#include "teno_sweep.hpp"

namespace teno {

struct MarchArgs {
    SweepArgs s;
    int64_t ncol;        // columns: every (x, z) for y, every (x, y) for z
    int32_t ngrp;        // groups of 64 columns
    MarchCut cut;        // segments of a column
    double cst[19];      // decision constants for the lane table (launch_march)
};

#if defined(__HIP_DEVICE_COMPILE__)
using ArgsPtr = KernArgs<MarchArgs>;
#else
using ArgsPtr = const MarchArgs*;
#endif

// Element at a uniform address plus a lane's byte offset.  The empty asm keeps
// the uniform part in scalar registers (the optimizer would otherwise add the
// lane's offset to a row first and form 64-bit vector addresses from it).
__device__ __forceinline__ double ld(const double* base, uint32_t off) {
#if defined(__HIP_DEVICE_COMPILE__)
    auto p = (__attribute__((address_space(1))) const char*)base;
    __asm__("" : "+s"(p), "+v"(off));
    return *(__attribute__((address_space(1))) const double*)(p + off);
#else
    return *(const double*)((const char*)base + off);
#endif
}
__device__ __forceinline__ void st(double* base, uint32_t off, double v) {
#if defined(__HIP_DEVICE_COMPILE__)
    auto p = (__attribute__((address_space(1))) char*)base;
    __asm__("" : "+s"(p), "+v"(off));
    *(__attribute__((address_space(1))) double*)(p + off) = v;
#else
    *(double*)((char*)base + off) = v;
#endif
}

// LDS exchange within the wave: its LDS operations complete in order, so only
// the compiler has to keep them so.
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The eq 2.15 weights (entries 0 .. 23, 3 per mask), the cutoff ladder (entries
// 24 .. 44) and the decision constants (entries 45 .. 63) as one value per
// lane: a lookup reads another lane's register, so it waits for no memory (a
// vector load would also wait for the rows in flight before it, a scalar load
// for a few hundred cycles in a path that needs ten of them).  All lanes are
// active at every lookup.
__device__ __forceinline__ double lane_table(ArgsPtr args) {
    const int l = threadIdx.x;
    return l < 24 ? kOmega[l / 3][l % 3] : l < 45 ? kLadder[l - 24] : args->cst[l - 45];
}
__device__ __forceinline__ double lane_const(double tab, int entry) {
    const uint64_t b = (uint64_t)__double_as_longlong(tab);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, entry);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), entry);
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}
__device__ __forceinline__ double lane_lookup(double tab, int entry) {
    const uint64_t b = (uint64_t)__double_as_longlong(tab);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * entry, (int)(uint32_t)b);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * entry, (int)(uint32_t)(b >> 32));
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// Reconstruction of a stencil x that the smooth bound does not settle (all
// lanes active; `smooth` lanes keep every candidate).
template <bool A5>
__device__ __forceinline__ double rec_cut(ArgsPtr args, double tab, bool smooth, const Teno5Beta& B,
                                          const double (&x)[5]) {
    __asm__ __volatile__("" : "+v"(tab));  // the constants are read here, not held
    const uint32_t ints = (uint32_t)__double_as_longlong(lane_const(tab, 57));
    uint32_t mask = 7u;
    if ((ints & 3u) != 2u) {
        SchemeParams S;
        DecisionConsts K;
        S.scheme = (int)(ints & 3u);
        K.literal = (int)(ints >> 2 & 1u);
        K.need_m = 0;
        S.Bl = (int)(ints >> 8 & 255u);
        K.nthr = (int)(ints >> 16 & 255u);
        S.kA_nan = (int)(ints >> 24);
        K.eps4 = lane_const(tab, 45);
        K.hi_fac = lane_const(tab, 46);
        K.lo_fac = lane_const(tab, 47);
        K.inv_h = lane_const(tab, 48);
        K.nthr_d = lane_const(tab, 49);
        K.ymarg = lane_const(tab, 50);
        K.h_hi = lane_const(tab, 51);
        K.h_lo = lane_const(tab, 52);
        S.cr = lane_const(tab, 53);
        S.epsA = lane_const(tab, 54);
        S.a1 = lane_const(tab, 55);
        S.a2 = lane_const(tab, 56);
        bool sure;
        uint32_t cd = teno5_decide_fast<A5, true>(S, K, [tab](int k) { return lane_lookup(tab, 24 + k); },
                                                  B.b0, B.b1, B.b2, smooth, x[0], x[1], x[2], x[3], x[4],
                                                  &sure);
        if (!sure && !smooth) cd = teno5_decide_literal<A5>(args->s.sch, x[0], x[1], x[2], x[3], x[4]);
        mask = smooth ? 7u : cd >> 5;
    }
    const int e = 3 * (int)mask;
    return teno5_combine(lane_lookup(tab, e), lane_lookup(tab, e + 1), lane_lookup(tab, e + 2), x[0],
                         x[1], x[2], x[3], x[4]);
}

// Reconstruction with every candidate kept (constant weights).
__device__ __forceinline__ double combine7(const double (&x)[5]) {
    return teno5_combine(omega_of(7, 0), omega_of(7, 1), omega_of(7, 2), x[0], x[1], x[2], x[3], x[4]);
}

// MODE 0: Rout = Rin - dF; 1: first RK stage; 2: the later stages.
template <int ND, int DIR, bool A5, int MODE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_march(MarchArgs A) {
    constexpr int NC = ND + 2;
    using LO = LocalOrder<ND, DIR>;
    __shared__ double ring[2][ND + 2][64];  // sqrt(rho), u, H of rows phi and phi + 1
    __shared__ double fmr[5][NC][64];       // f- of rows phi - 2 .. phi + 2
    // Stencils that are not smooth, gathered from all lanes and fields of a face
    // (pairs f+, f-), so that a decision pass or two serve them all: a jump
    // crosses a dozen lanes of a wave in every field, and a pass per field and
    // sign made the waves on a jump take four times as long as the others
    // (2D 2048^2 with one oblique jump: y 0.30 ms against 0.19 without it).
    constexpr int kPairs = ND == 2 ? 64 : 32;  // what the LDS of two waves per SIMD leaves
    constexpr int kBits = ND == 2 ? 7 : 6;
    __shared__ double cut[5][2 * kPairs];
    if (A.s.ctrl != nullptr) {
        if (!A.s.ctrl->active || A.s.ctrl->status != 0) return;
    }
#if defined(__HIP_DEVICE_COMPILE__)
    const ArgsPtr args = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
#else
    const ArgsPtr args = &A;
#endif
    const auto& Ai = *args;
    const double smooth_t = Ai.s.dk.smooth_t, smooth_te = Ai.s.dk.smooth_te;
    const int lane = threadIdx.x;
    const double tab = lane_table(args);
    const int lb = (int)(gridDim.x - 1 - (ND == 2 ? xcd_logical_block(blockIdx.x, gridDim.x) : blockIdx.x));
    const int seg = __builtin_amdgcn_readfirstlane(lb / Ai.ngrp);
    const int grp = lb - seg * Ai.ngrp;
    const int64_t c0 = (int64_t)grp * 64;
    // lanes past the last column repeat it (the same values to the same place)
    const int64_t c = c0 + lane < Ai.ncol ? c0 + lane : Ai.ncol - 1;
    // first cell of this lane's column, from the wave's
    const int nx = Ai.s.nx;
    int64_t cb0 = c0;
    uint32_t loff = (uint32_t)(c - c0);
    if (DIR == 1) {
        const int64_t plane = (int64_t)nx * Ai.s.ny;
        const int z0 = __builtin_amdgcn_readfirstlane((int)(c0 / nx)), x0 = (int)(c0 - (int64_t)z0 * nx);
        const int t = x0 + (int)(c - c0);
        const int dz = t / nx;
        cb0 = z0 * plane + x0;
        loff = (uint32_t)((int64_t)dz * plane + (t - dz * nx) - x0);
    }
    const uint32_t lo8 = loff * 8u;
    // values of every iteration: opaque, so that they stay in scalar registers
    // (spilled to lanes at worst) instead of being loaded again
    const double* pU = Ai.s.U;
    const double* pR = Ai.s.Rin;
    const double* pN = Ai.s.Un;
    double* pO = MODE == 0 ? Ai.s.Rout : Ai.s.Uout;
    int64_t ncell = Ai.s.ncell, stride = Ai.s.stride;
#if defined(__HIP_DEVICE_COMPILE__)
    __asm__("" : "+s"(pU), "+s"(pR), "+s"(pN), "+s"(pO), "+s"(ncell), "+s"(stride));
#endif
    const int n = Ai.s.n;
    // rows j0 .. j0 + len - 1; a segment has at least 3 rows (march_cut)
    const MarchCut seg_cut = {Ai.cut.nseg, Ai.cut.period};
    const int j0 = __builtin_amdgcn_readfirstlane(march_row(seg_cut, n, seg));
    const int len = __builtin_amdgcn_readfirstlane(march_row(seg_cut, n, seg + 1)) - j0;
    const double alpha = uniform(Ai.s.alpha[DIR]);
    const double gm1 = Ai.s.sch.gamma - 1.0;

    // Conserved state of row j (ghost rows mapped to their source) of this
    // lane's column; *neg: the sign bit that a mirrored row's normal momentum
    // takes when it is staged.
    const bool has_bnd = Ai.s.bnd != nullptr;
    auto load_row = [&](int j, double* q, uint64_t* neg) {
        bool flip = false;
        const int src = ghost_src(has_bnd ? 1 : Ai.s.bc, n, j, &flip);
        *neg = flip ? 0x8000000000000000ull : 0ull;
        const double* row = pU + cb0 + (int64_t)src * stride;
#pragma unroll
        for (int k = 0; k < NC; ++k) q[k] = ld(row + k * ncell, lo8);
    };
    // Ghost row j under per-end boundaries: each lane has its own kind.  The
    // loads end here, so that the rows' own path does not wait for registers
    // that they might still fill.
    auto bnd_row = [&](int j, double* q) {
        bool flip = false;
        const double* fixed = nullptr;
        const double dxa[3] = {Ai.s.dxa[0], Ai.s.dxa[1], Ai.s.dxa[2]};
        const int kind = boundary_kind(Ai.s.bnd, Ai.s.ctrl, Ai.s.stage, DIR, j < 0 ? 0 : 1, cb0 + loff,
                                       nx, Ai.s.ny, dxa, &fixed);
        const int src = ghost_src(kind, n, j, &flip);
        const double* cell = pU + cb0 + loff + (int64_t)src * stride;
#pragma unroll
        for (int k = 0; k < NC; ++k) q[k] = fixed != nullptr ? fixed[k] : cell[k * ncell];
        if (fixed == nullptr && flip) q[1 + DIR] = -q[1 + DIR];
        __builtin_amdgcn_s_waitcnt(0x0f70);
    };

    double fp[6][NC], Fprev[NC], qn[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) {
        Fprev[k] = 0.0;
#pragma unroll
        for (int j = 0; j < 6; ++j) fp[j][k] = 0.0;
    }
    // The first five rows of the window: all their loads are in flight at once
    // and wait in the f- ring, where the staging below finds them.
    uint64_t neg;
    {
        double q[5][NC];
#pragma unroll
        for (int r = 0; r < 5; ++r) {
            uint64_t ng;
            load_row(j0 - 3 + r, q[r], &ng);
            q[r][1 + DIR] = __longlong_as_double(__double_as_longlong(q[r][1 + DIR]) ^ ng);
        }
#pragma unroll
        for (int r = 0; r < 5; ++r)
#pragma unroll
            for (int k = 0; k < NC; ++k) fmr[r][k][lane] = q[r][k];
    }
    if (__builtin_expect(has_bnd && j0 == 0, 0)) {
#pragma unroll 1
        for (int r = 0; r < 3; ++r) {
            double q[NC];
            bnd_row(r - 3, q);
#pragma unroll
            for (int k = 0; k < NC; ++k) fmr[r][k][lane] = q[k];
        }
    }
    int s5 = 0, sr = 0;  // slots of the row being staged
    double rl[ND + 2];   // Roe inputs of row phi - 1
    auto stage = [&]() {
        qn[1 + DIR] = __longlong_as_double(__double_as_longlong(qn[1 + DIR]) ^ neg);
        const CellStage<ND> C = stage_values<ND, DIR>(qn, alpha, gm1);
        double* rg = &ring[sr][0][lane];
        rg[0] = C.srho;
#pragma unroll
        for (int k = 0; k < ND; ++k) rg[64 * (1 + k)] = C.u[k];
        rg[64 * (ND + 1)] = C.H;
        double* fr = &fmr[s5][0][lane];
#pragma unroll
        for (int k = 0; k < NC; ++k) fr[64 * k] = C.fm[k];
#pragma unroll
        for (int k = 0; k < NC; ++k) {
#pragma unroll
            for (int j = 0; j < 5; ++j) fp[j][k] = fp[j + 1][k];
            fp[5][k] = C.fp[k];
        }
    };
    auto next_slot = [&]() {
        sr ^= 1;
        s5 = s5 == 4 ? 0 : s5 + 1;
    };
#pragma unroll 1
    for (int it = -5; it < 0; ++it) {
        neg = 0ull;
#pragma unroll
        for (int k = 0; k < NC; ++k) qn[k] = fmr[s5][k][lane];
#pragma unroll
        for (int k = 0; k < ND + 2; ++k) rl[k] = ring[sr][k][lane];  // (of the last pass: row phi - 1)
        stage();
        next_slot();
    }
    // The loads of the next row and then five stores, as at the end of every
    // face below (row j0 of the output, unchanged).
    {
        const int64_t row = cb0 + (int64_t)j0 * stride;
        double keep[NC];
#pragma unroll
        for (int k = 0; k < NC; ++k) keep[k] = ld(pO + k * ncell + row, lo8);
        load_row(j0 + 2, qn, &neg);
#pragma unroll
        for (int k = 0; k < NC; ++k) st(pO + k * ncell + row, lo8, keep[k]);
    }
    const double h = MODE != 0 ? uniform(*Ai.s.dtp) : 0.0;
    const double w0 = Ai.s.rk == 3 ? 1.0 / 3.0 : 0.75, w1 = Ai.s.rk == 3 ? 2.0 / 3.0 : 0.25;
#pragma unroll 1
    for (int it = 0; it <= len; ++it) {
        // face j0 + it, between rows j0 + it - 1 and j0 + it
        FaceRoe<ND> R;
        {
            double rr[ND + 2];
#pragma unroll
            for (int k = 0; k < ND + 2; ++k) rr[k] = ring[sr][k][lane];  // row phi, two before the staged
            R = roe_average<ND, DIR>(rl[0], rl + 1, rl[ND + 1], rr[0], rr + 1, rr[ND + 1], gm1);
#pragma unroll
            for (int k = 0; k < ND + 2; ++k) rl[k] = rr[k];
        }
        stage();
        const double* fmp[5];  // f- of rows phi + 2 .. phi - 2
#pragma unroll
        for (int j = 0; j < 5; ++j) fmp[j] = &fmr[s5 - j < 0 ? s5 - j + 5 : s5 - j][0][lane];
        next_slot();
        // The first face finishes no cell: it stores row j0 unchanged (by selects:
        // a flux or a stage input that is not finite changes nothing either), so
        // that no store is behind a branch -- loads and stores share one in-order
        // counter, and a path that may have skipped the stores makes the wait for
        // the next row wait for them too.  (The output may be the buffer of U^n or
        // of the partial right-hand side, whose row j0 the next face reads again;
        // a first stage's output is neither and takes any value.)
        const bool none = it == 0;
        double r_in[NC], base[NC], u_n[NC];
        const int64_t row = cb0 + (int64_t)(j0 + (it > 0 ? it - 1 : 0)) * stride;
        double fh[NC];        // reconstructed characteristic fluxes
        uint32_t done = 0;    // fields of this lane that a decision pass has settled
        uint32_t todo = (1u << NC) - 1;  // fields of this pass (uniform)
        uint32_t rest = 0;    // fields of later passes (uniform)
        bool first = true;
        do {
            // once per pass: the left eigenvector's scalars, so that none stays
            // in registers through a decision pass
#if defined(__HIP_DEVICE_COMPILE__)
            __asm__ __volatile__("" : "+v"(R.Hb), "+v"(R.hq2), "+v"(R.cs), "+v"(R.un));
#endif
            left_scalars<ND>(R, gm1);
            uint32_t where = 0;  // kBits per field: kPairs | pair of this lane in `cut`
            uint32_t left = 0;   // fields that need another pass (uniform)
            int pairs = 0;       // pairs gathered (uniform)
#pragma unroll
            for (int s = 0; s < NC; ++s) {
                const bool acoustic = (s == 0 || s == NC - 1), entropy = (s == 1);
                if (s == 1 && first) {
#pragma unroll
                    for (int k = 0; k < NC; ++k) {
                        r_in[k] = ld(pR + k * ncell + row, lo8);
                        if (MODE >= 1) base[k] = ld(pU + k * ncell + row, lo8);
                        if (MODE == 2) u_n[k] = ld(pN + k * ncell + row, lo8);
                    }
                }
                if (s == NC - 2 && first) {
                    // the state part of eq 4.2, 4.3, before the next row's loads are
                    // in flight (a wait for the older loads alone)
                    if (MODE == 2) {
#pragma unroll
                        for (int k = 0; k < NC; ++k)
                            base[k] = none ? u_n[k] : w0 * u_n[k] + w1 * base[k];
                    }
                    const int jn = j0 + it + 3;
                    load_row(jn < n + 2 ? jn : n + 2, qn, &neg);
                    if (__builtin_expect(has_bnd && jn >= n, 0)) bnd_row(jn < n + 2 ? jn : n + 2, qn);
                }
                if (!(todo & (1u << s))) continue;
                __asm__ __volatile__("" ::: "memory");  // re-read f- per field
                double Lr[NC];
                left_row<ND>(R, s, Lr);
                double v[5], w[5];
                if (!acoustic && !entropy) {
#pragma unroll
                    for (int j = 0; j < 5; ++j) {
                        v[j] = Lr[0] * fp[j][0] + fp[j][s];
                        w[j] = Lr[0] * fmp[j][0] + fmp[j][64 * s];
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < 5; ++j) {
                        double a = Lr[0] * fp[j][0], b = Lr[0] * fmp[j][0];
#pragma unroll
                        for (int k = 1; k < NC; ++k) {
                            a = __builtin_fma(Lr[k], fp[j][k], a);
                            b = __builtin_fma(Lr[k], fmp[j][64 * k], b);
                        }
                        v[j] = a;
                        w[j] = b;
                    }
                }
                const bool sp = teno5_smooth(smooth_t, smooth_te, teno5_beta4(v[0], v[1], v[2], v[3], v[4]));
                const bool sm = teno5_smooth(smooth_t, smooth_te, teno5_beta4(w[0], w[1], w[2], w[3], w[4]));
                const bool cutl = !(sp && sm) && !(done & (1u << s));
                const uint64_t bm = __builtin_amdgcn_ballot_w64(cutl);
                if (__builtin_expect(bm != 0, 0)) {
                    const int at = pairs + (int)__builtin_amdgcn_mbcnt_hi(
                                               (uint32_t)(bm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bm, 0u));
                    if (cutl && at < kPairs) {
#pragma unroll
                        for (int j = 0; j < 5; ++j) {
                            cut[j][2 * at] = v[j];
                            cut[j][2 * at + 1] = w[j];
                        }
                        where |= (uint32_t)(kPairs | at) << (kBits * s);
                    }
                    pairs += __builtin_popcountll(bm);
                    if (pairs > kPairs) {
                        pairs = kPairs;
                        left |= 1u << s;
                    }
                }
                if (first) fh[s] = combine7(v) + combine7(w);
            }
            if (__builtin_expect(pairs != 0, 0)) {
                // A wave on a jump has several times the work of the others: it
                // issues first from here on, so that it is not the last to end.
                __builtin_amdgcn_s_setprio(3);
                wave_fence();
#pragma unroll 1
                for (int e = lane; e - lane < 2 * pairs; e += 64) {
                    double x[5];
#pragma unroll
                    for (int j = 0; j < 5; ++j) x[j] = cut[j][e];
                    const Teno5Beta B = teno5_beta4(x[0], x[1], x[2], x[3], x[4]);
                    const bool smooth = e >= 2 * pairs || teno5_smooth(smooth_t, smooth_te, B);
                    const double f = rec_cut<A5>(args, tab, smooth, B, x);
                    wave_fence();
                    cut[0][e] = f;
                }
                wave_fence();
#pragma unroll
                for (int s = 0; s < NC; ++s) {
                    const int at = (int)(where >> (kBits * s)) & (2 * kPairs - 1);
                    if (at & kPairs) {
                        fh[s] = cut[0][2 * (at - kPairs)] + cut[0][2 * (at - kPairs) + 1];
                        done |= 1u << s;
                    }
                }
                wave_fence();
            }
            // the two lowest fields next (a field may fill a pass by itself, and
            // each is projected again)
            rest |= left;
            const uint32_t low = rest & (0u - rest), up = rest ^ low;
            todo = low | (up & (0u - up));
            rest ^= todo;
            first = false;
        } while (__builtin_expect(todo != 0, 0));
        // R * fh in local order, one field after the other (unit entries: plain adds)
        double Fh[NC];
#pragma unroll
        for (int k = 0; k < NC; ++k) Fh[k] = 0.0;
#pragma unroll
        for (int s = 0; s < NC; ++s) add_right<ND>(R, s, fh[s], Fh);
        double diff[NC], dq[NC], ro[NC];
#pragma unroll
        for (int k = 0; k < NC; ++k) diff[LO::nat(k)] = Fh[k] - Fprev[k];
        cr_div_n<NC>(diff, Ai.s.dx, Ai.s.rdx, Ai.s.rdx_ok != 0, dq);
#pragma unroll
        for (int k = 0; k < NC; ++k) ro[k] = MODE == 0 && none ? r_in[k] : r_in[k] - dq[k];
        if (Ai.s.add_source && it > 0) {
            const double* g = Ai.s.bnd->gravity;
            const double rho = ld(pU + row, lo8);
            double sE = 0.0;
#pragma unroll
            for (int d = 0; d < ND; ++d) {
                ro[1 + d] = ro[1 + d] + rho * g[d];
                const double mg = ld(pU + (1 + d) * ncell + row, lo8) * g[d];
                sE = d == 0 ? mg : sE + mg;
            }
            ro[NC - 1] = ro[NC - 1] + sE;
            __builtin_amdgcn_s_waitcnt(0x0f70);  // see load_row
        }
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            if (MODE == 1) ro[k] = base[k] + h * ro[k];
            if (MODE == 2) ro[k] = none ? base[k] : base[k] + w1 * (h * ro[k]);
            st(pO + k * ncell + row, lo8, ro[k]);
        }
#pragma unroll
        for (int k = 0; k < NC; ++k) Fprev[k] = Fh[k];
    }
}

bool march_takes(const teno_grid* g, int dir, const SweepArgs& A, bool digest) {
    return !digest && A.dump == nullptr && A.Rin != nullptr && march_grid(g, dir, A.rk != 0);
}

hipError_t launch_march(const teno_grid* g, int dir, const SweepArgs& A0, hipStream_t st) {
    MarchArgs A;
    memset(&A, 0, sizeof(A));
    A.s = A0;
    if (g->scheme == TENO_SCHEME_LINEAR5) {  // every stencil kept: the smooth test always holds
        A.s.dk.smooth_t = 0.0;
        A.s.dk.smooth_te = INFINITY;
    }
    // entries 45 .. 57 of the lane table (rec_cut reads them)
    const DecisionConsts& K = A.s.dk;
    const SchemeParams& S = A.s.sch;
    const uint64_t ints = (uint64_t)(uint32_t)S.scheme | (uint64_t)(K.literal ? 4 : 0) |
                          (uint64_t)(uint32_t)S.Bl << 8 | (uint64_t)(uint32_t)K.nthr << 16 |
                          (uint64_t)(uint32_t)S.kA_nan << 24;
    const double cst[12] = {K.eps4, K.hi_fac, K.lo_fac, K.inv_h, K.nthr_d, K.ymarg,
                            K.h_hi, K.h_lo,   S.cr,     S.epsA,  S.a1,     S.a2};
    memcpy(A.cst, cst, sizeof(cst));
    memcpy(&A.cst[12], &ints, sizeof(ints));
    A.ncol = march_cols(g, dir);
    A.ngrp = (int32_t)((A.ncol + 63) / 64);
    const int n = g->n[dir];
    A.cut = march_cut(A.ngrp, n, g->ndim == 2);
    const dim3 grid((unsigned)(A.ngrp * A.cut.nseg)), blk(64);
    const bool a5 = g->scheme == TENO_SCHEME_TENO5A;
    const int mode = A.s.rk >= 2 ? 2 : A.s.rk;
    switch ((g->ndim * 4 + dir + (a5 ? 16 : 0)) * 4 + mode) {
#define TENO_MARCH(nd, d, m)                                                                    \
    case (nd * 4 + d) * 4 + m:                                                                  \
        hipLaunchKernelGGL((k_march<nd, d, false, m>), grid, blk, 0, st, A); break;             \
    case (nd * 4 + d + 16) * 4 + m:                                                             \
        hipLaunchKernelGGL((k_march<nd, d, true, m>), grid, blk, 0, st, A); break;
        TENO_MARCH(2, 1, 0) TENO_MARCH(2, 1, 1) TENO_MARCH(2, 1, 2)
        TENO_MARCH(3, 1, 0)
        TENO_MARCH(3, 2, 0) TENO_MARCH(3, 2, 1) TENO_MARCH(3, 2, 2)
#undef TENO_MARCH
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace teno
