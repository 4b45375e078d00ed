// Whole steps of a short 1D line in one block: no launch between the stages
// (eq 4.1-4.3), the speeds, the time step and the bookkeeping of teno_step.
//
// A thread owns a cell, whose u^n and stage state stay in its registers, and
// the face on its left; the cells' split fluxes go through LDS, as in the
// face-stream sweep.  A stage of such a line is a chain of latencies: as
// launches of its own (three a step, and ten before the sweeps did a stage's
// bookkeeping themselves) each stage takes 13 us, of which about 4 us are the
// launch and the rest first touches of arguments, code and state that lie
// elsewhere.  Here they are touched once per launch, and a stage is bound by
// its chain of FP64 instructions, three waves per SIMD at most.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include "../../include/teno.h"
#include "teno_device.hpp"
#include "teno_face.hpp"
#include "teno_host.hpp"
#include "teno_stage.hpp"
#include "teno_sweep.hpp"

namespace teno {

constexpr int kLineThreads = 576;  // of the longest line, with its six ghost cells

// Doubles of LDS of an n-cell line: weights, four reduction slots per wave, the
// staged cells, the stage state and the face fluxes.
constexpr size_t line_lds(int n) {
    return 24 + 4 * (kLineThreads / 64) + 9 * (size_t)(n + 6) + 3 * (size_t)n + 3 * (size_t)(n + 1);
}
static_assert(line_lds(kLineThreads - 6) * sizeof(double) <= 80 * 1024, "half of a CU's LDS");

struct LineArgs {
    SweepArgs s;  // geometry, scheme and boundaries; U
    double* U;
    teno_ctrl* ctrl;
    int32_t nsteps;
};

template <bool A5>
__global__ __launch_bounds__(kLineThreads) void k_line(LineArgs A) {
    constexpr int NC = 3, NV = 9;
    extern __shared__ double smem[];
    const SweepArgs& S = A.s;
    const int n = S.n, cap = n + 6, tid = threadIdx.x;
    double* omega = smem;          // 24: eq 2.15 weights per cutoff mask
    double* red = omega + 24;      // 4 per wave
    double* ext = red + 4 * (kLineThreads / 64);
    double* su = ext + NV * cap;   // stage state
    double* fh = su + NC * n;      // face fluxes
    const double gamma = S.sch.gamma, gm1 = gamma - 1.0;
    teno_ctrl now = *A.ctrl;
    if (tid < 24) omega[tid] = kOmega[tid / 3][tid % 3];
    const bool cell = tid < n;
    double un[NC], u[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) un[c] = u[c] = cell ? A.U[c * n + tid] : 1.0;
    // the ext cell this thread stages: ghost cells by the line's own kind
    const int j = tid - 3;

    bool run = true;
    for (int step = 0; run && step < A.nsteps; ++step) {
        now.active = 0;
#pragma unroll 1
        for (int stage = 0; run && stage < 3; ++stage) {
            double r[4] = {0.0, 0.0, 0.0, 0.0};
            if (cell) {
                double amax[1] = {0.0};
                bool bad = false;
                cell_speeds<1>(u, gamma, gm1, amax, bad);
                r[0] = amax[0];
                r[3] = bad ? 1.0 : 0.0;
#pragma unroll
                for (int c = 0; c < NC; ++c) su[c * n + tid] = u[c];
            }
            block_max4<1>(r, red);  // (its barriers publish su)
            double dt;
            run = stage_decide(nullptr, now, r, stage, 1, S.dxa[0], 0.0, 0.0, false, &dt);
            if (!run) {
                const bool asked = stage != 0 || (now.status == 0 && now.t < now.t_end);
                if (asked && r[3] > 0.0) now.status = TENO_ERR_NONPHYSICAL;
                now.active = 0;
                break;
            }
            if (stage == 0) {
                now.active = 1;
                now.dt = dt;
            }
            double alpha = r[0];
            if (now.replay) {
                alpha = A.ctrl->alpha[stage][0];
            } else if (tid == 0) {
                A.ctrl->alpha[stage][0] = r[0];
                A.ctrl->alpha[stage][1] = A.ctrl->alpha[stage][2] = 0.0;
            }
            alpha = uniform(alpha);
            if (tid < n + 6) {
                bool flip = false;
                int kind = S.bc;
                const double* fixed = nullptr;
                if (S.bnd != nullptr && (j < 0 || j >= n))
                    kind = boundary_kind(S.bnd, &now, stage, 0, j < 0 ? 0 : 1, 0, n, 1, S.dxa, &fixed);
                double q[NC];
                if (fixed != nullptr) {
#pragma unroll
                    for (int c = 0; c < NC; ++c) q[c] = fixed[c];
                } else {
                    const int src = ghost_src(kind, n, j, &flip);
#pragma unroll
                    for (int c = 0; c < NC; ++c) q[c] = su[c * n + src];
                    if (flip) q[1] = -q[1];
                }
                stage_cell<1, 0, false>(q, alpha, gm1, ext, cap, tid);
            }
            __syncthreads();
            if (tid <= n) {
                double Fh[NC];
                face_flux<1, 0, A5, false>(ext, cap, tid, gm1, S.sch, S.dk, omega, nullptr, Fh, nullptr);
#pragma unroll
                for (int c = 0; c < NC; ++c) fh[c * (n + 1) + tid] = Fh[c];
            }
            __syncthreads();
            if (cell) {
                double diff[NC], dq[NC], rr[NC];
#pragma unroll
                for (int c = 0; c < NC; ++c) diff[c] = fh[c * (n + 1) + tid + 1] - fh[c * (n + 1) + tid];
                cr_div_n<NC>(diff, S.dx, S.rdx, S.rdx_ok != 0, dq);
#pragma unroll
                for (int c = 0; c < NC; ++c) rr[c] = 0.0 - dq[c];
                if (S.bnd != nullptr) {
                    const double g = S.bnd->gravity[0];
                    rr[1] = rr[1] + u[0] * g;
                    rr[2] = rr[2] + u[1] * g;
                }
                const double h = now.dt;
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    if (stage == 0)
                        u[c] = u[c] + h * rr[c];
                    else if (stage == 1)
                        u[c] = (0.75 * un[c] + 0.25 * u[c]) + 0.25 * (h * rr[c]);
                    else
                        u[c] = ((1.0 / 3.0) * un[c] + (2.0 / 3.0) * u[c]) + (2.0 / 3.0) * (h * rr[c]);
                }
                if (stage == 2) {
#pragma unroll
                    for (int c = 0; c < NC; ++c) un[c] = u[c];
                }
            }
        }
        if (run) step_end(&now);
    }
    if (cell) {
#pragma unroll
        for (int c = 0; c < NC; ++c) A.U[c * n + tid] = un[c];
    }
    if (tid == 0) {
        A.ctrl->t = now.t;
        A.ctrl->dt = now.dt;
        A.ctrl->status = now.status;
        A.ctrl->nsteps = now.nsteps;
        A.ctrl->active = now.active;
    }
}

// The line kernel takes 1D grids whose cells and ghost cells fit one block of
// nine waves (two or three per SIMD, and 67.7 KB of the CU's 160 KB of LDS),
// without the mask digest: a step of 200 cells takes 27.5 us in it and 38.6 in
// launches of its own, of 570 cells 38 to 40 and 42; the gain shrinks with the waves
// that share the one CU.
bool line_takes(const teno_grid* g) {
    return g->ndim == 1 && g->n[0] + 6 <= kLineThreads && (g->flags & TENO_FLAG_MASK_DIGEST) == 0;
}

hipError_t launch_line(const teno_grid* g, double* U, teno_ctrl* ctrl, int nsteps, hipStream_t st) {
    LineArgs A;
    memset(&A, 0, sizeof(A));
    const int n = g->n[0];
    A.U = U;
    A.ctrl = ctrl;
    A.nsteps = nsteps;
    A.s.n = n;
    A.s.bc = g->bc[0];
    A.s.dx = g->dx[0];
    A.s.rdx = 1.0 / A.s.dx;
    A.s.rdx_ok = (A.s.dx >= 0x1p-400 && A.s.dx < 0x1p400) ? 1 : 0;
    A.s.bnd = g->boundary_dev;
    for (int k = 0; k < 3; ++k) A.s.dxa[k] = g->dx[k];
    A.s.sch = scheme_of(g);
    A.s.dk = decision_consts(g, false);
    const int threads = (n + 6 + 63) / 64 * 64;
    const size_t lds = sizeof(double) * line_lds(n);
    if (g->scheme == TENO_SCHEME_TENO5A)
        hipLaunchKernelGGL(k_line<true>, dim3(1), dim3((unsigned)threads), lds, st, A);
    else
        hipLaunchKernelGGL(k_line<false>, dim3(1), dim3((unsigned)threads), lds, st, A);
    return hipGetLastError();
}

}  // namespace teno
