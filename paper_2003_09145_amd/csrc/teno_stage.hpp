// What an RK stage takes from its input state: the Lax-Friedrichs speeds, the
// time step, and whether it runs at all.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "../../include/teno.h"
#include "teno_device.hpp"

namespace teno {

// LF speeds |u_d| + c of one cell, as maxima with amax; bad: a cell with
// rho <= 0, p <= 0 or a non-finite sound speed.
template <int ND>
__device__ __forceinline__ void cell_speeds(const double (&q)[ND + 2], double gamma, double gm1,
                                            double (&amax)[ND], bool& bad) {
    constexpr int NC = ND + 2;
    const double rho = q[0];
    double u[ND];
    double y, m[ND];
    const bool rok = rcp_exact(rho, &y);
#pragma unroll
    for (int k = 0; k < ND; ++k) m[k] = q[1 + k];
    cr_div_n<ND>(m, rho, y, rok, u);
    double mu = q[1] * u[0];
#pragma unroll
    for (int k = 1; k < ND; ++k) mu = mu + q[1 + k] * u[k];
    const double ke = 0.5 * mu;
    const double p = gm1 * (q[NC - 1] - ke);
    double c2[1];
    const double gp[1] = {gamma * p};
    cr_div_n<1>(gp, rho, y, rok, c2);
    const double cs = cr_sqrt(c2[0]);
    if (!(rho > 0.0) || !(p > 0.0) || !isfinite(cs)) bad = true;
#pragma unroll
    for (int k = 0; k < ND; ++k) {
        const double s = fabs(u[k]) + cs;
        if (s > amax[k]) amax[k] = s;
    }
}

// Maxima of v[0 .. ND - 1] and the flag v[3] (0 or 1) over the wave, in every lane.
template <int ND>
__device__ __forceinline__ void wave_max4(double (&v)[4]) {
#pragma unroll
    for (int k = 0; k < ND; ++k) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const double o = __shfl_xor(v[k], off, 64);
            if (o > v[k]) v[k] = o;
        }
    }
    v[3] = __ballot(v[3] > 0.0) != 0 ? 1.0 : 0.0;
}

// Maxima of v over the block, in every thread; red: 4 doubles of LDS per wave,
// free again on return.
template <int ND>
__device__ __forceinline__ void block_max4(double (&v)[4], double* red) {
    wave_max4<ND>(v);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < 4; ++k) red[4 * wv + k] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        v[k] = red[k];
        for (int w = 1; w < (int)(blockDim.x >> 6); ++w)
            if (red[4 * w + k] > v[k]) v[k] = red[4 * w + k];
    }
    __syncthreads();
}

// Maxima of `npart` partials of 4 doubles (every thread of the block; up to 64:
// each wave by itself, without a barrier).
template <int ND>
__device__ __forceinline__ void reduce_partials(const double* __restrict__ part, int npart,
                                                double (&v)[4], double* red) {
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = 0.0;
    if (npart <= 64) {
        const int b = (int)(threadIdx.x & 63);
        if (b < npart) {
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = part[4 * b + k];
        }
        wave_max4<ND>(v);
        return;
    }
    for (int b = threadIdx.x; b < npart; b += blockDim.x) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double x = part[4 * b + k];
            if (x > v[k]) v[k] = x;
        }
    }
    block_max4<ND>(v, red);
}

// What stage `stage` of a step does, from the speeds r[0..2] of its input and
// r[3] > 0 if that is non-physical (sticky): false when it does not run; at
// stage 0 *dt from eq dt1 / dt2 (3D: the harmonic form) clipped to t_end.
// `was`: the control block before the launch; every block of a launch may ask,
// and one (write) records it: the fields read change, within the launch, only
// to what sends a later reader the same way.
__device__ __forceinline__ bool stage_decide(teno_ctrl* ctrl, const teno_ctrl& was,
                                             const double (&r)[4], int stage, int ndim,
                                             double dx0, double dx1, double dx2, bool write,
                                             double* dt_out) {
    const bool bad = r[3] > 0.0;
    const int replay = was.replay;
    if (stage == 0) {
        const double t = was.t, t_end = was.t_end;
        const bool go = was.status == 0 && t < t_end;
        double dt = was.dt;
        if (!replay) {
            if (ndim == 1) {
                dt = cr_div(was.cfl * dx0, r[0]);
            } else if (ndim == 2) {
                const double dtx = cr_div(dx0, r[0]);
                const double dty = cr_div(dx1, r[1]);
                dt = cr_div(was.cfl * (dtx * dty), dtx + dty);
            } else {
                dt = cr_div(was.cfl, (cr_div(r[0], dx0) + cr_div(r[1], dx1)) + cr_div(r[2], dx2));
            }
            if (t + dt > t_end) dt = t_end - t;
        }
        if (write) {
            ctrl->active = go && !bad ? 1 : 0;
            if (go && bad) ctrl->status = TENO_ERR_NONPHYSICAL;
            if (go && !bad && !replay) {
                ctrl->dt = dt;
                for (int k = 0; k < 3; ++k) ctrl->alpha[0][k] = r[k];
            }
        }
        *dt_out = dt;
        return go && !bad;
    }
    if (!was.active) return false;
    const bool ok = !bad && was.status == 0;
    if (write) {
        if (bad) ctrl->status = TENO_ERR_NONPHYSICAL;
        if (!ok) ctrl->active = 0;
        if (ok && !replay)
            for (int k = 0; k < 3; ++k) ctrl->alpha[stage][k] = r[k];
    }
    return ok;
}

__device__ __forceinline__ void step_end(teno_ctrl* ctrl) {
    if (ctrl->active && ctrl->status == 0) {
        ctrl->t = ctrl->t + ctrl->dt;
        ctrl->nsteps += 1;
    }
    ctrl->active = 0;
}

}  // namespace teno
