// Launch description of one sweep (one axis of L(U), eq 2.2), shared by the
// sweep kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/teno.h"
#include "teno_device.hpp"

namespace teno {

// Work around an RK stage (or a right-hand side) that a small grid's sweeps do
// themselves instead of kernels of their own (step_impl, rhs_with_scratch).
struct StageWork {
    // first axis: every block takes the LF speeds from `npart` partials at
    // `part` (npart = 0: from all cells of U) and decides what the stage does;
    // the first block records it
    int32_t begin;           // 0: none; 1: a stage of teno_step; 2: a right-hand side
    int32_t npart;
    const double* part;
    teno_ctrl* ctrl;         // begin = 1
    const double* alpha_in;  // begin = 2: nullable, frozen speeds
    double* alpha_used;
    double* alpha_out;       // nullable
    int32_t* status;         // nullable
    // last axis of stages 1 and 2: the speeds of the stage output, as maxima
    // over kSpeedSlots slots of 4 doubles that were zeroed before
    double* speeds;          // nullable
    // last sweep of a step: blocks that are done, zeroed by the first sweep;
    // the last one ends the step
    uint32_t* done;          // nullable
    int32_t end;
};
constexpr int kSpeedSlots = 64;

// Per-launch description of one sweep.
struct SweepArgs {
    const double* U;        // state the stencils read (stage input)
    const double* Rin;      // partial RHS of earlier axes (nullable: start from 0)
    double* Rout;           // RHS output (rk == 0)
    const double* Un;       // u^n (rk == 2, 3)
    double* Uout;           // RK stage output (rk > 0)
    const double* alpha;    // LF speeds, 3 doubles (indexed by axis)
    const teno_ctrl* ctrl;  // nullable: the sweep runs only while ctrl->active and OK
    const double* dtp;      // dt of the fused RK stage (rk > 0)
    unsigned long long* digest;  // nullable: cutoff-mask digest accumulator
    int32_t axis;
    int32_t small;          // 1: a small grid, whose blocks read the arguments ahead (touch_args)
    uint8_t* dump;          // nullable: decision bytes of this axis
    int64_t ncell;
    int64_t line_step;      // cell-index step between consecutive lines of a column
    int64_t stride;         // cell-index step along the swept axis
    int64_t col_step;       // cell-index step between columns
    int64_t ftot;           // faces per column = lines_per_col * (n + 1)
    int64_t nchunks;        // chunks per column * ncols
    int64_t ncols;
    int32_t n;              // cells along the swept axis
    int32_t bc;
    int32_t rk;             // 0: write RHS; 1..3: fused RK stage
    int32_t stage;          // RK stage of this sweep (digest key; with ctrl->nsteps)
    int32_t ext_cap;        // LDS ext cells per wave
    double dx, rdx;         // spacing along the axis and RN(1 / dx)
    int32_t rdx_ok;         // 1: dx is in the range of the fast quotients
    SchemeParams sch;
    DecisionConsts dk;
    const teno_boundary* bnd;  // nullable: per-end boundaries and gravity
    int32_t add_source;        // 1 on the last axis when bnd is set
    int32_t nx, ny;            // grid sizes (boundary split coordinates)
    double dxa[3];             // spacings per axis (boundary split coordinates)
    // multiply-and-shift division by n + 1, n + 6 and ncols (dividends < 2^31);
    // div32: every face and ext index of a column is below 2^31
    uint32_t m1, s1, m6, s6, mc, sc;
    int32_t div32;
    StageWork work;
};

// Boundary kind of the ghost cells at end `end` of axis `dir` for the line
// whose interior cells start at global index cell0 (per-end boundaries): the
// split coordinate along the side's split axis, the split position at the
// stage time (teno_step: t, t + dt, t + dt/2 by stage; teno_rhs: t_rhs), and
// the fixed state when the selected part is TENO_BC_FIXED (*fixed, else null).
__device__ __forceinline__ int boundary_kind(const teno_boundary* bnd, const teno_ctrl* ctrl,
                                             int stage, int dir, int end, int64_t cell0, int nx,
                                             int ny, const double* dxa, const double** fixed) {
    const teno_side* sd = &bnd->side[dir][end];
    int which = 0;
    const int ax = sd->split_axis;
    if (ax >= 0) {
        const int64_t nxy = (int64_t)nx * ny;
        const int64_t ia = (ax == 0) ? cell0 % nx : (ax == 1) ? (cell0 / nx) % ny : cell0 / nxy;
        double t = bnd->t_rhs;
        if (ctrl != nullptr) {
            t = ctrl->t;
            if (stage == 1) t = ctrl->t + ctrl->dt;
            if (stage == 2) t = ctrl->t + 0.5 * ctrl->dt;
        }
        const double coord = ((double)ia + 0.5) * dxa[ax];
        const double split = sd->split[0] + sd->split[1] * t;
        if (!(coord < split)) which = 1;
    }
    const int kind = sd->kind[which];
    *fixed = (kind == TENO_BC_FIXED) ? sd->state[which] : nullptr;
    return kind;
}

// A value that is the same in every lane, in scalar registers.
__device__ __forceinline__ double uniform(double x) {
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// A pointer to a kernel's argument segment (constant address space).
template <class T>
using KernArgs = __attribute__((address_space(4))) const T*;

// Reads one word of every cache line of the kernel's arguments at entry.  Scalar
// loads of the arguments are issued where their values are used; on a small grid
// each first touch of a line is then a full memory latency in a serial chain.
// Without and with it: a step of 128 x 512 cells 87 / 84 us, of 2048 48 / 47,
// a right-hand side of 200 11.3 / 10.9; but of 2048^2 1159 / 1167.
template <class T>
__device__ __forceinline__ void touch_args() {
#if defined(__HIP_DEVICE_COMPILE__)
    const auto p = (KernArgs<uint32_t>)__builtin_amdgcn_kernarg_segment_ptr();
    uint32_t x = 0;
#pragma unroll
    for (int k = 0; k < (int)(sizeof(T) / 4); k += 16) x |= p[k];
    __asm__ __volatile__("" ::"s"(x));
#endif
}

// The marching sweep (teno_march.hip): true when it takes this launch.
bool march_takes(const teno_grid* g, int dir, const SweepArgs& A, bool digest);
hipError_t launch_march(const teno_grid* g, int dir, const SweepArgs& A, hipStream_t st);

// Whole steps of a short 1D line in one launch (teno_line.hip).
bool line_takes(const teno_grid* g);
hipError_t launch_line(const teno_grid* g, double* U, teno_ctrl* ctrl, int nsteps, hipStream_t st);

}  // namespace teno
