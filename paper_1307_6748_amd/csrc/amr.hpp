// Refinement boundaries with masks (Sec. 3.3.1, 3.4.1): the operator, its
// Newton-Gauss-Seidel smoother and its defect on a refinement patch.
//
// A patch is an n^3 grid (spacing h, indices periodic) whose cells carry a
// mask: m > 0 inside the refinement (these cells are relaxed), m <= 0 outside
// (m = -1: the cell does not exist on this level, its value u^Int comes from
// the coarser grid; -1 < m <= 0: it exists with its centre outside the
// boundary, u^Int is its own pre-iteration value).  An inside cell c with a
// masked neighbour f sees the ghost value
//     u_G = u_f^Int + (m_f / m_c) (u_c - u_c^Pre)          (eq. ueq),
// the linear extrapolation through u_c and the boundary value at the mask's
// zero crossing; u^Pre is the field when the boundary values were set.  The
// model's operator then runs on the ghost-substituted neighbours (for the
// non-canonical models the face coefficient is b(u_G)), and the Newton
// denominator gains each ghost's dependence on u_c (model.ghost_dD).  Cells
// with m <= 0 are neither relaxed nor counted in the defect.  Patches keep a
// layer of m = -1 cells around their inside, so the periodic wrap never joins
// inside cells.  Double precision; per-cell grid-stride kernels (patches are
// small next to the uniform grid).
#pragma once
#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace isis {

template <class M>
__device__ __forceinline__ void masked_op(const M& m, int n, double ih2,
                                          const double* __restrict__ phi,
                                          const double* __restrict__ eta,
                                          const double* __restrict__ mask,
                                          const double* __restrict__ u_int,
                                          const double* __restrict__ u_pre, int i, int j, int k,
                                          double& L, double& D)
{
    const long c = cell(n, i, j, k);
    const long q[6] = {cell(n, wrap_dec(i, n), j, k), cell(n, wrap_inc(i, n), j, k),
                       cell(n, i, wrap_dec(j, n), k), cell(n, i, wrap_inc(j, n), k),
                       cell(n, i, j, wrap_dec(k, n)), cell(n, i, j, wrap_inc(k, n))};
    // everything but the rare ghosts' values in one round of loads (asking
    // each neighbour's mask before its value made three dependent rounds)
    const double p = phi[c], mc = mask[c], pre = u_pre[c], e = eta[c];
    double v[6], r[6], mf[6];
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        mf[f] = mask[q[f]];
        v[f] = phi[q[f]];
        r[f] = 0.0;
    }
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        if (!(mf[f] > 0.0)) {
            const double ui = mf[f] > -1.0 ? u_pre[q[f]] : u_int[q[f]];  // eq. bpsi
            r[f] = mf[f] / mc;
            v[f] = ui + r[f] * (p - pre);                                  // eq. ueq
        }
    }
    m.op(p, v, e, ih2, L, D);
#pragma unroll
    for (int f = 0; f < 6; ++f)
        if (r[f] != 0.0) D += m.ghost_dD(p, v[f], r[f], ih2);
}

// Control block of a patch solve on the device (in its workspace).
struct PatchState {
    double rms;   // of the defect over the inside cells, at the last judged block
    int sweeps;   // made until then
    int stop;     // 1: converged, out of sweeps or not finite; later launches do nothing
};

// One colour of the red-black Newton-Gauss-Seidel sweep over the inside
// cells; masked cells keep their values and cost a mask (a refinement fills
// what it will of its patch's box: 128^3 f(R) with 3 % inside, 8.5 us; 22.0
// with the operator formed everywhere).  With state: nothing is done once
// state->stop is set.
// Bound: launch and two rounds of cache latency.  (A byte per cell saying
// whether it is inside and has ghosts, so that cells without any need not read
// the masks, split every wave in two paths, for a row has ghosts at its ends:
// per launch of a 68^3 symmetron patch 7.5 us, now 6.9; f(R) 9.2, 8.0; 128^3
// f(R) half inside 21, 17.  Only where the masks' traffic counts did it gain:
// 128^3 symmetron, all inside, 17.4, now 18.7.  Both colours, or two sweeps,
// in one launch on LDS blocks with a halo took 15.5 and 43 us: each thread's
// few cells are a chain of LDS and double-precision latency.)
template <class M>
__global__ __launch_bounds__(kBlock) void k_masked_halfsweep(
    M m, int n, double ih2, double* __restrict__ phi, const double* __restrict__ eta,
    const double* __restrict__ sigma, const double* __restrict__ mask,
    const double* __restrict__ u_int, const double* __restrict__ u_pre, int colour,
    const PatchState* __restrict__ state)
{
    const int stop = state ? state->stop : 0;
    for_planes(n, n, n >> 1, [&](int i, int j, int kk) __attribute__((always_inline)) {
        const int k = 2 * kk + ((i + j + colour) & 1);
        const long c = cell(n, i, j, k);
        if (!(mask[c] > 0.0) || stop) return;
        double L, D;
        masked_op(m, n, ih2, phi, eta, mask, u_int, u_pre, i, j, k, L, D);
        const double eps = L - (sigma ? sigma[c] : 0.0);
        phi[c] = phi[c] - m.limit(eps / D);
    });
}

// out = L - sigma at inside cells, 0 elsewhere (out may be NULL); with
// partial, per-block sums of out^2 in partial[block] and of the inside cells
// in partial[nblocks + block] (for the RMS over the inside); with snap, the
// field is copied there (the next block's pre-iteration values).
template <class M>
__global__ __launch_bounds__(kBlock) void k_masked_defect(
    M m, int n, double ih2, const double* phi, const double* __restrict__ eta,
    const double* __restrict__ sigma, const double* __restrict__ mask,
    const double* __restrict__ u_int, const double* u_pre, double* __restrict__ out,
    double* __restrict__ partial, double* __restrict__ snap)
{
    double acc = 0.0, cnt = 0.0;
    for_planes(n, n, n, [&](int i, int j, int k) __attribute__((always_inline)) {
        const long c = cell(n, i, j, k);
        double res = 0.0;
        if (mask[c] > 0.0) {
            double L, D;
            masked_op(m, n, ih2, phi, eta, mask, u_int, u_pre, i, j, k, L, D);
            res = L - (sigma ? sigma[c] : 0.0);
            cnt += 1.0;
        }
        if (out) out[c] = res;
        if (snap) snap[c] = phi[c];
        acc += res * res;
    });
    if (partial) {
        const double s = block_sum(acc);
        const double q = block_sum(cnt);
        if (threadIdx.x == 0) {
            const int b = blockIdx.y * gridDim.x + blockIdx.x;
            partial[b] = s;
            partial[gridDim.x * gridDim.y + b] = q;
        }
    }
}

__global__ void k_patch_begin(PatchState* state) { *state = PatchState{0.0, 0, 0}; }

// The stop test of a patch solve after `sweeps` more sweeps (one block): the
// RMS from the partial sums, summed in k_reduce's order.
__global__ __launch_bounds__(kBlock) void k_patch_judge(const double* __restrict__ partial,
                                                        int count, int sweeps, int max_sweeps,
                                                        double tol, PatchState* __restrict__ state)
{
    const double s = reduce_runs(partial, count), q = reduce_runs(partial + count, count);
    if (threadIdx.x == 0 && !state->stop) {
        const double rms = q > 0.0 ? sqrt(s / q) : 0.0;
        state->rms = rms;
        state->sweeps += sweeps;
        state->stop = !(rms > tol) || (state->sweeps > 0 && !isfinite(rms)) ||
                              state->sweeps >= max_sweeps ? 1 : 0;
    }
}

}  // namespace isis
