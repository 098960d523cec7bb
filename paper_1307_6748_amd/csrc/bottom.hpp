// The bottom of a V-cycle in one workgroup: from the first level of side
// <= 16 down to the 4^3 coarsest grid and back (Sec. 3.2), with every field
// these levels touch held in LDS.  On the device each of these levels is a
// dozen launches of a few microseconds each, almost all launch and drain;
// here they are one launch whose phases are separated by workgroup barriers.
// Each phase computes per cell what the per-level kernels compute, with the
// same terms in the same order: k_halfsweep, k_defect_restrict (or the fine
// defect then k_restrict_fw for full weighting), k_fas_sigma,
// k_prolong_correct (with its weights PW) and the coarsest grid's sweeps of
// k_coarse_solve.  Only the first level's field is written back; the coarser
// levels' fields are rebuilt by every descent.
//
// Bound: the one CU's latency and VALU.  So the sides are compile-time (the
// indices are shifts and masks; with runtime sides every cell paid five
// integer divisions), the first level's density and source stay in the
// registers of the thread that owns the cell, f(R)'s e^phi is computed once
// per value beside the field instead of seven times per update, the defect is
// computed once per fine cell, and the 4^3 grid lives in one wave's registers
// (coarsest_sweeps).
// First level 16^3, per call, before and with this: symmetron FP64 67 -> 27 us,
// f(R) FP32 78 -> 42 and FP64 139 -> 71, chameleon FP32 70 -> 34 and FP64
// 128 -> 61.
#pragma once
#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace isis {

constexpr int kBottomMaxN = 16;      // side of the first level handled
constexpr int kBottomMaxLevels = 3;  // 16, 8, 4
// Threads: 1024 (16 waves hide the LDS latency on the one CU; up to 128
// registers), 512 where the double-precision exponentials need more.
template <class T, class M>
constexpr int bottom_threads()
{
    return sizeof(T) == 8 && StageOp<T, M>::kStaged ? 512 : 1024;
}

template <class T>
struct BottomArgs {
    int nu_pre, nu_post, nu_coarse;
    T* phi0;                         // the first level's field, updated in place
    const T* sigma0;                 // the first level's FAS source (may be NULL: zero)
    int from_rr;                     // sigma0 is its restricted defect: sigma = L(phi0) - rr
    const T* eta[kBottomMaxLevels];  // densities
    T ih2[kBottomMaxLevels];         // 1/h^2 per level
};

// LDS elements: the first level's field and defect; per coarser level the
// field, its restriction, density and FAS source; staged models: e^phi of
// every level's field.  Sides 4 << (nlev - 1 - q), q < nlev.
template <class T, class M>
constexpr int bottom_lds_elems(int nlev)
{
    int e = 0;
    for (int q = 0; q < nlev; ++q) {
        const int n = 4 << (nlev - 1 - q);
        e += ((q == 0 ? 2 : 4) + (StageOp<T, M>::kStaged ? 1 : 0)) * n * n * n;
    }
    return e;
}

// Value of lane `lane ^ ...` patterns on the 4^3 grid in one wave (lane = 16 i
// + 4 j + k): the k neighbours by a quad permutation, the j neighbours by a
// rotation of the 16-lane row, the i neighbours through the LDS crossbar.
// CTRL: DPP control word.
template <int CTRL>
__device__ __forceinline__ float lane_move(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double lane_move(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
// order x-, x+, y-, y+, z-, z+ (x = i); every lane of the wave must call it
template <class T>
__device__ __forceinline__ void lane_neighbours(T v, int lane, T nb[6])
{
    nb[0] = __shfl(v, (lane - 16) & 63, 64);
    nb[1] = __shfl(v, (lane + 16) & 63, 64);
    nb[2] = lane_move<0x124>(v);  // row_ror:4: lane takes lane - 4 of its row
    nb[3] = lane_move<0x12c>(v);  // row_ror:12
    nb[4] = lane_move<0x93>(v);   // quad_perm [3, 0, 1, 2]
    nb[5] = lane_move<0x39>(v);   // quad_perm [1, 2, 3, 0]
}

// nu red-black sweeps on the 4^3 grid in one wave64, one cell per lane, all in
// registers.  Once a sweep leaves every value as it was, the remaining sweeps
// would too, and are skipped (their safeguard activations, those of that
// sweep again, are added).  Returns the lane's value.
template <class T, class M>
__device__ __forceinline__ T coarsest_sweeps(const M& m, T ih2, T p, T e, T s, int nu,
                                             unsigned& hits)
{
    using SO = StageOp<T, M>;
    const int lane = threadIdx.x & 63;
    const int par = ((lane >> 4) + (lane >> 2) + lane) & 1;
    T ep = SO::stage(p);
    for (int it = 0; it < nu; ++it) {
        bool moved = false;
        unsigned h = 0;
#pragma unroll
        for (int colour = 0; colour < 2; ++colour) {
            T nb[6], enb[6];
            lane_neighbours(p, lane, nb);
            if constexpr (SO::kStaged) lane_neighbours(ep, lane, enb);
            if (par == colour) {
                T L, D;
                SO::eval(m, p, nb, ep, enb, e, ih2, L, D);
                if constexpr (M::kGuard) h += m.guarded(p, e);
                const T v = p - m.limit((L - s) / D);
                moved = moved || v != p;
                p = v;
                if constexpr (SO::kStaged) ep = SO::stage(p);
            }
        }
        hits += h;
        if (__ballot(moved) == 0) {
            hits += h * (unsigned)(nu - 1 - it);
            break;
        }
    }
    return p;
}

// PW: the prolongation's weights (k_prolong_correct).
template <class T, class M, int NLEV, bool FW, int PW = 0>
__global__ __launch_bounds__((bottom_threads<T, M>())) void k_bottom_cycle(M m, BottomArgs<T> a)
{
    using SO = StageOp<T, M>;
    constexpr bool STAGED = SO::kStaged;
    constexpr int NT = bottom_threads<T, M>();
    constexpr int N0 = 4 << (NLEV - 1), N3 = N0 * N0 * N0;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T* base = reinterpret_cast<T*>(smem_raw);
    const int tid = threadIdx.x;
    T *phi[NLEV], *ex[NLEV], *eta[NLEV], *sig[NLEV], *hat[NLEV];
    T* dfine = base;  // the defect of the level being restricted
    {
        int off = N3;
#pragma unroll
        for (int q = 0; q < NLEV; ++q) {
            const int n3 = N3 >> (3 * q);
            phi[q] = base + off;
            off += n3;
            ex[q] = base + off;
            if (STAGED) off += n3;
            eta[q] = sig[q] = hat[q] = nullptr;
            if (q > 0) {
                eta[q] = base + off;
                sig[q] = base + off + n3;
                hat[q] = base + off + 2 * n3;
                off += 3 * n3;
            }
        }
    }
    // cell t of a colour's list on a side-n grid (t < n^3 / 2)
    auto cell_of = [](int n, int t, int colour, int& i, int& j, int& k)
        __attribute__((always_inline)) {
        const int ln = 31 - __builtin_clz(n);
        const int kk = t & ((n >> 1) - 1);
        j = (t >> (ln - 1)) & (n - 1);
        i = t >> (2 * ln - 1);
        k = 2 * kk + ((i + j + colour) & 1);
    };
    // operator of cell (i, j, k) of level q's field
    auto oper = [&](int q, int n, int i, int j, int k, T e, T ih2, T& p, T& L, T& D)
        __attribute__((always_inline)) {
        const int w = n - 1, r = (i * n + j) * n;
        const int c = r + k;
        const int o[6] = {(((i - 1) & w) * n + j) * n + k, (((i + 1) & w) * n + j) * n + k,
                          (i * n + ((j - 1) & w)) * n + k, (i * n + ((j + 1) & w)) * n + k,
                          r + ((k - 1) & w), r + ((k + 1) & w)};
        T nb[6], enb[6];
#pragma unroll
        for (int f = 0; f < 6; ++f) nb[f] = phi[q][o[f]];
        p = phi[q][c];
        T ep = T(0);
        if constexpr (STAGED) {
#pragma unroll
            for (int f = 0; f < 6; ++f) enb[f] = ex[q][o[f]];
            ep = ex[q][c];
        }
        SO::eval(m, p, nb, ep, enb, e, ih2, L, D);
    };
    auto put = [&](int q, int c, T v) __attribute__((always_inline)) {
        phi[q][c] = v;
        if constexpr (STAGED) ex[q][c] = SO::stage(v);
    };

    // the first level's cells of this thread: density and source, per colour
    constexpr int PER = (N3 / 2 + NT - 1) / NT;
    T eta0[2][PER], sig0[2][PER];
#pragma unroll
    for (int colour = 0; colour < 2; ++colour)
#pragma unroll
        for (int r = 0; r < PER; ++r) {
            const int t = min(tid + r * NT, N3 / 2 - 1);
            int i, j, k;
            cell_of(N0, t, colour, i, j, k);
            const int c = (i * N0 + j) * N0 + k;
            eta0[colour][r] = a.eta[0][c];
            sig0[colour][r] = a.sigma0 ? a.sigma0[c] : T(0);
        }
    for (int c = tid; c < N3; c += NT) put(0, c, a.phi0[c]);
#pragma unroll
    for (int q = 1; q < NLEV; ++q)
        for (int c = tid; c < (N3 >> (3 * q)); c += NT) eta[q][c] = a.eta[q][c];
    __syncthreads();
    if (a.from_rr) {
#pragma unroll
        for (int colour = 0; colour < 2; ++colour)
#pragma unroll
            for (int r = 0; r < PER; ++r) {
                int i, j, k;
                cell_of(N0, min(tid + r * NT, N3 / 2 - 1), colour, i, j, k);
                T p, L, D;
                oper(0, N0, i, j, k, eta0[colour][r], a.ih2[0], p, L, D);
                sig0[colour][r] = L - sig0[colour][r];
            }
        __syncthreads();
    }
    unsigned hits = 0;

    // f(cell, density, source) for this thread's cells of one colour of level q
    auto each = [&](auto qc, int colour, auto&& f) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value, n = N0 >> q, half = n * n * n / 2;
        if constexpr (q == 0) {
#pragma unroll
            for (int r = 0; r < PER; ++r)
                if ((r + 1) * NT <= half || tid + r * NT < half) {
                    int i, j, k;
                    cell_of(n, tid + r * NT, colour, i, j, k);
                    f(i, j, k, eta0[colour][r], sig0[colour][r]);
                }
        } else {
            static_assert(half <= NT, "one cell per thread");
            if (tid < half) {
                int i, j, k;
                cell_of(n, tid, colour, i, j, k);
                const int c = (i * n + j) * n + k;
                f(i, j, k, eta[q][c], sig[q][c]);
            }
        }
    };
    auto sweep = [&](auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value, n = N0 >> q;
#pragma unroll
        for (int colour = 0; colour < 2; ++colour) {
            each(qc, colour, [&](int i, int j, int k, T e, T s) __attribute__((always_inline)) {
                T p, L, D;
                oper(q, n, i, j, k, e, a.ih2[q], p, L, D);
                if constexpr (M::kGuard) hits += m.guarded(p, e);
                put(q, (i * n + j) * n + k, p - m.limit((L - s) / D));
            });
            __syncthreads();
        }
    };

    auto descend = [&](auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value, nf = N0 >> q, nc = nf / 2, c3 = nc * nc * nc;
        constexpr int lc = nc == 8 ? 3 : nc == 4 ? 2 : 1;
#pragma unroll
        for (int colour = 0; colour < 2; ++colour)
            each(qc, colour, [&](int i, int j, int k, T e, T s) __attribute__((always_inline)) {
                T p, L, D;
                oper(q, nf, i, j, k, e, a.ih2[q], p, L, D);
                dfine[(i * nf + j) * nf + k] = L - s;
            });
        __syncthreads();
        const int K = tid & (nc - 1), J = (tid >> lc) & (nc - 1), I = tid >> (2 * lc);
        T rr = T(0);
        if (tid < c3) {
            T sr = T(0), sp = T(0);
#pragma unroll
            for (int di = 0; di < 2; ++di)
#pragma unroll
                for (int dj = 0; dj < 2; ++dj)
#pragma unroll
                    for (int dk = 0; dk < 2; ++dk) {
                        const int c = ((2 * I + di) * nf + 2 * J + dj) * nf + 2 * K + dk;
                        sr += dfine[c];
                        sp += phi[q][c];
                    }
            const T pc = sp / T(8);
            put(q + 1, tid, pc);
            hat[q + 1][tid] = pc;
            rr = sr / T(8);
            if constexpr (FW) {
                const T w[4] = {T(0.125), T(0.375), T(0.375), T(0.125)};
                rr = T(0);
#pragma unroll
                for (int aa = 0; aa < 4; ++aa) {
                    const int i = (2 * I - 1 + aa) & (nf - 1);
                    T sy = T(0);
#pragma unroll
                    for (int bb = 0; bb < 4; ++bb) {
                        const int j = (2 * J - 1 + bb) & (nf - 1);
                        const T* row = dfine + (i * nf + j) * nf;
                        T sz = T(0);
#pragma unroll
                        for (int cc = 0; cc < 4; ++cc) sz += w[cc] * row[(2 * K - 1 + cc) & (nf - 1)];
                        sy += w[bb] * sz;
                    }
                    rr += w[aa] * sy;
                }
            }
        }
        __syncthreads();
        // Sigma_c = L_c(phi_c) - rr
        if (tid < c3) {
            T p, L, D;
            oper(q + 1, nc, I, J, K, eta[q + 1][tid], a.ih2[q + 1], p, L, D);
            sig[q + 1][tid] = L - rr;
        }
        __syncthreads();
    };

    // one thread per coarse cell updates its 8 children (see k_prolong_pairs)
    auto prolong = [&](auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value, nf = N0 >> q, nc = nf / 2, c3 = nc * nc * nc;
        constexpr int lc = nc == 8 ? 3 : nc == 4 ? 2 : 1;
        const T* co = phi[q + 1];
        const T* ch = hat[q + 1];
        const T w[2] = {T(0.75), T(0.25)};
        if (tid < c3) {
            const int K = tid & (nc - 1), J = (tid >> lc) & (nc - 1), I = tid >> (2 * lc);
            const int Ix[3] = {(I - 1) & (nc - 1), I, (I + 1) & (nc - 1)};
            const int Jy[3] = {(J - 1) & (nc - 1), J, (J + 1) & (nc - 1)};
            const int Kz[3] = {(K - 1) & (nc - 1), K, (K + 1) & (nc - 1)};
            T d[3][3][3];
#pragma unroll
            for (int x = 0; x < 3; ++x)
#pragma unroll
                for (int y = 0; y < 3; ++y)
#pragma unroll
                    for (int z = 0; z < 3; ++z) {
                        const int c = (Ix[x] * nc + Jy[y]) * nc + Kz[z];
                        d[x][y][z] = co[c] - ch[c];
                    }
            T wo[3][2] = {{w[1], w[1]}, {w[1], w[1]}, {w[1], w[1]}};
            if constexpr (PW != 0) {
                const T hp = ch[tid];
#pragma unroll
                for (int sd = 0; sd < 2; ++sd) {
                    wo[0][sd] = prolong_weight<PW>(hp, ch[(Ix[2 * sd] * nc + J) * nc + K]);
                    wo[1][sd] = prolong_weight<PW>(hp, ch[(I * nc + Jy[2 * sd]) * nc + K]);
                    wo[2][sd] = prolong_weight<PW>(hp, ch[(I * nc + J) * nc + Kz[2 * sd]]);
                }
            }
#pragma unroll
            for (int di = 0; di < 2; ++di)
#pragma unroll
                for (int dj = 0; dj < 2; ++dj)
#pragma unroll
                    for (int dk = 0; dk < 2; ++dk) {
                        const int ai[2] = {1, 2 * di}, bj[2] = {1, 2 * dj}, ck[2] = {1, 2 * dk};
                        const T wx[2] = {PW ? T(1) - wo[0][di] : w[0], PW ? wo[0][di] : w[1]};
                        const T wy[2] = {PW ? T(1) - wo[1][dj] : w[0], PW ? wo[1][dj] : w[1]};
                        const T wz[2] = {PW ? T(1) - wo[2][dk] : w[0], PW ? wo[2][dk] : w[1]};
                        T s = T(0);
#pragma unroll
                        for (int x = 0; x < 2; ++x)
#pragma unroll
                            for (int y = 0; y < 2; ++y)
#pragma unroll
                                for (int z = 0; z < 2; ++z)
                                    s += wx[x] * wy[y] * wz[z] * d[ai[x]][bj[y]][ck[z]];
                        const int c = ((2 * I + di) * nf + 2 * J + dj) * nf + 2 * K + dk;
                        put(q, c, phi[q][c] + s);
                    }
        }
        __syncthreads();
    };

    static_for<0, NLEV - 1>([&](auto qc) {
        for (int it = 0; it < a.nu_pre; ++it) sweep(qc);
        descend(qc);
    });
    if (tid < 64) {  // the 4^3 grid in the first wave
        constexpr int q = NLEV - 1;
        phi[q][tid] = coarsest_sweeps(m, a.ih2[q], phi[q][tid], eta[q][tid], sig[q][tid],
                                      a.nu_coarse, hits);
    }
    __syncthreads();
    static_for<0, NLEV - 1>([&](auto rc) {
        constexpr std::integral_constant<int, NLEV - 2 - decltype(rc)::value> qc{};
        prolong(qc);
        for (int it = 0; it < a.nu_post; ++it) sweep(qc);
    });
    for (int c = tid; c < N3; c += NT) a.phi0[c] = phi[0][c];
    guard_flush(m, hits);
}

}  // namespace isis
