// One red-black Newton-Gauss-Seidel sweep of a small level (sides 32 and 64) in
// one launch, out of place, with the steps around it in the V-cycle: the FAS
// source from the restricted defect before it, the coarse-grid correction
// before it, or the defect and its restriction after it.
//
// A workgroup owns an 8 x 8 x 16 block of cells and stages it with a halo of
// two cells (three in x and y, four in z, with the restriction) in LDS, with
// e^phi beside it for the staged models.  Both colours then run there: the red
// stage on the block and a ring around it, the black stage one cell further
// in, every neighbour at the stage the sequential sweep sees.  A thread keeps
// the same z-pairs of cells throughout, their densities and sources in
// registers.
//
// Why: on these levels a launch is mostly launch and drain (4.7 us, whatever
// it does).  Per level and cycle this makes three launches (four with two
// post-smoothing sweeps) of what were eight or ten: 1.9 to 2.5 times the
// updates (the halo's), which the device has room for.
// 32^3 and 64^3: 6 to 11 us per launch.  Not from 128^3 on: 55, 45 and 23 us for
// the three launches in double precision (symmetron) against 36 and 21 in fused
// passes, 34, 24 and 18 in single precision against six half-sweeps of 9.1 us, a
// restriction of 10 and a prolongation of 9.
//
// Per cell the arithmetic is that of k_halfsweep, k_fas_sigma, k_prolong_pairs
// and k_defect_restrict_pairs, in their order.
#pragma once
#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace isis {

template <bool DESC, bool PROL>
struct BlockTile {
    static constexpr int TX = 8, TY = 8, TZ = 16, NT = 512;
    static constexpr int H = DESC ? 3 : 2, HZ = (H + 1) & ~1;  // pairs start even
    static constexpr int EX = TX + 2 * H, EY = TY + 2 * H, EZ = TZ + 2 * HZ, NP = EZ / 2;
    static constexpr int CELLS = EX * EY * EZ, PAIRS = CELLS / 2;
    static constexpr int PER = (PAIRS + NT - 1) / NT;
    // coarse window of the correction: the parents and their neighbours
    static constexpr int CX = EX / 2 + 2, CY = EY / 2 + 2, CZ = EZ / 2 + 2, CWIN = CX * CY * CZ;
    static_assert(!(DESC && PROL), "the correction comes before post-smoothing only");
};

template <class T, class M, bool DESC, bool PROL>
constexpr int block_lds_bytes()
{
    using G = BlockTile<DESC, PROL>;
    int e = G::CELLS * (StageOp<T, M>::kStaged ? 2 : 1);
    if (DESC) e += G::TX * G::TY * G::TZ;
    if (PROL) e += 2 * G::CWIN;
    return e * (int)sizeof(T);
}

template <class T>
struct BlockArgs {
    int n;
    T ih2;
    const T* in;
    T* out;
    const T* eta;
    T* sigma;         // FAS source (NULL: zero); written where rr is given
    const T* rr;      // restricted defect: sigma = L(in) - rr first (or NULL)
    const T* cphi;    // PROL: the coarse field and its restriction, side n / 2
    const T* cphat;
    T* phi_c;         // DESC: restricted field, twice, and restricted defect
    T* phihat_c;
    T* rr_c;
};

// PW: the prolongation's weights (k_prolong_correct).
template <class T, class M, bool DESC, bool PROL, int PW = 0>
__global__ __launch_bounds__(512) void k_block_sweep(M m, BlockArgs<T> a)
{
    using G = BlockTile<DESC, PROL>;
    using V = typename Vec2<T>::type;
    using SO = StageOp<T, M>;
    constexpr bool STAGED = SO::kStaged;
    constexpr int SX = G::EY * G::EZ, SY = G::EZ;  // LDS strides
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T* ph = reinterpret_cast<T*>(smem_raw);
    T* ex = ph + G::CELLS;
    T* aux = ph + G::CELLS * (STAGED ? 2 : 1);  // DESC: the block's defect; PROL: the coarse window

    const int tid = threadIdx.x;
    const int n = a.n, msk = n - 1;
    int b = blockIdx.x;
    const int nb = gridDim.x;
    if ((nb & 7) == 0) b = (b & 7) * (nb >> 3) + (b >> 3);  // contiguous blocks per XCD
    const int nz = n / G::TZ, ny = n / G::TY;
    const int z0 = (b % nz) * G::TZ, y0 = (b / nz) % ny * G::TY, x0 = b / (nz * ny) * G::TX;

    // this thread's pairs: local x, y and the local column of the first cell
    int lx[G::PER], ly[G::PER], lz[G::PER];
    V e2[G::PER], s2[G::PER], f2[G::PER], r2[G::PER];
#pragma unroll
    for (int q = 0; q < G::PER; ++q) {
        const int e = min(tid + q * G::NT, G::PAIRS - 1);
        lz[q] = 2 * (e % G::NP);
        ly[q] = e / G::NP % G::EY;
        lx[q] = e / (G::NP * G::EY);
        const size_t g = ((size_t)((x0 - G::H + lx[q]) & msk) * n + ((y0 - G::H + ly[q]) & msk)) * n +
                         ((z0 - G::HZ + lz[q]) & msk);
        f2[q] = *reinterpret_cast<const V*>(a.in + g);
        e2[q] = *reinterpret_cast<const V*>(a.eta + g);
        s2[q] = V{T(0), T(0)};
        r2[q] = V{T(0), T(0)};
        if (a.rr)
            r2[q] = *reinterpret_cast<const V*>(a.rr + g);
        else if (a.sigma)
            s2[q] = *reinterpret_cast<const V*>(a.sigma + g);
    }
    if constexpr (PROL) {
        const int nc = n >> 1, cm = nc - 1;
        T* cd = aux;            // coarse differences
        T* ch = aux + G::CWIN;  // restricted field
        for (int e = tid; e < G::CWIN; e += G::NT) {
            const int cz = e % G::CZ, cy = e / G::CZ % G::CY, cx = e / (G::CZ * G::CY);
            const size_t g = ((size_t)((((x0 - G::H) >> 1) - 1 + cx) & cm) * nc +
                              ((((y0 - G::H) >> 1) - 1 + cy) & cm)) * nc +
                             ((((z0 - G::HZ) >> 1) - 1 + cz) & cm);
            const T h = a.cphat[g];
            cd[e] = a.cphi[g] - h;
            ch[e] = h;
        }
        __syncthreads();
        const T w[2] = {T(0.75), T(0.25)};
#pragma unroll
        for (int q = 0; q < G::PER; ++q) {
            // parent's window index; the other cell towards the child's side
            const int cx = (lx[q] >> 1) + 1, cy = (ly[q] >> 1) + 1, cz = (lz[q] >> 1) + 1;
            const int c0 = (cx * G::CY + cy) * G::CZ + cz;
            const int ox = ((lx[q] & 1) ? 1 : -1) * G::CY * G::CZ, oy = ((ly[q] & 1) ? 1 : -1) * G::CZ;
            T wx[2] = {w[0], w[1]}, wy[2] = {w[0], w[1]};
            if constexpr (PW != 0) {
                wx[1] = prolong_weight<PW>(ch[c0], ch[c0 + ox]);
                wy[1] = prolong_weight<PW>(ch[c0], ch[c0 + oy]);
                wx[0] = T(1) - wx[1];
                wy[0] = T(1) - wy[1];
            }
#pragma unroll
            for (int dk = 0; dk < 2; ++dk) {
                const int oz = dk ? 1 : -1;
                T wz[2] = {w[0], w[1]};
                if constexpr (PW != 0) {
                    wz[1] = prolong_weight<PW>(ch[c0], ch[c0 + oz]);
                    wz[0] = T(1) - wz[1];
                }
                T s = T(0);
#pragma unroll
                for (int x = 0; x < 2; ++x)
#pragma unroll
                    for (int y = 0; y < 2; ++y)
#pragma unroll
                        for (int z = 0; z < 2; ++z)
                            s += wx[x] * wy[y] * wz[z] * cd[c0 + x * ox + y * oy + z * oz];
                f2[q][dk] += s;
            }
        }
    }
#pragma unroll
    for (int q = 0; q < G::PER; ++q) {
        const int o = lx[q] * SX + ly[q] * SY + lz[q];
        if ((q + 1) * G::NT <= G::PAIRS || tid + q * G::NT < G::PAIRS) {
            *reinterpret_cast<V*>(ph + o) = f2[q];
            if constexpr (STAGED)
                *reinterpret_cast<V*>(ex + o) = V{SO::stage(f2[q].x), SO::stage(f2[q].y)};
        }
    }
    __syncthreads();

    // operator at LDS offset o
    auto oper = [&](int o, T e, T& p, T& L, T& D) __attribute__((always_inline)) {
        T nbv[6], enb[6];
        nbv[0] = ph[o - SX];
        nbv[1] = ph[o + SX];
        nbv[2] = ph[o - SY];
        nbv[3] = ph[o + SY];
        nbv[4] = ph[o - 1];
        nbv[5] = ph[o + 1];
        p = ph[o];
        T ep = T(0);
        if constexpr (STAGED) {
            enb[0] = ex[o - SX];
            enb[1] = ex[o + SX];
            enb[2] = ex[o - SY];
            enb[3] = ex[o + SY];
            enb[4] = ex[o - 1];
            enb[5] = ex[o + 1];
            ep = ex[o];
        }
        SO::eval(m, p, nbv, ep, enb, e, a.ih2, L, D);
    };
    // whether pair q's rows, or its cell at column z, lie within `ring` cells of the block
    auto rows_in = [&](int q, int ring) __attribute__((always_inline)) {
        return lx[q] >= G::H - ring && lx[q] < G::H + G::TX + ring && ly[q] >= G::H - ring &&
               ly[q] < G::H + G::TY + ring &&
               ((q + 1) * G::NT <= G::PAIRS || tid + q * G::NT < G::PAIRS);
    };
    auto col_in = [&](int z, int ring) __attribute__((always_inline)) {
        return z >= G::HZ - ring && z < G::HZ + G::TZ + ring;
    };
    auto own = [&](int q) __attribute__((always_inline)) { return rows_in(q, 0) && col_in(lz[q], 0); };
    // global index of an own pair
    auto gidx = [&](int q) __attribute__((always_inline)) {
        return ((size_t)(x0 - G::H + lx[q]) * n + (y0 - G::H + ly[q])) * n + z0 - G::HZ + lz[q];
    };

    constexpr int R1 = G::H - 1;  // ring of the red stage
    if (a.rr) {                   // the FAS source, from the field as restricted
#pragma unroll
        for (int q = 0; q < G::PER; ++q)
            if (rows_in(q, R1)) {
#pragma unroll
                for (int dk = 0; dk < 2; ++dk)
                    if (col_in(lz[q] + dk, R1)) {
                        T p, L, D;
                        oper(lx[q] * SX + ly[q] * SY + lz[q] + dk, e2[q][dk], p, L, D);
                        s2[q][dk] = L - r2[q][dk];
                    }
                if (own(q)) *reinterpret_cast<V*>(a.sigma + gidx(q)) = s2[q];
            }
        __syncthreads();
    }
    unsigned hits = 0;
#pragma unroll
    for (int colour = 0; colour < 2; ++colour) {
#pragma unroll
        for (int q = 0; q < G::PER; ++q) {
            // (x0, y0, z0 and the z halo are even: the parity is local)
            const int dk = (lx[q] + ly[q] + 2 * G::H + colour) & 1;
            const int z = lz[q] + dk;
            if (rows_in(q, R1 - colour) && col_in(z, R1 - colour)) {
                const int o = lx[q] * SX + ly[q] * SY + z;
                const T e = dk ? e2[q].y : e2[q].x, s = dk ? s2[q].y : s2[q].x;
                T p, L, D;
                oper(o, e, p, L, D);
                if constexpr (M::kGuard) {
                    if (own(q)) hits += m.guarded(p, e);
                }
                const T v = p - m.limit((L - s) / D);
                ph[o] = v;
                if constexpr (STAGED) {
                    if (DESC || colour == 0) ex[o] = SO::stage(v);
                }
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < G::PER; ++q)
        if (own(q)) {
            const int o = lx[q] * SX + ly[q] * SY + lz[q];
            *reinterpret_cast<V*>(a.out + gidx(q)) = *reinterpret_cast<const V*>(ph + o);
            if constexpr (DESC) {
                V d;
#pragma unroll
                for (int dk = 0; dk < 2; ++dk) {
                    T p, L, D;
                    oper(o + dk, e2[q][dk], p, L, D);
                    d[dk] = L - s2[q][dk];
                }
                *reinterpret_cast<V*>(aux + ((lx[q] - G::H) * G::TY + ly[q] - G::H) * G::TZ +
                                      lz[q] - G::HZ) = d;
            }
        }
    if constexpr (DESC) {
        __syncthreads();
        constexpr int KC = G::TZ / 2, JC = G::TY / 2, IC = G::TX / 2;
        static_assert(IC * JC * KC <= G::NT, "one coarse cell per thread");
        if (tid < IC * JC * KC) {
            const int K = tid % KC, J = tid / KC % JC, I = tid / (KC * JC);
            T sr = T(0), sp = T(0);
#pragma unroll
            for (int di = 0; di < 2; ++di)
#pragma unroll
                for (int dj = 0; dj < 2; ++dj) {
                    const V d = *reinterpret_cast<const V*>(aux + ((2 * I + di) * G::TY + 2 * J + dj) * G::TZ + 2 * K);
                    const V p = *reinterpret_cast<const V*>(
                        ph + (G::H + 2 * I + di) * SX + (G::H + 2 * J + dj) * SY + G::HZ + 2 * K);
                    sr += d[0];
                    sr += d[1];
                    sp += p[0];
                    sp += p[1];
                }
            const int nc = n >> 1;
            const size_t g = ((size_t)(x0 / 2 + I) * nc + y0 / 2 + J) * nc + z0 / 2 + K;
            const T pc = sp / T(8);
            a.phi_c[g] = pc;
            a.phihat_c[g] = pc;
            a.rr_c[g] = sr / T(8);
        }
    }
    guard_flush(m, hits);
}

}  // namespace isis
