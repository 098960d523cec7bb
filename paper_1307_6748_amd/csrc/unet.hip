// Learned warm start: a 3D U-Net in BF16 with FP32 accumulation on MFMA.
//
// The network maps (log density, expansion factor, cold-start field) to the
// correction phi* - phi_cold; its prediction initialises the FAS solve, which
// stays the judge of its error (the caller falls back to the cold start when
// the predicted field's residual is not below the cold start's).
//
// Architecture (4 levels, channels 16/32/64/64, periodic 3x3x3 convolutions,
// ReLU, 2x2x2 average pooling, nearest upsampling, skip concatenation
// [upsampled, skip], 1x1x1 head):
//   enc0 16->16, 16->16 | enc1 pool, 16->32, 32->32 | enc2 pool, 32->64, 64->64
//   bot pool, 64->64, 64->64 | dec2 up+cat 128->64, 64->64
//   dec1 up+cat 96->32, 32->32 | dec0 up+cat 48->16, 16->16 | head 16->1
// Tensors are channels-last [x][y][z][c] in bfloat16 (raw uint16 bits).
// Convolution weights W[t][cout][cin], t = (di+1)*9 + (dj+1)*3 + (dk+1) for
// the input read at (i+di, j+dj, k+dk); the flat FP32 parameter vector holds
// the 14 convolutions (weights then bias) in the order above, then the head.
//
// Convolutions are implicit GEMMs: M = voxels, N = output channels,
// K = 27 * input channels, on the bf16 MFMAs of 16 x 16 outputs, with the input
// and mostly the weights staged in LDS: sides >= 64 in k_conv3_ring (16 input
// channels, streaming along x, v_mfma_f32_16x16x16), k_conv3_planes (16 output
// channels, streaming along x) and k_conv3_lds (the others), both on
// v_mfma_f32_16x16x32; sides 8 to 32 in k_conv3_small and below in k_conv3, one
// tile straight from memory, both on 16x16x16.  The data gradient is the same
// kernels on flipped, transposed weights; the weight gradient is a split-K GEMM
// over regions of the grid with a fixed-order reduction of the partial sums
// (deterministic).  The prediction's last decoder stage reads its upsampled and
// skip inputs directly instead of a materialised concatenation.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <cstring>

#include "../../include/isis_mg.h"
#include "device.hpp"

namespace {

thread_local char u_err[512];

void uerr(const char* fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(u_err, sizeof(u_err), fmt, ap);
    va_end(ap);
}

using bf16_t = uint16_t;
typedef short s4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));  // (HIP's uint4 arrays go to scratch)
// The convolutions' inputs and weights: callers' tensors, aligned as their bf16
// elements are.  (The same one load instruction.)
typedef s4 s4_any __attribute__((aligned(2)));
typedef u4 u4_any __attribute__((aligned(2)));

constexpr int kThreads = 256;
constexpr int kMaxGrid = 65536;

int grid_of(long work) { return (int)std::max(1L, std::min((work + kThreads - 1) / kThreads, (long)kMaxGrid)); }

__device__ __forceinline__ float bf2f(bf16_t b) { return __uint_as_float((uint32_t)b << 16); }

// Round to nearest even (NaN kept quiet).
__device__ __forceinline__ bf16_t f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x7fffffu)) return (bf16_t)((u >> 16) | 0x40);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}

// ---------------------------------------------------------------------------
// Convolution (forward; also the data gradient with prepared weights).
// ---------------------------------------------------------------------------

// Four consecutive channels of one voxel (element offset o, a multiple of 4):
// ReLU, then to the bf16 and / or FP32 output; vec: as one 8- and 16-byte
// store (the outputs' base addresses are that much aligned).
__device__ __forceinline__ void store4(f4 v, int relu, int vec, bf16_t* y, float* yf, size_t o)
{
    if (relu) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = fmaxf(v[r], 0.f);
    }
    if (vec) {
        if (y) *reinterpret_cast<bf4v*>(y + o) = __builtin_convertvector(v, bf4v);
        if (yf) *reinterpret_cast<f4*>(yf + o) = v;
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (y) y[o + r] = f2bf(v[r]);
            if (yf) yf[o + r] = v[r];
        }
    }
}

__device__ __forceinline__ f4 bias4(const float* bias, int co)
{
    f4 b = f4{0.f, 0.f, 0.f, 0.f};
    if (bias) {
#pragma unroll
        for (int r = 0; r < 4; ++r) b[r] = bias[co + r];
    }
    return b;
}

// y[v][co] = sum_t sum_ci x[v + d_t][ci] * w[t][co][ci] (+ bias, ReLU), sides
// below 8.  Any power-of-two side n >= 2; each wave owns 16 consecutive
// voxels and 16 output channels (a few hundred waves at most: these grids are
// all latency).  Lanes past the last voxel load voxel 0 and store nothing.
//   64 -> 64 at 4^3: 0.085 -> 0.025 ms
template <int CIN>
__global__ __launch_bounds__(kThreads) void k_conv3(const bf16_t* __restrict__ x, int n,
                                                    const bf16_t* __restrict__ w,
                                                    const float* __restrict__ bias, int cout,
                                                    int relu, int vec, bf16_t* __restrict__ y,
                                                    float* __restrict__ yf)
{
    const int lane = threadIdx.x & 63;
    const int wave = blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    const int nco = cout >> 4;
    const int co0 = (wave % nco) * 16, v0 = (wave / nco) * 16;
    const int nvox = n * n * n, msk = n - 1;
    if (v0 >= nvox) return;
    const int m = lane & 15, g = lane >> 4;
    const int v = v0 + m < nvox ? v0 + m : 0;
    const int ck = v & msk, cj = (v / n) & msk, ci = v / (n * n);
    constexpr int NS = CIN / 16;
    // three taps (dk = -1, 0, 1) at a time, the next three in flight
    s4 xa[2][3][NS], wa[2][3][NS];
    auto load = [&](int t9, int p) __attribute__((always_inline)) {
        const int di = t9 / 3 - 1, dj = t9 % 3 - 1;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const bf16_t* xs = x + (((((ci + di) & msk) * n + ((cj + dj) & msk)) * n + ((ck + k - 1) & msk)) * CIN + 4 * g);
            const bf16_t* wt = w + ((3 * t9 + k) * cout + co0 + m) * CIN + 4 * g;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                xa[p][k][s] = *reinterpret_cast<const s4_any*>(xs + 16 * s);
                wa[p][k][s] = *reinterpret_cast<const s4_any*>(wt + 16 * s);
            }
        }
    };
    f4 acc = f4{0.f, 0.f, 0.f, 0.f};
    load(0, 0);
#pragma unroll
    for (int t9 = 0; t9 < 9; ++t9) {
        if (t9 < 8) load(t9 + 1, (t9 + 1) & 1);
        __builtin_amdgcn_sched_barrier(0);  // keep the loads ahead of these MFMAs
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int s = 0; s < NS; ++s)
                acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(wa[t9 & 1][k][s], xa[t9 & 1][k][s], acc, 0, 0, 0);
    }
    // the weights are the row operand: D[row = 4g + r][col = m] is channel
    // co0 + 4g + r of voxel v0 + m
    if (v0 + m < nvox)
        store4(acc + bias4(bias, co0 + 4 * g), relu, vec, y, yf, (size_t)(v0 + m) * cout + co0 + 4 * g);
}

// The same convolution on sides 8, 16 and 32 (Z), all input channels staged in
// LDS: a workgroup computes 16 NT output channels of TY rows of one x-plane,
// MW M tiles of 16 voxels per wave.  LDS holds the 3 x (TY + 2) x (Z + 2)
// voxels as arrays of 4-channel units, one per k-group of the 16x16x16 MFMA
// (see k_conv3_ring), and two buffers of the weights of TPB taps each, filled
// one stage ahead.  (Weight operands read from memory by every wave, 16 lines
// of 32 bytes each, held 64 -> 64 at 32^3 at 0.058 ms.)  Taps, then channels
// are added in the order of k_conv3.  Bound: at 32^3 one workgroup per CU,
// LDS reads and MFMAs in about equal parts; at 16^3 latency.
//   64 -> 64 at 32^3: 0.109 -> 0.024 ms; at 16^3: 0.107 -> 0.009 ms
template <int CIN, int NT, int Z, int TY, int TPB>
struct ConvSmall {
    static constexpr int NS = CIN / 16;
    static constexpr int ZP = Z + 2, VOX = 3 * (TY + 2) * ZP;
    static constexpr int VP = VOX + (48 - VOX % 32) % 32;  // = 16 mod 32: groups 128 bytes out of phase
    static constexpr int WU = TPB * 16 * NT * (CIN / 8);   // 16-byte units of weights per stage
    static constexpr int WPT = (WU + kThreads - 1) / kThreads;
    static constexpr int LDS = VP * CIN * 2 + 2 * WU * 16;
    static constexpr int MW = TY * Z / 64;                 // M tiles (16 voxels of the tile's rows) per wave
    static_assert(MW >= 1 && TY * Z % 64 == 0 && 27 % TPB == 0, "four waves share the tile");
    static_assert(LDS <= 160 * 1024, "LDS overflow");
};
template <int CIN, int NT, int Z, int TY, int TPB>
__global__ __launch_bounds__(kThreads, 1) void k_conv3_small(const bf16_t* __restrict__ x,
                                                             const bf16_t* __restrict__ w,
                                                             const float* __restrict__ bias,
                                                             int cout, int relu, int vec,
                                                             bf16_t* __restrict__ y,
                                                             float* __restrict__ yf)
{
    using G = ConvSmall<CIN, NT, Z, TY, TPB>;
    constexpr int n = Z, msk = n - 1, NS = G::NS;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    s4* tile = reinterpret_cast<s4*>(smem_raw);  // [slice][4-channel group][plane][row][z]
    s4* wl = tile + G::VP * (CIN / 4);           // [buffer][tap][slice][16 channels][group][channel]
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int m = lane & 15, g = lane >> 4;
    const int nco = cout / (16 * NT);
    int b = blockIdx.x;
    const int co0 = (b % nco) * 16 * NT;
    b /= nco;
    const int y0 = (b % (n / TY)) * TY, x0 = b / (n / TY);
    u4 wr[G::WPT];
    // stage st's weights; unit e: 8 channels 8q .. of output channel co0 + c, tap t
    auto load_w = [&](int st) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < G::WPT; ++k) {
            const int e = min(tid + k * kThreads, G::WU - 1);
            const int q = e % (CIN / 8), c = (e / (CIN / 8)) % (16 * NT), t = e / (CIN / 8 * 16 * NT);
            wr[k] = *reinterpret_cast<const u4_any*>(w + (size_t)((st * TPB + t) * cout + co0 + c) * CIN + 8 * q);
        }
    };
    // channel c of group gg sits at position c ^ 2 (q mod 8), q = 8-channel
    // index: the units of one output channel fall on different banks
    auto put_w = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < G::WPT; ++k) {
            const int e = tid + k * kThreads;
            if ((k + 1) * kThreads <= G::WU || e < G::WU) {
                const int q = e % (CIN / 8), c = (e / (CIN / 8)) % (16 * NT), t = e / (CIN / 8 * 16 * NT);
                s4* d = wl + buf * 2 * G::WU +
                        (((t * NS + (q >> 1)) * NT + (c >> 4)) * 4 + 2 * (q & 1)) * 16 +
                        ((c & 15) ^ (2 * (q & 7)));
                d[0] = __builtin_bit_cast(s4, __builtin_shufflevector(wr[k], wr[k], 0, 1));
                d[16] = __builtin_bit_cast(s4, __builtin_shufflevector(wr[k], wr[k], 2, 3));
            }
        }
    };
    load_w(0);
#pragma unroll 4
    for (int e = tid; e < G::VOX * (CIN / 8); e += kThreads) {
        const int q = e % (CIN / 8), v = e / (CIN / 8);  // 8 channels 8q .. of staged voxel v
        const int zz = v % G::ZP, rr = (v / G::ZP) % (TY + 2), pp = v / (G::ZP * (TY + 2));
        const int vox = (((x0 - 1 + pp) & msk) * n + ((y0 - 1 + rr) & msk)) * n + ((zz - 1) & msk);
        const u4 r = *reinterpret_cast<const u4_any*>(x + (size_t)vox * CIN + 8 * q);
        s4* d = tile + 2 * q * G::VP + v;
        d[0] = __builtin_bit_cast(s4, __builtin_shufflevector(r, r, 0, 1));
        d[G::VP] = __builtin_bit_cast(s4, __builtin_shufflevector(r, r, 2, 3));
    }
    f4 acc[G::MW][NT];
#pragma unroll
    for (int t = 0; t < G::MW; ++t)
#pragma unroll
        for (int u = 0; u < NT; ++u) acc[t][u] = f4{0.f, 0.f, 0.f, 0.f};
    const s4* base[G::MW];  // this lane's voxel in its wave's tiles
#pragma unroll
    for (int t = 0; t < G::MW; ++t) {
        const int q = (wv * G::MW + t) * 16 + m;
        base[t] = tile + g * G::VP + (q / Z) * G::ZP + q % Z;
    }
    int wp[NS];  // this lane's weight position per slice
#pragma unroll
    for (int s = 0; s < NS; ++s) wp[s] = g * 16 + (m ^ (2 * ((2 * s + (g >> 1)) & 7)));
    put_w(0);
    if (27 / TPB > 1) load_w(1);
    __syncthreads();
    for (int st = 0; st < 27 / TPB; ++st) {
        if (st + 1 < 27 / TPB) {
            put_w((st + 1) & 1);
            load_w(min(st + 2, 27 / TPB - 1));
        }
        const s4* ws = wl + (st & 1) * 2 * G::WU;
#pragma unroll
        for (int tt = 0; tt < TPB; ++tt) {
            const int tap = st * TPB + tt;
            const int off = ((tap / 9) * (TY + 2) + (tap / 3) % 3) * G::ZP + tap % 3;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                s4 wq[NT];
#pragma unroll
                for (int u = 0; u < NT; ++u) wq[u] = ws[((tt * NS + s) * NT + u) * 64 + wp[s]];
#pragma unroll
                for (int t = 0; t < G::MW; ++t) {
                    const s4 a = base[t][off + 4 * s * G::VP];
#pragma unroll
                    for (int u = 0; u < NT; ++u)
                        acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(wq[u], a, acc[t][u], 0, 0, 0);
                }
            }
        }
        __syncthreads();  // this stage's buffer is refilled next
    }
#pragma unroll
    for (int t = 0; t < G::MW; ++t) {
        const size_t v = ((size_t)x0 * n + y0) * n + (wv * G::MW + t) * 16 + m;
#pragma unroll
        for (int u = 0; u < NT; ++u) {
            const int co = co0 + 16 * u + 4 * g;
            store4(acc[t][u] + bias4(bias, co), relu, vec, y, yf, v * cout + co);
        }
    }
}

// The same convolution with its input and weights staged in LDS (sides n >=
// 64, 32 output channels and more).  A workgroup of NW waves computes 16 NT
// output channels of an NW (y) x 64 (z) tile of two x-planes, one z-row of 64 voxels of both planes per wave
// (eight M tiles of 16).  For each 16-channel slice of the input it stages the
// 4 x (NW + 2) x 66 voxels its 27 taps read and the slice's 27 x 16 NT
// weights.  LDS holds both as arrays of 16-byte units, one per half of 8
// channels ([half][plane][row][z], [tap][half][channel]), read by the 16x16x32
// BF16 MFMA two taps at a time: lane g = lane / 16 takes channel half g & 1 of
// tap 2p + (g >> 1), so the 16 lanes of one (half, tap) group read 256
// contiguous bytes.  The 27th tap is a 14th pair whose second half is zero, so
// every product runs on the 16x16x32 MFMA.  Tiles are dealt to the 8 XCDs in
// contiguous ranges with x fastest, so neighbouring planes share an L2.
// Bound: with one plane per wave and the weights read from memory by each
// wave, the weight reads (32 lines of 32 bytes per operand) held the kernel at
// 0.38-0.55 PFLOP/s; now it reaches 0.73 to 1.05, held by the LDS (NT = 2: one
// and a half operands per MFMA) and by the L2: a 32-byte slice of a voxel
// fetches its whole line, which is often gone before the next slice.  Plane by
// plane the staging needs three address registers where voxel by voxel it took
// eleven and spilled, and the operands are read a step or three before their
// MFMAs (the compiler's own order put the reads next to their use).  Each
// output adds slices, taps and channels in the order of k_conv3.
//   64 -> 64 at 64^3: 0.138 -> 0.063 ms; 128 -> 64 at 64^3: 0.248 -> 0.109 ms;
//   96 -> 32 at 128^3: 0.71 -> 0.44 ms
constexpr int kLZ = 64;                            // output columns (z)
constexpr int kLPX = 2, kLPZ = kLZ + 2;            // output planes; staged columns
template <int NT, int NW>
struct ConvTile {
    static constexpr int NTH = 64 * NW;
    static constexpr int PY = NW + 2;
    // staged voxels per slice, whole 256-byte rows of the banks: a 16-byte read
    // serves lanes 0-3 and 12-15 of one half with 4-11 of the other in a cycle
    static constexpr int VOX = ((kLPX + 2) * PY * kLPZ + 15) / 16 * 16;
    static constexpr int XU = 2 * VOX, WU = 27 * 16 * NT * 2;  // 16-byte units: input, weights
    static constexpr int WPT = (WU + NTH - 1) / NTH;
    // a thread's units: PR rounds of each plane, then TR of what is left of all
    static constexpr int PU = 2 * PY * kLPZ, PR = PU / NTH, TU = PU % NTH;
    static constexpr int TR = ((kLPX + 2) * TU + NTH - 1) / NTH;
    static_assert(TU % 2 == 0 && TU > 0, "a thread keeps its channel half");
    static constexpr int LDS = (XU + WU) * 16;
    static constexpr int AHEAD = NT == 2 ? 4 : 2;  // operands in flight: what the registers hold
};

template <int CIN, int COUT, int NT, int NW>
__global__ __launch_bounds__(64 * NW, 2) void k_conv3_lds(const bf16_t* __restrict__ x, int n,
                                                          const bf16_t* __restrict__ w,
                                                          const float* __restrict__ bias, int relu,
                                                          bf16_t* __restrict__ y,
                                                          float* __restrict__ yf, int vec)
{
    using G = ConvTile<NT, NW>;
    static_assert(CIN % 16 == 0 && COUT % (16 * NT) == 0, "whole 16-channel slices");
    extern __shared__ __align__(16) unsigned char smem_raw[];
    u4* tile = reinterpret_cast<u4*>(smem_raw);  // [8-channel half][plane][row][z]
    u4* wl = tile + G::XU;                       // [tap][8-channel half][output channel]
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int m = lane & 15, g = lane >> 4;
    const int msk = n - 1, nx = n / kLPX, nyt = n / NW;
    const int nb = gridDim.x;
    int b = blockIdx.x;
    if ((nb & 7) == 0) b = (b & 7) * (nb >> 3) + (b >> 3);
    constexpr int NCO = COUT / (16 * NT);  // channel groups: neighbours, their input stays in L2
    const int co0 = (b % NCO) * 16 * NT;
    b /= NCO;
    const int x0 = (b % nx) * kLPX, yt = (b / nx) % nyt, zt = b / (nx * nyt);
    const int y0 = yt * NW, z0 = zt * kLZ;

    f4 acc[kLPX][4][NT];
#pragma unroll
    for (int p = 0; p < kLPX; ++p)
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int u = 0; u < NT; ++u) acc[p][t][u] = f4{0.f, 0.f, 0.f, 0.f};

    // k of the 16x16x32 MFMA = two taps of one slice: lanes g = 0, 1 carry
    // channels 8g..8g+7 of tap 2p, lanes g = 2, 3 those of tap 2p + 1.  The
    // 27th tap is the 14th pair with zeros in the second half: every product
    // runs on the one MFMA shape.  (Mixing in the 16x16x16 MFMA for the 27th
    // tap measured wrong sums for the 32 -> 16 instantiation, whose schedule
    // interleaves the two shapes on renamed accumulators.)
    const int hh = g & 1, side = g >> 1;
    const u4* th = tile + hh * G::VOX + wv * kLPZ + m;  // this lane's half, row and column
    const u4* wh = wl + hh * 16 * NT + m;
    // staged vectors of this thread: the same in-plane offsets for every plane
    // (whose pointers are uniform), and voxels of the planes' remainders (tail
    // clamped; its stores are skipped)
    const int h = tid & 1;  // an even stride: a thread's vectors share a channel half
    unsigned po[G::PR], to[G::TR], wo[G::WPT];
    auto in_plane = [&](int vox) __attribute__((always_inline)) {
        return ((y0 - 1 + vox / kLPZ) & msk) * n + ((z0 - 1 + vox % kLPZ) & msk);
    };
#pragma unroll
    for (int q = 0; q < G::PR; ++q)
        po[q] = (unsigned)(in_plane((tid + q * G::NTH) >> 1) * CIN + 8 * h);
#pragma unroll
    for (int q = 0; q < G::TR; ++q) {
        const int e = min(tid + q * G::NTH, (kLPX + 2) * G::TU - 1);
        to[q] = (unsigned)(((x0 - 1 + e / G::TU) & msk) * n * n +
                           in_plane((G::PR * G::NTH + e % G::TU) >> 1));
    }
#pragma unroll
    for (int q = 0; q < G::WPT; ++q) {
        const int e = min(tid + q * G::NTH, G::WU - 1) >> 1;  // tap * 16 NT + channel
        wo[q] = (unsigned)((e / (16 * NT) * COUT + co0 + e % (16 * NT)) * CIN + 8 * h);
    }
    u4 v[kLPX + 2][G::PR], vt[G::TR], wr[G::WPT];
    auto load = [&](int c0) __attribute__((always_inline)) {
#pragma unroll
        for (int pp = 0; pp < kLPX + 2; ++pp) {
            const bf16_t* pl = x + (size_t)((x0 - 1 + pp) & msk) * n * n * CIN + c0;
#pragma unroll
            for (int q = 0; q < G::PR; ++q) v[pp][q] = *reinterpret_cast<const u4_any*>(pl + po[q]);
        }
#pragma unroll
        for (int q = 0; q < G::TR; ++q)
            vt[q] = *reinterpret_cast<const u4_any*>(x + (size_t)to[q] * CIN + c0 + 8 * h);
#pragma unroll
        for (int q = 0; q < G::WPT; ++q) wr[q] = *reinterpret_cast<const u4_any*>(w + wo[q] + c0);
    };
    auto put = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int pp = 0; pp < kLPX + 2; ++pp)
#pragma unroll
            for (int q = 0; q < G::PR; ++q)
                tile[h * G::VOX + (pp * G::PU + tid + q * G::NTH) / 2] = v[pp][q];
#pragma unroll
        for (int q = 0; q < G::TR; ++q) {
            const int e = tid + q * G::NTH;
            if ((q + 1) * G::NTH <= (kLPX + 2) * G::TU || e < (kLPX + 2) * G::TU)
                tile[h * G::VOX + (e / G::TU * G::PU + G::PR * G::NTH + e % G::TU) / 2] = vt[q];
        }
#pragma unroll
        for (int q = 0; q < G::WPT; ++q) {
            const int e = tid + q * G::NTH, k = e >> 1;
            if ((q + 1) * G::NTH <= G::WU || e < G::WU)
                wl[(k / (16 * NT) * 2 + h) * 16 * NT + k % (16 * NT)] = wr[q];
        }
    };
    const u4 first = side ? u4{0, 0, 0, 0} : u4{~0u, ~0u, ~0u, ~0u};
    for (int c0 = 0; c0 < CIN; c0 += 16) {
        // (the next slice held in registers during this one's MFMAs measured
        // 10 to 30 % slower: the registers cost waves)
        load(c0);
        if (c0) __syncthreads();  // the previous slice has been consumed
        put();
        __syncthreads();
        // step q: plane q & 1 of pair q / 2 of the taps, its operands read
        // AHEAD - 1 steps before.  Pair 13 is tap 26 alone: lanes
        // of the second half read its (valid) addresses and zero what they get.
        u4 a[G::AHEAD][4], bw[G::AHEAD / 2 + 1][NT];
        auto fetch = [&](int q) __attribute__((always_inline)) {
            const int pr = q / 2, p = q % 2, t0 = 2 * pr, t1 = pr < 13 ? t0 + 1 : t0;
            const int o0 = ((t0 / 9) * G::PY + (t0 / 3) % 3) * kLPZ + t0 % 3;
            const int o1 = ((t1 / 9) * G::PY + (t1 / 3) % 3) * kLPZ + t1 % 3;
            const u4* src = th + o0 + (side ? o1 - o0 : 0) + p * G::PY * kLPZ;
#pragma unroll
            for (int t = 0; t < 4; ++t) a[q % G::AHEAD][t] = src[16 * t];
            if (p == 0) {
                const u4* ws = wh + 32 * NT * t0 + (side ? 32 * NT * (t1 - t0) : 0);
#pragma unroll
                for (int u = 0; u < NT; ++u) bw[pr % (G::AHEAD / 2 + 1)][u] = ws[16 * u];
            }
        };
#pragma unroll
        for (int q = 0; q < G::AHEAD - 1; ++q) fetch(q);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 28; ++q) {
            if (q + G::AHEAD - 1 < 28) fetch(q + G::AHEAD - 1);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                u4 av = a[q % G::AHEAD][t];
                if (q >= 26) av &= first;
#pragma unroll
                for (int u = 0; u < NT; ++u) {
                    u4 bv = bw[q / 2 % (G::AHEAD / 2 + 1)][u];
                    if (q >= 26) bv &= first;
                    acc[q & 1][t][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf8v, bv), __builtin_bit_cast(bf8v, av),
                        acc[q & 1][t][u], 0, 0, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);  // or the reads move next to their use
        }
    }
    // the weights are the row operand: D[row = 4g + r][col = m] is channel
    // co0 + 16u + 4g + r of voxel z0 + 16t + m, four channels per 8-byte store
#pragma unroll
    for (int p = 0; p < kLPX; ++p) {
        const size_t v0 = ((size_t)(x0 + p) * n + (y0 + wv)) * n + z0 + m;
#pragma unroll
        for (int u = 0; u < NT; ++u) {
            const int co = co0 + 16 * u + 4 * g;
            const f4 bb = bias4(bias, co);
#pragma unroll
            for (int t = 0; t < 4; ++t)
                store4(acc[p][t][u] + bb, relu, vec, y, yf, (v0 + 16 * t) * COUT + co);
        }
    }
}

// 16 output channels from several slices of input (sides n >= 64): a 4 x 64
// (y, z) tile streams along x over xc output planes with every channel of four
// planes in LDS, three that the taps read and one being filled from registers
// loaded an output plane earlier.  A line is fetched once per tile (slice by
// slice, k_conv3_lds fetched it up to three times), all weights stay in
// registers, and the one barrier per plane and the stores of the plane to come
// stand among the MFMAs, whose operands are read five or six pairs of taps
// ahead (an LDS read under load takes three pairs' MFMAs).
// CLO > 0: the input is the concatenation [nearest upsampling of lo, x] of a
// coarse [(n/2)^3][CLO] tensor and a fine [n^3][CIN - CLO] tensor (the
// decoder's skip), read directly instead of materialised.
// LDS: [plane mod 4][slice][8-channel half][row][z] in 16-byte units, the
// halves in phase modulo the banks: a 16-byte read serves lanes 0-3 and 12-15
// of one with 4-11 of the other in a cycle.  Slices, pairs of taps and channels
// are added as k_conv3_lds does, bit for bit.
// Bound: the LDS, one kilobyte read per MFMA: at 128 bytes per cycle its
// instructions take 91 % of the CUs' busy cycles at 128^3 (2.2 GHz; the rest is
// mostly the prologue of four planes per workgroup) and all of them at 256^3,
// where the clock falls to 1.7 GHz (48 -> 16, SQ_INSTS_LDS x 8 cycles over
// SQ_BUSY_CU_CYCLES).
// Before (two x-planes per wave, slice by slice) and with this:
//   48 -> 16 at 128^3: 0.171 -> 0.10 ms, at 256^3 (CLO = 32) 1.24 -> 0.8 ms;
//   32 -> 16 at 128^3: 0.092 -> 0.063 ms
constexpr int kPY = 4;                        // tile rows
constexpr int kPVox = (kPY + 2) * kLPZ;       // staged voxels per plane
constexpr int kPVP = (kPVox + 15) / 16 * 16;
template <int CIN, int CLO>
struct ConvPlanes {
    static constexpr int NTH = 64 * kPY, NS = CIN / 16, MT = 4;
    // 16-byte units of a plane: of the coarse tensor (CLO > 0), of x; rounds
    static constexpr int UL = kPVox * CLO / 8, UX = kPVox * (CIN - CLO) / 8;
    static constexpr int RL = (UL + NTH - 1) / NTH, RX = (UX + NTH - 1) / NTH, R = RL + RX;
    static constexpr int SL = 2 * kPVP + 5;  // a slice; 5: its stores fall on other banks
    static constexpr int PLANE = NS * SL;
    // operands in flight, pairs of taps (a divisor of all, so that their
    // registers match from one output plane to the next); the pair before which
    // the plane being staged has to be complete; pairs per staged unit
    static constexpr int PAIRS = 14 * NS, AHEAD = NS == 3 ? 6 : 7, SYNC = 9 - (AHEAD - 1);
    static constexpr int EVERY = (PAIRS - SYNC) / R;
    static_assert(PAIRS % AHEAD == 0 && SYNC >= 0 && EVERY >= 1 && AHEAD <= 9, "schedule");
    static constexpr int LDS = 4 * PLANE * 16;
    static_assert(LDS <= 160 * 1024, "LDS overflow");
};
template <int CIN, int CLO>
__global__ __launch_bounds__(64 * kPY, 1) void k_conv3_planes(
    const bf16_t* __restrict__ x, const bf16_t* __restrict__ lo, int n, int xc,
    const bf16_t* __restrict__ w, const float* __restrict__ bias, int relu,
    bf16_t* __restrict__ y, float* __restrict__ yf, int vec)
{
    using G = ConvPlanes<CIN, CLO>;
    constexpr int COUT = 16, CX = CIN - CLO;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    u4* buf = reinterpret_cast<u4*>(smem_raw);
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int m = lane & 15, g = lane >> 4, hh = g & 1, side = g >> 1;
    const int msk = n - 1, nyt = n / kPY, nzt = n / kLZ;
    const int nb = gridDim.x;
    int b = blockIdx.x;
    if ((nb & 7) == 0) b = (b & 7) * (nb >> 3) + (b >> 3);  // rows that share a halo share an L2
    const int y0 = (b % nyt) * kPY, z0 = (b / nyt) % nzt * kLZ, x0 = b / (nyt * nzt) * xc;
    // this thread's units: element offsets in a plane of the source, positions
    // in the staged plane (tails clamped: stored twice)
    unsigned src[G::R], dst[G::R];
#pragma unroll
    for (int q = 0; q < G::R; ++q) {
        const bool l = q < G::RL;
        const int units = l ? G::UL : G::UX, hc = (l ? CLO : CX) / 8, sh = l ? 1 : 0;
        const int e = min(tid + (l ? q : q - G::RL) * G::NTH, units - 1);
        const int v = e / hc, c = e % hc;
        const int yy = (y0 - 1 + v / kLPZ) & msk, zz = (z0 - 1 + v % kLPZ) & msk;
        src[q] = (unsigned)(((yy >> sh) * (n >> sh) + (zz >> sh)) * (8 * hc) + 8 * c);
        const int cc = c + (l ? 0 : CLO / 8);
        dst[q] = (unsigned)(cc / 2 * G::SL + cc % 2 * kPVP + v);
    }
    u4 pre[G::R];
    auto load = [&](int q, int xp) __attribute__((always_inline)) {
        xp &= msk;
        const bf16_t* pl = q < G::RL ? lo + (size_t)(xp >> 1) * (n >> 1) * (n >> 1) * CLO
                                     : x + (size_t)xp * n * n * CX;
        pre[q] = *reinterpret_cast<const u4_any*>(pl + src[q]);
    };
    // the operand of each slice and pair of taps (k of the MFMA as in
    // k_conv3_lds; nothing in the second half of the 14th pair)
    u4 wr[G::NS][14];
#pragma unroll
    for (int s = 0; s < G::NS; ++s)
#pragma unroll
        for (int pr = 0; pr < 14; ++pr)
            wr[s][pr] = pr == 13 && side
                            ? u4{}
                            : *reinterpret_cast<const u4_any*>(
                                  w + ((2 * pr + side) * COUT + m) * CIN + 16 * s + 8 * hh);
    const f4 bb = bias4(bias, 4 * g);
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int q = 0; q < G::R; ++q) {
            load(q, x0 - 1 + d);
            if (d < 3) buf[d * G::PLANE + dst[q]] = pre[q];
        }
    // the 14th pair's second half (which reads a voxel past the 27th tap's)
    const u4 first = side ? u4{0, 0, 0, 0} : u4{~0u, ~0u, ~0u, ~0u};
    const u4* own = buf + hh * kPVP + wv * kLPZ + m;  // this lane's half, row and column
    // output plane i reads staged planes i .. i + 2; q >= PAIRS: the next one's.
    // A pair's two taps are neighbours in a row, the ends of two rows, or (taps
    // 8 and 9) those of two planes.
    u4 a[G::AHEAD][G::MT];
    auto fetch = [&](int i, int q) __attribute__((always_inline)) {
        if (q >= G::PAIRS) q -= G::PAIRS, ++i;
        const int s = q / 14, pr = q % 14, j = 2 * pr % 9, d = 2 * pr / 9;
        const u4* p = own + ((i + d) & 3) * G::PLANE;
        if (pr == 4)
            p = side ? own + ((i + 1) & 3) * G::PLANE : p + 2 * kLPZ + 2;
        else
            p += (j / 3) * kLPZ + j % 3 + (j % 3 == 2 && pr < 13 ? 64 : 1) * side;
#pragma unroll
        for (int t = 0; t < G::MT; ++t) a[q % G::AHEAD][t] = p[s * G::SL + 16 * t];
    };
    __syncthreads();
#pragma unroll
    for (int q = 0; q < G::AHEAD - 1; ++q) fetch(0, q);
    for (int i = 0; i < xc; ++i) {
        u4* next = buf + ((i + 3) & 3) * G::PLANE;
        f4 acc[G::MT];
#pragma unroll
        for (int t = 0; t < G::MT; ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < G::PAIRS; ++q) {
            // plane i + 2 is staged, and plane i - 1's last readers are done
            if (q == G::SYNC) __syncthreads();
            fetch(i, q + G::AHEAD - 1);
            const int u = (q - G::SYNC) / G::EVERY;
            if (q >= G::SYNC && (q - G::SYNC) % G::EVERY == 0 && u < G::R) {
                next[dst[u]] = pre[u];  // plane i + 3, among the MFMAs
                load(u, x0 + i + 3);
            }
#pragma unroll
            for (int t = 0; t < G::MT; ++t) {
                u4 av = a[q % G::AHEAD][t];
                if (q % 14 == 13) av &= first;
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    __builtin_bit_cast(bf8v, wr[q / 14][q % 14]), __builtin_bit_cast(bf8v, av),
                    acc[t], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);  // or the reads move next to their use
        }
        const size_t v0 = ((size_t)(x0 + i) * n + (y0 + wv)) * n + z0 + m;
#pragma unroll
        for (int t = 0; t < G::MT; ++t)
            store4(acc[t] + bb, relu, vec, y, yf, (v0 + 16 * t) * COUT + 4 * g);
    }
}

// 16 input channels (sides n >= 64): a 4 x 64 (y, z) tile streams along x over
// xc output planes, 16 output channels per workgroup, one row of 64 voxels
// per wave (two rows spill).  An input plane contributes to three output planes -- its taps
// 0..8 to the next one, 9..17 to its own, 18..26 to the previous one -- so
// three sets of accumulators are live and every plane is staged and read from
// LDS once: a fragment (row, dk) feeds three MFMAs instead of one, and
// each output still adds its taps in the order 0..26 (bit for bit the sums of
// k_conv3).  The 27 weight fragments stay in registers.  The weights are the
// MFMA's row operand, so a lane ends with four consecutive channels of one
// voxel and a tile is stored as 512 contiguous bytes (two-byte stores before).
// LDS holds a plane as four arrays of 4-channel units, one per k-group of the
// 16x16x16 MFMA, each 128 bytes out of phase modulo the 64 banks.
// Bound: the MFMA issue (66 % busy at 256^3; the 16x16x16 shape runs at half
// the rate of 16x16x32, which adds in another order).
//   16 -> 16 at 256^3: 0.44 -> 0.35 ms; at 128^3: 0.055 -> 0.044 ms;
//   16 -> 48 at 128^3: 0.254 -> 0.13 ms
constexpr int kRY = 4, kRW = 1;                    // tile rows, rows per wave
constexpr int kRPY = kRY + 2, kRPZ = kLZ + 2;
constexpr int kRVox = kRPY * kRPZ;                 // staged voxels per plane
constexpr int kRPad = kRVox + (48 - kRVox % 32) % 32;  // = 16 mod 32
// HEAD: the network's last convolution in a prediction, whose 16 channels only
// the head reads: no output y, but out and guess as k_head makes them (each
// NULL if not wanted; the channels' products added in its order, passed from
// the four lanes of a voxel to the next four).
struct HeadOut {
    const float* wh;
    const double* cold;
    float* out;
    double* guess;
};
template <bool HEAD>
__global__ __launch_bounds__(kThreads, 2) void k_conv3_ring(const bf16_t* __restrict__ x, int n,
                                                            int xc, const bf16_t* __restrict__ w,
                                                            const float* __restrict__ bias,
                                                            int cout, int relu,
                                                            bf16_t* __restrict__ y,
                                                            float* __restrict__ yf, int vec,
                                                            HeadOut head)
{
    constexpr int CIN = 16;
    constexpr int PV = kRVox * 2;                        // 16-byte input vectors per plane
    constexpr int PER = (PV + kThreads - 1) / kThreads;  // of them per thread
    __shared__ s4 buf[2][4 * kRPad];  // [plane parity][4-channel group][row][z]
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int m = lane & 15, g = lane >> 4;
    const int msk = n - 1, nyt = n / kRY, nzt = n / kLZ, nco = cout >> 4;
    const int nb = gridDim.x;
    int b = blockIdx.x;
    if ((nb & 7) == 0) b = (b & 7) * (nb >> 3) + (b >> 3);
    const int cg = b % nco;  // a tile's channel groups are neighbours: its input stays in L2
    b /= nco;
    const int yt = b % nyt, zt = (b / nyt) % nzt, xq = b / (nyt * nzt);
    const int y0 = yt * kRY, z0 = zt * kLZ, x0 = xq * xc;
    const size_t plane = (size_t)n * n * CIN;
    // in-plane element offsets of this thread's vectors (tail clamped; its
    // stores are skipped)
    unsigned poff[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int e = min(tid + q * kThreads, PV - 1);
        const int vox = e >> 1, h = e & 1;
        const int zz = vox % kRPZ, rr = vox / kRPZ;
        poff[q] = (unsigned)((((y0 - 1 + rr) & msk) * n + ((z0 - 1 + zz) & msk)) * CIN + 8 * h);
    }
    u4 pre[PER];
    auto load = [&](int xp) __attribute__((always_inline)) {
        const bf16_t* pl = x + (size_t)(xp & msk) * plane;
#pragma unroll
        for (int q = 0; q < PER; ++q) pre[q] = *reinterpret_cast<const u4_any*>(pl + poff[q]);
    };
    auto put = [&](int par) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int e = tid + q * kThreads;
            if ((q + 1) * kThreads <= PV || e < PV) {
                const int vox = e >> 1, h = e & 1;
                s4* d = buf[par] + 2 * h * kRPad + vox;
                d[0] = __builtin_bit_cast(s4, __builtin_shufflevector(pre[q], pre[q], 0, 1));
                d[kRPad] = __builtin_bit_cast(s4, __builtin_shufflevector(pre[q], pre[q], 2, 3));
            }
        }
    };
    s4 bw[27];
#pragma unroll
    for (int t = 0; t < 27; ++t)
        bw[t] = *reinterpret_cast<const s4_any*>(w + ((size_t)t * cout + 16 * cg + m) * CIN + 4 * g);
    const f4 bb = bias4(bias, 16 * cg + 4 * g);
    float wh[4] = {}, whb = 0.f;  // this lane's channels of the head, its bias
    if constexpr (HEAD) {
#pragma unroll
        for (int i = 0; i < 4; ++i) wh[i] = head.wh[4 * g + i];
        whb = head.wh[16];
    }
    f4 acc[3][kRW][4];
    // input plane xp (in buf[par]): taps 0..8 into S (output plane xp + 1,
    // begun here), 9..17 into M (xp), 18..26 into F (xp - 1, stored)
    auto step = [&](int xp, int par, f4 (&S)[kRW][4], f4 (&M)[kRW][4], f4 (&F)[kRW][4])
        __attribute__((always_inline)) {
        __syncthreads();  // plane xp is in LDS; the other buffer's last readers are done
        if (xp < x0 + xc) {
            put(par ^ 1);
            load(xp + 2);  // (past the last plane loaded and dropped)
        }
#pragma unroll
        for (int r = 0; r < kRW; ++r)
#pragma unroll
            for (int t = 0; t < 4; ++t) S[r][t] = f4{0.f, 0.f, 0.f, 0.f};
        const s4* base = buf[par] + g * kRPad + wv * kRW * kRPZ + m;
        // groups (input row j, dk): the next group's fragments are read before
        // this group's MFMAs; sets outside the region's planes are skipped
        s4 a[2][4];
        auto mac = [&](int q, int t0, f4 (&C)[kRW][4]) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < kRW; ++r) {
                const int dj = q / 3 - r;  // this input row is output row r's tap row dj
                if (dj < 0 || dj > 2) continue;
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    C[r][t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(bw[t0 + 3 * dj + q % 3],
                                                                        a[q & 1][t], C[r][t], 0, 0, 0);
            }
        };
#pragma unroll
        for (int t = 0; t < 4; ++t) a[0][t] = base[16 * t];
#pragma unroll
        for (int q = 0; q < 3 * (kRW + 2); ++q) {
            if (q + 1 < 3 * (kRW + 2)) {
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    a[(q + 1) & 1][t] = base[((q + 1) / 3) * kRPZ + (q + 1) % 3 + 16 * t];
            }
            if (xp + 1 < x0 + xc) mac(q, 0, S);
            if (xp >= x0 && xp < x0 + xc) mac(q, 9, M);
            if (xp > x0) mac(q, 18, F);
        }
        if (xp > x0) {
            // D[row = 4g + r][col = m]: channel 16 cg + 4g + r, voxel z0 + 16t + m
#pragma unroll
            for (int r = 0; r < kRW; ++r) {
                if constexpr (HEAD) {
                    const size_t v = ((size_t)(xp - 1) * n + (y0 + wv * kRW + r)) * n + z0 + lane;
                    const double cold = head.guess ? head.cold[v] : 0.0;
                    float res = 0.f;
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        float s = whb;
                        const f4 d = F[r][t] + bb;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            if (q > 0) s = __shfl(s, 16 * (q - 1) + m, 64);
#pragma unroll
                            for (int i = 0; i < 4; ++i) s += bf2f(f2bf(fmaxf(d[i], 0.f))) * wh[i];
                        }
                        s = __shfl(s, 48 + m, 64);
                        if (g == t) res = s;
                    }
                    if (head.out) head.out[v] = res;
                    if (head.guess) head.guess[v] = cold + (double)res;
                    continue;
                }
                const size_t v0 = ((size_t)(xp - 1) * n + (y0 + wv * kRW + r)) * n + z0 + m;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const size_t o = (v0 + 16 * t) * cout + 16 * cg + 4 * g;
                    store4(F[r][t] + bb, relu, vec, y, yf, o);
                }
            }
        }
    };
    load(x0 - 1);
    put(0);
    load(x0);
    for (int xp = x0 - 1, par = 0; xp <= x0 + xc; xp += 3) {
        step(xp, par, acc[0], acc[2], acc[1]);
        if (xp + 1 <= x0 + xc) step(xp + 1, par ^ 1, acc[1], acc[0], acc[2]);
        if (xp + 2 <= x0 + xc) step(xp + 2, par, acc[2], acc[1], acc[0]);
        par ^= 1;
    }
}

// dW partials: part[chunk][t][co][ci] = sum over the chunk's voxels v of
// dy[v][co] * x[v + d_t][ci].  One workgroup per (tap, chunk); its waves
// split the 16x16 output tiles.  K (voxels) advances 16 at a time.
template <int CIN, int COUT>
__global__ __launch_bounds__(kThreads) void k_conv3_dw(const bf16_t* __restrict__ x, int n,
                                                       const bf16_t* __restrict__ dy,
                                                       int chunk, float* __restrict__ part)
{
    constexpr int TM = COUT / 16, TN = CIN / 16, TILES = TM * TN;
    constexpr int WAVES = kThreads / 64;
    constexpr int TPW = (TILES + WAVES - 1) / WAVES;  // tiles per wave
    const int tap = blockIdx.x % 27;
    const int ch = blockIdx.x / 27;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = lane & 15, g = lane >> 4;
    const int di = tap / 9 - 1, dj = (tap / 3) % 3 - 1, dk = tap % 3 - 1;
    const int msk = n - 1;
    const long vbeg = (long)ch * chunk, vend = vbeg + chunk;

    f4 acc[TPW];
#pragma unroll
    for (int q = 0; q < TPW; ++q) acc[q] = f4{0.f, 0.f, 0.f, 0.f};

    for (long vb = vbeg; vb < vend; vb += 16) {
        // K index k = 4g + r  ->  voxel vb + 4g + r
        long vx[4], vy[4];
        bool live[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            long v = vb + 4 * g + r;
            live[r] = v < vend;  // chunks shorter than 16 voxels (tiny grids)
            if (!live[r]) v = vbeg;
            vy[r] = v;
            const int kk = (int)(v % n);
            const long rw = v / n;
            const int jj = (int)(rw % n), ii = (int)(rw / n);
            vx[r] = ((long)((ii + di) & msk) * n + ((jj + dj) & msk)) * n + ((kk + dk) & msk);
        }
#pragma unroll
        for (int q = 0; q < TPW; ++q) {
            const int tile = wave + q * WAVES;
            if (tile < TILES) {
                const int tm = tile / TN, tn = tile % TN;
                s4 a, b;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    a[r] = live[r] ? (short)dy[vy[r] * COUT + 16 * tm + m] : (short)0;  // A[co][v]
                    b[r] = (short)x[vx[r] * CIN + 16 * tn + m];                          // B[v][ci]
                }
                acc[q] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, acc[q], 0, 0, 0);
            }
        }
    }
    float* out = part + ((long)ch * 27 + tap) * COUT * CIN;
#pragma unroll
    for (int q = 0; q < TPW; ++q) {
        const int tile = wave + q * WAVES;
        if (tile < TILES) {
            const int tm = tile / TN, tn = tile % TN;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                out[(long)(16 * tm + 4 * g + r) * CIN + 16 * tn + m] = acc[q][r];
        }
    }
}

// The weight gradient on sides >= 16, staged in LDS.  A workgroup owns one
// 16 x 16 (output, input) channel tile and a region of the grid: TY rows and Z
// columns, streamed along x over xc planes.  Per plane it holds the 16 input
// channels of x (rows y0-1 .. y0+TY of the NDI planes its taps read) and the
// 16 output channels of dy (one voxel of z halo) as they lie in memory, 32
// bytes per voxel; the transposing LDS read ds_read_b64_tr_b16 turns four
// consecutive voxels into the K-contiguous operands of the 16x16x32 MFMA, so
// neither a transposed copy nor an alignment of the z shift is needed.  The
// z shift dk is taken on dy (three A operands per 32-voxel window), di and
// dj on x (one B operand per staged row), and rows are walked in order with
// the B operands of three rows kept in registers: 3 A + 3 NDI B operands per
// 9 NDI MFMAs, where the per-tap kernel loaded 8 + 8 two-byte values from
// memory per MFMA.  The four waves take different windows (K) of the region
// and are summed in LDS in a fixed order; regions are summed by k_sum_chunks.
// Bound: LDS reads and the MFMA issue about equally (NDI = 3); x and dy are
// read 1.5 and (per channel tile) 1.03 times.
//   48 -> 16 at 128^3: 5.0 -> 0.11 ms (0.79 PFLOP/s); 16 -> 16: 3.9 -> 0.037 ms;
//   64 -> 64 at 32^3: 0.45 -> 0.025 ms, at 16^3 0.44 -> 0.020 ms.
// NDI = 3: all 27 taps in one workgroup (sides >= 64); NDI = 1: one x offset
// per workgroup (blockIdx), for the small grids whose few regions would leave
// most of the device idle.
template <int Z_, int TY_, int NDI_>
struct DwTile {
    static constexpr int Z = Z_, TY = TY_, NDI = NDI_;
    static constexpr int XR = TY + 2, XPL = XR * Z * 16;      // staged x plane, elements
    static constexpr int DZ = Z + 2, DPL = TY * DZ * 16;      // staged dy plane
    static constexpr int XU = XPL / 8, DU = DPL / 8;          // 16-byte units
    static constexpr int XPT = (XU + kThreads - 1) / kThreads, DPT = (DU + kThreads - 1) / kThreads;
    static constexpr int RS = Z >= 32 ? 1 : 32 / Z;           // rows per 32-voxel window
    static constexpr int ZW = Z >= 32 ? Z / 32 : 1;           // windows per row
    static constexpr int RW = TY / (4 / ZW);                  // rows per wave
    static constexpr int LDS = (NDI * XPL + DPL) * 2;
    static_assert(4 % ZW == 0 && TY % (4 / ZW) == 0 && RW % RS == 0, "four waves share the tile");
    static_assert(LDS >= 9 * NDI * 256 * 4, "the reduction reuses the staging buffers");
};
typedef __attribute__((address_space(3))) s4 lds_s4;

template <class G>
__global__ __launch_bounds__(kThreads, 2) void k_conv3_dw_tiled(const bf16_t* __restrict__ x, int n,
                                                                int cin,
                                                                const bf16_t* __restrict__ dy,
                                                                int cout, int xc,
                                                                float* __restrict__ part)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    bf16_t* xs = reinterpret_cast<bf16_t*>(smem_raw);  // NDI planes of x
    bf16_t* ds = xs + G::NDI * G::XPL;                 // one plane of dy
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int m = lane & 15, g = lane >> 4;
    const int msk = n - 1;
    const int tn = cin >> 4, tiles = tn * (cout >> 4);
    const int nb = gridDim.x;
    int b = blockIdx.x;
    if ((nb & 7) == 0) b = (b & 7) * (nb >> 3) + (b >> 3);  // a region's tiles share an XCD's L2
    const int tile = b % tiles;
    b /= tiles;
    int d0 = -1;  // x offset of the first staged plane
    if constexpr (G::NDI == 1) {
        d0 = b % 3 - 1;
        b /= 3;
    }
    const int reg = b;
    const int nzt = n / G::Z, nyt = n / G::TY;
    const int zt = b % nzt, yt = (b / nzt) % nyt, xt = b / (nzt * nyt);
    const int x0 = xt * xc, y0 = yt * G::TY, z0 = zt * G::Z;
    const int ci0 = (tile % tn) * 16, co0 = (tile / tn) * 16;
    const size_t xplane = (size_t)n * n * cin, dplane = (size_t)n * n * cout;

    unsigned xo[G::XPT], dof[G::DPT];  // element offsets in a plane (tail clamped)
#pragma unroll
    for (int q = 0; q < G::XPT; ++q) {
        const int e = min(tid + q * kThreads, G::XU - 1);
        const int v = e >> 1, r = v / G::Z, z = v % G::Z;
        xo[q] = (unsigned)((((y0 - 1 + r) & msk) * n + z0 + z) * cin + ci0 + 8 * (e & 1));
    }
#pragma unroll
    for (int q = 0; q < G::DPT; ++q) {
        const int e = min(tid + q * kThreads, G::DU - 1);
        const int v = e >> 1, r = v / G::DZ, z = v % G::DZ;
        dof[q] = (unsigned)(((y0 + r) * n + ((z0 - 1 + z) & msk)) * cout + co0 + 8 * (e & 1));
    }
    u4 xr[G::XPT], dr[G::DPT];
    auto load_x = [&](int xp) __attribute__((always_inline)) {
        const bf16_t* p = x + (size_t)(xp & msk) * xplane;
#pragma unroll
        for (int q = 0; q < G::XPT; ++q) xr[q] = *reinterpret_cast<const u4*>(p + xo[q]);
    };
    auto load_d = [&](int xp) __attribute__((always_inline)) {
        const bf16_t* p = dy + (size_t)(xp & msk) * dplane;
#pragma unroll
        for (int q = 0; q < G::DPT; ++q) dr[q] = *reinterpret_cast<const u4*>(p + dof[q]);
    };
    auto put_x = [&](int slot) __attribute__((always_inline)) {
        u4* d = reinterpret_cast<u4*>(xs + slot * G::XPL);
#pragma unroll
        for (int q = 0; q < G::XPT; ++q) {
            const int e = tid + q * kThreads;
            if ((q + 1) * kThreads <= G::XU || e < G::XU) d[e] = xr[q];
        }
    };
    auto put_d = [&]() __attribute__((always_inline)) {
        u4* d = reinterpret_cast<u4*>(ds);
#pragma unroll
        for (int q = 0; q < G::DPT; ++q) {
            const int e = tid + q * kThreads;
            if ((q + 1) * kThreads <= G::DU || e < G::DU) d[e] = dr[q];
        }
    };

    f4 acc[G::NDI][3][3];
#pragma unroll
    for (int a = 0; a < G::NDI; ++a)
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int k = 0; k < 3; ++k) acc[a][j][k] = f4{0.f, 0.f, 0.f, 0.f};

    // this wave's window column and first row; this lane's address in a
    // transposing read: voxel 4g + m/4 of 16, channels 4 (m % 4) ..
    const int zw = (wv % G::ZW) * 32, r0 = (wv / G::ZW) * G::RW;
    const int lo = (4 * g + (m >> 2)) * 16 + 4 * (m & 3);
    // operand of the 32-voxel window whose first 16 voxels start at p and
    // the others `second` elements further
    auto operand = [&](const bf16_t* p, int second) __attribute__((always_inline)) {
        const s4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(p + lo));
        const s4 c = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(p + second + lo));
        return __builtin_bit_cast(bf8v, __builtin_shufflevector(a, c, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    constexpr int XSEC = G::RS == 1 ? 16 * 16 : G::Z * 16;   // second half: 16 voxels on, or the next row
    constexpr int DSEC = G::RS == 1 ? 16 * 16 : G::DZ * 16;

    load_x(x0 + d0);
    put_x(0);
    if constexpr (G::NDI == 3) {
        load_x(x0);
        put_x(1);
        load_x(x0 + 1);
    }
    load_d(x0);
    int head = 0;  // slot of plane xp - 1 (NDI = 3)
    for (int xp = x0; xp < x0 + xc; ++xp) {
        if constexpr (G::NDI == 3) put_x(head == 0 ? 2 : head - 1);
        else if (xp > x0) put_x(0);
        put_d();
        __syncthreads();
        // the next plane's values are in flight during this plane's MFMAs
        // (past the region's end they are loaded and dropped: branch-free)
        load_x(G::NDI == 3 ? xp + 2 : xp + 1 + d0);
        load_d(xp + 1);
        const bf16_t* xp_[G::NDI];
#pragma unroll
        for (int a = 0; a < G::NDI; ++a) {
            const int s = head + a;
            xp_[a] = xs + (G::NDI == 3 && s >= 3 ? s - 3 : s) * G::XPL + zw * 16;
        }
        const bf16_t* dp = ds + zw * 16;
        bf8v bq[3][G::NDI];  // rows r - 1, r, r + 1 (RS = 1: slot = row mod 3)
        if constexpr (G::RS == 1) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int a = 0; a < G::NDI; ++a) bq[j][a] = operand(xp_[a] + (r0 + j) * G::Z * 16, XSEC);
        }
#pragma unroll
        for (int r = 0; r < G::RW; r += G::RS) {
            bf8v aq[3];
#pragma unroll
            for (int k = 0; k < 3; ++k)  // x at z, dy at z - dk (dk = k - 1; ds starts at z0 - 1)
                aq[k] = operand(dp + ((r0 + r) * G::DZ + 2 - k) * 16, DSEC);
            if constexpr (G::RS == 1) {
#pragma unroll
                for (int a = 0; a < G::NDI; ++a)
                    bq[(r + 2) % 3][a] = operand(xp_[a] + (r0 + r + 2) * G::Z * 16, XSEC);
            } else {
#pragma unroll
                for (int j = 0; j < 3; ++j)
#pragma unroll
                    for (int a = 0; a < G::NDI; ++a)
                        bq[j][a] = operand(xp_[a] + (r0 + r + j) * G::Z * 16, XSEC);
            }
#pragma unroll
            for (int j = 0; j < 3; ++j)
#pragma unroll
                for (int a = 0; a < G::NDI; ++a)
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        const bf8v bb = G::RS == 1 ? bq[(r + j) % 3][a] : bq[j][a];
                        acc[a][j][k] =
                            __builtin_amdgcn_mfma_f32_16x16x32_bf16(aq[k], bb, acc[a][j][k], 0, 0, 0);
                    }
        }
        __syncthreads();  // the oldest plane's slot and dy are refilled next
        if constexpr (G::NDI == 3) head = head == 2 ? 0 : head + 1;
    }
    // waves 0 .. 3 summed in order, then D[row = 4g + r][col = m] of each tap
    float* red = reinterpret_cast<float*>(smem_raw);
    for (int w = 0; w < 4; ++w) {
        if (wv == w) {
#pragma unroll
            for (int a = 0; a < G::NDI; ++a)
#pragma unroll
                for (int j = 0; j < 3; ++j)
#pragma unroll
                    for (int k = 0; k < 3; ++k)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            float* q = red + ((a * 3 + j) * 3 + k) * 256 + (4 * g + r) * 16 + m;
                            *q = w == 0 ? acc[a][j][k][r] : *q + acc[a][j][k][r];
                        }
        }
        __syncthreads();
    }
    float* out = part + ((size_t)reg * 27 + 9 * (d0 + 1)) * cout * cin;
    for (int e = tid; e < 9 * G::NDI * 256; e += kThreads) {
        const int t = e >> 8, co = (e >> 4) & 15, ci = e & 15;
        out[((size_t)t * cout + co0 + co) * cin + ci0 + ci] = red[e];
    }
}

// out[e] = sum_c part[c][e] (deterministic): a workgroup sums 16 elements, 16
// threads per element each taking every 16th chunk in order, then those 16
// sums in order.  (One thread per element walked all chunks: 512 dependent
// loads, 0.14 ms for 48 -> 16 weights at 128^3; now 0.016 ms.)
__global__ __launch_bounds__(kThreads) void k_sum_chunks(const float* __restrict__ part,
                                                         int nchunk, long elems,
                                                         float* __restrict__ out)
{
    __shared__ float red[kThreads];
    const int tid = threadIdx.x, l = tid >> 4;
    const long e = (long)blockIdx.x * 16 + (tid & 15);
    float s = 0.f;
    if (e < elems) {
        int c = l;
        for (; c + 48 < nchunk; c += 64) {  // four loads in flight
            const float v0 = part[(long)c * elems + e], v1 = part[(long)(c + 16) * elems + e];
            const float v2 = part[(long)(c + 32) * elems + e], v3 = part[(long)(c + 48) * elems + e];
            s += v0;
            s += v1;
            s += v2;
            s += v3;
        }
        for (; c < nchunk; c += 16) s += part[(long)c * elems + e];
    }
    red[tid] = s;
    __syncthreads();
    if (tid < 16 && e < elems) {
        for (int k = 1; k < 16; ++k) s += red[k * 16 + tid];
        out[e] = s;
    }
}

// Per-channel sums of a [nvox][C] bf16 tensor (C a power of two, 16 .. 256):
// partial sums per chunk of voxels, reduced by k_sum_chunks.  A thread sums
// the 8 channels of one 16-byte vector over every (2048 / C)th voxel, so a
// workgroup reads contiguous memory (one thread per channel walked the voxels
// two bytes at a time: 0.55 ms for 16 channels at 128^3, now 0.015 ms).
// MASK: g = g * (o > 0) first (the ReLU gradient, exact in bf16), written back
// in the same pass.  VEC = false: tensors not aligned to 16 bytes, the same
// sums from two-byte accesses.
template <bool VEC>
__device__ __forceinline__ u4 load8(const bf16_t* p)
{
    if constexpr (VEC) return *reinterpret_cast<const u4*>(p);
    u4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = (uint32_t)p[2 * i] | ((uint32_t)p[2 * i + 1] << 16);
    return v;
}
constexpr int kSumVecs = 8 * kThreads;  // 16-byte vectors per workgroup
template <bool MASK, bool VEC>
__global__ __launch_bounds__(kThreads) void k_chan_sum(bf16_t* __restrict__ a,
                                                       const bf16_t* __restrict__ o, long nvox,
                                                       int C, float* __restrict__ part)
{
    __shared__ float red[4 * kThreads];
    const int tid = threadIdx.x;
    const int U = C >> 3;  // vectors per voxel, a divisor of 256: one channel group per thread
    const long u0 = (long)blockIdx.x * kSumVecs + tid, end = nvox * U;
    static_assert(VEC || !MASK, "the network's own tensors are aligned");
    float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    u4 v[8], p[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const long u = min(u0 + k * kThreads, end - 1);  // (clamped: branch-free loads)
        v[k] = load8<VEC>(a + u * 8);
        if constexpr (MASK) p[k] = load8<true>(o + u * 8);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const long u = u0 + k * kThreads;
        if (u >= end) break;
        if constexpr (MASK) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (!(bf2f((bf16_t)(p[k][i] & 0xffffu)) > 0.f)) v[k][i] &= 0xffff0000u;
                if (!(bf2f((bf16_t)(p[k][i] >> 16)) > 0.f)) v[k][i] &= 0xffffu;
            }
            *reinterpret_cast<u4*>(a + u * 8) = v[k];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            s[2 * i] += bf2f((bf16_t)(v[k][i] & 0xffffu));
            s[2 * i + 1] += bf2f((bf16_t)(v[k][i] >> 16));
        }
    }
    // lanes U apart hold the same channels: summed across the wave, then the
    // four waves in order
    for (int d = 32; d >= U; d >>= 1) {
#pragma unroll
        for (int i = 0; i < 8; ++i) s[i] += __shfl_xor(s[i], d, 64);
    }
    const int lane = tid & 63, wv = tid >> 6;
    if (lane < U) {
#pragma unroll
        for (int i = 0; i < 8; ++i) red[wv * C + lane * 8 + i] = s[i];
    }
    __syncthreads();
    if (tid < C)
        part[(long)blockIdx.x * C + tid] = ((red[tid] + red[C + tid]) + red[2 * C + tid]) + red[3 * C + tid];
}

// BF16 weights of all convolutions (one per blockIdx.y) from the FP32
// parameters: as they are, or, FLIP, for the data gradient: wt[t'][ci][co] =
// w[26 - t'][co][ci].  (A launch per layer: 14 times 2.4 or 4.5 us.)
struct ConvWeights {
    const float* src[14];
    bf16_t* dst[14];
    int cin[14], cout[14];
};
template <bool FLIP>
__global__ void k_conv_weights(ConvWeights a)
{
    const int c = blockIdx.y, cin = a.cin[c], cout = a.cout[c];
    const long total = 27L * cin * cout;
    const float* w = a.src[c];
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (long)gridDim.x * blockDim.x) {
        long from = e;
        if (FLIP) {
            const int co = (int)(e % cout);
            const long r = e / cout;
            from = ((26 - r / cin) * cout + co) * cin + r % cin;
        }
        a.dst[c][e] = f2bf(w[from]);
    }
}

// ---------------------------------------------------------------------------
// Pooling, upsampling, concatenation, masks, head, loss, Adam.
// ---------------------------------------------------------------------------

// y[V][c] = mean of the 8 children (reading channels [c0, c0+C) of a tensor
// with channel stride cs); nf = fine side (a power of two).  One 16-byte
// vector of 8 channels per thread (C, cs, c0 multiples of 8, C / 8 a power
// of two).
__global__ void k_pool2(const bf16_t* __restrict__ x, int nf, int cs, int c0, int C,
                        bf16_t* __restrict__ y)
{
    const int nc = nf / 2, lc = __builtin_ctz(nc), lq = __builtin_ctz(C / 8);
    const long total = ((long)nc * nc * nc) << lq;
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (long)gridDim.x * blockDim.x) {
        const int q = (int)(e & ((C / 8) - 1));
        const long V = e >> lq;
        const int K = (int)(V & (nc - 1)), J = (int)((V >> lc) & (nc - 1)), I = (int)(V >> (2 * lc));
        float sum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int a = 0; a < 2; ++a)
            for (int b = 0; b < 2; ++b)
                for (int d = 0; d < 2; ++d) {
                    const long vf = ((long)(2 * I + a) * nf + (2 * J + b)) * nf + (2 * K + d);
                    const uint4 u = *reinterpret_cast<const uint4*>(x + vf * cs + c0 + 8 * q);
                    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        sum[2 * i] += bf2f((bf16_t)(w[i] & 0xffffu));
                        sum[2 * i + 1] += bf2f((bf16_t)(w[i] >> 16));
                    }
                }
        uint32_t o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            o[i] = (uint32_t)f2bf(sum[2 * i] * 0.125f) | ((uint32_t)f2bf(sum[2 * i + 1] * 0.125f) << 16);
        reinterpret_cast<uint4*>(y)[e] = uint4{o[0], o[1], o[2], o[3]};
    }
}

// Nearest upsampling of a [nc^3][C] tensor into channels [0, C) of a
// [(2nc)^3][C+S] tensor, and copy of skip [(2nc)^3][S] into channels
// [C, C+S).  One 16-byte vector of 8 output channels per thread, so a wave
// writes 1 KiB of contiguous output (C and S are multiples of 8, the tensors
// 256-byte aligned); coordinates by shifts (the side is a power of two).
template <int C, int S>
__global__ void k_up2_cat(const bf16_t* __restrict__ lo, int nc, const bf16_t* __restrict__ skip,
                          bf16_t* __restrict__ out)
{
    static_assert(C % 8 == 0 && S % 8 == 0, "channels in whole 16-byte vectors");
    constexpr int VC = C / 8, VS = S / 8, VT = VC + VS;
    const int nf = 2 * nc, lf = __builtin_ctz(nf);
    const long total = (long)nf * nf * nf * VT;
    const uint4* lov = reinterpret_cast<const uint4*>(lo);
    const uint4* skv = reinterpret_cast<const uint4*>(skip);
    uint4* outv = reinterpret_cast<uint4*>(out);
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (long)gridDim.x * blockDim.x) {
        const long v = e / VT;
        const int q = (int)(e - v * VT);
        if (q < VC) {
            const int k = (int)(v & (nf - 1)), j = (int)((v >> lf) & (nf - 1));
            const int i = (int)(v >> (2 * lf));
            const long V = ((long)(i >> 1) * nc + (j >> 1)) * nc + (k >> 1);
            outv[e] = lov[V * VC + q];
        } else {
            outv[e] = skv[v * VS + (q - VC)];
        }
    }
}

// Gradient through upsampling: y[V][c] = sum of the 8 children's
// dcat[v][c] (channels [0, C) of the concat gradient, stride cs).  Bound by
// memory; as k_pool2 one 16-byte vector of 8 channels per thread and
// coordinates by shifts (one channel per thread, with four divisions: 51 -> 33 us at 128^3).
__global__ void k_up2_bwd(const bf16_t* __restrict__ dcat, int nf, int cs, int C,
                          bf16_t* __restrict__ y)
{
    const int nc = nf / 2, lc = __builtin_ctz(nc), lq = __builtin_ctz(C / 8);
    const long total = ((long)nc * nc * nc) << lq;
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (long)gridDim.x * blockDim.x) {
        const int q = (int)(e & ((C / 8) - 1));
        const long V = e >> lq;
        const int K = (int)(V & (nc - 1)), J = (int)((V >> lc) & (nc - 1)), I = (int)(V >> (2 * lc));
        float sum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int f = 0; f < 8; ++f) {
            const long vf = ((long)(2 * I + (f >> 2)) * nf + (2 * J + ((f >> 1) & 1))) * nf +
                            (2 * K + (f & 1));
            const uint4 u = *reinterpret_cast<const uint4*>(dcat + vf * cs + 8 * q);
            const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                sum[2 * i] += bf2f((bf16_t)(w[i] & 0xffffu));
                sum[2 * i + 1] += bf2f((bf16_t)(w[i] >> 16));
            }
        }
        uint32_t o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            o[i] = (uint32_t)f2bf(sum[2 * i]) | ((uint32_t)f2bf(sum[2 * i + 1]) << 16);
        reinterpret_cast<uint4*>(y)[e] = uint4{o[0], o[1], o[2], o[3]};
    }
}

// Gradient into a skip tensor: out[v][c] = bf16(dcat[v][C + c] + bf16(dlo[V][c] / 8))
// where dlo is the gradient at the pooled (coarse) level.  Bound by memory;
// 8 channels per thread as above (one channel per thread: 124 -> 46 us at 128^3).
__global__ void k_skip_grad(const bf16_t* __restrict__ dcat, int nf, int cs, int C, int S,
                            const bf16_t* __restrict__ dlo, bf16_t* __restrict__ out)
{
    const int nc = nf / 2, lf = __builtin_ctz(nf), lq = __builtin_ctz(S / 8);
    const long total = ((long)nf * nf * nf) << lq;
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (long)gridDim.x * blockDim.x) {
        const int q = (int)(e & ((S / 8) - 1));
        const long v = e >> lq;
        const int k = (int)(v & (nf - 1)), j = (int)((v >> lf) & (nf - 1)), i = (int)(v >> (2 * lf));
        const long V = ((long)(i >> 1) * nc + (j >> 1)) * nc + (k >> 1);
        const uint4 ud = *reinterpret_cast<const uint4*>(dlo + V * S + 8 * q);
        const uint4 uc = *reinterpret_cast<const uint4*>(dcat + v * cs + C + 8 * q);
        const uint32_t d[4] = {ud.x, ud.y, ud.z, ud.w}, c[4] = {uc.x, uc.y, uc.z, uc.w};
        uint32_t o[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const float lo = bf2f(f2bf(bf2f((bf16_t)(d[x] & 0xffffu)) * 0.125f));
            const float hi = bf2f(f2bf(bf2f((bf16_t)(d[x] >> 16)) * 0.125f));
            o[x] = (uint32_t)f2bf(bf2f((bf16_t)(c[x] & 0xffffu)) + lo) |
                   ((uint32_t)f2bf(bf2f((bf16_t)(c[x] >> 16)) + hi) << 16);
        }
        reinterpret_cast<uint4*>(out)[e] = uint4{o[0], o[1], o[2], o[3]};
    }
}

// Input channels: log(eta)/2, a, phi_cold, zeros (16 channels).
__global__ void k_make_input(const double* __restrict__ eta, const double* __restrict__ cold,
                             double a, long nvox, bf16_t* __restrict__ x)
{
    for (long v = (long)blockIdx.x * blockDim.x + threadIdx.x; v < nvox;
         v += (long)gridDim.x * blockDim.x) {
        // channels 0, 1, 2 = log(eta)/2, a, cold; 3..15 zero (two 16-byte stores)
        uint4* o = reinterpret_cast<uint4*>(x + v * 16);
        const uint32_t c01 = (uint32_t)f2bf((float)(log(eta[v]) * 0.5)) |
                             ((uint32_t)f2bf((float)a) << 16);
        o[0] = uint4{c01, (uint32_t)f2bf((float)cold[v]), 0u, 0u};
        o[1] = uint4{0u, 0u, 0u, 0u};
    }
}

// out[v] = sum_c d[v][c] wh[c] + bh (fp32); guess[v] = cold[v] + out[v] if
// guess != NULL.
__global__ void k_head(const bf16_t* __restrict__ d, const float* __restrict__ wh, long nvox,
                       float* __restrict__ out, const double* __restrict__ cold,
                       double* __restrict__ guess)
{
    for (long v = (long)blockIdx.x * blockDim.x + threadIdx.x; v < nvox;
         v += (long)gridDim.x * blockDim.x) {
        const uint4* dv = reinterpret_cast<const uint4*>(d + v * 16);
        const uint4 u0 = dv[0], u1 = dv[1];
        const uint32_t w[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
        float s = wh[16];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            s += bf2f((bf16_t)(w[i] & 0xffffu)) * wh[2 * i];
            s += bf2f((bf16_t)(w[i] >> 16)) * wh[2 * i + 1];
        }
        if (out) out[v] = s;
        if (guess) guess[v] = cold[v] + (double)s;
    }
}

// Loss pieces: dout[v] = 2 (out - target) / nvox; per-block partials of
// (out - target)^2 and of dout and of dout * d[v][c] (head gradient).  Bound by
// memory: the 16 channels in two 16-byte loads and stores, and the block's sums
// by shuffles (channel by channel, with 18 threads adding up 256 rows: 108 -> 35 us at 128^3).
__global__ __launch_bounds__(kThreads) void k_head_bwd(const float* __restrict__ out,
                                                       const double* __restrict__ phi_t,
                                                       const double* __restrict__ cold,
                                                       const bf16_t* __restrict__ d,
                                                       const float* __restrict__ wh, long nvox,
                                                       int chunk, float* __restrict__ part,
                                                       bf16_t* __restrict__ dh)
{
    // part[b][0..15] = sum dout*d[:,c], part[b][16] = sum dout, part[b][17] = sum err^2
    __shared__ float red[kThreads / 64][18];
    float acc[18], w[16];
    for (int q = 0; q < 18; ++q) acc[q] = 0.f;
    for (int c = 0; c < 16; ++c) w[c] = wh[c];
    const long v0 = (long)blockIdx.x * chunk;
    const float scale = 2.0f / (float)nvox;
    for (long v = v0 + threadIdx.x; v < v0 + chunk && v < nvox; v += blockDim.x) {
        const float err = out[v] - (float)(phi_t[v] - cold[v]);
        const float go = scale * err;
        const uint4* dv = reinterpret_cast<const uint4*>(d + v * 16);
        const uint4 u0 = dv[0], u1 = dv[1];
        const uint32_t x[8] = {u0.x, u0.y, u0.z, u0.w, u1.x, u1.y, u1.z, u1.w};
        uint32_t o[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            acc[2 * i] += go * bf2f((bf16_t)(x[i] & 0xffffu));
            acc[2 * i + 1] += go * bf2f((bf16_t)(x[i] >> 16));
            o[i] = (uint32_t)f2bf(go * w[2 * i]) | ((uint32_t)f2bf(go * w[2 * i + 1]) << 16);
        }
        uint4* hv = reinterpret_cast<uint4*>(dh + v * 16);
        hv[0] = uint4{o[0], o[1], o[2], o[3]};
        hv[1] = uint4{o[4], o[5], o[6], o[7]};
        acc[16] += go;
        acc[17] += err * err;
    }
#pragma unroll
    for (int q = 0; q < 18; ++q) {
        for (int f = 32; f; f >>= 1) acc[q] += __shfl_xor(acc[q], f, 64);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][q] = acc[q];
    }
    __syncthreads();
    if (threadIdx.x < 18) {
        float s = 0.f;
        for (int t = 0; t < kThreads / 64; ++t) s += red[t][threadIdx.x];
        part[(long)blockIdx.x * 18 + threadIdx.x] = s;
    }
}

__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, long total, float lr, float b1, float b2, float eps,
                       float c1, float c2)
{
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (long)gridDim.x * blockDim.x) {
        const float gg = g[e];
        const float mm = b1 * m[e] + (1.f - b1) * gg;
        const float vv = b2 * v[e] + (1.f - b2) * gg * gg;
        m[e] = mm;
        v[e] = vv;
        p[e] -= lr * (mm / c1) / (sqrtf(vv / c2) + eps);
    }
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------

struct ConvSpec {
    int cin, cout;
};
constexpr ConvSpec kConvs[14] = {{16, 16},  {16, 16}, {16, 32}, {32, 32}, {32, 64},
                                 {64, 64},  {64, 64}, {64, 64}, {128, 64}, {64, 64},
                                 {96, 32},  {32, 32}, {48, 16}, {16, 16}};
constexpr int kHeadIn = 16;

long param_offset(int layer)
{
    long off = 0;
    for (int l = 0; l < layer; ++l) off += 27L * kConvs[l].cin * kConvs[l].cout + kConvs[l].cout;
    return off;
}
long param_total() { return param_offset(14) + kHeadIn + 1; }

#define UCHECK(call)                                                                  \
    do {                                                                              \
        hipError_t e_ = (call);                                                       \
        if (e_ != hipSuccess) {                                                       \
            uerr("%s: %s", #call, hipGetErrorString(e_));                             \
            return ISIS_ERR_HIP;                                                      \
        }                                                                             \
    } while (0)
#define ULAUNCH(name)                                                                 \
    do {                                                                              \
        hipError_t e_ = hipGetLastError();                                            \
        if (e_ != hipSuccess) {                                                       \
            uerr("%s: %s", name, hipGetErrorString(e_));                              \
            return ISIS_ERR_HIP;                                                      \
        }                                                                             \
    } while (0)

// Whether four-channel stores to these outputs are aligned.
int vec_ok(const bf16_t* y, const float* yf)
{
    return ((uintptr_t)y & 7) == 0 && ((uintptr_t)yf & 15) == 0;
}

template <int CIN, int COUT>
int launch_conv_lds(const bf16_t* x, int n, const bf16_t* w, const float* bias, int relu,
                    bf16_t* y, float* yf, hipStream_t s)
{
    // output channels per workgroup: 16 NT; eight waves where the weights
    // fill most of the LDS (one workgroup per CU), four otherwise (two per CU)
    constexpr int NT = COUT == 32 ? 2 : COUT == 96 ? 3 : 4;
    constexpr int NW = NT >= 3 ? 8 : 4;
    using G = ConvTile<NT, NW>;
    static std::atomic<unsigned> lds_done{0};  // per instantiation: devices set up
    auto kern = k_conv3_lds<CIN, COUT, NT, NW>;
    UCHECK(isis::ensure_dynamic_lds((const void*)kern, G::LDS, lds_done));
    const long blocks = (long)(n / kLPX) * (n / NW) * (n / kLZ) * (COUT / (16 * NT));
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(G::NTH), G::LDS, s, x, n, w, bias, relu,
                       y, yf, vec_ok(y, yf));
    ULAUNCH("k_conv3_lds");
    return ISIS_OK;
}

template <int CIN, int CLO>
int launch_conv_planes(const bf16_t* x, const bf16_t* lo, int n, const bf16_t* w,
                       const float* bias, int relu, bf16_t* y, float* yf, hipStream_t s)
{
    using G = ConvPlanes<CIN, CLO>;
    static std::atomic<unsigned> lds_done{0};  // per instantiation: devices set up
    auto kern = k_conv3_planes<CIN, CLO>;
    UCHECK(isis::ensure_dynamic_lds((const void*)kern, G::LDS, lds_done));
    // planes per workgroup: as many as leave one workgroup per CU
    const long cols = (long)(n / kPY) * (n / kLZ);
    int xc = n;
    while (xc > 2 && cols * (n / xc) < 256) xc /= 2;
    hipLaunchKernelGGL(kern, dim3((unsigned)(cols * (n / xc))), dim3(G::NTH), G::LDS, s, x, lo, n,
                       xc, w, bias, relu, y, yf, vec_ok(y, yf));
    ULAUNCH("k_conv3_planes");
    return ISIS_OK;
}

template <int CIN, int NT, int Z, int TY, int TPB>
int launch_conv_small(const bf16_t* x, const bf16_t* w, const float* bias, int cout, int relu,
                      bf16_t* y, float* yf, hipStream_t s)
{
    constexpr int lds = ConvSmall<CIN, NT, Z, TY, TPB>::LDS;
    static std::atomic<unsigned> lds_done{0};  // per instantiation: devices set up
    auto kern = k_conv3_small<CIN, NT, Z, TY, TPB>;
    UCHECK(isis::ensure_dynamic_lds((const void*)kern, lds, lds_done));
    hipLaunchKernelGGL(kern, dim3(Z * (Z / TY) * (cout / (16 * NT))), dim3(kThreads), lds, s, x, w,
                       bias, cout, relu, vec_ok(y, yf), y, yf);
    ULAUNCH("k_conv3_small");
    return ISIS_OK;
}

template <bool HEAD>
int launch_conv_ring(const bf16_t* x, int n, const bf16_t* w, const float* bias, int cout,
                     int relu, bf16_t* y, float* yf, const HeadOut& head, hipStream_t s)
{
    // planes per workgroup: a power of two up to 64 that leaves >= 512
    // workgroups (two per CU)
    const long cols = (long)(n / kRY) * (n / kLZ) * (cout / 16);
    int xc = 2;
    while (xc < 64 && cols * (n / (2 * xc)) >= 512) xc *= 2;
    hipLaunchKernelGGL(k_conv3_ring<HEAD>, dim3((unsigned)(cols * (n / xc))), dim3(kThreads), 0, s,
                       x, n, xc, w, bias, cout, relu, y, yf, vec_ok(y, yf), head);
    ULAUNCH("k_conv3_ring");
    return ISIS_OK;
}

int launch_conv(const bf16_t* x, int n, int cin, const bf16_t* w, const float* bias, int cout,
                int relu, bf16_t* y, float* yf, hipStream_t s)
{
    const bool lds = n >= kLZ;  // powers of two: whole tiles
    if (lds && cin == 16 && (cout == 16 || cout == 32 || cout == 48))
        return launch_conv_ring<false>(x, n, w, bias, cout, relu, y, yf, HeadOut{}, s);
#define CONV_CASE(CI, CO)                                                                   \
    if (cin == CI && cout == CO) {                                                          \
        if constexpr (CI > 16)                                                              \
            if (lds) {                                                                      \
                if constexpr (CO == 16)                                                     \
                    return launch_conv_planes<CI, 0>(x, nullptr, n, w, bias, relu, y, yf, s); \
                else                                                                        \
                    return launch_conv_lds<CI, CO>(x, n, w, bias, relu, y, yf, s); \
            }                                                                               \
        if (n == 32)  /* rows per workgroup: what fits the LDS */                           \
            return launch_conv_small<CI, (CO % 64 == 0 ? 4 : CO % 32 == 0 ? 2 : 1), 32,     \
                                     (CI > 64 ? 2 : 4), 1>(x, w, bias, CO, relu, y, yf, s); \
        if (n == 16)                                                                        \
            return launch_conv_small<CI, 1, 16, 4, 9>(x, w, bias, CO, relu, y, yf, s);      \
        if (n == 8)                                                                         \
            return launch_conv_small<CI, 1, 8, 8, 9>(x, w, bias, CO, relu, y, yf, s);       \
        const int waves = (n * n * n + 15) / 16 * (CO / 16);                                \
        hipLaunchKernelGGL((k_conv3<CI>), dim3((waves + 3) / 4), dim3(kThreads), 0, s, x,   \
                           n, w, bias, CO, relu, vec_ok(y, yf), y, yf);                     \
        ULAUNCH("k_conv3");                                                                 \
        return ISIS_OK;                                                                     \
    }
    CONV_CASE(16, 16) CONV_CASE(16, 32) CONV_CASE(32, 32) CONV_CASE(32, 64) CONV_CASE(64, 64)
    CONV_CASE(128, 64) CONV_CASE(96, 32) CONV_CASE(48, 16)
    // data-gradient shapes (channels swapped)
    CONV_CASE(32, 16) CONV_CASE(64, 32) CONV_CASE(64, 128) CONV_CASE(32, 96) CONV_CASE(16, 48)
#undef CONV_CASE
    uerr("no convolution kernel for %d -> %d channels", cin, cout);
    return ISIS_ERR_UNSUPPORTED;
}

// Convolution of [nearest upsampling of lo (n/2)^3 x clo, skip n^3 x (cin -
// clo)] without materialising the concatenation (sides n >= 64).
int launch_conv_cat(const bf16_t* lo, const bf16_t* skip, int n, int cin, int clo,
                    const bf16_t* w, const float* bias, int cout, int relu, bf16_t* y,
                    hipStream_t s)
{
    if (n < kLZ || !(cin == 48 && clo == 32 && cout == 16)) {
        uerr("no fused decoder convolution for %d (%d upsampled) -> %d channels at side %d", cin,
             clo, cout, n);
        return ISIS_ERR_UNSUPPORTED;
    }
    return launch_conv_planes<48, 32>(skip, lo, n, w, bias, relu, y, nullptr, s);
}

int dw_chunk(long nvox) { return (int)std::min<long>(nvox, 4096); }

size_t dw_part_floats(long nvox, int cin, int cout)
{
    return (size_t)(nvox / dw_chunk(nvox)) * 27 * cin * cout;
}

// dw = sum over the nchunk partial sums in part.
int launch_sum_chunks(const float* part, int nchunk, long elems, float* out, hipStream_t s)
{
    hipLaunchKernelGGL(k_sum_chunks, dim3((unsigned)((elems + 15) / 16)), dim3(kThreads), 0, s, part,
                       nchunk, elems, out);
    ULAUNCH("k_sum_chunks");
    return ISIS_OK;
}

// One k_conv3_dw_tiled launch: regions of xc planes; one region writes dw itself.
template <class G>
int launch_dw_tiled(const bf16_t* x, int n, int cin, const bf16_t* dy, int cout, int xc,
                    float* part, float* dw, hipStream_t s)
{
    static std::atomic<unsigned> lds_done{0};  // per instantiation: devices set up
    auto kern = k_conv3_dw_tiled<G>;
    UCHECK(isis::ensure_dynamic_lds((const void*)kern, G::LDS, lds_done));
    const int regions = (n / G::Z) * (n / G::TY) * (n / xc);
    const int blocks = regions * (cin / 16) * (cout / 16) * (3 / G::NDI);
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(kThreads), G::LDS, s, x, n, cin, dy, cout, xc,
                       regions == 1 ? dw : part);
    ULAUNCH("k_conv3_dw_tiled");
    return regions == 1 ? (int)ISIS_OK : launch_sum_chunks(part, regions, 27L * cin * cout, dw, s);
}

int launch_conv_dw(const bf16_t* x, int n, int cin, const bf16_t* dy, int cout, float* part,
                   float* dw, hipStream_t s)
{
    const long nvox = (long)n * n * n;
    bool known = false;  // the network's layer shapes
    for (const ConvSpec& c : kConvs) known = known || (c.cin == cin && c.cout == cout);
    if (!known) {
        uerr("no weight-gradient kernel for %d -> %d channels", cin, cout);
        return ISIS_ERR_UNSUPPORTED;
    }
    // Regions per launch stay within the caller's n^3 / 4096 partial sums.
    // Planes per region: 8 up to 128^3 (512 regions there, two workgroups per
    // CU for one channel tile), 16 at 256^3, 32 above (fewer partial sums).
    const bool vec = (((uintptr_t)x | (uintptr_t)dy) & 15) == 0;  // 16-byte loads
    if (vec && n >= 64) {
        const int xc = n <= 128 ? 8 : n == 256 ? 16 : 32;
        return launch_dw_tiled<DwTile<64, 8, 3>>(x, n, cin, dy, cout, xc, part, dw, s);
    }
    if (vec && n == 32) return launch_dw_tiled<DwTile<32, 8, 1>>(x, n, cin, dy, cout, 16, part, dw, s);
    if (vec && n == 16) return launch_dw_tiled<DwTile<16, 16, 1>>(x, n, cin, dy, cout, 16, part, dw, s);
    // sides below 16 (no 16-voxel windows along z) and unaligned tensors
    // (one chunk, sides up to 16: its sum is dw)
    const int chunk = dw_chunk(nvox);
    const int nchunk = (int)(nvox / chunk);
    float* sums = nchunk == 1 ? dw : part;
#define DW_CASE(CI, CO)                                                                     \
    if (cin == CI && cout == CO)                                                            \
        hipLaunchKernelGGL((k_conv3_dw<CI, CO>), dim3(27 * nchunk), dim3(kThreads), 0, s, x, \
                           n, dy, chunk, sums);
    DW_CASE(16, 16) DW_CASE(16, 32) DW_CASE(32, 32) DW_CASE(32, 64) DW_CASE(64, 64)
    DW_CASE(128, 64) DW_CASE(96, 32) DW_CASE(48, 16)
#undef DW_CASE
    ULAUNCH("k_conv3_dw");
    return nchunk == 1 ? (int)ISIS_OK : launch_sum_chunks(part, nchunk, 27L * cin * cout, dw, s);
}

// out[c] = sum of channel c of a (C = 16, 32, 64); with o: a = a * (o > 0) first.
// Scratch: one partial sum per kSumVecs vectors, less than the weight gradient's.
int launch_chan_sum(bf16_t* a, const bf16_t* o, long nvox, int C, float* part, float* out,
                    hipStream_t s)
{
    const int nb = (int)((nvox * (C / 8) + kSumVecs - 1) / kSumVecs);
    if (o)
        hipLaunchKernelGGL((k_chan_sum<true, true>), dim3(nb), dim3(kThreads), 0, s, a, o, nvox, C, part);
    else if (((uintptr_t)a & 15) == 0)
        hipLaunchKernelGGL((k_chan_sum<false, true>), dim3(nb), dim3(kThreads), 0, s, a, o, nvox, C, part);
    else
        hipLaunchKernelGGL((k_chan_sum<false, false>), dim3(nb), dim3(kThreads), 0, s, a, o, nvox, C, part);
    ULAUNCH("k_chan_sum");
    return launch_sum_chunks(part, nb, (long)C, out, s);
}

// ---------------------------------------------------------------------------
// The network: workspace plan, forward, backward.
// ---------------------------------------------------------------------------

int level_of(int layer)
{
    static const int lv[14] = {0, 0, 1, 1, 2, 2, 3, 3, 2, 2, 1, 1, 0, 0};
    return lv[layer];
}

struct Plan {
    int n[4];
    long nv[4];
    bf16_t *in, *o[14], *p1, *p2, *p3, *c8, *c10, *c12;  // forward tensors
    float* out;                                            // head output (fp32)
    bf16_t* wf[14];                                        // bf16 weights
    // training only
    bf16_t *ga, *gb;            // ping-pong gradients (largest: nv0 x 16)
    bf16_t *gc8, *gc10, *gc12;  // gradients of the concatenations (kept for the skips)
    bf16_t* wb[14];             // flipped, transposed bf16 weights (data gradient)
    float *part, *grad, *hpart, *hsum, *loss;
    size_t bytes;
};

Plan make_plan(int n, int training, char* base)
{
    Plan P;
    memset(&P, 0, sizeof(P));
    size_t off = 0;
    auto take = [&](size_t bytes) -> char* {
        off = (off + 255) & ~(size_t)255;
        char* p = base ? base + off : nullptr;
        off += bytes;
        return p;
    };
    for (int l = 0; l < 4; ++l) {
        P.n[l] = n >> l;
        P.nv[l] = (long)P.n[l] * P.n[l] * P.n[l];
    }
    P.in = (bf16_t*)take(P.nv[0] * 16 * 2);
    for (int c = 0; c < 14; ++c) P.o[c] = (bf16_t*)take(P.nv[level_of(c)] * kConvs[c].cout * 2);
    P.p1 = (bf16_t*)take(P.nv[1] * 16 * 2);
    P.p2 = (bf16_t*)take(P.nv[2] * 32 * 2);
    P.p3 = (bf16_t*)take(P.nv[3] * 64 * 2);
    P.c8 = (bf16_t*)take(P.nv[2] * 128 * 2);
    P.c10 = (bf16_t*)take(P.nv[1] * 96 * 2);
    P.c12 = (bf16_t*)take(P.nv[0] * 48 * 2);
    P.out = (float*)take(P.nv[0] * 4);
    for (int c = 0; c < 14; ++c) P.wf[c] = (bf16_t*)take(27L * kConvs[c].cin * kConvs[c].cout * 2);
    if (training) {
        P.ga = (bf16_t*)take(P.nv[0] * 16 * 2);
        P.gb = (bf16_t*)take(P.nv[0] * 16 * 2);
        P.gc8 = (bf16_t*)take(P.nv[2] * 128 * 2);
        P.gc10 = (bf16_t*)take(P.nv[1] * 96 * 2);
        P.gc12 = (bf16_t*)take(P.nv[0] * 48 * 2);
        for (int c = 0; c < 14; ++c)
            P.wb[c] = (bf16_t*)take(27L * kConvs[c].cin * kConvs[c].cout * 2);
        size_t part = 0;
        for (int c = 0; c < 14; ++c)
            part = std::max(part, dw_part_floats(P.nv[level_of(c)], kConvs[c].cin, kConvs[c].cout));
        for (int l = 0; l < 4; ++l) part = std::max(part, (size_t)((P.nv[l] + 4095) / 4096) * 128);
        P.part = (float*)take(part * 4);
        P.grad = (float*)take(param_total() * 4);
        P.hpart = (float*)take((size_t)((P.nv[0] + 4095) / 4096) * 18 * 4);
        P.hsum = (float*)take(18 * 4);
        P.loss = (float*)take(4);
    }
    P.bytes = off + 256;
    return P;
}

#define TRY(x)                       \
    do {                             \
        int r_ = (x);                \
        if (r_ != ISIS_OK) return r_; \
    } while (0)

// All convolutions' weights in bf16, FLIP: the data gradient's.
template <bool FLIP>
int launch_conv_weights(const float* params, bf16_t* const* dst, hipStream_t s)
{
    ConvWeights a;
    for (int c = 0; c < 14; ++c) {
        a.src[c] = params + param_offset(c);
        a.dst[c] = dst[c];
        a.cin[c] = kConvs[c].cin;
        a.cout[c] = kConvs[c].cout;
    }
    hipLaunchKernelGGL(k_conv_weights<FLIP>, dim3(54, 14), dim3(kThreads), 0, s, a);
    ULAUNCH("k_conv_weights");
    return ISIS_OK;
}

// predict: out and guess come from the head, which joins the last convolution
// on sides that k_conv3_ring takes, as the last decoder stage's concatenation
// joins its convolution; no activation is then kept for a backward pass
// (training keeps the concatenation for the weight gradient).
int run_forward(const Plan& P, const float* params, const double* phi_cold, float* out,
                double* guess, bool predict, hipStream_t s)
{
    TRY(launch_conv_weights<false>(params, P.wf, s));
    auto conv = [&](int c, const bf16_t* x) -> int {
        const int lv = level_of(c);
        return launch_conv(x, P.n[lv], kConvs[c].cin, P.wf[c],
                           params + param_offset(c) + 27L * kConvs[c].cin * kConvs[c].cout,
                           kConvs[c].cout, 1, P.o[c], nullptr, s);
    };
    auto pool = [&](const bf16_t* x, int lvf, int C, bf16_t* y) -> int {
        hipLaunchKernelGGL(k_pool2, dim3(grid_of(P.nv[lvf + 1] * C / 8)), dim3(kThreads), 0, s, x,
                           P.n[lvf], C, 0, C, y);
        ULAUNCH("k_pool2");
        return (int)ISIS_OK;
    };
    auto upcat = [&](const bf16_t* lo, int lvc, int C, const bf16_t* skip, int S, bf16_t* out) -> int {
        const dim3 g(grid_of(P.nv[lvc - 1] * (C + S) / 8));
        if (C == 64 && S == 64)
            hipLaunchKernelGGL((k_up2_cat<64, 64>), g, dim3(kThreads), 0, s, lo, P.n[lvc], skip, out);
        else if (C == 64 && S == 32)
            hipLaunchKernelGGL((k_up2_cat<64, 32>), g, dim3(kThreads), 0, s, lo, P.n[lvc], skip, out);
        else if (C == 32 && S == 16)
            hipLaunchKernelGGL((k_up2_cat<32, 16>), g, dim3(kThreads), 0, s, lo, P.n[lvc], skip, out);
        else {
            uerr("k_up2_cat: no instance for %d + %d channels", C, S);
            return (int)ISIS_ERR_INVALID_ARG;
        }
        ULAUNCH("k_up2_cat");
        return (int)ISIS_OK;
    };
    TRY(conv(0, P.in));
    TRY(conv(1, P.o[0]));
    TRY(pool(P.o[1], 0, 16, P.p1));
    TRY(conv(2, P.p1));
    TRY(conv(3, P.o[2]));
    TRY(pool(P.o[3], 1, 32, P.p2));
    TRY(conv(4, P.p2));
    TRY(conv(5, P.o[4]));
    TRY(pool(P.o[5], 2, 64, P.p3));
    TRY(conv(6, P.p3));
    TRY(conv(7, P.o[6]));
    TRY(upcat(P.o[7], 3, 64, P.o[5], 64, P.c8));
    TRY(conv(8, P.c8));
    TRY(conv(9, P.o[8]));
    TRY(upcat(P.o[9], 2, 64, P.o[3], 32, P.c10));
    TRY(conv(10, P.c10));
    TRY(conv(11, P.o[10]));
    const bool fuse = predict && P.n[0] >= kLZ;
    if (fuse) {
        TRY(launch_conv_cat(P.o[11], P.o[1], P.n[0], 48, 32, P.wf[12],
                            params + param_offset(12) + 27L * 48 * 16, 16, 1, P.o[12], s));
    } else {
        TRY(upcat(P.o[11], 1, 32, P.o[1], 16, P.c12));
        TRY(conv(12, P.c12));
    }
    const HeadOut head{params + param_offset(14), phi_cold, out, guess};
    if (fuse)
        return launch_conv_ring<true>(P.o[12], P.n[0], P.wf[13],
                                      params + param_offset(13) + 27L * 16 * 16, 16, 1, nullptr,
                                      nullptr, head, s);
    TRY(conv(13, P.o[12]));
    hipLaunchKernelGGL(k_head, dim3(grid_of(P.nv[0])), dim3(kThreads), 0, s, P.o[13], head.wh,
                       P.nv[0], out, phi_cold, guess);
    ULAUNCH("k_head");
    return ISIS_OK;
}

// Backward from d(o13) in P.ga; writes the 14 convolutions' gradients into
// P.grad (the head's part is written by the caller).
int run_backward(const Plan& P, const float* params, hipStream_t s)
{
    TRY(launch_conv_weights<true>(params, P.wb, s));
    // back(c, g, x, dx): g = d(o_c) (masked in place), weight and bias
    // gradients from the layer input x, dx = d(x) (skipped when NULL).
    auto back = [&](int c, bf16_t* g, const bf16_t* x, bf16_t* dx) -> int {
        const int lv = level_of(c);
        const long nv = P.nv[lv];
        const int ci = kConvs[c].cin, co = kConvs[c].cout;
        float* gw = P.grad + param_offset(c);
        int rr = launch_chan_sum(g, P.o[c], nv, co, P.part, gw + 27L * ci * co, s);
        if (rr) return rr;
        rr = launch_conv_dw(x, P.n[lv], ci, g, co, P.part, gw, s);
        if (rr) return rr;
        if (!dx) return ISIS_OK;
        return launch_conv(g, P.n[lv], co, P.wb[c], nullptr, ci, 0, dx, nullptr, s);
    };
    // gradient of the upsampled half of a concatenation (level lvf fine)
    auto upb = [&](const bf16_t* dcat, int lvf, int cs, int C, bf16_t* y) -> int {
        hipLaunchKernelGGL(k_up2_bwd, dim3(grid_of(P.nv[lvf + 1] * C / 8)), dim3(kThreads), 0, s,
                           dcat, P.n[lvf], cs, C, y);
        ULAUNCH("k_up2_bwd");
        return (int)ISIS_OK;
    };
    // gradient of a skip tensor: concat part + pooled path
    auto skipg = [&](const bf16_t* dcat, int lvf, int cs, int C, int S, const bf16_t* dlo,
                     bf16_t* y) -> int {
        hipLaunchKernelGGL(k_skip_grad, dim3(grid_of(P.nv[lvf] * S / 8)), dim3(kThreads), 0, s,
                           dcat, P.n[lvf], cs, C, S, dlo, y);
        ULAUNCH("k_skip_grad");
        return (int)ISIS_OK;
    };
    TRY(back(13, P.ga, P.o[12], P.gb));               // gb = d o12
    TRY(back(12, P.gb, P.c12, P.gc12));               // gc12 = d c12 [nv0][48]
    TRY(upb(P.gc12, 0, 48, 32, P.ga));                // ga = d o11 [nv1][32]
    TRY(back(11, P.ga, P.o[10], P.gb));               // gb = d o10
    TRY(back(10, P.gb, P.c10, P.gc10));               // gc10 = d c10 [nv1][96]
    TRY(upb(P.gc10, 1, 96, 64, P.ga));                // ga = d o9 [nv2][64]
    TRY(back(9, P.ga, P.o[8], P.gb));                 // gb = d o8
    TRY(back(8, P.gb, P.c8, P.gc8));                  // gc8 = d c8 [nv2][128]
    TRY(upb(P.gc8, 2, 128, 64, P.ga));                // ga = d o7 [nv3][64]
    TRY(back(7, P.ga, P.o[6], P.gb));                 // gb = d o6
    TRY(back(6, P.gb, P.p3, P.ga));                   // ga = d p3 [nv3][64]
    TRY(skipg(P.gc8, 2, 128, 64, 64, P.ga, P.gb));    // gb = d o5 [nv2][64]
    TRY(back(5, P.gb, P.o[4], P.ga));                 // ga = d o4
    TRY(back(4, P.ga, P.p2, P.gb));                   // gb = d p2 [nv2][32]
    TRY(skipg(P.gc10, 1, 96, 64, 32, P.gb, P.ga));    // ga = d o3 [nv1][32]
    TRY(back(3, P.ga, P.o[2], P.gb));                 // gb = d o2
    TRY(back(2, P.gb, P.p1, P.ga));                   // ga = d p1 [nv1][16]
    TRY(skipg(P.gc12, 0, 48, 32, 16, P.ga, P.gb));    // gb = d o1 [nv0][16]
    TRY(back(1, P.gb, P.o[0], P.ga));                 // ga = d o0
    TRY(back(0, P.ga, P.in, nullptr));
    return ISIS_OK;
}

bool valid_unet_n(int n) { return n >= 16 && n <= 2048 && (n & (n - 1)) == 0; }

}  // namespace

// ---------------------------------------------------------------------------
// C ABI.
// ---------------------------------------------------------------------------

extern "C" {

size_t isis_unet_param_count(void) { return (size_t)param_total(); }

size_t isis_unet_workspace_size(int n, int training)
{
    if (!valid_unet_n(n)) return 0;
    return make_plan(n, training, nullptr).bytes;
}

const char* isis_unet_last_error(void) { return u_err; }

int isis_unet_predict(const float* params, const double* eta, const double* phi_cold, double a,
                      int n, double* guess, float* out, void* workspace, size_t workspace_bytes,
                      void* stream)
{
    u_err[0] = 0;
    if (!valid_unet_n(n) || !params || !eta || !phi_cold || !workspace || !(a > 0.0)) {
        uerr("unet_predict: need n a power of two in [16, 2048], a > 0, non-NULL arrays");
        return ISIS_ERR_INVALID_ARG;
    }
    Plan P = make_plan(n, 0, (char*)workspace);
    if (workspace_bytes < P.bytes || ((uintptr_t)workspace & 255)) {
        uerr("unet_predict: workspace must be 256-byte aligned and >= %zu bytes", P.bytes);
        return ISIS_ERR_INVALID_ARG;
    }
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(k_make_input, dim3(grid_of(P.nv[0])), dim3(kThreads), 0, s, eta, phi_cold,
                       a, P.nv[0], P.in);
    ULAUNCH("k_make_input");
    return run_forward(P, params, phi_cold, out, guess, true, s);
}

int isis_unet_forward(const float* params, const double* eta, const double* phi_cold, double a,
                      int n, float* out, void* workspace, size_t workspace_bytes, void* stream)
{
    u_err[0] = 0;
    if (!valid_unet_n(n) || !params || !eta || !phi_cold || !workspace || !(a > 0.0)) {
        uerr("unet_forward: need n a power of two in [16, 2048], a > 0, non-NULL arrays");
        return ISIS_ERR_INVALID_ARG;
    }
    Plan P = make_plan(n, 1, (char*)workspace);
    if (workspace_bytes < P.bytes || ((uintptr_t)workspace & 255)) {
        uerr("unet_forward: workspace must be 256-byte aligned and >= %zu bytes (training size)",
             P.bytes);
        return ISIS_ERR_INVALID_ARG;
    }
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(k_make_input, dim3(grid_of(P.nv[0])), dim3(kThreads), 0, s, eta, phi_cold,
                       a, P.nv[0], P.in);
    ULAUNCH("k_make_input");
    TRY(run_forward(P, params, nullptr, P.out, nullptr, false, s));
    if (out) UCHECK(hipMemcpyAsync(out, P.out, P.nv[0] * sizeof(float), hipMemcpyDeviceToDevice, s));
    return ISIS_OK;
}

int isis_unet_backward(const float* params, const double* phi_cold, const double* phi_target,
                       int n, void* workspace, size_t workspace_bytes, float* grad,
                       float* loss_out, void* stream)
{
    u_err[0] = 0;
    if (!valid_unet_n(n) || !params || !phi_cold || !phi_target || !workspace) {
        uerr("unet_backward: need n a power of two in [16, 2048] and non-NULL arrays");
        return ISIS_ERR_INVALID_ARG;
    }
    Plan P = make_plan(n, 1, (char*)workspace);
    if (workspace_bytes < P.bytes || ((uintptr_t)workspace & 255)) {
        uerr("unet_backward: workspace must be 256-byte aligned and >= %zu bytes (training size)",
             P.bytes);
        return ISIS_ERR_INVALID_ARG;
    }
    hipStream_t s = (hipStream_t)stream;
    const float* head = params + param_offset(14);
    const int hchunk = 4096;
    const int hb = (int)((P.nv[0] + hchunk - 1) / hchunk);
    hipLaunchKernelGGL(k_head_bwd, dim3(hb), dim3(kThreads), 0, s, P.out, phi_target, phi_cold,
                       P.o[13], head, P.nv[0], hchunk, P.hpart, P.ga);
    ULAUNCH("k_head_bwd");
    TRY(launch_sum_chunks(P.hpart, hb, 18L, P.hsum, s));
    // head gradient (16 weights, 1 bias) into the flat gradient
    UCHECK(hipMemcpyAsync(P.grad + param_offset(14), P.hsum, 17 * sizeof(float),
                          hipMemcpyDeviceToDevice, s));
    TRY(run_backward(P, params, s));
    if (grad && grad != P.grad)
        UCHECK(hipMemcpyAsync(grad, P.grad, param_total() * sizeof(float), hipMemcpyDeviceToDevice,
                              s));
    if (loss_out) {
        float h[18];
        UCHECK(hipMemcpyAsync(h, P.hsum, sizeof(h), hipMemcpyDeviceToHost, s));
        UCHECK(hipStreamSynchronize(s));
        *loss_out = h[17] / (float)P.nv[0];
    }
    return ISIS_OK;
}

int isis_unet_adam_step(float* params, const float* grad, float* adam_m, float* adam_v,
                        long count, int step, float lr, void* stream)
{
    u_err[0] = 0;
    if (!params || !grad || !adam_m || !adam_v || count < 0 || step < 1 || !(lr >= 0.f)) {
        uerr("unet_adam_step: invalid arguments");
        return ISIS_ERR_INVALID_ARG;
    }
    if (count == 0) return ISIS_OK;
    const float b1 = 0.9f, b2 = 0.999f;
    const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3(grid_of(count)), dim3(kThreads), 0, (hipStream_t)stream,
                       params, grad, adam_m, adam_v, count, lr, b1, b2, 1e-8f, c1, c2);
    ULAUNCH("k_adam");
    return ISIS_OK;
}

int isis_unet_train_step(float* params, float* adam_m, float* adam_v, int step, float lr,
                         const double* eta, const double* phi_cold, const double* phi_target,
                         double a, int n, void* workspace, size_t workspace_bytes,
                         float* loss_out, float* grad_out, void* stream)
{
    u_err[0] = 0;
    if (!valid_unet_n(n) || !params || !adam_m || !adam_v || step < 1 || !(lr >= 0.f) || !eta ||
        !phi_cold || !phi_target || !workspace || !(a > 0.0)) {
        uerr("unet_train_step: invalid arguments");
        return ISIS_ERR_INVALID_ARG;
    }
    TRY(isis_unet_forward(params, eta, phi_cold, a, n, nullptr, workspace, workspace_bytes,
                          stream));
    Plan P = make_plan(n, 1, (char*)workspace);
    TRY(isis_unet_backward(params, phi_cold, phi_target, n, workspace, workspace_bytes, grad_out,
                           loss_out, stream));
    return isis_unet_adam_step(params, P.grad, adam_m, adam_v, param_total(), step, lr, stream);
}

int isis_unet_tensor(void* workspace, int n, int id, void** ptr, long* voxels, int* channels)
{
    u_err[0] = 0;
    if (!valid_unet_n(n) || !workspace || !ptr || id < 0 || id > 21) {
        uerr("unet_tensor: need n a power of two in [16, 2048], a workspace and 0 <= id <= 21");
        return ISIS_ERR_INVALID_ARG;
    }
    Plan P = make_plan(n, 1, (char*)workspace);
    void* q = nullptr;
    int lv = 0, C = 0;
    if (id < 14) {
        q = P.o[id];
        lv = level_of(id);
        C = kConvs[id].cout;
    } else if (id == 14) {
        q = P.in;
        C = 16;
    } else if (id <= 17) {
        lv = id - 14;
        q = id == 15 ? P.p1 : id == 16 ? P.p2 : P.p3;
        C = id == 15 ? 16 : id == 16 ? 32 : 64;
    } else if (id == 18) {
        q = P.c8;
        lv = 2;
        C = 128;
    } else if (id == 19) {
        q = P.c10;
        lv = 1;
        C = 96;
    } else if (id == 20) {
        q = P.c12;
        lv = 0;
        C = 48;
    } else {
        q = P.out;
        lv = 0;
        C = 1;
    }
    *ptr = q;
    if (voxels) *voxels = P.nv[lv];
    if (channels) *channels = C;
    return ISIS_OK;
}

int isis_conv3_fwd(const uint16_t* x, int n, int cin, const uint16_t* w, const float* bias,
                   int cout, int relu, uint16_t* y, float* yf, void* stream)
{
    u_err[0] = 0;
    if (!valid_unet_n(n) && !(n >= 2 && (n & (n - 1)) == 0)) {
        uerr("conv3_fwd: n must be a power of two >= 2");
        return ISIS_ERR_INVALID_ARG;
    }
    if (!x || !w || (!y && !yf)) {
        uerr("conv3_fwd: NULL array");
        return ISIS_ERR_INVALID_ARG;
    }
    return launch_conv(x, n, cin, w, bias, cout, relu, y, yf, (hipStream_t)stream);
}

size_t isis_conv3_bwd_weight_workspace(int n, int cin, int cout)
{
    if (n < 2 || (n & (n - 1))) return 0;
    const long nv = (long)n * n * n;
    return std::max(dw_part_floats(nv, cin, cout), (size_t)((nv + 4095) / 4096) * cout) * 4 + 256;
}

int isis_conv3_bwd_weight(const uint16_t* x, int n, int cin, const uint16_t* dy, int cout,
                          float* dw, float* db, void* workspace, size_t workspace_bytes,
                          void* stream)
{
    u_err[0] = 0;
    if (n < 2 || (n & (n - 1)) || !x || !dy || !dw || !workspace) {
        uerr("conv3_bwd_weight: invalid arguments");
        return ISIS_ERR_INVALID_ARG;
    }
    if (workspace_bytes < isis_conv3_bwd_weight_workspace(n, cin, cout)) {
        uerr("conv3_bwd_weight: workspace too small");
        return ISIS_ERR_INVALID_ARG;
    }
    hipStream_t s = (hipStream_t)stream;
    TRY(launch_conv_dw(x, n, cin, dy, cout, (float*)workspace, dw, s));
    if (db)  // (dy is only read)
        TRY(launch_chan_sum(const_cast<uint16_t*>(dy), nullptr, (long)n * n * n, cout,
                            (float*)workspace, db, s));
    return ISIS_OK;
}

int isis_conv3_flip_weights(const float* w, int cin, int cout, uint16_t* wt, void* stream)
{
    u_err[0] = 0;
    if (!w || !wt || cin <= 0 || cout <= 0) {
        uerr("conv3_flip_weights: invalid arguments");
        return ISIS_ERR_INVALID_ARG;
    }
    ConvWeights a{};
    a.src[0] = w;
    a.dst[0] = wt;
    a.cin[0] = cin;
    a.cout[0] = cout;
    hipLaunchKernelGGL(k_conv_weights<true>, dim3(grid_of(27L * cin * cout)), dim3(kThreads), 0,
                       (hipStream_t)stream, a);
    ULAUNCH("k_conv_weights");
    return ISIS_OK;
}

}  // extern "C"
