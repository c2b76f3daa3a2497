// mg_bottom.hpp -- the coarse levels of the psi V-cycle in one workgroup.
//
// From the first level of at most kBottomMax (16) cells per axis down to
// the coarsest solve and back, every step of the V-cycle runs in one workgroup of 16 waves on
// arrays in LDS.  As separate launches each of these steps costs a launch and a round of
// memory latency (3-4 us for a colour pass of 8^3 or 16^3 cells, 19 launches from 16^3 to 4^3
// and back: 75 us and the gaps between them in a 128^3 FP32 cycle).  Here the whole V(1,3)
// from 16^3 to 4^3 and back takes 40 us (FP64 43, Robin 71 and 92): the 4^3 solve 11 (Robin 20), the
// 8^3 level around it 9 (Robin 18 and 20), the 16^3 level 21 to 23 (Robin 34 and 51).  With the scratch
// of the coarsest solve behind generic pointers it took 1 to 5 us more (10^3 over 5^3: 33 -> 26 us,
// Robin 149 -> 72).
//
// Corrections d live in padded arrays of (n + 4)^3 values whose ghost layers hold what the
// boundary rule gives there, so that every tap is a fixed offset from its cell whatever the
// rule; a thread that writes a cell near a face writes its ghosts along the axes with it.
// Threads own z pairs and keep the pair's right-hand side, coefficient and reciprocal diagonal
// in registers through all passes of a level.  A colour pass forms the new values of its cells
// from the old array, waits, and writes them: the values of the double-buffered grid pass.
#pragma once

#include "mg_kernels.hpp"

namespace grtmg {

constexpr int kBottomThreads = kGjWaves * kWave;
constexpr int kBottomLevels = 5;
constexpr int kBottomBytes = 150 * 1024;
template <typename T>
constexpr int kBottomMax = 16;

template <typename T>
struct BottomArgs {
    int nl;              // levels, the last one is the coarsest
    int nu_pre, nu_post; // sweeps
    int cubic;           // corrections prolonged by the 4-point cubic, else trilinearly
    Geo geo[kBottomLevels];
    const T *r0, *c0; // first level: right-hand side and coefficient
    T *d0;            // first level: the correction (output)
    double *flag;     // set when the coarsest matrix is singular
};

// LDS of a level: padded d, then (below the first level) r and c.
__host__ __device__ inline int bottom_padded(int n) { return (n + 4) * (n + 4) * (n + 4); }
__host__ __device__ inline int bottom_level_values(int n, bool first)
{
    return (bottom_padded(n) + (first ? 0 : 2 * n * n * n) + 3) / 4 * 4;
}
// Values of the shared scratch below a level of n cells: the pair sums of a restriction, or
// the two stages of the cubic prolongation from n / 2.
__host__ __device__ inline int bottom_scratch_values(int n)
{
    const int p = n / 2 + 4, cub = p * p * n + p * n * n, pairs = n * n * n;
    return cub > pairs ? cub : pairs;
}
// Robin weights of a level kept in LDS (FP32; the FP64 arrays leave no room for them).
template <int BC, typename T>
constexpr bool kBottomWeights = BC == kBcRobin && sizeof(T) == 4;
template <typename T>
inline bool bottom_fits(const int *n, int nl)
{
    if (nl < 2 || nl > kBottomLevels || n[0] > kBottomMax<T>) return false;
    // more cells than one wave solves take the block's Krylov steps, whose registers (taps and
    // vectors of two cells a thread) this kernel does not have beside its own: 14^3 over 7^3 in
    // here, 56^3 solves took 2 to 3 times as long
    if (n[nl - 1] * n[nl - 1] * n[nl - 1] > kWaveMax) return false;
    size_t b = 0;
    for (int l = 0; l < nl; l++) b += (size_t)bottom_level_values(n[l], l == 0) * sizeof(T);
    for (int l = 0; l + 1 < nl && sizeof(T) == 4; l++) b += 12 * (size_t)n[l] * n[l] * sizeof(double);
    const size_t coarse = (size_t)n[nl - 1] * n[nl - 1] * n[nl - 1] * sizeof(T) + 32 + sizeof(CoarseScratch);
    return b + std::max((size_t)bottom_scratch_values(n[0]) * sizeof(T), coarse) <= (size_t)kBottomBytes;
}

// The z pairs of a level that a thread owns, with their pointwise values.
constexpr int kBottomPairs = 2;

// Diagonals of the unscaled Laplacian sum at both members of a pair (lap_diag_sum's values); the
// Robin weights are loaded whether or not a cell lies on a face, so that the loads of all pairs
// are in flight together.
template <int BC>
__device__ __forceinline__ void bottom_diagonals(const Geo &g, const double *gw, int i, int j, int k, double (&ds)[2])
{
    ds[0] = ds[1] = -90.0;
    if constexpr (BC == kBcRobin) {
        const int n = g.n, nn = n * n;
        const double *wx = gw + (i ? 2 : 0) * nn + j * n + k, *wy = gw + (j ? 6 : 4) * nn + i * n + k,
                     *wz = gw + (k ? 10 : 8) * nn + i * n + j;
        const bool ex = i == 0 || i == n - 1, ey = j == 0 || j == n - 1;
#pragma unroll
        for (int e = 0; e < 2; e++) {
            const double x1 = wx[e], x2 = wx[nn + e], y1 = wy[e], y2 = wy[nn + e], z1 = wz[0], z2 = wz[nn];
            const bool ez = k + e == 0 || k + e == n - 1;
            ds[e] += (ex ? 16.0 * x1 - x2 : 0.0) + (ey ? 16.0 * y1 - y2 : 0.0) + (ez ? 16.0 * z1 - z2 : 0.0);
        }
    } else if constexpr (BC == kBcReflect || BC == kBcExtrap) {
#pragma unroll
        for (int e = 0; e < 2; e++) ds[e] = lap_diag_sum<BC>(g, i, j, k + e);
    }
}

template <typename T>
struct BottomPairs {
    int a[kBottomPairs];            // word of the even member in the padded array
    int i[kBottomPairs], j[kBottomPairs], k[kBottomPairs];
    T r[kBottomPairs][2], c[kBottomPairs][2], iv[kBottomPairs][2]; // right-hand side, coefficient, 1 / diagonal
};

// D (padded, all zero on entry of the level) += prolongation of the level below (padded DC, all
// ghosts filled), with the ghosts of the result.
template <int BC, typename T>
__device__ __forceinline__ void bottom_prolong(const Geo &g, const double *gw, T *D, const T *DC, T *scratch, bool cubic)
{
    const int n = g.n, nc = n >> 1, P = n + 4, Q = nc + 4;
    const T w[2][4] = {{T(-5.0 / 128.0), T(35.0 / 128.0), T(105.0 / 128.0), T(-7.0 / 128.0)},
                       {T(-7.0 / 128.0), T(105.0 / 128.0), T(35.0 / 128.0), T(-5.0 / 128.0)}};
    T *t1 = scratch, *t2 = scratch + Q * Q * n;
    // child f of coarse cell f / 2 reads nodes f / 2 - 2 + (f & 1) .. + 3, padded index + 2
    auto sum4 = [&](const T *s, int step, int par) {
        T o = T(0);
#pragma unroll
        for (int e = 0; e < 4; e++) o += (par ? w[1][e] : w[0][e]) * s[e * step];
        return o;
    };
    if (cubic) {
        for (int t = threadIdx.x; t < Q * Q * n; t += kBottomThreads) {
            const int row = t / n, f = t - row * n;
            t1[t] = sum4(DC + row * Q + (f >> 1) + (f & 1), 1, f & 1);
        }
        __syncthreads();
        for (int t = threadIdx.x; t < Q * n * n; t += kBottomThreads) {
            const int x = t / (n * n), rem = t - x * n * n, f = rem / n, z = rem - f * n;
            t2[t] = sum4(t1 + (x * Q + (f >> 1) + (f & 1)) * n + z, n, f & 1);
        }
        __syncthreads();
    }
    for (int t = threadIdx.x; t < n * n * n; t += kBottomThreads) {
        const int row = t / n, k = t - row * n, i = row / n, j = row - i * n;
        T v;
        if (cubic) {
            v = sum4(t2 + (((i >> 1) + (i & 1)) * n + j) * n + k, n * n, i & 1);
        } else {
            const T a = T(0.75), b = T(0.25);
            const int s0 = (((i >> 1) + 2) * Q + (j >> 1) + 2) * Q + (k >> 1) + 2;
            const int dx = (i & 1 ? 1 : -1) * Q * Q, dy = (j & 1 ? 1 : -1) * Q, dz = k & 1 ? 1 : -1;
            auto C = [&](int o) { return DC[s0 + o]; };
            v = a * (a * (a * C(0) + b * C(dz)) + b * (a * C(dy) + b * C(dy + dz))) +
                b * (a * (a * C(dx) + b * C(dx + dz)) + b * (a * C(dx + dy) + b * C(dx + dy + dz)));
        }
        const int at = ((i + 2) * P + j + 2) * P + k + 2;
        v += D[at];
        T gv[3][2];
        padded_ghosts<BC>(n, gw, i, j, k, v, gv);
        padded_store<BC>(D, at, n, i, j, k, v, gv);
    }
    __syncthreads();
}

// Every ghost of a padded array, edges and corners included (the cubic and trilinear stencils
// read them).
template <int BC, typename T>
__device__ __forceinline__ void bottom_fill_ghosts(const Geo &g, T *D)
{
    const int n = g.n, P = n + 4;
    for (int t = threadIdx.x; t < P * P * P; t += kBottomThreads) {
        const int row = t / P, k = t - row * P - 2, i = row / P - 2, j = row % P - 2;
        if ((unsigned)i < (unsigned)n && (unsigned)j < (unsigned)n && (unsigned)k < (unsigned)n) continue;
        int bi, bj, bk;
        const double w = ghost_source<BC>(g, i, j, k, bi, bj, bk);
        const T v = D[((bi + 2) * P + bj + 2) * P + bk + 2];
        D[t] = BC == kBcRobin ? (T)((double)v * w) : BC == kBcZero ? T(0) : v;
    }
    __syncthreads();
}

// One pass of the code below runs every level on the way down (leg = level) and again on the
// way up (leg = 2 (L - 1) - 1 - level): one copy of the smoother serves all of them.  FP64 from
// 16^3: the vector units issue in half of a SIMD's cycles (four waves each); the rest is waiting, a
// quarter of the time for the one wave of the coarsest solve, else at barriers.
template <int BC, typename T>
__global__ void __launch_bounds__(kBottomThreads) k_bottom_psi(const BottomArgs<T> A)
{
    static_assert(kBottomMax<T> * kBottomMax<T> * kBottomMax<T> <= 2 * kBottomPairs * kBottomThreads, "pairs of the first level");
    __shared__ __align__(16) char lds[kBottomBytes];
    T *buf = reinterpret_cast<T *>(lds);
    const int L = A.nl, tid = (int)threadIdx.x;
    const long long zs = A.geo[0].zs;
    const T *gr0 = zsh(A.r0, zs), *gc0 = zsh(A.c0, zs);
    int end = 0; // of the levels' arrays
    for (int l = 0; l < L; l++) end += bottom_level_values(A.geo[l].n, l == 0);
    double *weights = reinterpret_cast<double *>(buf + end); // of every smoothed level (kBottomWeights)
    int scratch_at = end;
    for (int t = tid; t < end; t += kBottomThreads) buf[t] = T(0);
    if constexpr (kBottomWeights<BC, T>) {
        int o = 0;
        for (int l = 0; l + 1 < L; l++) {
            const int cw = 12 * A.geo[l].n * A.geo[l].n;
            for (int t = tid; t < cw; t += kBottomThreads) weights[o + t] = A.geo[l].gw[t];
            o += cw;
        }
        scratch_at += o * (int)(sizeof(double) / sizeof(T));
    }
    T *scratch = buf + scratch_at;
    __syncthreads();
    T *D = buf; // the current level's padded array
#pragma unroll 1
    for (int leg = 0; leg < 2 * (L - 1); leg++) {
        const bool down = leg < L - 1;
        const int l = down ? leg : 2 * (L - 1) - 1 - leg;
        const Geo &g = A.geo[l];
        const int n = g.n, np = n >> 1, P = n + 4, cnt = n * n * np, m = 2 * cnt, mc = m / 8;
        T *below = D + bottom_level_values(n, l == 0); // the next level's arrays
        const double *gw = g.gw;
        if constexpr (kBottomWeights<BC, T>) {
            gw = weights;
            for (int q = 0; q < l; q++) gw += 12 * A.geo[q].n * A.geo[q].n;
        }
        if (!down) {
            bottom_fill_ghosts<BC>(A.geo[l + 1], below);
            bottom_prolong<BC>(g, gw, D, below, scratch, A.cubic != 0);
        }
        BottomPairs<T> B;
        // (a copy for each address space: a pointer that may be either makes generic loads)
        auto load = [&](const T *R, const T *C) {
#pragma unroll
            for (int q = 0; q < kBottomPairs; q++) {
                const int it = min(tid + q * kBottomThreads, cnt - 1);
#pragma unroll
                for (int e = 0; e < 2; e++) {
                    B.r[q][e] = R[2 * it + e];
                    B.c[q][e] = C[2 * it + e];
                }
            }
        };
        if (l)
            load(D + bottom_padded(n), D + bottom_padded(n) + m);
        else
            load(gr0, gc0);
#pragma unroll
        for (int q = 0; q < kBottomPairs; q++) {
            const int it = min(tid + q * kBottomThreads, cnt - 1);
            const int row = it / np;
            B.k[q] = 2 * (it - row * np);
            B.i[q] = row / n;
            B.j[q] = row - B.i[q] * n;
            B.a[q] = ((B.i[q] + 2) * P + B.j[q] + 2) * P + B.k[q] + 2;
        }
#pragma unroll
        for (int q = 0; q < kBottomPairs; q++) {
            double ds[2];
            bottom_diagonals<BC>(g, gw, B.i[q], B.j[q], B.k[q], ds);
#pragma unroll
            for (int e = 0; e < 2; e++) B.iv[q][e] = T(1) / (pinned((T)(ds[e] * g.inv12h2)) + B.c[q][e]);
        }
        const T h2 = (T)g.inv12h2;
        const int passes = 2 * (down ? A.nu_pre : A.nu_post);
#pragma unroll 1
        for (int s = 0; s < passes; s++) {
            const bool from_zero = down && s == 0;
            T val[kBottomPairs], gv[kBottomPairs][3][2];
#pragma unroll
            for (int q = 0; q < kBottomPairs; q++)
                if (tid + q * kBottomThreads < cnt) {
                    const int e = (B.i[q] + B.j[q] + s) & 1, at = B.a[q] + e;
                    const T rr = e ? B.r[q][1] : B.r[q][0], cc = e ? B.c[q][1] : B.c[q][0];
                    const T v = D[at]; // 0 on the first pass, whose neighbours are 0 too
                    val[q] = v + (rr - (from_zero ? T(0) : padded_lap(D, at, P, v) * h2 + cc * v)) *
                                     (e ? B.iv[q][1] : B.iv[q][0]);
                    padded_ghosts<BC>(n, gw, B.i[q], B.j[q], B.k[q] + e, val[q], gv[q]);
                }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < kBottomPairs; q++)
                if (tid + q * kBottomThreads < cnt) {
                    const int e = (B.i[q] + B.j[q] + s) & 1;
                    padded_store<BC>(D, B.a[q] + e, n, B.i[q], B.j[q], B.k[q] + e, val[q], gv[q]);
                }
            __syncthreads();
        }
        if (!down) {
            if (l) D -= bottom_level_values(A.geo[l - 1].n, l == 1);
            continue;
        }
        // the defect and the coefficient, summed over the pair, then over the four pairs of a
        // coarse cell
        T *Rc = below + bottom_padded(n >> 1);
#pragma unroll
        for (int q = 0; q < kBottomPairs; q++)
            if (tid + q * kBottomThreads < cnt) {
                T s = T(0);
#pragma unroll
                for (int e = 0; e < 2; e++) {
                    const T v = D[B.a[q] + e];
                    s += B.r[q][e] - (padded_lap(D, B.a[q] + e, P, v) * h2 + B.c[q][e] * v);
                }
                scratch[tid + q * kBottomThreads] = s;
                scratch[cnt + tid + q * kBottomThreads] = B.c[q][0] + B.c[q][1];
            }
        __syncthreads();
        for (int t = tid; t < mc; t += kBottomThreads) {
            const int row = t / np, K = t - row * np, I = row / np, J = row - I * np;
            const T *s0 = scratch + (2 * I * n + 2 * J) * np + K, *s1 = s0 + n * np; // rows (2I, 2J), (2I + 1, 2J)
            Rc[t] = (s0[0] + s0[np] + s1[0] + s1[np]) * T(0.125);
            s0 += cnt;
            s1 += cnt;
            Rc[mc + t] = (s0[0] + s0[np] + s1[0] + s1[np]) * T(0.125);
        }
        __syncthreads();
        if (l + 2 < L) {
            D = below;
            continue;
        }
        // the coarsest level: solved into the scratch, then into its padded array
        // (at a constant offset at the end of lds: of an address rounded up as an integer the
        // compiler does not know any more that it is in LDS)
        CoarseScratch &cs = *reinterpret_cast<CoarseScratch *>(lds + kBottomBytes - (sizeof(CoarseScratch) + 15) / 16 * 16);
        for (int t = tid; t < mc; t += kBottomThreads) scratch[t] = T(0); // stays 0 if singular
        __syncthreads();
        coarse_psi_solve<BC, T>(A.geo[l + 1], mc, Rc + mc, Rc, scratch, zsh(A.flag, zs), cs);
        __syncthreads();
        const int Q = np + 4;
        for (int t = tid; t < mc; t += kBottomThreads) {
            const int row = t / np, k = t - row * np, i = row / np, j = row - i * np;
            below[((i + 2) * Q + j + 2) * Q + k + 2] = scratch[t];
        }
        __syncthreads();
    }
    T *out = zsh(A.d0, zs);
    const int n = A.geo[0].n, P = n + 4;
    for (int t = tid; t < n * n * n; t += kBottomThreads) {
        const int row = t / n, k = t - row * n, i = row / n, j = row - i * n;
        out[t] = buf[((i + 2) * P + j + 2) * P + k + 2];
    }
}

} // namespace grtmg
