// mg_refine.hpp -- kernels of the static mesh refinement by nested boxes (Key
// features, "Adaptive Mesh Refinement": refined boxes over the base grid; "Fast").
//
// Levels: a base grid, then boxes, each refined by 2 over m^3 cells of its parent
// whose corner is parent cell (b0, b0, b0) (nf = 2m cells per axis).  A parent
// cell under a box holds the average of its 8 children; a box's two ghost layers
// are the children of the parent cells around it by the 4-point cubic (weights
// (-5, 35, 105, -7)/128 and mirror).  A box is solved as a grid of its own under
// the zero ghost rule with a forcing that carries the interpolated ghosts,
// f = sum over stencil taps outside the box of w g / (12 h_box^2); a parent takes
// the FAS forcing tau = R H_box - H_parent(R u_box) on the cells under the box.  A
// box keeps a margin of at least 3 parent cells, so every cubic stencil stays inside
// the parent and no boundary rule is needed here.  BoxGeo names a parent-box pair:
// nc is the parent's cells per axis.
#pragma once

#include "mg_kernels.hpp"

namespace grtmg {

struct BoxGeo {
    int nc;   // base cells per axis
    int b0;   // base index of the box's first cell on every axis
    int m;    // base cells covered per axis (the box has 2m fine cells per axis)
};

__device__ __forceinline__ int64_t cidx(int n, int i, int j, int k) { return ((int64_t)i * n + j) * n + k; }

// Cubic weights of the child of parity p (0: nearer the lower neighbour) on the four
// base nodes I - 2 + p .. I + 1 + p.
__device__ __forceinline__ double cubic_w(int p, int e)
{
    const double w0[4] = {-5.0 / 128.0, 35.0 / 128.0, 105.0 / 128.0, -7.0 / 128.0};
    const double w1[4] = {-7.0 / 128.0, 105.0 / 128.0, 35.0 / 128.0, -5.0 / 128.0};
    return p ? w1[e] : w0[e];
}

// Base cells under the box take the average of their 8 children: uc[b0 + I..] = R uf.
__global__ void __launch_bounds__(kBlock) k_box_restrict(BoxGeo bx, const double *__restrict__ uf,
                                                         double *__restrict__ uc)
{
    const int m = bx.m, nf = 2 * m;
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (t >= (int64_t)m * m * m) return;
    const int K = (int)(t % m), J = (int)((t / m) % m), I = (int)(t / ((int64_t)m * m));
    double s = 0.0;
#pragma unroll
    for (int di = 0; di < 2; di++)
#pragma unroll
        for (int dj = 0; dj < 2; dj++)
#pragma unroll
            for (int dk = 0; dk < 2; dk++) s += uf[cidx(nf, 2 * I + di, 2 * J + dj, 2 * K + dk)];
    uc[cidx(bx.nc, bx.b0 + I, bx.b0 + J, bx.b0 + K)] = 0.125 * s;
}

// The box's ghosts across its faces, from the cubic of the base field: one thread per face and
// line (blockIdx.y: face x-, x+, y-, y+, z-, z+; two in-face coordinates) forms both layers,
// the two children of the base cell beside the face, from that cell's 5 nodes along the normal
// and the 4 x 4 in-face nodes of the line.  gv: layer l of face f at (2 f + l) nf^2.  (Formed
// per fine cell instead, every wave of a z line waited for its few boundary lanes' 64-node
// sums: 24 us for a 64^3 box, 14 us with this and the forcing kernel below.)
__global__ void __launch_bounds__(kBlock) k_box_ghosts(BoxGeo bx, const double *__restrict__ uc, double *__restrict__ gv)
{
    const int nf = 2 * bx.m, nc = bx.nc, t = (int)(blockIdx.x * kBlock + threadIdx.x);
    if (t >= nf * nf) return;
    const int face = (int)blockIdx.y, ax = face >> 1, hi = face & 1;
    const int64_t st[3] = {(int64_t)nc * nc, nc, 1};
    const int64_t sn = st[ax], sa = ax == 0 ? st[1] : st[0], sb = ax == 2 ? st[1] : st[2];
    const int a = t / nf, b = t - a * nf;
    // base cell beside the face, and the first in-face nodes
    const int I = hi ? bx.b0 + bx.m : bx.b0 - 1, pa = a & 1, pb = b & 1;
    const double *q = uc + (I - 2) * sn + (bx.b0 + (a >> 1) - 2 + pa) * sa + (bx.b0 + (b >> 1) - 2 + pb) * sb;
    double v[5];
#pragma unroll
    for (int e = 0; e < 5; e++) {
        double sy = 0.0;
#pragma unroll
        for (int x = 0; x < 4; x++) {
            double sz = 0.0;
#pragma unroll
            for (int y = 0; y < 4; y++) sz += cubic_w(pb, y) * q[e * sn + x * sa + y * sb];
            sy += cubic_w(pa, x) * sz;
        }
        v[e] = sy;
    }
#pragma unroll
    for (int c = 0; c < 2; c++) { // child c of the cell: layer 0 is the one next to the face
        double o = 0.0;
#pragma unroll
        for (int e = 0; e < 4; e++) o += cubic_w(c, e) * v[e + c];
        gv[(size_t)(2 * face + (hi ? c : 1 - c)) * nf * nf + t] = o;
    }
}

// Forcing of the box under the zero rule: the taps of every fine cell that fall
// outside the box, on the interpolated ghosts gv, times 1/(12 (h/2)^2), plus the box's
// own FAS forcing tau from a finer box inside it (null: none).
__global__ void __launch_bounds__(kBlock) k_box_ghost_forcing(BoxGeo bx, double inv12h2, const double *__restrict__ gv,
                                                              const double *__restrict__ tau, double *__restrict__ ff)
{
    const int nf = 2 * bx.m;
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const unsigned un = (unsigned)nf;
    if (t >= (int64_t)nf * nf * nf) return;
    const unsigned row = (unsigned)t / un;
    const int k = (int)((unsigned)t - row * un), i = (int)(row / un), j = (int)(row - (unsigned)i * un);
    const size_t nn = (size_t)nf * nf;
    const int c[3] = {i, j, k}, A[3] = {j, i, i}, B[3] = {k, k, j};
    double f = 0.0;
#pragma unroll
    for (int ax = 0; ax < 3; ax++) {
        const bool hi = c[ax] >= nf - 2;
        const int d = hi ? nf - 1 - c[ax] : c[ax]; // distance from the face
        if (d >= 2) continue;                      // every tap along this axis is inside
        const double *g = gv + 2 * (2 * ax + (hi ? 1 : 0)) * nn + (unsigned)(A[ax] * nf + B[ax]);
        f += d == 0 ? 16.0 * g[0] - g[nn] : -g[0];
    }
    ff[t] = f * inv12h2 + (tau ? tau[t] : 0.0);
}

// FAS forcing of the base grid: tau = R H_f - H_c on covered cells, zero elsewhere.
__global__ void __launch_bounds__(kBlock) k_box_tau(BoxGeo bx, const double *__restrict__ Hf,
                                                    const double *__restrict__ Hc, double *__restrict__ fc)
{
    const int nc = bx.nc, m = bx.m, nf = 2 * m;
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (t >= (int64_t)nc * nc * nc) return;
    const int K = (int)(t % nc) - bx.b0, J = (int)((t / nc) % nc) - bx.b0, I = (int)(t / ((int64_t)nc * nc)) - bx.b0;
    if ((unsigned)I >= (unsigned)m || (unsigned)J >= (unsigned)m || (unsigned)K >= (unsigned)m) {
        fc[t] = 0.0;
        return;
    }
    double s = 0.0;
#pragma unroll
    for (int di = 0; di < 2; di++)
#pragma unroll
        for (int dj = 0; dj < 2; dj++)
#pragma unroll
            for (int dk = 0; dk < 2; dk++) s += Hf[cidx(nf, 2 * I + di, 2 * J + dj, 2 * K + dk)];
    fc[t] = 0.125 * s - Hc[t];
}

// Box correction by the base grid's change: uf += cubic interpolation of uc - uc_old, one
// thread per covered base cell writing its 8 children from the tile's staged differences (tiles
// of k_prolong_cubic_add_staged; read through the caches, a thread took 1024 loads: 61 us for
// 32^3 covered cells, 7 us staged).
__global__ void __launch_bounds__(kBlock) k_box_correct(BoxGeo bx, const double *__restrict__ uc,
                                                        const double *__restrict__ uc_old, double *__restrict__ uf)
{
    using Q = CubicTile<8>;
    __shared__ double S[Q::kSX][Q::kSY][Q::kSZP];
    const int m = bx.m, nby = (m + Q::kY - 1) / Q::kY, nbz = (m + Q::kZ - 1) / Q::kZ;
    const int bz = blockIdx.x % nbz, by = (blockIdx.x / nbz) % nby, bxx = blockIdx.x / (nbz * nby);
    const int I0 = bxx * Q::kX, J0 = by * Q::kY, K0 = bz * Q::kZ;
    const int t = threadIdx.x, kz = t % Q::kZ, jy = (t / Q::kZ) % Q::kY, ix = t / (Q::kZ * Q::kY);
    for (int q = t; q < Q::kSX * Q::kSY * Q::kSZ; q += kBlock) {
        const int a = q / (Q::kSY * Q::kSZ), rem = q % (Q::kSY * Q::kSZ), b = rem / Q::kSZ, e = rem % Q::kSZ;
        const int I = I0 - 2 + a, J = J0 - 2 + b, K = K0 - 2 + e;
        if (I < m + 2 && J < m + 2 && K < m + 2) { // the margin of 3 cells keeps these inside the base grid
            const int64_t at = cidx(bx.nc, bx.b0 + I, bx.b0 + J, bx.b0 + K);
            S[a][b][e] = uc[at] - uc_old[at];
        }
    }
    __syncthreads();
    if (I0 + ix < m && J0 + jy < m && K0 + kz < m)
        cubic_children_add<double>([&](int a, int b, int e) { return S[ix + a][jy + b][kz + e]; }, uf, 2 * m, I0 + ix,
                                   J0 + jy, K0 + kz);
}

// Composite norm partials of one level: sum of H^2 times the cell volume over the
// cells no finer box covers (child.m = 0: no finer box), and max |H|; grid-stride.
__global__ void __launch_bounds__(kBlock) k_level_norm(int n, BoxGeo child, double vol, const double *__restrict__ H,
                                                       double *__restrict__ partials)
{
    const int64_t m3 = (int64_t)n * n * n;
    double v[2] = {0.0, 0.0};
    for (int64_t q = (int64_t)blockIdx.x * kBlock + threadIdx.x; q < m3; q += (int64_t)gridDim.x * kBlock) {
        const int K = (int)(q % n) - child.b0, J = (int)((q / n) % n) - child.b0, I = (int)(q / ((int64_t)n * n)) - child.b0;
        if ((unsigned)I < (unsigned)child.m && (unsigned)J < (unsigned)child.m && (unsigned)K < (unsigned)child.m)
            continue;
        const double h = H[q];
        v[0] += vol * h * h;
        v[1] = fmax(v[1], fabs(h));
    }
    block_reduce_store<2>(v, 0x2u, partials + 2 * (int64_t)blockIdx.x);
}

} // namespace grtmg
