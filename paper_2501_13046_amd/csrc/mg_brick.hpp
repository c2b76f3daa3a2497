// mg_brick.hpp -- psi kernels on LDS bricks of any even grid and boundary rule.
//
// A workgroup of 4 waves owns a brick of TX (x) x TYB (y) x BZ (z) cells (BZ = 64: 8 rows
// of y, two per wave; BZ = 32: 16 rows, four per wave) and stages it with a 2-cell halo
// once.  The grid need not be a multiple of the brick: staged positions past the grid hold
// values nobody uses, and only cells inside are written.
//
// Ghosts.  psi's operator reads along the axes only, so a ghost is one grid cell times a
// weight that depends on its place on a face and its layer.  The Robin weights
// |x_b| / |x_g| are formed once per level at set-up (Geo::gw, FP64); a brick is staged with
// the cells the rule reads and those next to a face weigh their ghosts in LDS afterwards, so
// no global load waits for another.  Formed in place, a ghost took two square roots and a
// division in FP64, and every wave paid for them in every row, since every z line has two
// ends.  Robin 256^3: colour pass 240 -> 85 us (268 MB, 3.2 TB/s), defect restriction 337 -> 76
// us, residual without W 486 -> 232 us; weights applied while staging left the pass at 106 us.
#pragma once

#include "mg_tiled.hpp"

namespace grtmg {

// Robin weights of every level of a context (blockIdx.z) in one launch: at (face * 2 + layer) n^2,
// then the two in-face coordinates, row-major.  A launch per level took 10 to 45 us of a context's
// set-up.
constexpr int kMaxLevels = 16;
struct GhostLevels {
    Geo g[kMaxLevels];
    double *gw[kMaxLevels];
};
__global__ void __launch_bounds__(kBlock) k_ghost_weights(GhostLevels lv)
{
    const Geo &g = lv.g[blockIdx.z];
    double *gw = lv.gw[blockIdx.z];
    const int n = g.n, t = (int)(blockIdx.x * kBlock + threadIdx.x);
    if (t >= n * n) return;
    const int a = t / n, b = t - a * n, face = (int)blockIdx.y >> 1, layer = (int)blockIdx.y & 1;
    const int out = face & 1 ? n + layer : -1 - layer;
    const int i = face < 2 ? out : a, j = face < 2 ? a : face < 4 ? out : b, k = face < 4 ? b : out;
    int bi, bj, bk;
    gw[(size_t)blockIdx.y * n * n + t] = ghost_source<kBcRobin>(g, i, j, k, bi, bj, bk);
}

template <int TX, int BZ>
struct BrickGeom {
    using G = ZGeom<BZ>;
    static constexpr int kPlane = G::kPYB * G::kPZB;
    // brick rows of a thread that shares its wave with adjacent rows (paired y rows meet
    // in a lane exchange); G::row() deals rows of one y parity to a wave instead
    __device__ static int adjacent_row() { return threadIdx.y * G::kRPW + (int)threadIdx.x / G::kLPR; }
};

template <int TX, int BZ>
__device__ __forceinline__ void brick_origin(const TileMap &t, int &x0, int &y0, int &z0)
{
    const int total = t.nx * t.ny * t.nz;
    const int b = blockIdx.x;
    int logical = b;
    if (total % kXCD == 0) logical = (b % kXCD) * (total / kXCD) + b / kXCD;
    const int bz = logical % t.nz, rest = logical / t.nz;
    x0 = (rest / t.ny) * TX;
    y0 = (rest % t.ny) * ZGeom<BZ>::kTYB;
    z0 = bz * BZ;
}

// Grid index that position i reads along one axis (positions past the ghost layers, which
// only bricks that overhang the grid have, read some cell of the grid).
template <int BC>
__device__ __forceinline__ int brick_src(int i, int n)
{
    if constexpr (BC == kBcPeriodic) return wrap(i, n);
    if constexpr (BC == kBcReflect) return clampc(mirror(i, n), n);
    return clampc(i, n);
}

// Staged values at (x, y, z) and (x, y, z + 1), z even, of plane brick_src(x) (ap): the grid
// cells the boundary rule reads there; the weights of the Robin and zero rules are applied in
// LDS by weigh_ghosts, so that no load waits for another one.
template <int BC, typename T>
__device__ __forceinline__ typename Vec2<T>::type brick_pair(const Geo &g, const T *ap, int y, int z)
{
    using V2 = typename Vec2<T>::type;
    const int n = g.n;
    const T *row = ap + (unsigned)(brick_src<BC>(y, n) * n);
    if constexpr (BC == kBcPeriodic) {
        return *reinterpret_cast<const V2 *>(row + wrap(z, n));
    } else {
        const int zs = z < 0 ? 0 : (z >= n ? n - 2 : z);
        const V2 v = *reinterpret_cast<const V2 *>(row + zs);
        V2 o = v; // z ghosts: (-2, -1) or (n, n + 1)
        if constexpr (BC == kBcReflect) {
            o.x = zs != z ? v.y : v.x;
            o.y = zs != z ? v.x : v.y;
        } else {
            o.x = z >= n ? v.y : v.x;
            o.y = z < 0 ? v.x : v.y;
        }
        return o;
    }
}

// Ghost weights of a staged brick (Robin: the level's table; zero rule: 0), on the ghosts that
// the axis taps of the brick's cells read.  The branches are uniform: bricks away from the
// faces leave at once.  A brick that reaches a face holds both layers beyond it (the side, the
// brick's extents and its origin are even).
template <int BC, typename T, int TX, int BZ>
__device__ __forceinline__ void weigh_ghosts(T (*s)[ZGeom<BZ>::kPYB][ZGeom<BZ>::kPZB], const Geo &g, int x0, int y0,
                                             int z0)
{
    using G = ZGeom<BZ>;
    if constexpr (BC == kBcRobin || BC == kBcZero) {
        const int n = g.n, tid = threadIdx.y * kLanes + threadIdx.x;
        const int left[3] = {n - x0, n - y0, n - z0}, org[3] = {x0, y0, z0}, ext[3] = {TX, G::kTYB, BZ};
        if (x0 && y0 && z0 && left[0] > TX && left[1] > G::kTYB && left[2] > BZ) return;
        __syncthreads();
        static_for<6>([&](auto ff) {
            constexpr int f = decltype(ff)::value, ax = f / 2;
            constexpr int A = ax == 0 ? 1 : 0, B = ax == 2 ? 1 : 2;          // the in-face axes
            constexpr int EB = B == 2 ? BZ : G::kTYB, CNT = (A == 0 ? TX : G::kTYB) * EB;
            if (f & 1 ? left[ax] > ext[ax] : org[ax] != 0) return;
            const double *w = g.gw + 2 * f * (size_t)n * n;
            for (int t = tid; t < CNT; t += kTY * kLanes) {
                const int a = t / EB, b = t % EB;
                if (a >= left[A] || b >= left[B]) continue;
                T *at[2];
#pragma unroll
                for (int l = 0; l < 2; l++) {
                    int i[3]; // staged index of layer l
                    i[A] = a + 2;
                    i[B] = b + 2;
                    i[ax] = f & 1 ? left[ax] + 2 + l : 1 - l;
                    at[l] = &s[i[0]][i[1]][(i[2] & 1) * G::kHalfB + (i[2] >> 1)];
                }
                if constexpr (BC == kBcZero) {
                    *at[0] = *at[1] = T(0);
                } else {
                    const unsigned q = (unsigned)((org[A] + a) * n + org[B] + b);
                    const double w1 = w[q], w2 = w[(size_t)n * n + q];
                    *at[0] = (T)((double)*at[0] * w1);
                    *at[1] = (T)((double)*at[1] * w2);
                }
            }
        });
    }
}

// The brick and its halo in LDS: row (xx, yy) holds z0 - 2 .. z0 + BZ + 1, even and odd z in
// separate halves.  All loads of a thread are issued before its first store.
template <int BC, typename T, int TX, int BZ>
__device__ __forceinline__ void stage_brick(T (*s)[ZGeom<BZ>::kPYB][ZGeom<BZ>::kPZB], const Geo &g,
                                            const T *__restrict__ a, int x0, int y0, int z0)
{
    using G = ZGeom<BZ>;
    using V2 = typename Vec2<T>::type;
    constexpr int NI = (G::kPYB + G::kTYB - 1) / G::kTYB;
    constexpr int NE = (TX + 4) * G::kPYB * 2, EPT = (NE + kTY * kLanes - 1) / (kTY * kLanes);
    const int n = g.n, ty = G::row(), p = G::pair(), tid = threadIdx.y * kLanes + threadIdx.x;
    const size_t nn = (size_t)n * n;
    V2 v[TX + 4][NI], e[EPT];
#pragma unroll
    for (int xx = 0; xx < TX + 4; xx++) {
        const int x = x0 + xx - 2;
        const T *ap = a + (size_t)brick_src<BC>(x, n) * nn;
#pragma unroll
        for (int i = 0; i < NI; i++) {
            const int yy = i * G::kTYB + ty;
            if (G::kPYB % G::kTYB == 0 || yy < G::kPYB) v[xx][i] = brick_pair<BC, T>(g, ap, y0 + yy - 2, z0 - 2 + 2 * p);
        }
    }
    // the two last pairs of every row
#pragma unroll
    for (int q = 0; q < EPT; q++) {
        const int t = tid + q * kTY * kLanes;
        if (NE % (kTY * kLanes) == 0 || t < NE) {
            const int row = t >> 1, x = x0 + row / G::kPYB - 2;
            e[q] = brick_pair<BC, T>(g, a + (size_t)brick_src<BC>(x, n) * nn, y0 + row % G::kPYB - 2,
                                     z0 - 2 + 2 * (G::kLPR + (t & 1)));
        }
    }
#pragma unroll
    for (int xx = 0; xx < TX + 4; xx++)
#pragma unroll
        for (int i = 0; i < NI; i++) {
            const int yy = i * G::kTYB + ty;
            if (G::kPYB % G::kTYB == 0 || yy < G::kPYB) {
                s[xx][yy][p] = v[xx][i].x;
                s[xx][yy][G::kHalfB + p] = v[xx][i].y;
            }
        }
#pragma unroll
    for (int q = 0; q < EPT; q++) {
        const int t = tid + q * kTY * kLanes;
        if (NE % (kTY * kLanes) == 0 || t < NE) {
            const int row = t >> 1, ep = G::kLPR + (t & 1);
            T *dst = s[row / G::kPYB][row % G::kPYB];
            dst[ep] = e[q].x;
            dst[G::kHalfB + ep] = e[q].y;
        }
    }
    weigh_ghosts<BC, T, TX, BZ>(s, g, x0, y0, z0);
}

// Taps around cell (x0 + TT, row, 2 p + PAR) of a staged brick; b points at word p of staged
// row (plane 0, row).
template <typename T, int PAR, int TT, int BZ>
struct BrickTaps {
    using G = ZGeom<BZ>;
    static constexpr bool kOrdered = true;
    const T *b;
    template <int DX, int DY, int DZ>
    __device__ __forceinline__ T at() const
    {
        return b[(TT + 2 + DX) * G::kPYB * G::kPZB + (2 + DY) * G::kPZB + G::template zoff<PAR, DZ>()];
    }
};

// ---------------------------------------------------------------------------------------
// psi smoother colour pass.  The lane owning a z pair updates the member of the active
// colour and copies the other; a wave's rows have one y parity, so the member is uniform.
// Bound by memory (16 B a cell).
// ---------------------------------------------------------------------------------------
template <int BC, typename T, int PAR, int TT, int BZ>
__device__ __forceinline__ void brick_psi_cell(const Geo &g, const T *row0, T rv, T cv, T *__restrict__ out, int x,
                                               int y, int z, T h2, T dlap)
{
    const BrickTaps<T, PAR, TT, BZ> S{row0};
    RegTaps<T> D;
    D.get_lap(S);
    const unsigned qrow = ((unsigned)x * (unsigned)g.n + (unsigned)y) * (unsigned)g.n + (unsigned)z;
    const unsigned qa = qrow + PAR, qb = qrow + (PAR ^ 1);
    const T v = D.c();
    const T Ad = (D.dxx(v) + D.dyy(v) + D.dzz(v)) * h2 + cv * v;
    T diag;
    if constexpr (BC == kBcPeriodic)
        diag = dlap + cv;
    else
        diag = pinned((T)(lap_diag_sum<BC>(g, x, y, z + PAR) * g.inv12h2)) + cv;
    out[qa] = v + (rv - Ad) / diag;
    out[qb] = D.template at<0, 0, (PAR ? -1 : 1)>();
}

template <int BC, typename T, int TX, int BZ>
__global__ void __launch_bounds__(kTY *kLanes) k_pass_psi_brick(Geo g, TileMap tm, const T *__restrict__ in,
                                                               T *__restrict__ out, const T *__restrict__ r,
                                                               const T *__restrict__ c, int colour)
{
    using G = ZGeom<BZ>;
    in = zsh(in, g.zs);
    out = zsh(out, g.zs);
    r = zsh(r, g.zs);
    c = zsh(c, g.zs);
    __shared__ T lds[TX + 4][G::kPYB][G::kPZB];
    int x0, y0, z0;
    brick_origin<TX, BZ>(tm, x0, y0, z0);
    const int n = g.n, ty = G::row(), p = G::pair(), y = y0 + ty, z = z0 + 2 * p;
    const int p0 = (colour + x0 + y) & 1; // z0 is even
    const bool in_grid = y < n && z < n;
    // r and c of the active cells, in flight with the brick's loads
    T rv[TX], cv[TX];
#pragma unroll
    for (int tt = 0; tt < TX; tt++) {
        rv[tt] = cv[tt] = T(0);
        if (in_grid && x0 + tt < n) {
            const unsigned q = ((unsigned)(x0 + tt) * (unsigned)n + (unsigned)y) * (unsigned)n + (unsigned)z +
                               (unsigned)((p0 ^ tt) & 1);
            rv[tt] = r[q];
            cv[tt] = c[q];
        }
    }
    stage_brick<BC, T, TX, BZ>(lds, g, in, x0, y0, z0);
    __syncthreads();
    if (!in_grid) return;
    const T h2 = (T)g.inv12h2;
    const T dlap = pinned((T)(-90.0 * g.inv12h2));
    const T *row0 = &lds[0][ty][p];
    static_for<TX>([&](auto tt) {
        constexpr int TT = decltype(tt)::value;
        const int x = x0 + TT;
        if (x < n) {
            if ((p0 ^ TT) & 1)
                brick_psi_cell<BC, T, 1, TT, BZ>(g, row0, rv[TT], cv[TT], out, x, y, z, h2, dlap);
            else
                brick_psi_cell<BC, T, 0, TT, BZ>(g, row0, rv[TT], cv[TT], out, x, y, z, h2, dlap);
        }
    });
}

// ---------------------------------------------------------------------------------------
// psi defect r - (L_h + c) d restricted to the next coarser level (mean of the 8 children),
// the coefficient restricted the same way (cc_out, may be null) and the coarse level's first
// colour pass from zero (d1_out, may be null; needs cc_out).  Each lane evaluates both
// members of its z pair on every plane of the brick; paired y rows are adjacent in the wave.
// ---------------------------------------------------------------------------------------
template <int BC, typename T, int TX, int BZ>
__global__ void __launch_bounds__(kTY *kLanes) k_defect_restrict_psi_brick(Geo g, TileMap tm, const T *__restrict__ d,
                                                                          const T *__restrict__ r,
                                                                          const T *__restrict__ c,
                                                                          T *__restrict__ rc_out, T *__restrict__ cc_out,
                                                                          T *__restrict__ d1_out, Geo gc)
{
    using G = ZGeom<BZ>;
    using V2 = typename Vec2<T>::type;
    static_assert(TX % 2 == 0 && G::kRPW % 2 == 0, "whole coarse cells per brick, paired rows in one wave");
    d = zsh(d, g.zs);
    r = zsh(r, g.zs);
    c = zsh(c, g.zs);
    rc_out = zsh(rc_out, g.zs);
    cc_out = zsh(cc_out, g.zs);
    d1_out = zsh(d1_out, g.zs);
    __shared__ T lds[TX + 4][G::kPYB][G::kPZB];
    int x0, y0, z0;
    brick_origin<TX, BZ>(tm, x0, y0, z0);
    const int n = g.n, ty = BrickGeom<TX, BZ>::adjacent_row(), p = G::pair(), y = y0 + ty, z = z0 + 2 * p;
    const bool in = y < n && z < n;
    V2 rv[TX], cv[TX]; // in flight with the brick's loads
#pragma unroll
    for (int tt = 0; tt < TX; tt++) {
        rv[tt].x = rv[tt].y = cv[tt].x = cv[tt].y = T(0);
        if (in && x0 + tt < n) {
            const unsigned q = ((unsigned)(x0 + tt) * (unsigned)n + (unsigned)y) * (unsigned)n + (unsigned)z;
            rv[tt] = *reinterpret_cast<const V2 *>(r + q);
            cv[tt] = *reinterpret_cast<const V2 *>(c + q);
        }
    }
    stage_brick<BC, T, TX, BZ>(lds, g, d, x0, y0, z0);
    __syncthreads();
    const T h2 = (T)g.inv12h2;
    const T *row0 = &lds[0][ty][p];
    T sd = T(0), sc = T(0);
    static_for<TX>([&](auto tt) {
        constexpr int TT = decltype(tt)::value;
        const int x = x0 + TT;
        if (x < n) { // uniform; n is even, so plane pairs are whole
            if (in) {
                auto defect = [&](auto par, T rr, T cc) {
                    constexpr int PAR = decltype(par)::value;
                    RegTaps<T> D;
                    D.get_lap(BrickTaps<T, PAR, TT, BZ>{row0});
                    const T v = D.c();
                    return rr - ((D.dxx(v) + D.dyy(v) + D.dzz(v)) * h2 + cc * v);
                };
                sd += defect(std::integral_constant<int, 0>{}, rv[TT].x, cv[TT].x) +
                      defect(std::integral_constant<int, 1>{}, rv[TT].y, cv[TT].y);
                sc += cv[TT].x + cv[TT].y;
            }
            if constexpr (TT & 1) {
                sd += __shfl_xor(sd, G::kLPR, kWave);
                sc += __shfl_xor(sc, G::kLPR, kWave);
                if (in && !(ty & 1)) {
                    const int nc = n >> 1, I = x >> 1, J = y >> 1, K = z >> 1;
                    const unsigned qc = ((unsigned)I * (unsigned)nc + (unsigned)J) * (unsigned)nc + (unsigned)K;
                    const T rcv = sd * T(0.125), ccv = sc * T(0.125);
                    rc_out[qc] = rcv;
                    if (cc_out) cc_out[qc] = ccv;
                    if (d1_out) d1_out[qc] = first_pass_psi<BC, T>(gc, I, J, K, rcv, ccv);
                }
                sd = sc = T(0);
            }
        }
    });
}

// ---------------------------------------------------------------------------------------
// Residual of eq. Ham without W (psi-only contexts, FP64): outputs as k_residual.  Each lane
// owns a z pair of every plane of its brick; bound by FP64 arithmetic (a square root and
// two divisions per cell with a puncture) and memory.
// ---------------------------------------------------------------------------------------
template <int BC, typename T, int TX, int BZ>
__global__ void __launch_bounds__(kTY *kLanes) k_residual_psi_brick(Geo g, TileMap tm, ResArgs a)
{
    using G = ZGeom<BZ>;
    a = res_shift(a, g.zs);
    __shared__ double lds[TX + 4][G::kPYB][G::kPZB];
    int x0, y0, z0;
    brick_origin<TX, BZ>(tm, x0, y0, z0);
    using V2 = typename Vec2<T>::type;
    const int n = g.n, ty = G::row(), p = G::pair(), y = y0 + ty, z = z0 + 2 * p;
    const bool in = y < n && z < n;
    const unsigned q0 = ((unsigned)x0 * (unsigned)n + (unsigned)y) * (unsigned)n + (unsigned)z;
    const size_t nn = (size_t)n * n;
    // the pointwise fields, in flight with the brick's loads
    double2 r5[TX], r1[TX], bp[TX], ba[TX], ff[TX];
#pragma unroll
    for (int t = 0; t < TX; t++) {
        r5[t] = r1[t] = bp[t] = ba[t] = ff[t] = make_double2(0.0, 0.0);
        if (in && x0 + t < n) {
            const size_t q = q0 + t * nn;
            r5[t] = *reinterpret_cast<const double2 *>(a.rho5 + q);
            r1[t] = *reinterpret_cast<const double2 *>(a.rho1 + q);
            if (a.psi0f) bp[t] = *reinterpret_cast<const double2 *>(a.psi0f + q);
            if (a.A2bg) ba[t] = *reinterpret_cast<const double2 *>(a.A2bg + q);
            if (a.f) ff[t] = *reinterpret_cast<const double2 *>(a.f + q);
        }
    }
    stage_brick<BC, double, TX, BZ>(lds, g, a.u, x0, y0, z0);
    __syncthreads();
    const double K2 = a.K2p ? *a.K2p : a.K2;
    const T dlap = pinned((T)(-90.0 * g.inv12h2));
    const double *row0 = &lds[0][ty][p];
    ResSums acc;
    if (in)
        static_for<TX>([&](auto tt) {
            constexpr int TT = decltype(tt)::value;
            const int x = x0 + TT;
            if (x < n) { // uniform
                double H[2], c[2];
                static_for<2>([&](auto par) {
                    constexpr int PAR = decltype(par)::value;
                    RegTaps<double> D;
                    D.get_lap(BrickTaps<double, PAR, TT, BZ>{row0});
                    const double uc = D.c();
                    const double psi = (a.psi0f ? (PAR ? bp[TT].y : bp[TT].x) : psi0_at(g, a.pmass, x, y, z + PAR)) + uc;
                    ham_point(g, a, K2, D.dxx(uc) + D.dyy(uc) + D.dzz(uc), psi, PAR ? r5[TT].y : r5[TT].x,
                              PAR ? r1[TT].y : r1[TT].x, PAR ? ba[TT].y : ba[TT].x, PAR ? ff[TT].y : ff[TT].x, H[PAR],
                              c[PAR]);
                    acc.hsum += H[PAR] * H[PAR];
                    acc.hmax = fmax(acc.hmax, fabs(H[PAR]));
                });
                const size_t q = q0 + TT * nn;
                if (a.H) *reinterpret_cast<double2 *>(a.H + q) = make_double2(H[0], H[1]);
                if (a.c) *reinterpret_cast<double2 *>(a.c + q) = make_double2(c[0], c[1]);
                V2 r, rc, d1;
                r.x = pinned((T)(-H[0]));
                r.y = pinned((T)(-H[1]));
                rc.x = pinned((T)c[0]);
                rc.y = pinned((T)c[1]);
                if (a.r) *reinterpret_cast<V2 *>((T *)a.r + q) = r;
                if (a.rc) *reinterpret_cast<V2 *>((T *)a.rc + q) = rc;
                if (a.d1) { // first colour pass from zero
                    const int act = (x + y) & 1; // the colour 0 member
                    T diag = dlap;
                    if constexpr (BC != kBcPeriodic) diag = pinned((T)(lap_diag_sum<BC>(g, x, y, z + act) * g.inv12h2));
                    d1.x = act ? T(0) : T(0) + (r.x - T(0)) / (diag + rc.x);
                    d1.y = act ? T(0) + (r.y - T(0)) / (diag + rc.y) : T(0);
                    *reinterpret_cast<V2 *>((T *)a.d1 + q) = d1;
                }
            }
        });
    if (a.partials) {
        double v[4] = {acc.hsum, acc.hmax, 0.0, 0.0};
        block_reduce_store<4>(v, 0xAu, a.partials + 4 * (int64_t)blockIdx.x);
    }
}

// Brick map of a psi kernel (overhanging the grid where it is no multiple of the brick).
template <int TX, int BZ>
inline TileMap make_brickmap(int n)
{
    TileMap t;
    constexpr int TYB = ZGeom<BZ>::kTYB;
    t.nx = (n + TX - 1) / TX;
    t.ny = (n + TYB - 1) / TYB;
    t.nz = (n + BZ - 1) / BZ;
    t.tx = TX;
    return t;
}

} // namespace grtmg
