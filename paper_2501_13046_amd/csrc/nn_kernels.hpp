// nn_kernels.hpp -- device kernels of the warm-start network.
//
// Activations are BF16, channels-last: element c of cell v = (i*n + j)*n + k
// of a C-channel tensor is at v*C + c (C a multiple of 8, so one channel
// octet is one aligned 16-byte load).  Convolutions are implicit GEMMs on
// the BF16 matrix cores (v_mfma_f32_16x16x32_bf16, FP32 accumulate):
//   M = output channels (16 per tile), N = cells (16 per tile), K = 27 taps x
//   input channels, enumerated as channel octets (see KOrder) and consumed
//   4 octets (32 values) per step.
// Lane l of a wave supplies row l%16 of A and column l%16 of B, each with
// the 8 consecutive K values of octet l/16 of the step; it receives rows
// 4*(l/16) .. 4*(l/16)+3 of column l%16 of the 16x16 result, that is four
// consecutive channels of one cell, stored as they are.
#pragma once

#include <utility>
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace grtnn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4))); // rows of any alignment
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16;

constexpr int kNBlock = 256; // threads per block (4 waves)

template <int... I, typename Fn>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, Fn &&f)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename Fn>
__device__ __forceinline__ void static_for(Fn &&f)
{
    static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

// ---- BF16 helpers -------------------------------------------------------------------

__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ float bf2f(u16 b) { return __uint_as_float((uint32_t)b << 16); }

// float -> bf16 bits, round to nearest even (NaN kept quiet): one v_cvt_pk_bf16_f32
__device__ __forceinline__ uint32_t pack2(float lo, float hi)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{lo, hi}), bf16x2));
}
__device__ __forceinline__ uint32_t f2bf(float f) { return pack2(f, 0.0f) & 0xffffu; }

// logistic function with the hardware reciprocal (about 1 ulp; the results are
// rounded to BF16)
__device__ __forceinline__ float sigm(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }
__device__ __forceinline__ float silu(float z) { return z * sigm(z); }
__device__ __forceinline__ float dsilu(float z)
{
    const float s = sigm(z);
    return s * (1.0f + z * (1.0f - s));
}

__device__ __forceinline__ u32x4 silu8(u32x4 w)
{
    u32x4 o;
#pragma unroll
    for (int q = 0; q < 4; q++) o[q] = pack2(silu(bf_lo(w[q])), silu(bf_hi(w[q])));
    return o;
}

__device__ __forceinline__ void unpack8(u32x4 w, float (&f)[8])
{
#pragma unroll
    for (int q = 0; q < 4; q++) {
        f[2 * q] = bf_lo(w[q]);
        f[2 * q + 1] = bf_hi(w[q]);
    }
}

__device__ __forceinline__ u32x4 pack8(const float (&f)[8])
{
    u32x4 o;
#pragma unroll
    for (int q = 0; q < 4; q++) o[q] = pack2(f[2 * q], f[2 * q + 1]);
    return o;
}

__device__ __forceinline__ int wrapn(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

__device__ __forceinline__ f32x4 mfma(u32x4 a, u32x4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// ---- K order shared by the packed weights and the convolution kernels --------------
//
// The input channels are processed in slices of cs channels (32, 16 or 8: the
// largest that divides both concatenated inputs).  K step ch belongs to slice
// ch / spp (spp = ceil(27 cs / 32) steps per slice); within the slice, lane
// group g of step ch takes octet o = 4 (ch % spp) + g (octets o >= 27 cs / 8
// are zero padding), i.e. tap o / (cs/8) and channels
// slice * cs + 8 (o % (cs/8)) .. + 7.  Tap t = 9 kx + 3 ky + kz is the offset
// (kx - 1, ky - 1, kz - 1).

struct KOrder {
    int cs, spp;
    __device__ __forceinline__ bool at(int ch, int g, int &tap, int &c0) const
    {
        const int sl = ch / spp, o = (ch - sl * spp) * 4 + g;
        const int per = cs >> 3;
        if (o >= 27 * per) return false;
        tap = o / per;
        c0 = sl * cs + (o - tap * per) * 8;
        return true;
    }
};

// ---- convolution (forward; backward data with mirrored transposed weights) ----------

enum { kEpStoreF32, kEpDsiluBf16, kEpSiluBf16 };

struct ConvArgs {
    const u16 *in1, *in2; // input = concatenation [in1, in2] along channels
    int c1, c2;           // channels (= strides) of in1 / in2 (c2 = 0: no in2)
    int act1, act2;       // apply SiLU to values read from in1 / in2
    const u32x4 *w;       // packed weights [tile][chunk][64 lanes] of 8 BF16
    const float *bias;    // per output channel, or null
    int n;                // cells per axis
    KOrder ko;            // K order of the packed weights
    int nchunk;           // K steps
    int ntile;            // 16-wide output channel tiles of the layer
    int cout;             // output channels written = oc1 + oc2
    int oc1, oc2;         // output channels [0, oc1) -> out1, [oc1, cout) -> out2
    int mode1, mode2;     // epilogue per destination (kEp*)
    void *out1, *out2;
    const u16 *zref1, *zref2; // pre-activations (layout of out1 / out2) for kEpDsiluBf16
    u16 *zout1;           // kEpSiluBf16: pre-activations of destination 1 (may be null)
};

// Epilogue of output channels co0 .. co0+3 of cell v (acc with the bias added)
__device__ __forceinline__ void conv_store4(const ConvArgs &a, int co0, int64_t v, f32x4 f)
{
    const bool first = co0 < a.oc1; // oc1 is a multiple of 8 where there is a second destination
    const int cc = first ? co0 : co0 - a.oc1;
    const int oc = first ? a.oc1 : a.oc2;
    const int mode = first ? a.mode1 : a.mode2;
    void *out = first ? a.out1 : a.out2;
    const int64_t idx = v * oc + cc;
    if (mode == kEpStoreF32) {
        if (co0 + 4 <= a.cout) {
            *(f32x4u *)((float *)out + idx) = f;
        } else {
#pragma unroll
            for (int j = 0; j < 3; j++)
                if (co0 + j < a.cout) ((float *)out)[idx + j] = f[j];
        }
        return;
    }
    // BF16 destinations have a multiple of 8 channels
    if (mode == kEpSiluBf16) {
        *(u32x2 *)((u16 *)out + idx) = u32x2{pack2(silu(f[0]), silu(f[1])), pack2(silu(f[2]), silu(f[3]))};
        if (a.zout1) *(u32x2 *)(a.zout1 + idx) = u32x2{pack2(f[0], f[1]), pack2(f[2], f[3])};
    } else {
        const u32x2 z = *(const u32x2 *)((first ? a.zref1 : a.zref2) + idx);
        *(u32x2 *)((u16 *)out + idx) = u32x2{pack2(f[0] * dsilu(bf_lo(z[0])), f[1] * dsilu(bf_hi(z[0]))),
                                             pack2(f[2] * dsilu(bf_lo(z[1])), f[3] * dsilu(bf_hi(z[1])))};
    }
}

__device__ __forceinline__ int brick_block(int nblocks)
{
    // consecutive bricks (which share halo cells) go to the same XCD
    const int b = blockIdx.x;
    return (nblocks % 8 == 0) ? (b % 8) * (nblocks / 8) + b / 8 : b;
}

// x / D for 0 <= x < 4096 and D <= 18, without a wide multiplication
template <int D>
__device__ __forceinline__ int div_small(int x)
{
    return __mul24(x, (65536 + D - 1) / D) >> 16;
}

// Brick of cells of one block of four waves, ROWS tiles of 16 cells per wave.  A
// tile is 16 / BZ rows of BZ cells.  ROWS = 4: 4 x 4 x 16 or 4 x 8 x 8 cells, wave
// w at x0 + w, tile q at row q of tiles.  ROWS = 1: 2 x 2 x 16 or 2 x 4 x 8 cells,
// one tile per wave.  The halo is one cell on every side; in LDS the octets
// of a cell are adjacent (P = 4: in pairs, the second pairs half a bank row off), which
// leaves both the operand reads (16 cells, lane groups on different octets) and the
// staging stores (16 / P cells, all octets) without bank conflicts.
template <int BZ, int ROWS, int P>
struct Brick {
    static constexpr int MY = 16 / BZ; // y rows of a tile
    static constexpr int BX = ROWS == 4 ? 4 : 2;
    static constexpr int BY = (ROWS == 4 ? 4 : 2) * MY;
    static constexpr int HX = BX + 2, HY = BY + 2, HZ = BZ + 2;
    static constexpr int kHalo = HX * HY * HZ;
    static constexpr int CW = P == 1 ? 1 : 2;                      // elements per cell and plane
    static constexpr int kPlane = (kHalo * CW + 15) / 16 * 16 + 8; // from the first to the second octet pair
    static constexpr int kTile = P == 4 ? kPlane + 2 * kHalo : kHalo * CW;
    static constexpr int NE = (kHalo * P + kNBlock - 1) / kNBlock; // staging loads per thread
    static constexpr int kSteps = (27 * P + 3) / 4;                // K steps of a slice

    // element of octet o relative to the cell's octet 0
    static __host__ __device__ constexpr int octet(int o) { return (o >> 1) * kPlane + (o & 1); }
    // halo cell of staging load k of this thread (past the halo: its last cell)
    static __device__ __forceinline__ int cell(int tid, int k) { return min((tid + k * kNBlock) / P, kHalo - 1); }
    static __device__ __forceinline__ void split(int hv, int &hx, int &hy, int &hz)
    {
        const int row = div_small<HZ>(hv);
        hz = hv - row * HZ;
        hx = div_small<HY>(row);
        hy = row - hx * HY;
    }
    static __device__ __forceinline__ void store(u32x4 *smem, const u32x4 (&stg)[NE])
    {
        const int tid = threadIdx.x;
#pragma unroll
        for (int k = 0; k < NE; k++)
            if ((k + 1) * kNBlock <= kHalo * P || tid + k * kNBlock < kHalo * P)
                smem[octet(tid % P) + (tid / P + k * (kNBlock / P)) * CW] = stg[k];
    }
    // cell of tile 0 of this lane, from the brick's first one
    static __device__ __forceinline__ void lane_cell(int wave, int r, int &x, int &y, int &z)
    {
        x = ROWS == 4 ? wave : wave >> 1;
        y = (ROWS == 4 ? 0 : (wave & 1) * MY) + r / BZ;
        z = r % BZ;
    }
    // element of K octet o relative to octet 0 of tap 0 (past the 27 taps: that one;
    // its operands are zeroed)
    static __host__ __device__ constexpr int tap(int o)
    {
        if (o >= 27 * P) return 0;
        const int t = o / P;
        return (((t / 9) * HY + (t / 3) % 3) * HZ + t % 3) * CW + octet(o % P);
    }
    // The operands of K step ST are read at row(ST) + tap(4 ST) + tile offset: the
    // second and third summand are constants, the first takes few values over the
    // steps (one for P = 4, four for P = 2)
    template <int ST>
    static __device__ __forceinline__ int row(int g)
    {
        constexpr int t0 = tap(4 * ST), d1 = tap(4 * ST + 1) - t0, d2 = tap(4 * ST + 2) - t0, d3 = tap(4 * ST + 3) - t0;
        if constexpr (P == 4)
            return octet(g);
        else if constexpr (P == 2 && 4 * ST + 3 < 27 * P)
            return (g & 1) + ((g & 2) ? d2 : 0);
        else
            return g == 0 ? 0 : g == 1 ? d1 : g == 2 ? d2 : d3;
    }
    // cell operands of step ST for the ROWS tiles of the lane (base: its first element)
    template <int ST>
    static __device__ __forceinline__ void operands(const u32x4 *base, int g, u32x4 (&av)[ROWS])
    {
        const u32x4 *ap = base + row<ST>(g);
#pragma unroll
        for (int q = 0; q < ROWS; q++) av[q] = ap[tap(4 * ST) + q * MY * HZ * CW];
        if constexpr (4 * ST + 3 >= 27 * P) {
            const bool pad = 4 * ST + g >= 27 * P;
#pragma unroll
            for (int q = 0; q < ROWS; q++)
#pragma unroll
                for (int j = 0; j < 4; j++) av[q][j] = pad ? 0u : av[q][j];
        }
    }
};

// A cell past the grid's wrapped one only feeds cells past the grid, which are not stored.
__device__ __forceinline__ int halo_at(int p, int n) { return wrapn(min(p, n), n); }

// The channel slice sl of the layer input: source of its first channel, stride, SiLU
struct SliceSrc {
    const u16 *p;
    int cs, act;
    template <class Args>
    __device__ __forceinline__ SliceSrc(const Args &a, int cb)
    {
        const bool one = cb < a.c1;
        p = one ? a.in1 + cb : a.in2 + (cb - a.c1);
        cs = one ? a.c1 : a.c2;
        act = one ? a.act1 : a.act2;
    }
};

__device__ __forceinline__ f32x4 conv_bias(const ConvArgs &a, int co0)
{
    f32x4 b = {0.f, 0.f, 0.f, 0.f};
    if (a.bias) {
#pragma unroll
        for (int j = 0; j < 4; j++) b[j] = a.bias[min(co0 + j, a.cout - 1)];
    }
    return b;
}

template <class B, int ROWS>
__device__ __forceinline__ void conv_write(const ConvArgs &a, int co0, int x, int y, int z, f32x4 (&acc)[ROWS],
                                           f32x4 bias)
{
    const int n = a.n;
#pragma unroll
    for (int q = 0; q < ROWS; q++) {
        const int yq = y + q * B::MY;
        if (co0 < a.cout && max(x, max(yq, z)) < n)
            conv_store4(a, co0, ((int64_t)x * n + yq) * n + z, acc[q] + bias);
        acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
}

// Convolution on small grids (any n: cells past the grid are not stored): one brick of
// ROWS = 1 and one tile of 16 output channels per block, so that the few cells spread
// over many blocks.  Per channel slice the block stages the brick's halo (wrapped
// periodically); a cell operand is then one 16-byte LDS read.  What bounds it is the
// chain of latencies of one block, so a whole slice of weights is in registers and is
// replaced step by step by the next slice's, whose halo is fetched meanwhile.
// 48 -> 48 channels at 16^3 12.9 -> 5.8 us, 64 -> 64 at 8^3 22 -> 6.0 us against
// two steps of weights in flight and operands from global memory at 8^3.
template <int CS, int BZ>
__global__ void __launch_bounds__(kNBlock, 2) k_conv3_small(ConvArgs a)
{
    using B = Brick<BZ, 1, CS / 8>;
    constexpr int P = CS / 8, spp = B::kSteps;
    __shared__ u32x4 smem[B::kTile];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g = lane >> 4, r = lane & 15;
    const int n = a.n, nbz = (n + BZ - 1) / BZ, nby = (n + B::BY - 1) / B::BY;
    int b = brick_block(gridDim.x);
    const int bz = b % nbz;
    b /= nbz;
    const int by = b % nby, bx = b / nby;
    const int x0 = bx * B::BX, y0 = by * B::BY, z0 = bz * BZ;
    int cell[B::NE];
#pragma unroll
    for (int k = 0; k < B::NE; k++) {
        int hx, hy, hz;
        B::split(B::cell(threadIdx.x, k), hx, hy, hz);
        cell[k] = (halo_at(x0 + hx - 1, n) * n + halo_at(y0 + hy - 1, n)) * n + halo_at(z0 + hz - 1, n);
    }
    u32x4 stg[B::NE];
    auto stage_load = [&](int sl) {
        const SliceSrc s(a, sl * CS);
#pragma unroll
        for (int k = 0; k < B::NE; k++)
            stg[k] = *(const u32x4 *)(s.p + ((int64_t)cell[k] * s.cs + 8 * (threadIdx.x % P)));
        if (s.act) {
#pragma unroll
            for (int k = 0; k < B::NE; k++) stg[k] = silu8(stg[k]);
        }
    };
    const u32x4 *w = a.w + (int64_t)blockIdx.y * a.nchunk * 64;
    auto wload = [&](int ch) { return *(const u32x4 *)((const char *)(w + ch * 64) + (uint32_t)(16 * lane)); };
    u32x4 bw[spp];
    stage_load(0);
    static_for<spp>([&](auto k) { bw[decltype(k)::value] = wload(decltype(k)::value); });
    const int co0 = blockIdx.y * 16 + 4 * g;
    const f32x4 bias = conv_bias(a, co0);
    f32x4 acc[1] = {f32x4{0.f, 0.f, 0.f, 0.f}};
    int cx, cy, cz;
    B::lane_cell(wave, r, cx, cy, cz);
    const u32x4 *base = smem + ((cx * B::HY + cy) * B::HZ + cz) * B::CW;
    auto consume = [&](auto reload, int sl) {
        static_for<spp>([&](auto stc) {
            constexpr int st = decltype(stc)::value;
            u32x4 av[1];
            B::template operands<st>(base, g, av);
            acc[0] = mfma(bw[st], av[0], acc[0]);
            if constexpr (decltype(reload)::value) bw[st] = wload((sl + 1) * spp + st);
        });
    };
    const int nslice = (a.c1 + a.c2) / CS;
    for (int sl = 0; sl < nslice; sl++) {
        __syncthreads(); // the slice staged before is consumed
        B::store(smem, stg);
        __syncthreads();
        if (sl + 1 < nslice) {
            stage_load(sl + 1);
            consume(std::true_type{}, sl);
        } else {
            consume(std::false_type{}, sl);
        }
    }
    conv_write<B, 1>(a, co0, x0 + cx, y0 + cy, z0 + cz, acc, bias);
}

// Convolution on large grids (any n): a block takes several bricks of ROWS = 4 and
// one tile of 16 output channels (blockIdx.y).  The slice's weights are in LDS, read
// there once per four products: from L2 into every wave they cost more of the vector
// cache's bandwidth than the halo (14 against 5 loads of 1 KB per wave and brick of 16
// channels).  Several bricks, so that the loads of the next are in flight: with
// one brick per block the same arithmetic waited 70 % of its time.  Blocks that run together
// work on neighbouring bricks, whose halos and whose further slices then come from the L2.  (With
// a run of consecutive bricks per block they fell out of step wherever the run and a row of
// bricks did not divide each other: 112 -> 48 channels at 64^3 250 us against 123, 40 -> 8 at 112^3
// 199 against 88, 32 -> 32 at 96^3 118 against 77.)  The next halo (of the next slice or
// brick) and, where the layer has several slices, the next weights are fetched into
// registers while this one is consumed.  The four layers with 16 output channels at 128^3 (one of them
// of three slices) 350 -> 291 us, 112 -> 48 channels at 32^3 32 -> 24 us.
template <int CS, int BZ>
__global__ void __launch_bounds__(kNBlock, CS == 32 ? 2 : 4) k_conv3_stream(ConvArgs a, int bricks)
{
    using B = Brick<BZ, 4, CS / 8>;
    constexpr int P = CS / 8, spp = B::kSteps;
    constexpr int NW = (spp * 64 + kNBlock - 1) / kNBlock; // weight loads per thread
    __shared__ u32x4 smem[B::kTile];
    __shared__ u32x4 wsm[spp * 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4, r = lane & 15;
    const int n = a.n, nbz = (n + BZ - 1) / BZ, nby = (n + B::BY - 1) / B::BY;
    // each XCD (block number modulo 8) walks an eighth of the bricks, its blocks side by side
    const int xcd = blockIdx.x % 8, step = gridDim.x / 8;
    const int first = (int)((int64_t)bricks * xcd / 8) + (int)blockIdx.x / 8;
    const int last = (int)((int64_t)bricks * (xcd + 1) / 8);
    if (first >= last) return;
    int off[B::NE]; // cells from the halo's first one, inside the grid
#pragma unroll
    for (int k = 0; k < B::NE; k++) {
        int hx, hy, hz;
        B::split(B::cell(tid, k), hx, hy, hz);
        off[k] = (hx * n + hy) * n + hz;
    }
    int x0, y0, z0; // first cell of the brick whose halo was fetched last
    auto brick_at = [&](int bi) {
        const int t = bi / nbz;
        z0 = (bi - t * nbz) * BZ;
        const int bx = t / nby;
        y0 = (t - bx * nby) * B::BY;
        x0 = bx * B::BX;
    };
    u32x4 stg[B::NE], wst[NW];
    auto stage_load = [&](int sl) {
        const SliceSrc s(a, sl * CS);
        if (min(x0, min(y0, z0)) > 0 && max(x0 + B::BX, max(y0 + B::BY, z0 + BZ)) < n) {
            const char *p = (const char *)(s.p + (((int64_t)(x0 - 1) * n + y0 - 1) * n + z0 - 1) * s.cs);
#pragma unroll
            for (int k = 0; k < B::NE; k++)
                stg[k] = *(const u32x4 *)(p + (uint32_t)(__mul24(off[k], 2 * s.cs) + 16 * (tid % P)));
        } else {
            int t = tid; // the cells are worked out anew, not kept in registers over the loop
            asm volatile("" : "+v"(t));
#pragma unroll
            for (int k = 0; k < B::NE; k++) {
                int hx, hy, hz;
                B::split(B::cell(t, k), hx, hy, hz);
                const int c = (halo_at(x0 + hx - 1, n) * n + halo_at(y0 + hy - 1, n)) * n + halo_at(z0 + hz - 1, n);
                stg[k] = *(const u32x4 *)(s.p + ((int64_t)c * s.cs + 8 * (tid % P)));
            }
        }
        if (s.act) {
#pragma unroll
            for (int k = 0; k < B::NE; k++) stg[k] = silu8(stg[k]);
        }
    };
    const u32x4 *w = a.w + (int64_t)blockIdx.y * a.nchunk * 64;
    auto weight_load = [&](int sl) {
#pragma unroll
        for (int k = 0; k < NW; k++) wst[k] = w[sl * spp * 64 + min(tid + k * kNBlock, spp * 64 - 1)];
    };
    auto weight_store = [&]() {
#pragma unroll
        for (int k = 0; k < NW; k++)
            if ((k + 1) * kNBlock <= spp * 64 || tid + k * kNBlock < spp * 64) wsm[tid + k * kNBlock] = wst[k];
    };
    const int nslice = (a.c1 + a.c2) / CS;
    int bi = first, sl = 0;
    brick_at(bi);
    weight_load(0);
    stage_load(0);
    const int co0 = blockIdx.y * 16 + 4 * g;
    const f32x4 bias = conv_bias(a, co0);
    f32x4 acc[4];
#pragma unroll
    for (int q = 0; q < 4; q++) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    int cx, cy, cz;
    B::lane_cell(wave, r, cx, cy, cz);
    const u32x4 *base = smem + ((cx * B::HY + cy) * B::HZ + cz) * B::CW;
    weight_store();
    for (;;) {
        B::store(smem, stg);
        if (nslice > 1) weight_store();
        __syncthreads();
        const int nsl = sl + 1 < nslice ? sl + 1 : 0, nbi = nsl ? bi : bi + step;
        const int px = x0 + cx, py = y0 + cy, pz = z0 + cz;
        if (nbi < last) {
            if (!nsl) brick_at(nbi);
            if (nslice > 1) weight_load(nsl);
            stage_load(nsl);
        }
        static_for<spp>([&](auto stc) {
            constexpr int st = decltype(stc)::value;
            const u32x4 wv = wsm[st * 64 + lane];
            u32x4 av[4];
            B::template operands<st>(base, g, av);
#pragma unroll
            for (int q = 0; q < 4; q++) acc[q] = mfma(wv, av[q], acc[q]);
        });
        if (!nsl) conv_write<B, 4>(a, co0, px, py, pz, acc, bias);
        if (nbi >= last) break;
        bi = nbi;
        sl = nsl;
        __syncthreads(); // the staged slice is consumed
    }
}

// ---- weight gradient ------------------------------------------------------------------
//
// dW[co][ci][t] = sum_v dy[v][co] a[v + d_t][ci]: an MFMA with M = input channels,
// N = output channels, K = cells (32 per step).  Block (co tile, ci tile, split) sums
// the cells of a range of bricks; its partial sums [tap][co][ci] are added over the
// splits in a fixed order afterwards.  Tap 27 is the bias (the same product with ones).
//
// A brick's halo and output gradients are staged as they are, channels last, and read
// with transposing LDS loads: lanes 16 g .. 16 g + 15 read the 16 channels of four
// consecutive cells (128 contiguous bytes) and lane 16 g + i receives channel i of the
// four.  The waves split the taps (seven each), not the cells: no sums between waves
// are left, and every wave keeps 7 accumulators instead of 27.  Bound by LDS reads
// (27 times the staged bytes) and their latency; 16 -> 16 channels at 64^3 49 -> 13 us,
// 64 -> 64 at 8^3 102 -> 6.3 us, against operands turned around while staging (and
// formed from single values in global memory at 8^3).

struct WgtArgs {
    const u16 *in1, *in2;
    int c1, c2, act1, act2; // layer input as in ConvArgs
    const u16 *dy;          // output gradient, BF16, stride cy
    int cy;
    int n;
    int bricks, per_split;
    int cot, cit;           // co / ci tiles of the layer
    float *part;            // [split][co tile][ci tile][28][16 co][16 ci]
};

constexpr int kWgtTile = 28 * 256; // partial sums of one pair of tiles

typedef short s16x4 __attribute__((ext_vector_type(4)));

// four cells (32 bytes apart) of one channel; see above
__device__ __forceinline__ u32x2 read_turned(const char *p)
{
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)p));
}

template <int BZ>
__global__ void __launch_bounds__(kNBlock, 2) k_conv3_wgrad(WgtArgs a)
{
    using B = Brick<BZ, 4, 2>;
    constexpr int BY = B::BY, kCells = 256;
    __shared__ u32x4 halo[B::kTile], dys[2 * kCells];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4, i = lane & 15, o = tid & 1;
    const int n = a.n, nbz = (n + BZ - 1) / BZ, nby = (n + BY - 1) / BY;
    const int first = blockIdx.z * a.per_split, last = min(a.bricks, first + a.per_split);
    // the octet this thread stages (absent ones are zero)
    const bool have = (int)blockIdx.y * 16 + 8 * o < a.c1 + a.c2, haved = (int)blockIdx.x * 16 + 8 * o < a.cy;
    const SliceSrc src(a, have ? blockIdx.y * 16 + 8 * o : 0);
    const u16 *dsrc = a.dy + (haved ? blockIdx.x * 16 + 8 * o : 0);
    const u32x4 zero = {0u, 0u, 0u, 0u};
    u32x4 stg[B::NE], dst[2];
    auto load = [&](int bi) {
        const int t = bi / nbz, bx = t / nby;
        const int x0 = bx * B::BX, y0 = (t - bx * nby) * BY, z0 = (bi - t * nbz) * BZ;
#pragma unroll
        for (int k = 0; k < B::NE; k++) {
            int hx, hy, hz;
            B::split(B::cell(tid, k), hx, hy, hz);
            const int c = (halo_at(x0 + hx - 1, n) * n + halo_at(y0 + hy - 1, n)) * n + halo_at(z0 + hz - 1, n);
            const u32x4 v = *(const u32x4 *)(src.p + (int64_t)c * src.cs);
            stg[k] = have ? v : zero;
        }
#pragma unroll
        for (int k = 0; k < 2; k++) {
            const int c = (tid >> 1) + k * (kNBlock / 2);
            const int x = x0 + (c >> 6), y = y0 + (c / BZ) % BY, z = z0 + c % BZ;
            const bool in = haved && max(x, max(y, z)) < n; // cells past the grid add nothing
            const u32x4 v = *(const u32x4 *)(dsrc + (in ? ((int64_t)x * n + y) * n + z : 0) * a.cy);
            dst[k] = in ? v : zero;
        }
        if (src.act) {
#pragma unroll
            for (int k = 0; k < B::NE; k++) stg[k] = silu8(stg[k]);
        }
    };
    // lane's piece of the 16 cells of a tile row: cell 4 g + i / 4 of them
    const int q = 4 * g + (i >> 2);
    const char *db = (const char *)dys + q * 32 + (i & 3) * 8;
    const char *hb[7];
#pragma unroll
    for (int t = 0; t < 7; t++) {
        const int tap = min(7 * wave + t, 26);
        const int c = ((tap / 9) * B::HY + tap / 3 % 3 + q / BZ) * B::HZ + tap % 3 + q % BZ;
        hb[t] = (const char *)halo + c * 32 + (i & 3) * 8;
    }
    constexpr uint32_t kOnes = 0x3f803f80u;
    f32x4 acc[7];
#pragma unroll
    for (int t = 0; t < 7; t++) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    // the products of a staged brick.  Past: cells of it lie past the grid (nx, ny and nz cells are
    // inside); the halo has grid cells' values there, whose product with the zero output gradient
    // is no zero where they are infinite, so they are taken as zeros too
    auto consume = [&](auto past, int nx, int ny, int nz) {
        constexpr bool Past = decltype(past)::value;
        uint32_t mz[2]; // inside along z: the two pairs of this lane's four cells
#pragma unroll
        for (int j = 0; j < 2; j++) {
            const int z = 4 * g % BZ + 2 * j;
            mz[j] = (z < nz ? 0xffffu : 0u) | (z + 1 < nz ? 0xffff0000u : 0u);
        }
        static_for<8>([&](auto sc) {
            constexpr int r0 = 2 * decltype(sc)::value, r1 = r0 + 1; // tile rows: x = r / 4, tile r % 4 of y
            constexpr int h0 = ((r0 / 4) * B::HY + (r0 % 4) * B::MY) * B::HZ * 32;
            constexpr int h1 = ((r1 / 4) * B::HY + (r1 % 4) * B::MY) * B::HZ * 32;
            const u32x2 d0 = read_turned(db + r0 * 512), d1 = read_turned(db + r1 * 512);
            const u32x4 dv = {d0[0], d0[1], d1[0], d1[1]};
            uint32_t mk[4] = {~0u, ~0u, ~0u, ~0u};
            if constexpr (Past) {
                const bool in0 = r0 / 4 < nx && (r0 % 4) * B::MY + 4 * g / BZ < ny;
                const bool in1 = r1 / 4 < nx && (r1 % 4) * B::MY + 4 * g / BZ < ny;
#pragma unroll
                for (int j = 0; j < 2; j++) {
                    mk[j] = in0 ? mz[j] : 0u;
                    mk[2 + j] = in1 ? mz[j] : 0u;
                }
            }
#pragma unroll
            for (int t = 0; t < 7; t++) {
                const u32x2 v0 = read_turned(hb[t] + h0), v1 = read_turned(hb[t] + h1);
                u32x4 av = {v0[0], v0[1], v1[0], v1[1]};
                if constexpr (Past) {
#pragma unroll
                    for (int j = 0; j < 4; j++) av[j] &= mk[j];
                }
                if (t == 6) {
#pragma unroll
                    for (int j = 0; j < 4; j++) av[j] = wave == 3 ? kOnes : av[j];
                }
                acc[t] = mfma(av, dv, acc[t]);
            }
        });
    };
    load(first);
    for (int bi = first; bi < last; bi++) {
        B::store(halo, stg);
        dys[tid] = dst[0];
        dys[tid + kNBlock] = dst[1];
        __syncthreads();
        if (bi + 1 < last) load(bi + 1);
        if constexpr (BZ == 16) {
            consume(std::false_type{}, B::BX, BY, BZ); // bricks of 16 divide the sides they serve
        } else {
            const int t = bi / nbz, bx = t / nby;
            const int nx = n - bx * B::BX, ny = n - (t - bx * nby) * BY, nz = n - (bi - t * nbz) * BZ;
            if (nx >= B::BX && ny >= BY && nz >= BZ)
                consume(std::false_type{}, nx, ny, nz);
            else
                consume(std::true_type{}, nx, ny, nz);
        }
        __syncthreads(); // the staged brick is consumed
    }
    float *out = a.part + (((int64_t)blockIdx.z * a.cot + blockIdx.x) * a.cit + blockIdx.y) * kWgtTile;
#pragma unroll
    for (int t = 0; t < 7; t++) *(f32x4 *)(out + (7 * wave + t) * 256 + i * 16 + 4 * g) = acc[t];
}

// gw[(co*cin + ci)*27 + t] (+)= sum_s part[s][co][ci][t], gb[co] (+)= tap 27, for all
// layers of a backward pass in one launch (one per layer left most of the chip idle
// and cost 4.7 us at least, 112 us of a training step at 64^3, now 41 us).  A block reduces 16
// quads of one layer with 16 threads each (thread k sums splits k, k + 16, ...) in FP64; the
// 16 sums are added in a fixed order.
constexpr int kMaxLayers = 15; // 4 levels: 8 encoder + 6 decoder convolutions + head

struct WgtSum {
    const float *part;
    float *gw, *gb;
    int first; // first block
    int nsplit, cot, cit, cin, cout;
};
struct WgtSums {
    WgtSum l[kMaxLayers];
    int count, accumulate;
};

__global__ void __launch_bounds__(kNBlock) k_wgrad_reduce(WgtSums w)
{
    __shared__ double sh[16][64];
    int li = 0;
    while (li + 1 < w.count && (int)blockIdx.x >= w.l[li + 1].first) li++;
    const WgtSum &l = w.l[li];
    const int el = threadIdx.x & 15, k = threadIdx.x >> 4;
    const int e = ((int)blockIdx.x - l.first) * 16 + el; // quad of [co tile][ci tile][28][16][4]
    const int64_t per = (int64_t)l.cot * l.cit * kWgtTile;
    double s[4] = {0., 0., 0., 0.};
    for (int q = k; q < l.nsplit; q += 16) {
        const f32x4 v = *(const f32x4 *)(l.part + q * per + 4 * e);
#pragma unroll
        for (int j = 0; j < 4; j++) s[j] += (double)v[j];
    }
#pragma unroll
    for (int j = 0; j < 4; j++) sh[k][4 * el + j] = s[j];
    __syncthreads();
    if (threadIdx.x >= 64) return;
    double d = 0.0;
    for (int q = 0; q < 16; q++) d += sh[q][threadIdx.x];
    const float t = (float)d;
    const int v = ((int)blockIdx.x - l.first) * 64 + threadIdx.x;
    const int tile = v / kWgtTile, tap = v % kWgtTile >> 8;
    const int co = tile / l.cit * 16 + (v >> 4 & 15), ci = tile % l.cit * 16 + (v & 15);
    if (co >= l.cout) return;
    if (tap == 27) {
        if (ci == 0) l.gb[co] = w.accumulate ? l.gb[co] + t : t;
    } else if (ci < l.cin) {
        float *dst = l.gw + ((int64_t)co * l.cin + ci) * 27 + tap;
        *dst = w.accumulate ? *dst + t : t;
    }
}

// ---- weight packing -------------------------------------------------------------------
//
// Forward pack of a layer W[co][ci][27] (cin_real real input channels):
// element (tile, chunk, lane) holds the 8 weights W[tile*16 + lane%16][c0 + j][tap]
// of the octet (tap, c0) that KOrder assigns to (chunk, lane/16), zero where
// the channel or the octet does not exist.  The transposed pack (backward
// data) does the same for W'[ci][co][26 - tap], i.e. the layer with inputs and
// outputs exchanged and the taps mirrored.
// All packs of a network in one launch (blockIdx.y: one pack), which also copies the
// biases: a launch per pack and a copy per bias took 160 us after every optimiser step, this 7.
struct PackJob {
    const float *W;
    u32x4 *out;
    const float *b; // biases to copy to bias, or null
    float *bias;
    int cin_real, cout;
    KOrder ko;
    int nchunk, ntile, transposed;
};
struct PackJobs {
    PackJob j[2 * kMaxLayers];
};

__global__ void __launch_bounds__(kNBlock) k_pack_weights(PackJobs jobs)
{
    const PackJob &p = jobs.j[blockIdx.y];
    const float *W = p.W;
    const int cin_real = p.cin_real, cout = p.cout, nchunk = p.nchunk;
    const KOrder ko = p.ko;
    const bool transposed = p.transposed != 0;
    const int64_t e = (int64_t)blockIdx.x * kNBlock + threadIdx.x;
    if (p.b && e < cout) p.bias[e] = p.b[e];
    const int64_t total = (int64_t)p.ntile * nchunk * 64;
    if (e >= total) return;
    const int lane = (int)(e % 64);
    const int64_t tc = e / 64;
    const int chunk = (int)(tc % nchunk), tile = (int)(tc / nchunk);
    const int col = tile * 16 + lane % 16; // output channel of the (possibly transposed) layer
    float f[8];
#pragma unroll
    for (int j = 0; j < 8; j++) f[j] = 0.0f;
    int tap, c0;
    if (ko.at(chunk, lane / 16, tap, c0)) {
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const int k = c0 + j; // input channel of the (possibly transposed) layer
            if (!transposed) {
                if (col < cout && k < cin_real) f[j] = W[((int64_t)col * cin_real + k) * 27 + tap];
            } else {
                // layer (cin_real -> cout) seen as (cout -> cin_real): col = ci, k = co
                if (col < cin_real && k < cout) f[j] = W[((int64_t)k * cin_real + col) * 27 + (26 - tap)];
            }
        }
    }
    p.out[e] = pack8(f);
}

// ---- pooling, upsampling and their adjoints ---------------------------------------------

// out[coarse][c] = mean of the 8 children of act(z); one thread per (coarse cell, octet)
__global__ void __launch_bounds__(kNBlock) k_pool(const u16 *z, int C, int nc, int act, u16 *out)
{
    const int oc = C / 8;
    const int64_t Vc = (int64_t)nc * nc * nc;
    const int64_t e = (int64_t)blockIdx.x * kNBlock + threadIdx.x;
    if (e >= Vc * oc) return;
    const int o = (int)(e % oc);
    const int64_t v = e / oc;
    const int k = (int)(v % nc), j = (int)((v / nc) % nc), i = (int)(v / ((int64_t)nc * nc));
    const int nf = 2 * nc;
    float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int a = 0; a < 2; a++)
        for (int b = 0; b < 2; b++)
            for (int c = 0; c < 2; c++) {
                const int64_t vf = ((int64_t)(2 * i + a) * nf + (2 * j + b)) * nf + (2 * k + c);
                u32x4 w = *(const u32x4 *)(z + vf * C + 8 * o);
                if (act) w = silu8(w);
                float f[8];
                unpack8(w, f);
#pragma unroll
                for (int q = 0; q < 8; q++) s[q] += f[q];
            }
#pragma unroll
    for (int q = 0; q < 8; q++) s[q] *= 0.125f;
    *(u32x4 *)(out + v * C + 8 * o) = pack8(s);
}

// Per-axis weights of cell-centred x2 interpolation: fine 2I+a takes 3/4 of
// coarse I and 1/4 of coarse I-1 (a = 0) or I+1 (a = 1).  One thread per
// (coarse cell, octet) fetches the 3 x 3 x 3 coarse neighbourhood once and
// writes the octet of all 8 children; each child sums its 8 terms in the order
// (own, neighbour) per axis, x outermost.
__global__ void __launch_bounds__(kNBlock) k_up(const u16 *z, int C, int nc, int act, u16 *out)
{
    const int oc = C / 8;
    const int64_t Vc = (int64_t)nc * nc * nc;
    const int64_t e = (int64_t)blockIdx.x * kNBlock + threadIdx.x;
    if (e >= Vc * oc) return;
    const int o = (int)(e % oc);
    const int64_t v = e / oc;
    const int K = (int)(v % nc), J = (int)((v / nc) % nc), I = (int)(v / ((int64_t)nc * nc));
    int xi[3], yj[3], zk[3];
#pragma unroll
    for (int d = 0; d < 3; d++) {
        xi[d] = wrapn(I + d - 1, nc);
        yj[d] = wrapn(J + d - 1, nc);
        zk[d] = wrapn(K + d - 1, nc);
    }
    u32x4 nb[3][3][3];
#pragma unroll
    for (int dx = 0; dx < 3; dx++)
#pragma unroll
        for (int dy = 0; dy < 3; dy++)
#pragma unroll
            for (int dz = 0; dz < 3; dz++) {
                const int64_t vc = ((int64_t)xi[dx] * nc + yj[dy]) * nc + zk[dz];
                u32x4 w = *(const u32x4 *)(z + vc * C + 8 * o);
                nb[dx][dy][dz] = act ? silu8(w) : w;
            }
    const float wt[2] = {0.75f, 0.25f};
    const int nf = 2 * nc;
#pragma unroll
    for (int ca = 0; ca < 2; ca++)
#pragma unroll
        for (int cb = 0; cb < 2; cb++)
#pragma unroll
            for (int cc = 0; cc < 2; cc++) {
                float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
                for (int a = 0; a < 2; a++)
#pragma unroll
                    for (int b = 0; b < 2; b++)
#pragma unroll
                        for (int c = 0; c < 2; c++) {
                            // own cell (index 1) or the neighbour on the child's side
                            const int dx = a ? (ca ? 2 : 0) : 1, dy = b ? (cb ? 2 : 0) : 1, dz = c ? (cc ? 2 : 0) : 1;
                            float f[8];
                            unpack8(nb[dx][dy][dz], f);
                            const float ww = wt[a] * wt[b] * wt[c];
#pragma unroll
                            for (int q = 0; q < 8; q++) s[q] += ww * f[q];
                        }
                const int64_t vf = ((int64_t)(2 * I + ca) * nf + (2 * J + cb)) * nf + (2 * K + cc);
                *(u32x4 *)(out + vf * C + 8 * o) = pack8(s);
            }
}

// The same interpolation with one thread per (fine cell, octet), each reading
// its 8 coarse cells (the same sums in the same order as k_up).
__global__ void __launch_bounds__(kNBlock) k_up_fine(const u16 *z, int C, int nc, int act, u16 *out)
{
    const int oc = C / 8;
    const int nf = 2 * nc;
    const int64_t Vf = (int64_t)nf * nf * nf;
    const int64_t e = (int64_t)blockIdx.x * kNBlock + threadIdx.x;
    if (e >= Vf * oc) return;
    const int o = (int)(e % oc);
    const int64_t v = e / oc;
    const int k = (int)(v % nf), j = (int)((v / nf) % nf), i = (int)(v / ((int64_t)nf * nf));
    int ci[2], cj[2], ck[2];
    ci[0] = i >> 1;
    ci[1] = wrapn((i >> 1) + ((i & 1) ? 1 : -1), nc);
    cj[0] = j >> 1;
    cj[1] = wrapn((j >> 1) + ((j & 1) ? 1 : -1), nc);
    ck[0] = k >> 1;
    ck[1] = wrapn((k >> 1) + ((k & 1) ? 1 : -1), nc);
    const float wt[2] = {0.75f, 0.25f};
    float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int a = 0; a < 2; a++)
        for (int b = 0; b < 2; b++)
            for (int c = 0; c < 2; c++) {
                const int64_t vc = ((int64_t)ci[a] * nc + cj[b]) * nc + ck[c];
                u32x4 w = *(const u32x4 *)(z + vc * C + 8 * o);
                if (act) w = silu8(w);
                float f[8];
                unpack8(w, f);
                const float ww = wt[a] * wt[b] * wt[c];
#pragma unroll
                for (int q = 0; q < 8; q++) s[q] += ww * f[q];
            }
    *(u32x4 *)(out + v * C + 8 * o) = pack8(s);
}

// (z[0..3] of SiLU') * s, rounded
__device__ __forceinline__ u32x2 dsilu4(f32x4 s, u32x2 z)
{
    return u32x2{pack2(s[0] * dsilu(bf_lo(z[0])), s[1] * dsilu(bf_hi(z[0]))),
                 pack2(s[2] * dsilu(bf_lo(z[1])), s[3] * dsilu(bf_hi(z[1])))};
}

// Adjoint of k_up followed by the SiLU derivative: for coarse cell I and
// channel c, sum over the 4 fine cells per axis that read I (2I-1, 2I, 2I+1,
// 2I+2 with weights 1/4, 3/4, 3/4, 1/4) of g_fine, times SiLU'(zref[I][c]).
// Bound by the vector cache; a thread takes four channels of two coarse cells along z
// (6 fine cells of a row instead of 8): 32 channels onto 32^3 32 -> 17 us.
__global__ void __launch_bounds__(kNBlock) k_up_adjoint_dsilu(const float *gf, int C, int nc, const u16 *zref,
                                                             u16 *dz)
{
    const int64_t e = (int64_t)blockIdx.x * kNBlock + threadIdx.x;
    const int qc = C / 4, nk = (nc + 1) / 2;
    if (e >= (int64_t)nc * nc * nk * qc) return;
    const int c = (int)(e % qc) * 4;
    const int64_t t = e / qc;
    const int k = 2 * (int)(t % nk), j = (int)(t / nk % nc), i = (int)(t / ((int64_t)nk * nc));
    const int nf = 2 * nc;
    const float wt[4] = {0.25f, 0.75f, 0.75f, 0.25f};
    int fk[6];
#pragma unroll
    for (int q = 0; q < 6; q++) fk[q] = wrapn(wrapn(2 * k - 1 + q, nf), nf);
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
    for (int a = 0; a < 4; a++) {
        const int fi = wrapn(2 * i - 1 + a, nf);
#pragma unroll
        for (int b = 0; b < 4; b++) {
            const int fj = wrapn(2 * j - 1 + b, nf);
            const float wab = wt[a] * wt[b];
            const float *row = gf + ((int64_t)fi * nf + fj) * nf * C + c;
            f32x4 g[6];
#pragma unroll
            for (int q = 0; q < 6; q++) g[q] = *(const f32x4 *)(row + (int64_t)fk[q] * C);
#pragma unroll
            for (int q = 0; q < 4; q++) {
                s0 += wab * wt[q] * g[q];
                s1 += wab * wt[q] * g[q + 2];
            }
        }
    }
    const int64_t v = (((int64_t)i * nc + j) * nc + k) * C + c;
    *(u32x2 *)(dz + v) = dsilu4(s0, *(const u32x2 *)(zref + v));
    if (k + 1 < nc) *(u32x2 *)(dz + v + C) = dsilu4(s1, *(const u32x2 *)(zref + v + C));
}

// dz[fine] = (skip[fine] + g_coarse[parent] / 8) * SiLU'(zref[fine]); skip may be null;
// four channels per thread
__global__ void __launch_bounds__(kNBlock) k_pool_adjoint_dsilu(const float *gc, const float *skip, int C, int nc,
                                                               const u16 *zref, u16 *dz)
{
    const int nf = 2 * nc, qc = C / 4;
    const int64_t Vf = (int64_t)nf * nf * nf;
    const int64_t e = (int64_t)blockIdx.x * kNBlock + threadIdx.x;
    if (e >= Vf * qc) return;
    const int c = (int)(e % qc) * 4;
    const int64_t v = e / qc;
    const int k = (int)(v % nf), j = (int)((v / nf) % nf), i = (int)(v / ((int64_t)nf * nf));
    const int64_t vc = ((int64_t)(i >> 1) * nc + (j >> 1)) * nc + (k >> 1);
    f32x4 s = 0.125f * *(const f32x4 *)(gc + vc * C + c);
    if (skip) s += *(const f32x4 *)(skip + v * C + c);
    *(u32x2 *)(dz + v * C + c) = dsilu4(s, *(const u32x2 *)(zref + v * C + c));
}

// ---- loss, optimiser, packing of fields -------------------------------------------------

// dz[v][c] = 2 (out - t) / (V * cout) for c < cout, 0 for cout <= c < 8 (BF16);
// block partial sums of (out - t)^2.
__global__ void __launch_bounds__(kNBlock) k_mse(const float *out, const u16 *target, int cout, int64_t V,
                                                u16 *dz, double *partials)
{
    __shared__ double sh[kNBlock / 64];
    const int64_t e = (int64_t)blockIdx.x * kNBlock + threadIdx.x;
    const float scale = (float)(2.0 / ((double)V * cout));
    double sq = 0.0;
    if (e < V * 8) {
        const int c = (int)(e % 8);
        const int64_t v = e / 8;
        float d = 0.0f;
        if (c < cout) {
            d = out[v * cout + c] - bf2f(target[v * cout + c]);
            sq = (double)d * d;
        }
        dz[e] = (u16)f2bf(scale * d);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = sq;
    __syncthreads();
    if (threadIdx.x == 0) partials[blockIdx.x] = sh[0] + sh[1] + sh[2] + sh[3];
}

// Deterministic sum of count doubles by one block; out[0] = sum.  Four loads of a
// thread in flight and 1024 threads: 8192 values 9.4 -> 3.8 us.
constexpr int kSumBlock = 1024;
__global__ void __launch_bounds__(kSumBlock) k_sum_final(const double *x, int64_t count, double *out)
{
    __shared__ double sh[kSumBlock / 64];
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    int64_t q = threadIdx.x;
    for (; q + 3 * kSumBlock < count; q += 4 * kSumBlock)
#pragma unroll
        for (int k = 0; k < 4; k++) s[k] += x[q + k * kSumBlock];
    for (; q < count; q += kSumBlock) s[0] += x[q];
    double t = (s[0] + s[1]) + (s[2] + s[3]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
        double u = 0.0;
        for (int w = 0; w < kSumBlock / 64; w++) u += sh[w];
        out[0] = u;
    }
}

// Block partial sums of v and v^2, v = x + y (y may be null), grid-stride:
// partials[block] and partials[gridDim.x + block]
__global__ void __launch_bounds__(kNBlock) k_moments(const double *x, const double *y, int64_t count,
                                                    double *partials)
{
    __shared__ double sh[2][kNBlock / 64];
    double s = 0.0, s2 = 0.0;
    for (int64_t q = (int64_t)blockIdx.x * kNBlock + threadIdx.x; q < count; q += (int64_t)gridDim.x * kNBlock) {
        const double v = y ? x[q] + y[q] : x[q];
        s += v;
        s2 += v * v;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        s += __shfl_xor(s, o, 64);
        s2 += __shfl_xor(s2, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        sh[0][threadIdx.x >> 6] = s;
        sh[1][threadIdx.x >> 6] = s2;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        partials[blockIdx.x] = sh[0][0] + sh[0][1] + sh[0][2] + sh[0][3];
        partials[gridDim.x + blockIdx.x] = sh[1][0] + sh[1][1] + sh[1][2] + sh[1][3];
    }
}

__global__ void __launch_bounds__(kNBlock) k_adam(float *p, const float *g, float *m, float *v, int64_t count,
                                                 float lr, float b1, float b2, float eps, float c1, float c2,
                                                 float gscale)
{
    const int64_t e = (int64_t)blockIdx.x * kNBlock + threadIdx.x;
    if (e >= count) return;
    const float gr = gscale * g[e];
    const float mm = b1 * m[e] + (1.0f - b1) * gr;
    const float vv = b2 * v[e] + (1.0f - b2) * gr * gr;
    m[e] = mm;
    v[e] = vv;
    p[e] -= lr * (mm / c1) / (sqrtf(vv / c2) + eps);
}

struct Norm8 {
    float in_mean[4], in_inv[4], out_mean[4], out_std[4];
};

// x[v][c]: (rho5 + rho1, S_x, S_y, S_z) standardised, channels 4..7 zero
__global__ void __launch_bounds__(kNBlock) k_pack_input(const double *rho5, const double *rho1, const double *S,
                                                       int64_t V, Norm8 nm, u16 *x)
{
    const int64_t v = (int64_t)blockIdx.x * kNBlock + threadIdx.x;
    if (v >= V) return;
    float f[8];
    f[0] = (float)((rho5[v] + rho1[v] - nm.in_mean[0]) * nm.in_inv[0]);
    for (int a = 0; a < 3; a++) f[1 + a] = (float)((S[a * V + v] - nm.in_mean[1 + a]) * nm.in_inv[1 + a]);
    f[4] = f[5] = f[6] = f[7] = 0.0f;
    *(u32x4 *)(x + v * 8) = pack8(f);
}

__global__ void __launch_bounds__(kNBlock) k_pack_target(const double *u, const double *W, int64_t V, Norm8 nm,
                                                        u16 *t)
{
    const int64_t v = (int64_t)blockIdx.x * kNBlock + threadIdx.x;
    if (v >= V) return;
    float f[4];
    f[0] = (float)((u[v] - nm.out_mean[0]) / nm.out_std[0]);
    for (int a = 0; a < 3; a++) f[1 + a] = (float)((W[a * V + v] - nm.out_mean[1 + a]) / nm.out_std[1 + a]);
    uint2 o;
    o.x = pack2(f[0], f[1]);
    o.y = pack2(f[2], f[3]);
    *(uint2 *)(t + v * 4) = o;
}

__global__ void __launch_bounds__(kNBlock) k_unpack_output(const float *out, int64_t V, Norm8 nm, double *u,
                                                          double *W)
{
    const int64_t v = (int64_t)blockIdx.x * kNBlock + threadIdx.x;
    if (v >= V) return;
    u[v] = (double)out[v * 4] * nm.out_std[0] + nm.out_mean[0];
    for (int a = 0; a < 3; a++) W[a * V + v] = (double)out[v * 4 + 1 + a] * nm.out_std[1 + a] + nm.out_mean[1 + a];
}

} // namespace grtnn
