// colorsum.hpp -- the colour-matrix contraction, batched over events: on the matrix cores in the mixed
// forms, as fused multiply-adds in the lane in FP64.
//
// For every (event, helicity) column the amplitude kernel leaves the colour-flow
// amplitudes J_c (c < NC, real and imaginary rows) in HBM, layout
// jamp[h][2c + re/im][column], column = event within the chunk, row stride ld.  Here
//     ME_h = (1/D) sum_{c,c'} (Re J_c Chat_{cc'} Re J_c' + Im J_c Chat_{cc'} Im J_c')
// with Chat = D * C the integer colour matrix; in the mixed forms as the matrix product Chat x J
// over 16 event columns per wavefront, followed by the column dot product and the sum over the
// filtered helicities in FP64.
//
// Symmetry (mixed forms): Chat is symmetric, so with the colour index cut into blocks of 16 the
// contraction equals J^T A J for the block upper-triangular A with A = Chat on diagonal
// blocks, 2 Chat above them and 0 below; only the tiles of A that touch the upper triangle
// are multiplied (36 of 64 blocks for 120 flows).  The host prepares A in that form.
//
// Helicity groups: blockIdx.y selects a group of consecutive filtered helicities.  With one
// group the kernel writes the averaged result; with several, each group writes its partial
// sum to part[group][event] and hel_reduce adds the groups in a fixed order, so every
// event's result is independent of the batch it came in.
//
// FP64 form: up to six flows as row chains, 24 and 120 flows through the block-diagonal form below.
// (The FP64 matrix cores run at the rate of the FP64 vector units, and the block form leaves 52 and 964
// of the 576 and 14400 products.)
// Mixed forms: the FP32 real (imaginary) rows of one (event, helicity) column are scaled by
// a power of two so that their largest |J| lies in [1/2, 1), split exactly into two 16-bit
// terms hi + lo * 2^-p (p = 11 for FP16, 8 for BF16), and contracted with
// v_mfma_f32_16x16x32_{f16,bf16} (FP32 accumulation); the dot product with the scaled FP32
// jamps is formed in FP64, unscaled exactly, and summed over helicities in FP64.  Colour
// numerators that a 16-bit type cannot hold exactly (BF16 keeps 8 significant bits) are
// split the same way on the host into A_hi + A_lo, both exact; tiles whose A_lo vanishes
// are skipped by a per-tile mask.
//
// MFMA operand layouts (lane l, i = l % 16, g = l / 16):
//   16x16x32:      A[i][8g + t], B[8g + t][i] (t = 0..7), D[4g + r][i]
// In the 16x16x32 form the k slot (kb, 8g + t) carries colour 16 (2 kb + t / 4) + 4 g + t % 4,
// so that the B elements a lane holds are exactly the D rows it receives (the dot product
// then needs no data exchange between lanes).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "flows.hpp"
#include "generated/colour_blocks.hpp"
#include "helas.hpp"
#include "process.hpp"

namespace me {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

__device__ __forceinline__ double sum_lane_groups(double x)
{
    x += __shfl_xor(x, 16, 64);
    x += __shfl_xor(x, 32, 64);
    return x;
}
__device__ __forceinline__ float max_lane_groups(float x)
{
    x = fmaxf(x, __shfl_xor(x, 16, 64));
    x = fmaxf(x, __shfl_xor(x, 32, 64));
    return x;
}

// tile count of the block upper-triangular colour matrix in the mixed forms
__host__ __device__ constexpr int cs16_tiles(int nc)
{
    int n = 0;
    for (int mt = 0; mt < (nc + 15) / 16; ++mt)
        for (int kb = mt / 2; kb < ((nc + 15) / 16 + 1) / 2; ++kb) ++n;
    return n;
}

// the colour-matrix operands are re-read from the cache for every helicity: hiding the table
// pointer from loop-invariant code motion keeps the compiler from hoisting all of them into
// registers (which would leave one wave per SIMD for the large matrix)
template <class P>
__device__ __forceinline__ const P* opaque(const P* p)
{
    __asm__ volatile("" : "+s"(p));
    return p;
}

// store or accumulate the helicity-group result of one event
__device__ __forceinline__ void cs_store(double me, int64_t e, int64_t n_evt, double scale_avg, double* out,
                                         double* part)
{
    if (gridDim.y == 1)
        out[e] = me * scale_avg;
    else
        part[(int64_t)blockIdx.y * n_evt + e] = me;
}

// One colour flow (the e+e- processes): D |M_h|^2 = Chat_00 (Re J^2 + Im J^2), a scalar, with
// one rounding sequence wherever it is formed (the colour-sum kernel, the amplitude kernels
// that do the colour sum themselves); the empty asm keeps the compiler from fusing the last
// multiply into a later addition.  c00 = aop[0], the one operand of the 1x1 table.
__device__ __forceinline__ double cs1(double jr, double ji, double c00)
{
    double v = c00 * __builtin_fma(jr, jr, ji * ji);
    asm volatile("" : "+v"(v));
    return v;
}

// One colour flow in a mixed form, as the 16-bit tile computes it for that column: the jamp
// scaled by a power of two into [1/2, 1), split into hi + lo * 2^-p, both multiplied by the one
// operand (exact in FP32, the only non-zero products the tile adds), and the dot product formed
// in FP64 and unscaled.  Bitwise the tile's value (16-bit element types below).
template <class T>
__device__ __forceinline__ double cs1_h16_part(float x, float a00)
{
    float mx = fabsf(x);
    int ex = 0;
    if (mx > 0.0f) frexpf(mx, &ex);
    const float s = ldexpf(1.0f, -ex);
    const float v = x * s;
    const typename T::elem hi = T::round(v);
    const typename T::elem lo = T::round((v - T::value(hi)) * T::LO);
    const float dh = a00 * T::value(hi), dl = a00 * T::value(lo);
    double acc = 0.0;
    acc += (double)v * ((double)dh + (double)dl * (1.0 / T::LO));
    return acc / ((double)s * (double)s);
}
template <class T>
__device__ __forceinline__ double cs1_h16(float jr, float ji, const typename T::elem* aop)
{
    const float a00 = T::value(aop[0]);
    double part = 0.0;
    part += cs1_h16_part<T>(jr, a00);
    part += cs1_h16_part<T>(ji, a00);
    asm volatile("" : "+v"(part));
    return part;
}

// Two colour flows (gg -> tt~): D |M_h|^2 = sum over re/im of J^T Chat J with the 2x2 integer
// matrix, as a scalar in one fixed rounding sequence (rows of Chat J by fused multiply-adds, then
// the dot product); Chat_rc = aop[r + 16 c], the diagonal tile of the 16x4 table.
__device__ __forceinline__ double cs2_part(double a, double b, double c00, double c01, double c10, double c11)
{
    const double r0 = __builtin_fma(c01, b, c00 * a), r1 = __builtin_fma(c11, b, c10 * a);
    return __builtin_fma(b, r1, a * r0);
}
__device__ __forceinline__ double cs2(double j0r, double j0i, double j1r, double j1i, const double* aop)
{
    const double c00 = aop[0], c10 = aop[1], c01 = aop[16], c11 = aop[17];
    double v = cs2_part(j0r, j1r, c00, c01, c10, c11) + cs2_part(j0i, j1i, c00, c01, c10, c11);
    asm volatile("" : "+v"(v));
    return v;
}
// Up to 16 flows as a scalar (gg -> tt~g: 6): for re and im, each row of Chat J as a chain of
// fused multiply-adds over c, then the dot product with J as another; Chat_rc is
// aop[(c / 4) * 64 + r + 16 (c % 4)], the diagonal 16-block of the table (A = Chat there).
// j(c, ri) gives the jamps.
template <int NC, class Jget>
__device__ __forceinline__ double csn(const Jget& j, const double* aop)
{
    static_assert(NC <= 16, "one diagonal tile");
    double v = 0.0;
#pragma unroll
    for (int ri = 0; ri < 2; ++ri) {
        double s = 0.0;
#pragma unroll
        for (int r = 0; r < NC; ++r) {
            double row = aop[r] * j(0, ri);
#pragma unroll
            for (int c = 1; c < NC; ++c) row = __builtin_fma(aop[(c / 4) * 64 + r + 16 * (c % 4)], j(c, ri), row);
            s = __builtin_fma(j(r, ri), row, s);
        }
        v += s;
    }
    asm volatile("" : "+v"(v));
    return v;
}
// the scalar forms from a lane's own jamps Jr[2 c + re/im] (amplitude kernels with register jamps)
template <int NC>
__device__ __forceinline__ double colour_sum_regs(const double* Jr, const double* __restrict__ aop)
{
    static_assert(NC <= 6, "scalar colour sums up to six flows");
    if constexpr (NC == 1)
        return cs1(Jr[0], Jr[1], aop[0]);
    else if constexpr (NC == 2)
        return cs2(Jr[0], Jr[1], Jr[2], Jr[3], aop);
    else
        return csn<NC>([&](int c, int ri) { return Jr[2 * c + ri]; }, aop);
}

// 24 and 120 flows (gg -> tt~gg, gg -> tt~ggg) in FP64: the colour matrix in its block form
// (flows.hpp), D |M_h|^2 = sum over re/im and over the eight blocks of z^T B z, as scalar fused
// multiply-adds on one lane's own jamps.  The blocks leave 80 (1808) of the 576 (14400) products of
// the full matrix, and their symmetry 52 (964), so the sum is cheaper here than as matrix-core
// tiles of the full matrix (which took 64 (512) 16x16x4 tiles per 64 events), and needs no exchange
// between lanes.  The entries are compile-time integers: as scalar loads from a table, each batch
// of them was waited for (120 flows: 390 us per 4096 events x 128 helicities).  The rounding
// sequence is fixed: no contraction beyond the written ones.
//
// y of the orbit O for the signs numbered S = 0 .. 3, (chi01, chi23) = (+,+), (+,-), (-,+), (-,-),
// from its four flows (relabelled by neither, (01), (23), both)
template <int S>
__device__ __forceinline__ double orbit_sum(double m00, double m10, double m01, double m11)
{
#pragma clang fp contract(off)
    const double a = S < 2 ? m00 + m10 : m00 - m10, c = S < 2 ? m01 + m11 : m01 - m11;
    return S % 2 ? a - c : a + c;
}
// the two blocks of the signs S from their y over all orbits (of the real or imaginary parts)
template <int NG, int S>
__device__ __forceinline__ double sign_blocks(const double (&y)[FlowBlocks<NG>::NO])
{
#pragma clang fp contract(off)
    constexpr int NP = flow_blocks<NG>.n_pair, NF = flow_blocks<NG>.n_fix;
    double q = 0.0;
    static_for<2>([&](auto K) {
        constexpr int rho = K ? -1 : 1, chi = (S == 0 || S == 3) ? 1 : -1;
        constexpr int nz = NP + (rho == chi ? NF : 0);
        // table entries before this block: of the signs before (a block with the fixed orbits and one
        // without, each), and of this sign's first block
        constexpr int T0 = NP * (NP + 1) / 2, T1 = (NP + NF) * (NP + NF + 1) / 2;
        constexpr int t0 = S * (T0 + T1) + (K ? (chi > 0 ? T1 : T0) : 0);
        double z[nz];
        static_for<nz>([&](auto I) {
            if constexpr (I < NP) {
                const double u = y[flow_blocks<NG>.pair[I][0]], v = y[flow_blocks<NG>.pair[I][1]];
                z[I] = rho * chi > 0 ? u + v : u - v;
            } else {
                z[I] = y[flow_blocks<NG>.fix[I - NP]];
            }
        });
        static_for<nz>([&](auto I) {
            constexpr int t = t0 + I * nz - I * (I - 1) / 2;
            double r = ColourBlocks<NG>::table[t] * z[I];
            static_for<nz - I - 1>([&](auto J) {
                constexpr int c = ColourBlocks<NG>::table[t + 1 + J];
                if constexpr (c != 0) r = __builtin_fma((double)c, z[I + 1 + J], r);
            });
            q = __builtin_fma(z[I], r, q);
        });
    });
    return q;
}
template <int NG, int S, class Get>
__device__ __forceinline__ double colour_blocks_part(const Get& x)
{
    double y[FlowBlocks<NG>::NO];
    static_for<FlowBlocks<NG>::NO>([&](auto O) {
        y[O] = orbit_sum<S>(x(std::integral_constant<int, flow_blocks<NG>.member[O][0][0]>{}),
                            x(std::integral_constant<int, flow_blocks<NG>.member[O][1][0]>{}),
                            x(std::integral_constant<int, flow_blocks<NG>.member[O][0][1]>{}),
                            x(std::integral_constant<int, flow_blocks<NG>.member[O][1][1]>{}));
    });
    return sign_blocks<NG, S>(y);
}
// the blocks of all signs of the real or the imaginary parts, and D |M_h|^2 from both
template <int NG, class Get>
__device__ __forceinline__ double colour_blocks_signs(const Get& x)
{
#pragma clang fp contract(off)
    return (colour_blocks_part<NG, 0>(x) + colour_blocks_part<NG, 1>(x)) +
           (colour_blocks_part<NG, 2>(x) + colour_blocks_part<NG, 3>(x));
}
__device__ __forceinline__ double colour_blocks_total(double r, double i)
{
    double v = (r + i) * (1.0 / 64.0);
    asm volatile("" : "+v"(v));
    return v;
}
template <int NG>
__device__ __forceinline__ double colour_blocks(const cx<double> (&J)[factorial(NG)])
{
    const auto re = [&](auto F) { return J[F].r; };
    const auto im = [&](auto F) { return J[F].i; };
    return colour_blocks_total(colour_blocks_signs<NG>(re), colour_blocks_signs<NG>(im));
}

// |M_h|^2 of row h to the helicities that it stands for
template <bool PAIRS = true>
__device__ __forceinline__ void store_hel(double* __restrict__ out, const int2* __restrict__ members, int h, double v)
{
    if constexpr (!PAIRS) {
        out[h] = v;
    } else {
        const int2 m = members[h];
        if (m.x >= 0) out[m.x] = v;
        if (m.y >= 0) out[m.y] = v;
    }
}

// The separate colour sum in FP64: one lane per event, the rows (good helicities, or pairs) of the
// group blockIdx.y in turn.  aop: the 16x4 tile table (up to six flows).
template <int NC, bool PAIRS>
__global__ __launch_bounds__(NC > 6 ? 64 : 256) void colour_sum_f64(
    const double* __restrict__ J, int64_t ld, int n_good, int hel_per_group, int64_t n_evt,
    const double* __restrict__ aop, double scale_hel, double scale_avg, double* __restrict__ out,
    double* __restrict__ out_hel, double* __restrict__ part, const int2* __restrict__ members, int n_hel)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n_evt) return;
    const int h0 = blockIdx.y * hel_per_group, h1 = min(n_good, h0 + hel_per_group);
    double me = 0.0;
    for (int h = h0; h < h1; ++h) {
        const double* Jh = J + (int64_t)h * (2 * NC) * ld + e;
        double me_h;
        if constexpr (NC <= 6) {
            double Jr[2 * NC];
#pragma unroll
            for (int s = 0; s < 2 * NC; ++s) Jr[s] = Jh[(int64_t)s * ld];
            me_h = colour_sum_regs<NC>(Jr, aop);
        } else {
            static_assert(NC == 24, "120 flows: colour_sum_f64_120");
            cx<double> Jr[NC];
            static_for<NC>([&](auto F) { Jr[F] = {Jh[(int64_t)(2 * F) * ld], Jh[(int64_t)(2 * F + 1) * ld]}; });
            me_h = colour_blocks<4>(Jr);
        }
        if (out_hel) store_hel<PAIRS>(out_hel + e * n_hel, members, h, me_h * scale_hel);
        me += members_of<PAIRS>(members, h) * me_h;
    }
    cs_store(me, e, n_evt, scale_avg, out, part);
}
// 16-bit element types of the mixed colour sum
struct Fp16Terms {
    typedef _Float16 elem;
    typedef v8h vec;
    static constexpr float LO = 2048.0f;  // hi keeps 11 significant bits
    static __device__ __forceinline__ elem round(float v) { return (_Float16)v; }
    static __device__ __forceinline__ float value(elem x) { return (float)x; }
    static __device__ __forceinline__ v4f mfma(vec a, vec b, v4f c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
    }
};
struct Bf16Terms {
    typedef __bf16 elem;
    typedef v8bf vec;
    static constexpr float LO = 256.0f;  // hi keeps 8 significant bits
    static __device__ __forceinline__ elem round(float v) { return (__bf16)v; }
    static __device__ __forceinline__ float value(elem x) { return (float)x; }
    static __device__ __forceinline__ v4f mfma(vec a, vec b, v4f c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
};

// One (16-event tile, helicity) column block of the mixed forms: this lane's share of
// D * |M_h|^2 for event column i, from the FP32 jamps load(c, ri) of its column.
template <int NC, class T, bool AREG, class Load>
__device__ __forceinline__ double cs16_column(const Load& load, const typename T::vec* A,
                                              const typename T::elem* aop, const typename T::elem* aop_lo,
                                              uint64_t lo_mask, int lane)
{
    typedef typename T::vec vec;
    typedef typename T::elem elem;
    constexpr int MT = (NC + 15) / 16, KB = (MT + 1) / 2;
    const int g = lane >> 4;
    double part_h = 0.0;
#pragma unroll 1
    for (int ri = 0; ri < 2; ++ri) {
        // x[kb][t]: colour 16 (2 kb + t / 4) + 4 g + t % 4 of column i
        float x[KB][8];
        float mx = 0.0f;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const int c = 16 * (2 * kb + t / 4) + 4 * g + t % 4;
                const float v = (c < NC) ? (float)load(c, ri) : 0.0f;
                x[kb][t] = v;
                mx = fmaxf(mx, fabsf(v));
            }
        mx = max_lane_groups(mx);
        // power-of-two scale: largest |J| of the column into [1/2, 1)
        int ex = 0;
        if (mx > 0.0f) frexpf(mx, &ex);
        const float s = ldexpf(1.0f, -ex);
        vec bh[KB], bl[KB];
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const float v = x[kb][t] * s;
                const elem hi = T::round(v);
                bh[kb][t] = hi;
                bl[kb][t] = T::round((v - T::value(hi)) * T::LO);
                x[kb][t] = v;
            }
        double acc = 0.0;  // the column dot product, in FP64 (colour sums can cancel)
        int q = 0;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const elem* ap = opaque(aop);
            const elem* ap_lo = opaque(aop_lo);
            v4f dh = {0.f, 0.f, 0.f, 0.f}, dl = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kb = mt / 2; kb < KB; ++kb, ++q) {
                const vec a = AREG ? A[q] : *reinterpret_cast<const vec*>(ap + (q * 64 + lane) * 8);
                dh = T::mfma(a, bh[kb], dh);
                dl = T::mfma(a, bl[kb], dl);
                if ((lo_mask >> q) & 1) {
                    const vec alo = *reinterpret_cast<const vec*>(ap_lo + (q * 64 + lane) * 8);
                    dh = T::mfma(alo, bh[kb], dh);
                }
            }
            // D rows 16 mt + 4 g + r are this lane's x[mt / 2][4 (mt % 2) + r]
#pragma unroll
            for (int r = 0; r < 4; ++r)
                acc += (double)x[mt / 2][4 * (mt % 2) + r] * ((double)dh[r] + (double)dl[r] * (1.0 / T::LO));
        }
        part_h += acc / ((double)s * (double)s);
    }
    return part_h;
}

// A operands, per lane, in the kernel's tile order (mt ascending, then kb >= mt / 2):
// aop[(q * 64 + l) * 8 + t] = A[16 mt + l % 16][colour of k slot (kb, 8 (l / 16) + t)].
// aop_lo (A_lo, same layout) is read for the tiles whose bit is set in lo_mask.
template <int NC, class T>
__global__ __launch_bounds__(256) void colour_sum_h16(const float* __restrict__ J, int64_t ld, int n_good,
                                                      int hel_per_group, int64_t n_evt,
                                                      const typename T::elem* __restrict__ aop,
                                                      const typename T::elem* __restrict__ aop_lo, uint64_t lo_mask,
                                                      double scale_hel, double scale_avg, double* __restrict__ out,
                                                      double* __restrict__ out_hel, double* __restrict__ part)
{
    typedef typename T::vec vec;
    constexpr int NT = cs16_tiles(NC);
    constexpr bool AREG = NT <= 8;
    const int lane = threadIdx.x & 63;
    const int64_t e0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 16;
    if (e0 >= n_evt) return;
    const int i = lane & 15, g = lane >> 4;
    const int64_t e = e0 + i;
    const bool valid = e < n_evt;
    const int64_t ec = valid ? e : n_evt - 1;
    const int h0 = blockIdx.y * hel_per_group, h1 = min(n_good, h0 + hel_per_group);
    vec A[AREG ? NT : 1];
    if (AREG) {
#pragma unroll
        for (int q = 0; q < NT; ++q) A[q] = *reinterpret_cast<const vec*>(aop + (q * 64 + lane) * 8);
    }
    double me = 0.0;
    for (int h = h0; h < h1; ++h) {
        const float* Jh = J + (int64_t)h * (2 * NC) * ld;
        const auto load = [&](int c, int ri) { return Jh[(int64_t)(2 * c + ri) * ld + ec]; };
        double part_h = sum_lane_groups(cs16_column<NC, T, AREG>(load, A, aop, aop_lo, lo_mask, lane));
        if (out_hel && g == 0 && valid) out_hel[e * n_good + h] = part_h * scale_hel;
        me += part_h;
    }
    if (g == 0 && valid) cs_store(me, e, n_evt, scale_avg, out, part);
}

// The same contractions inside an amplitude kernel whose wave (64 events of one helicity) holds
// its jamps in LDS, Jl[(2c + re/im) * 64 + event]: for each of the four 16-event tiles the lanes
// load the B operands from the other lanes' slots and run the same column body as the separate
// kernels (so each |M_h|^2 is bitwise the same).  Returns this lane's event's D * |M_h|^2.  The
// caller must have completed all jamp updates of the wave (a barrier) before the call.
template <int NC, class T>
__device__ __forceinline__ double colour_sum_lds_h16(const float* Jl, const typename T::elem* __restrict__ aop,
                                                     const typename T::elem* __restrict__ aop_lo, uint64_t lo_mask,
                                                     int lane)
{
    typedef typename T::vec vec;
    constexpr int NT = cs16_tiles(NC);
    static_assert(NT <= 8, "operands held in registers");
    const int i = lane & 15, g = lane >> 4;
    vec A[NT];
#pragma unroll
    for (int q = 0; q < NT; ++q) A[q] = *reinterpret_cast<const vec*>(aop + (q * 64 + lane) * 8);
    double mine = 0.0;
#pragma unroll 1
    for (int j = 0; j < 4; ++j) {
        const auto load = [&](int c, int ri) { return Jl[(2 * c + ri) * 64 + 16 * j + i]; };
        const double part_h = sum_lane_groups(cs16_column<NC, T, true>(load, A, aop, aop_lo, lo_mask, lane));
        if (g == j) mine = part_h;
    }
    return mine;
}

// The helicity sum after the fused colour sum, in the order of the separate colour-sum kernel
// with the same helicity groups: within each group of hel_per_group consecutive rows from
// zero, then the groups in order (so the result is bitwise that of the separate kernels).
// part_h[row][e] = D |M_h|^2.  PAIRS: the rows stand for one or two helicities (members); HEL: also the
// helicities' own |M_h|^2 to out_hel.  Instances, not tests per row: a short loop of dependent additions, with the
// tests in it a mixed gg -> tt~g call of 4000 events took 25.0 us instead of 24.7.
template <bool PAIRS, bool HEL>
__global__ __launch_bounds__(256) void hel_reduce_grouped(const double* __restrict__ part_h, int n_rows,
                                                          int hel_per_group, int64_t n_evt, double scale,
                                                          double* __restrict__ out, const int2* __restrict__ members,
                                                          double* __restrict__ out_hel, int n_hel, double scale_hel)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= n_evt) return;
    double s = 0.0;
    for (int h0 = 0; h0 < n_rows; h0 += hel_per_group) {
        const int h1 = min(n_rows, h0 + hel_per_group);
        double m = 0.0;
        for (int h = h0; h < h1; ++h) {
            const double v = part_h[(int64_t)h * n_evt + e];
            if constexpr (HEL) store_hel<PAIRS>(out_hel + e * n_hel, members, h, v * scale_hel);
            m += members_of<PAIRS>(members, h) * v;
        }
        s += m;
    }
    out[e] = s * scale;
}

// out[e] = scale * sum over helicity groups of part[group][e], groups in order
static __global__ __launch_bounds__(256) void hel_reduce(const double* __restrict__ part, int groups, int64_t n_evt,
                                                  double scale, double* __restrict__ out)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= n_evt) return;
    double s = 0.0;
    for (int k = 0; k < groups; ++k) s += part[(int64_t)k * n_evt + e];
    out[e] = s * scale;
}

}  // namespace me
