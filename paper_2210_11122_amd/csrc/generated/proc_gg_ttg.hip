// Generated by paper_2210_11122_amd.gen for the process gg_ttg; do not edit.
// 16 Feynman diagrams (18 vertex contractions), 6 colour flows, 32 helicity combinations.
#include "../helas.hpp"
#include "../process.hpp"
#include "../colorsum.hpp"
#include "me.h"
namespace me {
namespace proc_gg_ttg {
constexpr int NPAR = 5;
constexpr int NC = 6;
constexpr int NSLOT = 0;
template <class R, bool SDE>
__global__ __launch_bounds__(64 * 4, 3) void amp_kernel(const double* __restrict__ mom, int64_t n_evt, int64_t ld, const signed char* __restrict__ hel, int n_good, double mt, double gs, R* __restrict__ jamp, const int* __restrict__ chan, double* __restrict__ sde, FusedColour fc)
{
    constexpr int WG = 4;  // waves per workgroup
    __shared__ double lds[4 * NPAR * 64];
    const int lane = threadIdx.x & 63;
    const int64_t w = xcd_remap(blockIdx.x, gridDim.x);
    const int hpb = (n_good + WG - 1) / WG;  // workgroups per event block
    const int64_t e0 = (w / hpb) * 64;
    const int hr = (int)(w % hpb) * WG + (int)(threadIdx.x >> 6);
    const bool live = hr < n_good;  // a spare wave of the last group repeats a helicity, writes nothing
    const int h = live ? hr : n_good - 1;
    const int64_t e = e0 + lane;  // < ld: ld is a multiple of 64 covering the grid
    stage_momenta<NPAR, WG>(mom, n_evt, e0, lds, threadIdx.x);
#define PM(i) lds_p4(lds, i, lane)
    int lam[NPAR];
#pragma unroll
    for (int i = 0; i < NPAR; ++i) lam[i] = hel[h * NPAR + i];
    // 3 external wavefunctions computed once: in LDS, private to the lane, or in registers
    constexpr int XWP[3] = {0, 1, -1};
    constexpr int NXL = 2;
    __shared__ R xw_wg[NXL > 0 ? WG * NXL * 8 * 64 : 1];
    R* const xw = xw_wg + (threadIdx.x >> 6) * (NXL * 8 * 64);
    [[maybe_unused]] W4<R> xwr[3];
    { const W4<R> t = ext_ubar<R>(PM(2), mt, lam[2]); if constexpr (XWP[0] >= 0) st_w4<R>(xw, XWP[0], lane, t); else xwr[0] = t; }
    { const W4<R> t = ext_v<R>(PM(3), mt, lam[3]); if constexpr (XWP[1] >= 0) st_w4<R>(xw, XWP[1], lane, t); else xwr[1] = t; }
    { const W4<R> t = ext_vec<R>(PM(1), lam[1], false); if constexpr (XWP[2] >= 0) st_w4<R>(xw, XWP[2], lane, t); else xwr[2] = t; }
#define XW(k) (XWP[k] >= 0 ? ld_w4<R>(xw, XWP[k], lane) : xwr[k])
    constexpr int NW = 6;
    R Jr[2 * NW];
#pragma unroll
    for (int s = 0; s < 2 * NW; ++s) Jr[s] = (R)0;
#define JADD(s, ri, v) (Jr[2 * (s) + (ri)] += (v))
#define JGET(s, ri) Jr[2 * (s) + (ri)]
    cx<R> a, sa;
    int ch = -1;
    double sde_ch = 0.0, sde_all = 0.0;
    if constexpr (SDE) ch = (e < n_evt) ? chan[e] : -1;
#define SDEACC(d, k) do { if constexpr (SDE) { const double w_ = (k) * ((double)a.r * (double)a.r + (double)a.i * (double)a.i); sde_all += w_; sde_ch += ((d) == ch) ? w_ : 0.0; } } while (0)
    P4 m0_0 = PM(0);
    P4 m0_2 = PM(2);
    P4 m0_3 = PM(3);
    P4 m0_4 = PM(4);
    W4<R> y0_0 = XW(0);
    W4<R> y0_1 = XW(1);
    W4<R> y0_2 = XW(2);
    pin_p4<R>(m0_0);
    pin_p4<R>(m0_2);
    pin_p4<R>(m0_3);
    pin_p4<R>(m0_4);
    pin_w4<R>(y0_0);
    pin_w4<R>(y0_1);
    pin_w4<R>(y0_2);
    const W4<R> w0 = ext_vec<R>(m0_0, lam[0], false);
    const W4<R> w1 = fstr_u<R>(y0_0, w0, m0_2 - (m0_0), mt, gs);
    const W4<R> w2 = ext_vec<R>(m0_4, lam[4], true);
    const W4<R> w3 = fstr_v<R>(y0_1, w2, ((-m0_4)) - m0_3, mt, gs);
    P4 m1_1 = PM(1);
    P4 m1_3 = PM(3);
    W4<R> y1_1 = XW(1);
    W4<R> y1_2 = XW(2);
    a = amp_ffv<R>(w1, w3, y0_2, gs);
    pin_cx<R>(a);
    SDEACC(0, 7.111111111111111);
    JADD(0, 0, a.r); JADD(0, 1, a.i);
    pin_p4<R>(m1_1);
    pin_p4<R>(m1_3);
    pin_w4<R>(y1_1);
    pin_w4<R>(y1_2);
    const W4<R> w4 = fstr_v<R>(y1_1, y1_2, (m1_1) - m1_3, mt, gs);
    P4 m2_1 = PM(1);
    P4 m2_4 = PM(4);
    W4<R> y2_1 = XW(1);
    W4<R> y2_2 = XW(2);
    a = amp_ffv<R>(w1, w4, w2, gs);
    pin_cx<R>(a);
    SDEACC(1, 7.111111111111111);
    JADD(1, 0, a.r); JADD(1, 1, a.i);
    pin_p4<R>(m2_1);
    pin_p4<R>(m2_4);
    pin_w4<R>(y2_1);
    pin_w4<R>(y2_2);
    const W4<R> w5 = vvv_cur<R>(y2_2, (m2_1), w2, ((-m2_4)), gs);
    P4 m3_1 = PM(1);
    P4 m3_2 = PM(2);
    W4<R> y3_0 = XW(0);
    W4<R> y3_2 = XW(2);
    a = amp_ffv<R>(w1, y2_1, w5, gs);
    pin_cx<R>(a);
    SDEACC(2, 16.0);
    JADD(0, 0, a.i); JADD(0, 1, -a.r);
    JADD(1, 0, -a.i); JADD(1, 1, a.r);
    pin_p4<R>(m3_1);
    pin_p4<R>(m3_2);
    pin_w4<R>(y3_0);
    pin_w4<R>(y3_2);
    const W4<R> w6 = fstr_u<R>(y3_0, y3_2, m3_2 - (m3_1), mt, gs);
    P4 m4_0 = PM(0);
    P4 m4_1 = PM(1);
    W4<R> y4_0 = XW(0);
    W4<R> y4_2 = XW(2);
    a = amp_ffv<R>(w6, w3, w0, gs);
    pin_cx<R>(a);
    SDEACC(3, 7.111111111111111);
    JADD(2, 0, a.r); JADD(2, 1, a.i);
    pin_p4<R>(m4_0);
    pin_p4<R>(m4_1);
    pin_w4<R>(y4_0);
    pin_w4<R>(y4_2);
    const W4<R> w7 = vvv_cur<R>(w0, (m4_0), y4_2, (m4_1), gs);
    P4 m5_0 = PM(0);
    P4 m5_3 = PM(3);
    W4<R> y5_1 = XW(1);
    a = amp_ffv<R>(y4_0, w3, w7, gs);
    pin_cx<R>(a);
    SDEACC(9, 16.0);
    JADD(0, 0, a.i); JADD(0, 1, -a.r);
    JADD(2, 0, -a.i); JADD(2, 1, a.r);
    pin_p4<R>(m5_0);
    pin_p4<R>(m5_3);
    pin_w4<R>(y5_1);
    const W4<R> w8 = fstr_v<R>(y5_1, w0, (m5_0) - m5_3, mt, gs);
    W4<R> y6_0 = XW(0);
    a = amp_ffv<R>(w6, w8, w2, gs);
    pin_cx<R>(a);
    SDEACC(4, 7.111111111111111);
    JADD(3, 0, a.r); JADD(3, 1, a.i);
    pin_w4<R>(y6_0);
    P4 m7_0 = PM(0);
    P4 m7_4 = PM(4);
    W4<R> y7_1 = XW(1);
    a = amp_ffv<R>(y6_0, w8, w5, gs);
    pin_cx<R>(a);
    SDEACC(11, 16.0);
    JADD(3, 0, a.i); JADD(3, 1, -a.r);
    JADD(5, 0, -a.i); JADD(5, 1, a.r);
    pin_p4<R>(m7_0);
    pin_p4<R>(m7_4);
    pin_w4<R>(y7_1);
    const W4<R> w9 = vvv_cur<R>(w0, (m7_0), w2, ((-m7_4)), gs);
    W4<R> y8_0 = XW(0);
    a = amp_ffv<R>(w6, y7_1, w9, gs);
    pin_cx<R>(a);
    SDEACC(5, 16.0);
    JADD(2, 0, a.i); JADD(2, 1, -a.r);
    JADD(3, 0, -a.i); JADD(3, 1, a.r);
    pin_w4<R>(y8_0);
    P4 m9_2 = PM(2);
    P4 m9_4 = PM(4);
    W4<R> y9_0 = XW(0);
    a = amp_ffv<R>(y8_0, w4, w9, gs);
    pin_cx<R>(a);
    SDEACC(10, 16.0);
    JADD(1, 0, a.i); JADD(1, 1, -a.r);
    JADD(4, 0, -a.i); JADD(4, 1, a.r);
    pin_p4<R>(m9_2);
    pin_p4<R>(m9_4);
    pin_w4<R>(y9_0);
    const W4<R> w10 = fstr_u<R>(y9_0, w2, m9_2 - ((-m9_4)), mt, gs);
    W4<R> y10_2 = XW(2);
    a = amp_ffv<R>(w10, w4, w0, gs);
    pin_cx<R>(a);
    SDEACC(6, 7.111111111111111);
    JADD(4, 0, a.r); JADD(4, 1, a.i);
    pin_w4<R>(y10_2);
    W4<R> y11_1 = XW(1);
    a = amp_ffv<R>(w10, w8, y10_2, gs);
    pin_cx<R>(a);
    SDEACC(7, 7.111111111111111);
    JADD(5, 0, a.r); JADD(5, 1, a.i);
    pin_w4<R>(y11_1);
    P4 m12_0 = PM(0);
    P4 m12_1 = PM(1);
    P4 m12_4 = PM(4);
    W4<R> y12_0 = XW(0);
    W4<R> y12_1 = XW(1);
    a = amp_ffv<R>(w10, y11_1, w7, gs);
    pin_cx<R>(a);
    SDEACC(8, 16.0);
    JADD(4, 0, a.i); JADD(4, 1, -a.r);
    JADD(5, 0, -a.i); JADD(5, 1, a.r);
    pin_p4<R>(m12_0);
    pin_p4<R>(m12_1);
    pin_p4<R>(m12_4);
    pin_w4<R>(y12_0);
    pin_w4<R>(y12_1);
    const W4<R> w11 = jf<R>(y12_0, y12_1, (m12_0 + m12_1 + (-m12_4)), gs);
    W4<R> y13_2 = XW(2);
    a = amp_vvv<R>(w11, (-(m12_0 + m12_1 + (-m12_4))), w0, (m12_0), w5, (m12_1 + (-m12_4)), gs);
    pin_cx<R>(a);
    SDEACC(12, 36.0);
    sa = a;
    pin_w4<R>(y13_2);
    P4 m14_0 = PM(0);
    P4 m14_1 = PM(1);
    P4 m14_4 = PM(4);
    a = amp_vvvv<R, 0>(w11, w0, y13_2, w2, gs);
    pin_cx<R>(a);
    SDEACC(15, 36.0);
    sa.r += a.r; sa.i += a.i;
    JADD(0, 0, -sa.r); JADD(0, 1, -sa.i);
    JADD(1, 0, sa.r); JADD(1, 1, sa.i);
    JADD(3, 0, sa.r); JADD(3, 1, sa.i);
    JADD(5, 0, -sa.r); JADD(5, 1, -sa.i);
    pin_p4<R>(m14_0);
    pin_p4<R>(m14_1);
    pin_p4<R>(m14_4);
    W4<R> y15_2 = XW(2);
    a = amp_vvv<R>(w11, (-(m14_0 + m14_1 + (-m14_4))), w7, (m14_0 + m14_1), w2, ((-m14_4)), gs);
    pin_cx<R>(a);
    SDEACC(13, 36.0);
    sa = a;
    pin_w4<R>(y15_2);
    P4 m16_0 = PM(0);
    P4 m16_1 = PM(1);
    P4 m16_4 = PM(4);
    W4<R> y16_2 = XW(2);
    a = amp_vvvv<R, 2>(w11, w0, y15_2, w2, gs);
    pin_cx<R>(a);
    SDEACC(15, 36.0);
    sa.r -= a.r; sa.i -= a.i;
    JADD(0, 0, -sa.r); JADD(0, 1, -sa.i);
    JADD(2, 0, sa.r); JADD(2, 1, sa.i);
    JADD(4, 0, sa.r); JADD(4, 1, sa.i);
    JADD(5, 0, -sa.r); JADD(5, 1, -sa.i);
    pin_p4<R>(m16_0);
    pin_p4<R>(m16_1);
    pin_p4<R>(m16_4);
    pin_w4<R>(y16_2);
    W4<R> y17_2 = XW(2);
    a = amp_vvv<R>(w11, (-(m16_0 + m16_1 + (-m16_4))), w9, (m16_0 + (-m16_4)), y16_2, (m16_1), gs);
    pin_cx<R>(a);
    SDEACC(14, 36.0);
    sa = a;
    pin_w4<R>(y17_2);
    a = amp_vvvv<R, 1>(w11, w0, y17_2, w2, gs);
    pin_cx<R>(a);
    SDEACC(15, 36.0);
    sa.r -= a.r; sa.i -= a.i;
    JADD(1, 0, -sa.r); JADD(1, 1, -sa.i);
    JADD(2, 0, sa.r); JADD(2, 1, sa.i);
    JADD(3, 0, -sa.r); JADD(3, 1, -sa.i);
    JADD(4, 0, sa.r); JADD(4, 1, sa.i);
    if constexpr (SDE) {
        if (live && e < n_evt) {
            double* so = sde + (int64_t)h * 2 * ld + e;
            so[0] = sde_ch;
            so[ld] = sde_all;
        }
    }
    if (fc.aop) {  // colour sum here: D |M_h|^2 of this lane's event, to [h][event]
        double me_h;
        __syncthreads();
        R* Js = reinterpret_cast<R*>(lds);
        if constexpr (WG > 1) {  // the momentum area is shared: a staging area per wave
            __shared__ R Jst_wg[WG * 2 * NC * 64];
            Js = Jst_wg + (threadIdx.x >> 6) * (2 * NC * 64);
        }
#pragma unroll
        for (int s = 0; s < 2 * NC; ++s) Js[s * 64 + lane] = Jr[s];
        __syncthreads();
        if (fc.form == ME_MIXED_BF16)
            me_h = colour_sum_lds_h16<NC, Bf16Terms>(Js, static_cast<const __bf16*>(fc.aop), static_cast<const __bf16*>(fc.aop_lo), fc.lo_mask, lane);
        else
            me_h = colour_sum_lds_h16<NC, Fp16Terms>(Js, static_cast<const _Float16*>(fc.aop), static_cast<const _Float16*>(fc.aop), 0, lane);
        if (live && e < n_evt) reinterpret_cast<double*>(jamp)[(int64_t)h * n_evt + e] = me_h;
        return;
    }
    R jo[2 * NC];
#pragma unroll
    for (int s = 0; s < NC; ++s) {
        jo[2 * s] = JGET(s, 0);
        jo[2 * s + 1] = JGET(s, 1);
    }
    if (live && e < n_evt) {
        R* o = jamp + (int64_t)h * (2 * NC) * ld + e;
#pragma unroll
        for (int s = 0; s < 2 * NC; ++s) o[s * ld] = jo[s];
    }
#undef PM
#undef GB
#undef XW
#undef JADD
#undef JGET
#undef JZERO
#undef JTAKE
#undef JLAST
#undef JPUT
#undef SDEACC
}

static const int colour_num[NC * NC] = {64, -8, -8, 1, 1, 10, -8, 64, 1, 10, -8, 1, -8, 1, 64, -8, 10, 1, 1, 10, -8, 64, 1, -8, 1, -8, 10, 1, 64, -8, 10, 1, 1, -8, -8, 64};
static const int final_massive[NPAR - 2] = {1, 1, 0};
static const int orderings[] = {0, 1, 2, 0, 2, 1, 1, 0, 2, 1, 2, 0, 2, 0, 1, 2, 1, 0};
static const int diagram_lines[] = {24, 26, 10, 26, 18, 26, 6, 24, 6, 22, 6, 14, 10, 20, 20, 22, 20, 28, 24, 28, 10, 14, 18, 22, 12, 18, 12, 28, 12, 14, 12, 0};
template <class R>
static hipError_t launch(const double* mom, int64_t n_evt, int64_t ld, const signed char* hel, int n_good, double mt, double gs, R* jamp, const int* chan, double* sde, const FusedColour* fc, const HelicityGroups& hg, hipStream_t st)
{
    if (fc && ((chan && sizeof(R) == 4) || !fc->aop || (sizeof(R) == 8) != (fc->form == ME_FP64))) return hipErrorInvalidValue;
    const FusedColour none{nullptr, nullptr, 0, 0, nullptr, 0.0, 1};
    constexpr int WG = 4;  // waves (helicities) per workgroup
    int64_t blocks = ((n_evt + 63) / 64) * ((n_good + WG - 1) / WG);
    if (blocks == 0) return hipSuccess;
    if constexpr (sizeof(R) == 8) {  // the jamps and the channel weights by recursion
        return rec3::launch(mom, n_evt, ld, hg, mt, gs, jamp, chan, sde, fc, st);
    } else {
    if (chan)
        hipLaunchKernelGGL((amp_kernel<R, true>), dim3((unsigned)blocks), dim3(64 * WG), 0, st, mom, n_evt, ld, hel, n_good, mt, gs, jamp, chan, sde, none);
    else
        hipLaunchKernelGGL((amp_kernel<R, false>), dim3((unsigned)blocks), dim3(64 * WG), 0, st, mom, n_evt, ld, hel, n_good, mt, gs, jamp, nullptr, nullptr, fc ? *fc : none);
    }
    return hipGetLastError();
}
}  // namespace
const ProcessDesc* process_gg_ttg()
{
    static const ProcessDesc d = {
        "gg_ttg", proc_gg_ttg::NPAR, proc_gg_ttg::NC, 32, 256, 1, 1,
        proc_gg_ttg::colour_num, 9, proc_gg_ttg::final_massive, proc_gg_ttg::orderings, 3,
        16, 18, 3647.0, 3647.0, 24330.0, 169.0, proc_gg_ttg::NSLOT,
        proc_gg_ttg::diagram_lines, 2, 1, 1, 0, 4097, 0,
        nullptr, 1, 1, 0, 1,
        proc_gg_ttg::launch<double>, proc_gg_ttg::launch<float>,
    };
    return &d;
}
}  // namespace me
