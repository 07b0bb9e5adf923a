// Generated by paper_2210_11122_amd.gen for the process gg_gg; do not edit.
// 4 Feynman diagrams (6 vertex contractions), 6 colour flows, 16 helicity combinations.
#include "../helas.hpp"
#include "../process.hpp"
#include "../colorsum.hpp"
#include "me.h"
namespace me {
namespace proc_gg_gg {
constexpr int NPAR = 4;
constexpr int NC = 6;
constexpr int NSLOT = 0;
template <class R, bool SDE>
__global__ __launch_bounds__(64 * (sizeof(R) == 8 ? 4 : 4)) void amp_kernel(const double* __restrict__ mom, int64_t n_evt, int64_t ld, const signed char* __restrict__ hel, int n_good, double mt, double gs, R* __restrict__ jamp, const int* __restrict__ chan, double* __restrict__ sde, FusedColour fc)
{
    constexpr int WG = sizeof(R) == 8 ? 4 : 4;  // waves per workgroup
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
#define SDEACC(d, k) do { if constexpr (SDE) { const double w_ = (k) * ((double)a.r * (double)a.r + (double)a.i * (double)a.i); sde_all += w_; sde_ch += ((d) == ch) ? w_ : 0.0; if constexpr (sizeof(R) == 8) asm volatile("" : "+v"(sde_all), "+v"(sde_ch)); } } while (0)
    P4 m0_0 = PM(0);
    P4 m0_1 = PM(1);
    P4 m0_2 = PM(2);
    P4 m0_3 = PM(3);
    pin_p4<R>(m0_0);
    pin_p4<R>(m0_1);
    pin_p4<R>(m0_2);
    pin_p4<R>(m0_3);
    const W4<R> w0 = ext_vec<R>(m0_3, lam[3], true);
    const W4<R> w1 = ext_vec<R>(m0_0, lam[0], false);
    const W4<R> w2 = ext_vec<R>(m0_1, lam[1], false);
    const W4<R> w3 = ext_vec<R>(m0_2, lam[2], true);
    const W4<R> w4 = vvv_cur<R>(w2, (m0_1), w3, ((-m0_2)), gs);
    a = amp_vvv<R>(w0, ((-m0_3)), w1, (m0_0), w4, (m0_1 + (-m0_2)), gs);
    pin_cx<R>(a);
    sa = a;
    P4 m2_0 = PM(0);
    P4 m2_1 = PM(1);
    P4 m2_2 = PM(2);
    P4 m2_3 = PM(3);
    a = amp_vvvv<R, 0>(w0, w1, w2, w3, gs);
    pin_cx<R>(a);
    sa.r += a.r; sa.i += a.i;
    JADD(0, 0, (R)(-2) * sa.r - (R)(0) * sa.i); JADD(0, 1, (R)(-2) * sa.i + (R)(0) * sa.r);
    JADD(1, 0, (R)(2) * sa.r - (R)(0) * sa.i); JADD(1, 1, (R)(2) * sa.i + (R)(0) * sa.r);
    JADD(3, 0, (R)(2) * sa.r - (R)(0) * sa.i); JADD(3, 1, (R)(2) * sa.i + (R)(0) * sa.r);
    JADD(5, 0, (R)(-2) * sa.r - (R)(0) * sa.i); JADD(5, 1, (R)(-2) * sa.i + (R)(0) * sa.r);
    pin_p4<R>(m2_0);
    pin_p4<R>(m2_1);
    pin_p4<R>(m2_2);
    pin_p4<R>(m2_3);
    const W4<R> w5 = vvv_cur<R>(w1, (m2_0), w2, (m2_1), gs);
    a = amp_vvv<R>(w0, ((-m2_3)), w5, (m2_0 + m2_1), w3, ((-m2_2)), gs);
    pin_cx<R>(a);
    sa = a;
    P4 m4_0 = PM(0);
    P4 m4_1 = PM(1);
    P4 m4_2 = PM(2);
    P4 m4_3 = PM(3);
    a = amp_vvvv<R, 2>(w0, w1, w2, w3, gs);
    pin_cx<R>(a);
    sa.r -= a.r; sa.i -= a.i;
    JADD(0, 0, (R)(-2) * sa.r - (R)(0) * sa.i); JADD(0, 1, (R)(-2) * sa.i + (R)(0) * sa.r);
    JADD(2, 0, (R)(2) * sa.r - (R)(0) * sa.i); JADD(2, 1, (R)(2) * sa.i + (R)(0) * sa.r);
    JADD(4, 0, (R)(2) * sa.r - (R)(0) * sa.i); JADD(4, 1, (R)(2) * sa.i + (R)(0) * sa.r);
    JADD(5, 0, (R)(-2) * sa.r - (R)(0) * sa.i); JADD(5, 1, (R)(-2) * sa.i + (R)(0) * sa.r);
    pin_p4<R>(m4_0);
    pin_p4<R>(m4_1);
    pin_p4<R>(m4_2);
    pin_p4<R>(m4_3);
    const W4<R> w6 = vvv_cur<R>(w1, (m4_0), w3, ((-m4_2)), gs);
    a = amp_vvv<R>(w0, ((-m4_3)), w6, (m4_0 + (-m4_2)), w2, (m4_1), gs);
    pin_cx<R>(a);
    sa = a;
    a = amp_vvvv<R, 1>(w0, w1, w2, w3, gs);
    pin_cx<R>(a);
    sa.r -= a.r; sa.i -= a.i;
    JADD(1, 0, (R)(-2) * sa.r - (R)(0) * sa.i); JADD(1, 1, (R)(-2) * sa.i + (R)(0) * sa.r);
    JADD(2, 0, (R)(2) * sa.r - (R)(0) * sa.i); JADD(2, 1, (R)(2) * sa.i + (R)(0) * sa.r);
    JADD(3, 0, (R)(-2) * sa.r - (R)(0) * sa.i); JADD(3, 1, (R)(-2) * sa.i + (R)(0) * sa.r);
    JADD(4, 0, (R)(2) * sa.r - (R)(0) * sa.i); JADD(4, 1, (R)(2) * sa.i + (R)(0) * sa.r);
    if constexpr (SDE) {
        if (live && e < n_evt) {
            double* so = sde + (int64_t)h * 2 * ld + e;
            so[0] = sde_ch;
            so[ld] = sde_all;
        }
    }
    if (fc.aop) {  // colour sum here: D |M_h|^2 of this lane's event, to [h][event]
        double me_h;
        if constexpr (sizeof(R) == 8) {
            me_h = colour_sum_regs<NC>(Jr, static_cast<const double*>(fc.aop));
        } else {
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
        }
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

static const int colour_num[NC * NC] = {19, -2, -2, -2, -2, 4, -2, 19, -2, 4, -2, -2, -2, -2, 19, -2, 4, -2, -2, 4, -2, 19, -2, -2, -2, -2, 4, -2, 19, -2, 4, -2, -2, -2, -2, 19};
static const int final_massive[NPAR - 2] = {0, 0};
static const int orderings[] = {0, 1, 2, 0, 2, 1, 1, 0, 2, 1, 2, 0, 2, 0, 1, 2, 1, 0};
static const int diagram_lines[] = {0};
template <class R>
static hipError_t launch(const double* mom, int64_t n_evt, int64_t ld, const signed char* hel, int n_good, double mt, double gs, R* jamp, const int* chan, double* sde, const FusedColour* fc, const HelicityGroups& hg, hipStream_t st)
{
    if (fc && (chan || !fc->aop || (sizeof(R) == 8) != (fc->form == ME_FP64))) return hipErrorInvalidValue;
    const FusedColour none{nullptr, nullptr, 0, 0, nullptr, 0.0, 1};
    constexpr int WG = sizeof(R) == 8 ? 4 : 4;  // waves (helicities) per workgroup
    int64_t blocks = ((n_evt + 63) / 64) * ((n_good + WG - 1) / WG);
    if (blocks == 0) return hipSuccess;
    if (chan)
        hipLaunchKernelGGL((amp_kernel<R, true>), dim3((unsigned)blocks), dim3(64 * WG), 0, st, mom, n_evt, ld, hel, n_good, mt, gs, jamp, chan, sde, none);
    else
        hipLaunchKernelGGL((amp_kernel<R, false>), dim3((unsigned)blocks), dim3(64 * WG), 0, st, mom, n_evt, ld, hel, n_good, mt, gs, jamp, nullptr, nullptr, fc ? *fc : none);
    return hipGetLastError();
}
}  // namespace
const ProcessDesc* process_gg_gg()
{
    static const ProcessDesc d = {
        "gg_gg", proc_gg_gg::NPAR, proc_gg_gg::NC, 16, 256, 2, 1,
        proc_gg_gg::colour_num, 6, proc_gg_gg::final_massive, proc_gg_gg::orderings, 3,
        4, 6, 1462.0, 1462.0, 0.0, 0.0, proc_gg_gg::NSLOT,
        proc_gg_gg::diagram_lines, 1, 0, 1, 0, 0, 0,
        nullptr, 0, 0, 0, 0,
        proc_gg_gg::launch<double>, proc_gg_gg::launch<float>,
    };
    return &d;
}
}  // namespace me
