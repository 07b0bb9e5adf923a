// Generated by paper_2210_11122_amd.gen for the process gg_tt; do not edit.
// 3 Feynman diagrams (3 vertex contractions), 2 colour flows, 16 helicity combinations.
#include "../helas.hpp"
#include "../process.hpp"
#include "../colorsum.hpp"
#include "me.h"
namespace me {
namespace proc_gg_tt {
constexpr int NPAR = 4;
constexpr int NC = 2;
constexpr int NSLOT = 0;
template <class R, bool SDE>
__global__ __launch_bounds__(64 * 4, 6) void amp_kernel(const double* __restrict__ mom, int64_t n_evt, int64_t ld, const signed char* __restrict__ hel, int n_good, double mt, double gs, R* __restrict__ jamp, const int* __restrict__ chan, double* __restrict__ sde, FusedColour fc)
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
    constexpr int NW = 2;
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
    P4 m0_1 = PM(1);
    P4 m0_2 = PM(2);
    P4 m0_3 = PM(3);
    pin_p4<R>(m0_0);
    pin_p4<R>(m0_1);
    pin_p4<R>(m0_2);
    pin_p4<R>(m0_3);
    const W4<R> w0 = ext_ubar<R>(m0_2, mt, lam[2]);
    const W4<R> w1 = ext_v<R>(m0_3, mt, lam[3]);
    const W4<R> w2 = ext_vec<R>(m0_1, lam[1], false);
    const W4<R> w3 = fstr_v<R>(w1, w2, (m0_1) - m0_3, mt, gs);
    const W4<R> w4 = ext_vec<R>(m0_0, lam[0], false);
    P4 m1_0 = PM(0);
    P4 m1_3 = PM(3);
    a = amp_ffv<R>(w0, w3, w4, gs);
    pin_cx<R>(a);
    SDEACC(0, 5.333333333333333);
    JADD(0, 0, a.r); JADD(0, 1, a.i);
    pin_p4<R>(m1_0);
    pin_p4<R>(m1_3);
    const W4<R> w5 = fstr_v<R>(w1, w4, (m1_0) - m1_3, mt, gs);
    P4 m2_0 = PM(0);
    P4 m2_1 = PM(1);
    a = amp_ffv<R>(w0, w5, w2, gs);
    pin_cx<R>(a);
    SDEACC(1, 5.333333333333333);
    JADD(1, 0, a.r); JADD(1, 1, a.i);
    pin_p4<R>(m2_0);
    pin_p4<R>(m2_1);
    const W4<R> w6 = jf<R>(w0, w1, (m2_0 + m2_1), gs);
    a = amp_vvv<R>(w6, (-(m2_0 + m2_1)), w4, (m2_0), w2, (m2_1), gs);
    pin_cx<R>(a);
    SDEACC(2, 12.0);
    JADD(0, 0, a.i); JADD(0, 1, -a.r);
    JADD(1, 0, -a.i); JADD(1, 1, a.r);
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

static const int colour_num[NC * NC] = {16, -2, -2, 16};
static const int final_massive[NPAR - 2] = {1, 1};
static const int orderings[] = {0, 1, 1, 0};
static const int diagram_lines[] = {10, 6, 12};
template <class R>
static hipError_t launch(const double* mom, int64_t n_evt, int64_t ld, const signed char* hel, int n_good, double mt, double gs, R* jamp, const int* chan, double* sde, const FusedColour* fc, const HelicityGroups& hg, hipStream_t st)
{
    if (fc && ((chan && sizeof(R) == 4) || !fc->aop || (sizeof(R) == 8) != (fc->form == ME_FP64))) return hipErrorInvalidValue;
    const FusedColour none{nullptr, nullptr, 0, 0, nullptr, 0.0, 1};
    constexpr int WG = 4;  // waves (helicities) per workgroup
    int64_t blocks = ((n_evt + 63) / 64) * ((n_good + WG - 1) / WG);
    if (blocks == 0) return hipSuccess;
    if constexpr (sizeof(R) == 8) {  // the jamps and the channel weights by recursion
        return rec2::launch(mom, n_evt, ld, hg, mt, gs, jamp, chan, sde, fc, st);
    } else {
    if (chan)
        hipLaunchKernelGGL((amp_kernel<R, true>), dim3((unsigned)blocks), dim3(64 * WG), 0, st, mom, n_evt, ld, hel, n_good, mt, gs, jamp, chan, sde, none);
    else
        hipLaunchKernelGGL((amp_kernel<R, false>), dim3((unsigned)blocks), dim3(64 * WG), 0, st, mom, n_evt, ld, hel, n_good, mt, gs, jamp, nullptr, nullptr, fc ? *fc : none);
    }
    return hipGetLastError();
}
}  // namespace
const ProcessDesc* process_gg_tt()
{
    static const ProcessDesc d = {
        "gg_tt", proc_gg_tt::NPAR, proc_gg_tt::NC, 16, 256, 1, 1,
        proc_gg_tt::colour_num, 3, proc_gg_tt::final_massive, proc_gg_tt::orderings, 2,
        3, 3, 835.0, 835.0, 2451.0, 25.0, proc_gg_tt::NSLOT,
        proc_gg_tt::diagram_lines, 1, 1, 1, 0, 1, 0,
        nullptr, 1, 0, 0, 1,
        proc_gg_tt::launch<double>, proc_gg_tt::launch<float>,
    };
    return &d;
}
}  // namespace me
