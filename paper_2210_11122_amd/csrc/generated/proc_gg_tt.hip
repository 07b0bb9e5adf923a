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
__global__ __launch_bounds__(64 * (sizeof(R) == 8 ? 4 : 4), (sizeof(R) == 8 ? 4 : 6)) void amp_kernel(const double* __restrict__ mom, int64_t n_evt, int64_t ld, const signed char* __restrict__ hel, int n_good, double mt, double gs, R* __restrict__ jamp, const int* __restrict__ chan, double* __restrict__ sde, FusedColour fc)
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
template <class R>
__global__ __launch_bounds__(64, sizeof(R) == 8 ? 2 : 3) void amp_lanes(const double* __restrict__ mom, int64_t n_evt, const signed char* __restrict__ hel, int n_good, double mt, double gs, FusedColour fc)
{
    __shared__ double lds[4 * NPAR * 64];
    const int lane = threadIdx.x;
    const int64_t e0 = xcd_remap(blockIdx.x, gridDim.x) * 64;
    const int64_t e = e0 + lane;
    stage_momenta<NPAR, 1>(mom, n_evt, e0, lds, lane);
    // momenta re-read from LDS at each use, so that nothing computed from them is held
    // across the helicity loop
#define PM(i) lds_p4(lds, i, lane)
#define SDEACC(d, k) do { } while (0)
#define JADD(s, ri, v) (Jr[2 * (s) + (ri)] += (v))
    const W4<R> w0_p = ext_ubar<R>(PM(2), mt, 1), w0_m = ext_ubar<R>(PM(2), mt, -1);
    const W4<R> w1_p = ext_v<R>(PM(3), mt, 1), w1_m = ext_v<R>(PM(3), mt, -1);
    const W4<R> w2_p = ext_vec<R>(PM(1), 1, false), w2_m = ext_vec<R>(PM(1), -1, false);
    const W4<R> w4_p = ext_vec<R>(PM(0), 1, false), w4_m = ext_vec<R>(PM(0), -1, false);
    double s = 0.0, m = 0.0;
    int in_group = 0;
#pragma unroll 1
    for (int h = 0; h < n_good; ++h) {
        int lam[NPAR];
#pragma unroll
        for (int i = 0; i < NPAR; ++i) lam[i] = hel[h * NPAR + i];
        R Jr[2 * NC] = {};
        cx<R> a, sa;
        P4 m0_0 = PM(0);
        P4 m0_1 = PM(1);
        P4 m0_2 = PM(2);
        P4 m0_3 = PM(3);
        pin_p4<R>(m0_0);
        pin_p4<R>(m0_1);
        pin_p4<R>(m0_2);
        pin_p4<R>(m0_3);
        const W4<R> w0 = lam[2] > 0 ? w0_p : w0_m;
        const W4<R> w1 = lam[3] > 0 ? w1_p : w1_m;
        const W4<R> w2 = lam[1] > 0 ? w2_p : w2_m;
        const W4<R> w3 = fstr_v<R>(w1, w2, (m0_1) - m0_3, mt, gs);
        const W4<R> w4 = lam[0] > 0 ? w4_p : w4_m;
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
#pragma unroll
        for (int k = 0; k < 2 * NC; ++k) asm volatile("" : "+v"(Jr[k]));  // the jamps as the other paths hold them
        if constexpr (sizeof(R) == 8)
            m += colour_sum_regs<NC>(Jr, static_cast<const double*>(fc.aop));
        else if constexpr (NC == 1) {  // the 16-bit forms: one flow only
            if (fc.form == ME_MIXED_BF16)
                m += cs1_h16<Bf16Terms>(Jr[0], Jr[1], static_cast<const __bf16*>(fc.aop));
            else
                m += cs1_h16<Fp16Terms>(Jr[0], Jr[1], static_cast<const _Float16*>(fc.aop));
        }
        if (++in_group == fc.hel_per_group || h + 1 == n_good) {
            s += m;
            m = 0.0;
            in_group = 0;
        }
    }
    if (e < n_evt) fc.hsum_out[e] = s * fc.hsum_scale;
#undef PM
#undef SDEACC
#undef JADD
}

static const int colour_num[NC * NC] = {16, -2, -2, 16};
static const int final_massive[NPAR - 2] = {1, 1};
static const int orderings[] = {0, 1, 1, 0};
static const int diagram_lines[] = {10, 6, 12};
template <class R>
static hipError_t launch(const double* mom, int64_t n_evt, int64_t ld, const signed char* hel, int n_good, double mt, double gs, R* jamp, const int* chan, double* sde, const FusedColour* fc, const HelicityGroups& hg, hipStream_t st)
{
    if (fc && (chan || !fc->aop || (sizeof(R) == 8) != (fc->form == ME_FP64))) return hipErrorInvalidValue;
    const FusedColour none{nullptr, nullptr, 0, 0, nullptr, 0.0, 1};
    constexpr int WG = sizeof(R) == 8 ? 4 : 4;  // waves (helicities) per workgroup
    int64_t blocks = ((n_evt + 63) / 64) * ((n_good + WG - 1) / WG);
    if (blocks == 0) return hipSuccess;
    if (fc && fc->hsum_out) {  // the kernel also sums the helicities
        // batches large enough to fill the GPU with one lane per event (the mixed forms when
        // their one colour operand is exact in the 16-bit type, as the scalar form assumes)
        if (n_evt >= 65536 && (sizeof(R) == 8 || (NC == 1 && !(fc->lo_mask & 1)))) {
            hipLaunchKernelGGL((amp_lanes<R>), dim3((unsigned)((n_evt + 63) / 64)), dim3(64), 0, st, mom, n_evt, hel, n_good, mt, gs, *fc);
            return hipGetLastError();
        }
        return hipErrorInvalidValue;  // below the lane kernel's batch size: no such kernel
    }
    if (chan)
        hipLaunchKernelGGL((amp_kernel<R, true>), dim3((unsigned)blocks), dim3(64 * WG), 0, st, mom, n_evt, ld, hel, n_good, mt, gs, jamp, chan, sde, none);
    else
        hipLaunchKernelGGL((amp_kernel<R, false>), dim3((unsigned)blocks), dim3(64 * WG), 0, st, mom, n_evt, ld, hel, n_good, mt, gs, jamp, nullptr, nullptr, fc ? *fc : none);
    return hipGetLastError();
}
}  // namespace
const ProcessDesc* process_gg_tt()
{
    static const ProcessDesc d = {
        "gg_tt", proc_gg_tt::NPAR, proc_gg_tt::NC, 16, 256, 1, 1,
        proc_gg_tt::colour_num, 3, proc_gg_tt::final_massive, proc_gg_tt::orderings, 2,
        3, 3, 835.0, 835.0, proc_gg_tt::NSLOT,
        proc_gg_tt::diagram_lines, 1, 1, 1, 0, 65536,
        nullptr, 0,
        proc_gg_tt::launch<double>, proc_gg_tt::launch<float>,
    };
    return &d;
}
}  // namespace me
