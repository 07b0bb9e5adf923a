// Generated by paper_2210_11122_amd.gen for the process ee_mumu; do not edit.
// 1 Feynman diagrams (1 vertex contractions), 1 colour flows, 16 helicity combinations.
#include "../helas.hpp"
#include "../process.hpp"
#include "../colorsum.hpp"
#include "me.h"
namespace me {
namespace proc_ee_mumu {
constexpr int NPAR = 4;
constexpr int NC = 1;
constexpr int NSLOT = 0;
template <class R, bool SDE, bool HS = false>
__global__ __launch_bounds__(1024) void amp_kernel(const double* __restrict__ mom, int64_t n_evt, int64_t ld, const signed char* __restrict__ hel, int n_good, double mt, double gs, R* __restrict__ jamp, const int* __restrict__ chan, double* __restrict__ sde, FusedColour fc)
{
    constexpr int WG = 1;  // waves per workgroup
    __shared__ double lds[4 * NPAR * 64];
    const int lane = threadIdx.x & 63;
    const int64_t w = xcd_remap(blockIdx.x, gridDim.x);
    // with the helicity sum here, one workgroup holds all good helicities of its block
    constexpr bool hsum = HS && !SDE;
    const int wg = hsum ? n_good : WG;
    const int hpb = (n_good + wg - 1) / wg;  // workgroups per event block
    const int64_t e0 = (w / hpb) * 64;
    const int hr = (int)(w % hpb) * wg + (int)(threadIdx.x >> 6);
    const bool live = hr < n_good;  // a spare wave of the last group repeats a helicity, writes nothing
    const int h = live ? hr : n_good - 1;
    const int64_t e = e0 + lane;  // < ld: ld is a multiple of 64 covering the grid
    if constexpr (hsum)
        stage_momenta_n<NPAR>(mom, n_evt, e0, lds, threadIdx.x, 64 * wg);
    else
        stage_momenta<NPAR, WG>(mom, n_evt, e0, lds, threadIdx.x);
#define PM(i) lds_p4(lds, i, lane)
    int lam[NPAR];
#pragma unroll
    for (int i = 0; i < NPAR; ++i) lam[i] = hel[h * NPAR + i];
    constexpr int NW = 1;
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
    const W4<R> w0 = ext_vbar<R>(PM(0), 0.0, lam[0]);
    const W4<R> w1 = ext_u<R>(PM(1), 0.0, lam[1]);
    const W4<R> w2 = ext_v<R>(PM(2), 0.0, lam[2]);
    const W4<R> w3 = ext_ubar<R>(PM(3), 0.0, lam[3]);
    const W4<R> w4 = jf<R>(w0, w1, PM(0) + PM(1), gs);
    a = amp_ffv<R>(w3, w2, w4, gs);
    SDEACC(0, 1.0);
    JADD(0, 0, a.r); JADD(0, 1, a.i);
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
        if constexpr (hsum) {
            __shared__ R Jst[16 * 2 * NC * 64];
            Js = Jst + (threadIdx.x >> 6) * (2 * NC * 64);
        }
#pragma unroll
        for (int s = 0; s < 2 * NC; ++s) Js[s * 64 + lane] = Jr[s];
        __syncthreads();
        if (fc.form == ME_MIXED_BF16)
            me_h = colour_sum_lds_h16<NC, Bf16Terms>(Js, static_cast<const __bf16*>(fc.aop), static_cast<const __bf16*>(fc.aop_lo), fc.lo_mask, lane);
        else
            me_h = colour_sum_lds_h16<NC, Fp16Terms>(Js, static_cast<const _Float16*>(fc.aop), static_cast<const _Float16*>(fc.aop), 0, lane);
        if constexpr (hsum) {  // the helicity sum: the separate kernel's groups and order
            __shared__ double red[16 * 64];
            red[hr * 64 + lane] = me_h;
            __syncthreads();
            if (threadIdx.x < 64 && e < n_evt) {
                double s = 0.0;
                for (int h0 = 0; h0 < n_good; h0 += fc.hel_per_group) {
                    const int h1 = min(n_good, h0 + fc.hel_per_group);
                    double m = 0.0;
                    for (int k = h0; k < h1; ++k) m += red[k * 64 + lane];
                    s += m;
                }
                fc.hsum_out[e] = s * fc.hsum_scale;
            }
            return;
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
__global__ __launch_bounds__(64, 3) void amp_lanes(const double* __restrict__ mom, int64_t n_evt, const signed char* __restrict__ hel, int n_good, double mt, double gs, FusedColour fc)
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
    const W4<R> w0_p = ext_vbar<R>(PM(0), 0.0, 1), w0_m = ext_vbar<R>(PM(0), 0.0, -1);
    const W4<R> w1_p = ext_u<R>(PM(1), 0.0, 1), w1_m = ext_u<R>(PM(1), 0.0, -1);
    const W4<R> w2_p = ext_v<R>(PM(2), 0.0, 1), w2_m = ext_v<R>(PM(2), 0.0, -1);
    const W4<R> w3_p = ext_ubar<R>(PM(3), 0.0, 1), w3_m = ext_ubar<R>(PM(3), 0.0, -1);
    double s = 0.0, m = 0.0;
    int in_group = 0;
#pragma unroll 1
    for (int h = 0; h < n_good; ++h) {
        int lam[NPAR];
#pragma unroll
        for (int i = 0; i < NPAR; ++i) lam[i] = hel[h * NPAR + i];
        R Jr[2 * NC] = {};
        cx<R> a, sa;
        const W4<R> w0 = lam[0] > 0 ? w0_p : w0_m;
        const W4<R> w1 = lam[1] > 0 ? w1_p : w1_m;
        const W4<R> w2 = lam[2] > 0 ? w2_p : w2_m;
        const W4<R> w3 = lam[3] > 0 ? w3_p : w3_m;
        const W4<R> w4 = jf<R>(w0, w1, PM(0) + PM(1), gs);
        a = amp_ffv<R>(w3, w2, w4, gs);
        SDEACC(0, 1.0);
        JADD(0, 0, a.r); JADD(0, 1, a.i);
#pragma unroll
        for (int k = 0; k < 2 * NC; ++k) asm volatile("" : "+v"(Jr[k]));  // the jamps as the other paths hold them
        if constexpr (NC == 1) {  // the 16-bit forms: one flow only
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

static const int colour_num[NC * NC] = {1};
static const int final_massive[NPAR - 2] = {0, 0};
static const int orderings[] = {0};
static const int diagram_lines[] = {12};
template <class R>
static hipError_t launch(const double* mom, int64_t n_evt, int64_t ld, const signed char* hel, int n_good, double mt, double gs, R* jamp, const int* chan, double* sde, const FusedColour* fc, const HelicityGroups& hg, hipStream_t st)
{
    if (fc && ((chan && sizeof(R) == 4) || !fc->aop || (sizeof(R) == 8) != (fc->form == ME_FP64))) return hipErrorInvalidValue;
    const FusedColour none{nullptr, nullptr, 0, 0, nullptr, 0.0, 1};
    constexpr int WG = 1;  // waves (helicities) per workgroup
    int64_t blocks = ((n_evt + 63) / 64) * ((n_good + WG - 1) / WG);
    if (blocks == 0) return hipSuccess;
    if constexpr (sizeof(R) == 8) {  // the jamps and the channel weights by recursion
        return rec_ee::launch(mom, n_evt, ld, hg, mt, gs, jamp, chan, sde, fc, st);
    } else {
    if (fc && fc->hsum_out) {  // the kernel also sums the helicities
        // batches large enough to fill the GPU with one lane per event (the mixed forms when
        // their one colour operand is exact in the 16-bit type, as the scalar form assumes)
        if (n_evt >= 65536 && !(fc->lo_mask & 1)) {
            hipLaunchKernelGGL((amp_lanes<R>), dim3((unsigned)((n_evt + 63) / 64)), dim3(64), 0, st, mom, n_evt, hel, n_good, mt, gs, *fc);
            return hipGetLastError();
        }
        if (n_good > 16) return hipErrorInvalidValue;
        hipLaunchKernelGGL((amp_kernel<R, false, true>), dim3((unsigned)((n_evt + 63) / 64)), dim3(64 * n_good), 0, st, mom, n_evt, ld, hel, n_good, mt, gs, jamp, nullptr, nullptr, *fc);
        return hipGetLastError();
    }
    if (chan)
        hipLaunchKernelGGL((amp_kernel<R, true>), dim3((unsigned)blocks), dim3(64 * WG), 0, st, mom, n_evt, ld, hel, n_good, mt, gs, jamp, chan, sde, none);
    else
        hipLaunchKernelGGL((amp_kernel<R, false>), dim3((unsigned)blocks), dim3(64 * WG), 0, st, mom, n_evt, ld, hel, n_good, mt, gs, jamp, nullptr, nullptr, fc ? *fc : none);
    }
    return hipGetLastError();
}
}  // namespace
const ProcessDesc* process_ee_mumu()
{
    static const ProcessDesc d = {
        "ee_mumu", proc_ee_mumu::NPAR, proc_ee_mumu::NC, 16, 4, 1, 0,
        proc_ee_mumu::colour_num, 1, proc_ee_mumu::final_massive, proc_ee_mumu::orderings, 0,
        1, 1, 295.0, 295.0, 598.0, 9.0, proc_ee_mumu::NSLOT,
        proc_ee_mumu::diagram_lines, 1, 1, 1, 1, 1, 65536,
        nullptr, 1, 0, 0, 1,
        proc_ee_mumu::launch<double>, proc_ee_mumu::launch<float>,
    };
    return &d;
}
}  // namespace me
