// rec_ee_mumu.hip -- FP64 |M|^2 of e+e- -> mu+ mu- through a photon, one lane per event.
//
// The amplitude is the product of an electron and a muon current over s.  The spinors and currents
// of each helicity are formed once per event and every good combination is one product of two
// currents; the colour sum (one flow) and the helicity sum stay in the lane, one launch for any
// batch size.  2^20 events 92 -> 51 us per call with the momenta read from HBM (2.8 TB/s; the bytes take
// 28 us at the rate of a large copy), 69 -> 36 us where one batch is evaluated again and again and stays in
// the 256 MB last-level cache; 8192 events 8.6 us, host time.  (Cut to 128 registers for four waves per
// SIMD it spills.)
#include "colorsum.hpp"
#include "process.hpp"
#include "recursion.hpp"

namespace me {
namespace rec_ee {
using namespace rec;

constexpr int NPAR = 4, NC = 1;

// HSUM: |M|^2 to fc.hsum_out; else the jamps
template <bool HSUM>
__global__ __launch_bounds__(64, 2) void amp_rec(const double* __restrict__ mom, int64_t n_evt, int64_t ld,
                                                 const int* __restrict__ row, double g,
                                                 double* __restrict__ jamp, const int* __restrict__ chan,
                                                 double* __restrict__ sde, FusedColour fc)
{
    __shared__ double lds[4 * NPAR * 64];
    const unsigned lane = threadIdx.x;
    const int* const count = row + 8;   // good helicities of each combination's row
    const int64_t e0 = xcd_remap(blockIdx.x, gridDim.x) * 64, e = e0 + lane;
    stage_momenta<NPAR, 1>(mom, n_evt, e0, lds, lane);
    const P4 p0 = lds_p4(lds, 0, lane), p1 = lds_p4(lds, 1, lane), p2 = lds_p4(lds, 2, lane), p3 = lds_p4(lds, 3, lane);
    // (ubar gamma^mu s)(ubar' gamma_mu s') = 2 dot2(pair, pair')
    const double f = 2.0 * g * g * rcp(sq(lc(p0) + lc(p1)));
    const V4 ep = spinor(ext_vbar<double>(p0, 0.0, -1));   // the opposite combinations have equal |M_h|^2
    const V4 em[2] = {spinor(ext_u<double>(p1, 0.0, -1)), spinor(ext_u<double>(p1, 0.0, 1))};
    const V4 mp[2] = {spinor(ext_v<double>(p2, 0.0, -1)), spinor(ext_v<double>(p2, 0.0, 1))};
    const V4 mm[2] = {spinor(ext_ubar<double>(p3, 0.0, -1)), spinor(ext_ubar<double>(p3, 0.0, 1))};
    double s = 0.0, m = 0.0;
    int in_group = 0;
    static_for<2>([&](auto A) {
        // good combinations with these electron helicities?
        if (!(count[4 * A] | count[4 * A + 1] | count[4 * A + 2] | count[4 * A + 3])) return;
        const V4 c = pair(ep, em[A]);
        static_for<4>([&](auto B) {
            constexpr int h = 4 * A + B;
            if (!count[h]) return;
            C j = times(f, dot2(c, pair(mm[B % 2], mp[B / 2])));
            pin_cx(j);   // rounded the same way whatever uses it
            if constexpr (HSUM) {
                // in the groups and order of the separate helicity sum
                m += (double)count[h] * cs1(j.r, j.i, *static_cast<const double*>(fc.aop));
                if (++in_group == fc.hel_per_group) s += m, m = 0.0, in_group = 0;
            } else if (e < n_evt) {
                double* const o = jamp + (int64_t)row[h] * (2 * NC) * ld + e0;
                o[lane] = j.r;
                (o + ld)[lane] = j.i;
                if (chan) {   // one diagram: its square is the sum over all
                    ChannelSums w;
                    w.add(0, 1.0, chan[e], j);
                    double* const t = sde + (int64_t)row[h] * 2 * ld + e0;
                    t[lane] = w.ch;
                    (t + ld)[lane] = w.all;
                }
            }
        });
    });
    if (!HSUM || e >= n_evt) return;
    if (in_group) s += m;
    double r = s * fc.hsum_scale;
    if (chan && chan[e] > 0) r *= 0.0;   // one diagram, 0: its weight is 1, any other channel's 0
    (fc.hsum_out + e0)[lane] = r;
}

hipError_t launch(const double* mom, int64_t n_evt, int64_t ld, const HelicityGroups& hg, double, double g,
                  double* jamp, const int* chan, double* sde, const FusedColour* fc, hipStream_t st)
{
    if (fc && !fc->hsum_out) return hipErrorInvalidValue;   // the colour sum here includes the helicity sum
    const dim3 grid((unsigned)((n_evt + 63) / 64));
    if (fc)
        hipLaunchKernelGGL(amp_rec<true>, grid, dim3(64), 0, st, mom, n_evt, ld, hg.row, g, jamp, chan,
                           nullptr, *fc);
    else
        hipLaunchKernelGGL(amp_rec<false>, grid, dim3(64), 0, st, mom, n_evt, ld, hg.row, g, jamp, chan, sde,
                           FusedColour{nullptr, nullptr, 0, 0, nullptr, 0.0, 1});
    return hipGetLastError();
}
}  // namespace rec_ee
}  // namespace me
