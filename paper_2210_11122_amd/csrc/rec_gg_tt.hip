// rec_gg_tt.hip -- FP64 colour-flow amplitudes and |M|^2 of gg -> t t~ by colour-ordered recursion.
//
// One lane per event evaluates the 8 helicity combinations with gluon 0 at -, which stand for all 16:
// the polarisation vectors, strings and two-gluon currents of each helicity are formed once and shared
// by the combinations that have them in common (1.2k FP64 instructions per event; the diagram program
// took about 1k for each of the 12 good combinations).  The colour sum and the helicity sum stay in the
// lane: one launch, also for the smallest batch.  2^19 events 119 -> 37 us per call (67 with all 16
// evaluated; 49 us with the momenta read from HBM and not from the last-level cache; the bytes of momenta and
// results take 14 us), 256 events 11.7 -> 8.6 us (host time).
// The channel weight is applied in the same launch: 65000 events 43.5 -> 12.3 us per call (its sums are kept per row
// and added in the rows' order at the end; 2^19 events 43.8 us, 43.7 added as they came).
#include "colorsum.hpp"
#include "generated/channels.hpp"
#include "process.hpp"
#include "recursion.hpp"

namespace me {
namespace rec2 {
using namespace rec;

constexpr int NPAR = 4, NC = 2;

// HSUM: |M|^2 to fc.hsum_out; else the jamps.
// SDE: also the channel-weight sums, of each helicity to sde or, with HSUM, applied to |M|^2.
template <bool HSUM, bool SDE>
__global__ __launch_bounds__(64, 2) void amp_rec(const double* __restrict__ mom, int64_t n_evt, int64_t ld,
                                                 const int* __restrict__ row, double mt, double gs,
                                                 double* __restrict__ jamp, const int* __restrict__ chan,
                                                 double* __restrict__ sde, FusedColour fc)
{
    // the momenta, then (4 KB each) the two-gluon currents: kept in LDS so that two waves fit a SIMD
    __shared__ double lds[2 * 512];
    const unsigned lane = threadIdx.x;
    const int* const count = row + 8;   // good helicities of each combination's row
    const int64_t e0 = xcd_remap(blockIdx.x, gridDim.x) * 64, e = e0 + lane;
    stage_momenta<NPAR, 1>(mom, n_evt, e0, lds, lane);
    const P4 p0 = lds_p4(lds, 0, lane), p1 = lds_p4(lds, 1, lane), pt = lds_p4(lds, 2, lane), pu = lds_p4(lds, 3, lane);
    const K4 k0 = lc(p0), k1 = lc(p1);
    // gluon 0 has helicity - (the opposite combinations have equal |M_h|^2), gluon 1 either
    const E4 E0 = gluon(p0, -1, false, gs), E1 = gluon(p1, 1, false, gs);
    const auto g1 = [&](auto B) { return B ? E1 : flip(E1); };
    __syncthreads();   // the momenta are read
    {
        const double f = -rcp(sq(k0 + k1));
        static_for<2>([&](auto I) {
            const E4 B = g1(I);
            st_v(lds, I, lane, f * vvv_acc(zero4(), E0, k0, B, k1, dot2(E0, B)));
        });
    }
    __syncthreads();
    const V4 U[2] = {spinor(ext_ubar<double>(pt, mt, -1)), spinor(ext_ubar<double>(pt, mt, 1))};
    const Prop q0 = prop(k0 - lc(pu), mt), q1 = prop(k1 - lc(pu), mt);
    double me[8];
    [[maybe_unused]] ChannelSums weights[8];
    [[maybe_unused]] const int channel = SDE && e < n_evt ? chan[e] : -1;
    static_for<2>([&](auto SV) {
        // (formed here, so that only one antiquark spin's strings are held)
        P4 p = pu;
        asm volatile("" : "+v"(p.t), "+v"(p.x), "+v"(p.y), "+v"(p.z));
        const V4 S = spinor(ext_v<double>(p, mt, SV ? 1 : -1));
        V4 R0 = prop_col(q0, col(E0, S)), R1[2];   // the antiquark has taken gluon 0, gluon 1
        pin_v(R0);
        static_for<2>([&](auto B) {
            R1[B] = prop_col(q1, col(g1(B), S));
            pin_v(R1[B]);
        });
        static_for<2>([&](auto SU) {
            const V4 c = pair(U[SU], S);
            C j0[2], j1[2];   // [helicity of gluon 1]
            [[maybe_unused]] ChannelSums sums[2];
            static_for<2>([&](auto I) { j0[I] = rc(c, ld_v(lds, I, lane)); });
            static_for<2>([&](auto I) {
                j1[I] = neg(j0[I]);
                if constexpr (SDE) sums[I].add(channel_diagram[2], channel_weight[2], channel, j0[I]);
            });
            const V4 X0 = rec::row(U[SU], E0);
            static_for<2>([&](auto B) {
                const V4 X1 = rec::row(U[SU], g1(B));
                j0[B] = rc_acc(j0[B], X0, R1[B]);
                j1[B] = rc_acc(j1[B], X1, R0);
                if constexpr (SDE) {
                    sums[B].add(channel_diagram[0], channel_weight[0], channel, rc(X0, R1[B]));
                    sums[B].add(channel_diagram[1], channel_weight[1], channel, rc(X1, R0));
                }
            });
            static_for<2>([&](auto I) {
                constexpr int h = 4 * I + 2 * SU + SV;
                pin_cx(j0[I]), pin_cx(j1[I]);   // rounded the same way whatever uses them
                if constexpr (HSUM) {
                    if constexpr (SDE) weights[h] = sums[I];
                    me[h] = cs2(j0[I].r, j0[I].i, j1[I].r, j1[I].i, static_cast<const double*>(fc.aop));
                } else if (count[h] && e < n_evt) {
                    double* const o = jamp + (int64_t)row[h] * (2 * NC) * ld + e0;
                    o[lane] = j0[I].r;
                    (o + ld)[lane] = j0[I].i;
                    (o + 2 * ld)[lane] = j1[I].r;
                    (o + 3 * ld)[lane] = j1[I].i;
                    if constexpr (SDE) {
                        double* const t = sde + (int64_t)row[h] * 2 * ld + e0;
                        t[lane] = sums[I].ch;
                        (t + ld)[lane] = sums[I].all;
                    }
                }
            });
        });
    });
    if (!HSUM || e >= n_evt) return;
    // the rows in the groups and order of the separate helicity sum
    double s = 0.0, m = 0.0;
    int in_group = 0;
    static_for<8>([&](auto H) {
        if (!count[H]) return;
        m += (double)count[H] * me[H];
        if (++in_group == fc.hel_per_group) s += m, m = 0.0, in_group = 0;
    });
    if (in_group) s += m;
    double r = s * fc.hsum_scale;
    if (SDE && channel >= 0) {   // the rows in order, as where the weights are summed by a kernel of their own
        double num = 0.0, den = 0.0;
        static_for<8>([&](auto H) {
            const double w = (double)count[H];
            if (count[H]) num += w * weights[H].ch, den += w * weights[H].all;
        });
        r *= num / den;
    }
    (fc.hsum_out + e0)[lane] = r;
}

hipError_t launch(const double* mom, int64_t n_evt, int64_t ld, const HelicityGroups& hg, double mt, double gs,
                  double* jamp, const int* chan, double* sde, const FusedColour* fc, hipStream_t st)
{
    if (fc && !fc->hsum_out) return hipErrorInvalidValue;   // the colour sum here includes the helicity sum
    const FusedColour none{nullptr, nullptr, 0, 0, nullptr, 0.0, 1};
    const dim3 grid((unsigned)((n_evt + 63) / 64));
    const auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(64), 0, st, mom, n_evt, ld, hg.row, mt, gs, jamp, chan, sde, fc ? *fc : none);
    };
    if (fc && chan) go(amp_rec<true, true>);
    else if (fc) go(amp_rec<true, false>);
    else if (chan) go(amp_rec<false, true>);
    else go(amp_rec<false, false>);
    return hipGetLastError();
}
}  // namespace rec2
}  // namespace me
