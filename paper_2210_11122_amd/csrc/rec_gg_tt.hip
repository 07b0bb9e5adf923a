// rec_gg_tt.hip -- FP64 colour-flow amplitudes and |M|^2 of gg -> t t~ by colour-ordered recursion.
//
// One lane per event evaluates all 16 helicity combinations: the polarisation vectors, strings and
// two-gluon currents of each helicity are formed once and shared by the combinations that have them
// in common (2.3k FP64 instructions per event; the diagram program took about 1k for each of the 12
// good combinations).  The colour sum and the helicity sum stay in the lane: one launch, also for
// the smallest batch.  Bound by FP64 issue: 2^19 events 118.7 -> 67.4 us per call (the bytes of momenta
// and results take 14 us), 256 events 11.2 -> 9.0 us (host time).  The channel weight is applied in the
// same launch: 100 events 17.5 -> 11.5 us per call, 65000 43.5 -> 13.9 us.
#include "colorsum.hpp"
#include "generated/channels.hpp"
#include "process.hpp"
#include "recursion.hpp"

namespace me {
namespace rec2 {
using namespace rec;

constexpr int NPAR = 4, NC = 2;

// HSUM: |M|^2 to fc.hsum_out; else the jamps.  WAVES: waves per SIMD the registers are cut for.
// Two spill 180 B per lane and hide each other's waits (2^19 events 82.6 us with one, 67.4 with
// two).  While the batch has at most one wave for each of the 1024 SIMDs (2^16 events), one wave
// without spills is faster (256 events 9.0 us against 10.0 per call, 2^16 9.6 against 13.3).
// SDE: also the channel-weight sums, of each helicity to sde or, with HSUM, applied to |M|^2.
template <bool HSUM, int WAVES, bool SDE = false>
__global__ __launch_bounds__(64, WAVES) void amp_rec(const double* __restrict__ mom, int64_t n_evt, int64_t ld,
                                                 const int* __restrict__ index, double mt, double gs,
                                                 double* __restrict__ jamp, const int* __restrict__ chan,
                                                 double* __restrict__ sde, FusedColour fc)
{
    // the momenta, then (4 KB each) the four two-gluon currents: kept in LDS so that two waves fit a SIMD
    __shared__ double lds[4 * 512];
    const unsigned lane = threadIdx.x;
    const int64_t e0 = xcd_remap(blockIdx.x, gridDim.x) * 64, e = e0 + lane;
    stage_momenta<NPAR, 1>(mom, n_evt, e0, lds, lane);
    const P4 p0 = lds_p4(lds, 0, lane), p1 = lds_p4(lds, 1, lane), pt = lds_p4(lds, 2, lane), pu = lds_p4(lds, 3, lane);
    const K4 k0 = lc(p0), k1 = lc(p1);
    // polarisation vectors of helicity +; the others are their flips
    const E4 E0 = gluon(p0, 1, false, gs), E1 = gluon(p1, 1, false, gs);
    const auto g0 = [&](auto A) { return A ? E0 : flip(E0); };
    const auto g1 = [&](auto B) { return B ? E1 : flip(E1); };
    __syncthreads();   // the momenta are read
    {
        const double f = -rcp(sq(k0 + k1));
        static_for<4>([&](auto I) {
            const E4 A = g0(std::integral_constant<int, I / 2>{}), B = g1(std::integral_constant<int, I % 2>{});
            st_v(lds, I, lane, f * vvv_acc(zero4(), A, k0, B, k1, dot2(A, B)));
        });
    }
    __syncthreads();
    const V4 U[2] = {spinor(ext_ubar<double>(pt, mt, -1)), spinor(ext_ubar<double>(pt, mt, 1))};
    const Prop q0 = prop(k0 - lc(pu), mt), q1 = prop(k1 - lc(pu), mt);
    double me[16];
    [[maybe_unused]] double num = 0.0, den = 0.0;
    [[maybe_unused]] const int channel = SDE && e < n_evt ? chan[e] : -1;
    static_for<2>([&](auto SV) {
        // (formed here, so that only one antiquark spin's strings are held)
        P4 p = pu;
        asm volatile("" : "+v"(p.t), "+v"(p.x), "+v"(p.y), "+v"(p.z));
        const V4 S = spinor(ext_v<double>(p, mt, SV ? 1 : -1));
        V4 R0[2], R1[2];   // the antiquark has taken gluon 0, gluon 1
        static_for<2>([&](auto A) {
            R0[A] = prop_col(q0, col(g0(A), S));
            R1[A] = prop_col(q1, col(g1(A), S));
            pin_v(R0[A]), pin_v(R1[A]);
        });
        static_for<2>([&](auto SU) {
            const V4 c = pair(U[SU], S);
            C j0[4], j1[4];
            [[maybe_unused]] ChannelSums sums[4];
            static_for<4>([&](auto I) { j0[I] = rc(c, ld_v(lds, I, lane)); });
            static_for<4>([&](auto I) {
                j1[I] = neg(j0[I]);
                if constexpr (SDE) sums[I].add(channel_diagram[2], channel_weight[2], channel, j0[I]);
            });
            static_for<2>([&](auto A) {
                const V4 X = row(U[SU], g0(A));
                static_for<2>([&](auto B) {
                    j0[2 * A + B] = rc_acc(j0[2 * A + B], X, R1[B]);
                    if constexpr (SDE) sums[2 * A + B].add(channel_diagram[0], channel_weight[0], channel, rc(X, R1[B]));
                });
            });
            static_for<2>([&](auto B) {
                const V4 X = row(U[SU], g1(B));
                static_for<2>([&](auto A) {
                    j1[2 * A + B] = rc_acc(j1[2 * A + B], X, R0[A]);
                    if constexpr (SDE) sums[2 * A + B].add(channel_diagram[1], channel_weight[1], channel, rc(X, R0[A]));
                });
            });
            static_for<4>([&](auto I) {
                constexpr int h = 4 * I + 2 * SU + SV;
                pin_cx(j0[I]), pin_cx(j1[I]);   // rounded the same way whatever uses them
                if constexpr (HSUM) {
                    if constexpr (SDE) {
                        if (index[h] >= 0) num += sums[I].ch, den += sums[I].all;
                    }
                    me[h] = cs2(j0[I].r, j0[I].i, j1[I].r, j1[I].i, static_cast<const double*>(fc.aop));
                } else if (index[h] >= 0 && e < n_evt) {
                    double* const o = jamp + (int64_t)index[h] * (2 * NC) * ld + e0;
                    o[lane] = j0[I].r;
                    (o + ld)[lane] = j0[I].i;
                    (o + 2 * ld)[lane] = j1[I].r;
                    (o + 3 * ld)[lane] = j1[I].i;
                    if constexpr (SDE) {
                        double* const t = sde + (int64_t)index[h] * 2 * ld + e0;
                        t[lane] = sums[I].ch;
                        (t + ld)[lane] = sums[I].all;
                    }
                }
            });
        });
    });
    if (!HSUM || e >= n_evt) return;
    // the good helicities in the groups and order of the separate helicity sum
    double s = 0.0, m = 0.0;
    int in_group = 0;
    static_for<16>([&](auto H) {
        if (index[H] < 0) return;
        m += me[H];
        if (++in_group == fc.hel_per_group) s += m, m = 0.0, in_group = 0;
    });
    if (in_group) s += m;
    double r = s * fc.hsum_scale;
    if (SDE && channel >= 0) r *= num / den;
    (fc.hsum_out + e0)[lane] = r;
}

hipError_t launch(const double* mom, int64_t n_evt, int64_t ld, const HelicityGroups& hg, double mt, double gs,
                  double* jamp, const int* chan, double* sde, const FusedColour* fc, hipStream_t st)
{
    if (fc && !fc->hsum_out) return hipErrorInvalidValue;   // the colour sum here includes the helicity sum
    const FusedColour none{nullptr, nullptr, 0, 0, nullptr, 0.0, 1};
    const dim3 grid((unsigned)((n_evt + 63) / 64));
    constexpr int64_t ONE_WAVE = 65536;
    if (fc && chan)
        hipLaunchKernelGGL((amp_rec<true, 1, true>), grid, dim3(64), 0, st, mom, n_evt, ld, hg.index, mt, gs, jamp, chan,
                           nullptr, *fc);
    else if (fc && n_evt <= ONE_WAVE)
        hipLaunchKernelGGL((amp_rec<true, 1>), grid, dim3(64), 0, st, mom, n_evt, ld, hg.index, mt, gs, jamp,
                           nullptr, nullptr, *fc);
    else if (fc)
        hipLaunchKernelGGL((amp_rec<true, 2>), grid, dim3(64), 0, st, mom, n_evt, ld, hg.index, mt, gs, jamp,
                           nullptr, nullptr, *fc);
    else if (chan)
        hipLaunchKernelGGL((amp_rec<false, 1, true>), grid, dim3(64), 0, st, mom, n_evt, ld, hg.index, mt, gs, jamp,
                           chan, sde, none);
    else
        hipLaunchKernelGGL((amp_rec<false, 1>), grid, dim3(64), 0, st, mom, n_evt, ld, hg.index, mt, gs, jamp, nullptr,
                           nullptr, none);
    return hipGetLastError();
}
}  // namespace rec2
}  // namespace me
