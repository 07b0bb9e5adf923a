// rec_gg_ttg.hip -- FP64 colour-flow amplitudes and |M|^2 of gg -> t t~ g by colour-ordered recursion.
//
// One lane per (event, configuration of the three gluon helicities) evaluates the four quark spin
// configurations, which share the gluon currents and, two by two, the strings.  A workgroup's four waves
// hold the four configurations of 64 events and sum the helicities, with the channel weight where one is asked
// for (its diagrams' squares are formed from the same strings).  The diagram program took one lane per
// (event, helicity) and 24 of them made each gluon current anew.  Bound by FP64 issue: 2^20 events
// 2844 -> 862 us per call (1519 with all eight gluon configurations), 100003 events with channel weights
// 423 -> 140 us; the bytes (176 MB) take 35 us.
#include "colorsum.hpp"
#include "generated/channels.hpp"
#include "process.hpp"
#include "recursion.hpp"

namespace me {
namespace rec3 {
using namespace rec;

constexpr int NG = 3, NPAR = 5, NC = 6, MAX_ROWS = 16;
__host__ __device__ constexpr int flow(int a, int b, int c)
{
    Perm<3> x{};
    x.p[0] = a, x.p[1] = b, x.p[2] = c;
    return perm_rank<3>(x);
}

// HSUM: the workgroup takes its 64 events' configurations four at a time and writes |M|^2; else the
// workgroups of an event block take four configurations each, and every lane writes D |M_h|^2 (fc.aop
// set) or the jamps of its helicities.  N = 1 (not with HSUM): one spin configuration per lane, a
// workgroup's waves being the four of one gluon configuration.
// SDE: also the channel-weight sums, of each helicity to sde or, with HSUM, applied to |M|^2.
template <bool HSUM, int N, bool SDE = false>
__global__ __launch_bounds__(256, N == 1 ? 2 : 1) void amp_rec(const double* __restrict__ mom, int64_t n_evt, int64_t ld,
                                                  const int* __restrict__ cfg, int n_cfg,
                                                  const int2* __restrict__ members, int n_rows, double mt, double gs,
                                                  double* __restrict__ jamp, const int* __restrict__ chan,
                                                  double* __restrict__ sde, FusedColour fc)
{
    __shared__ double lds[4 * NPAR * 64];
    __shared__ double me_lds[HSUM ? MAX_ROWS * 64 : 1];
    // With the channel weights summed here (spills) the propagators of two gluons are made once for the
    // four waves and read from LDS: 100003 events take 4 % less than with them made in each lane.  Without
    // the weights they are made in each lane: from LDS 2^20 events take 1.5 % more
    constexpr bool SHARED_PROPS = HSUM && SDE;
    __shared__ double prop_lds[SHARED_PROPS ? 3 * 64 : 1];
    __shared__ double sde_lds[HSUM && SDE ? 2 * MAX_ROWS * 64 : 1];
    const unsigned lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int per_block = HSUM ? 1 : N == 1 ? n_cfg : (n_cfg + 3) / 4;
    const int64_t w = xcd_remap(blockIdx.x, gridDim.x);
    const int64_t e0 = (w / per_block) * 64, e = e0 + lane;
    stage_momenta<NPAR, 4>(mom, n_evt, e0, lds, threadIdx.x);
    if constexpr (SHARED_PROPS) {
        if (wave < 3) {   // (01), (02), (12)
            const P4 p = lds_p4(lds, wave == 2 ? 1 : 0, lane), q = lds_p4(lds, wave == 0 ? 1 : 4, lane);
            prop_lds[64 * wave + lane] = pair_prop(p, wave == 0 ? q : -q);
        }
        __syncthreads();
    }
    const int first = HSUM ? wave : N == 1 ? (int)(w % per_block) : (int)(w % per_block) * 4 + wave;
    const int step = HSUM ? 4 : n_cfg;
    // spins of the quark (antiquark): index i stands for spin i, or for the wave's one spin
    const auto spin = [&](int i, int bit) { return N == 1 ? ((wave >> bit) & 1 ? 1 : -1) : i ? 1 : -1; };
#pragma unroll 1
    for (int r = first; r < n_cfg; r += step) {
        const int* const row_cfg = cfg + r * 5;
        const int bits = row_cfg[0];
        const auto P = [&](int i) { return lc(lds_p4(lds, i, lane)); };
        const K4 k[3] = {P(0), P(1), -P(4)};
        const E4 E[3] = {gluon(lds_p4(lds, 0, lane), bits & 1 ? 1 : -1, false, gs),
                         gluon(lds_p4(lds, 1, lane), bits & 2 ? 1 : -1, false, gs),
                         gluon(lds_p4(lds, 4, lane), bits & 4 ? 1 : -1, true, gs)};
        V4 J2[3];   // (01), (02), (12)
        double f2[3];
        if constexpr (!SHARED_PROPS) {
            const P4 p0 = lds_p4(lds, 0, lane), p1 = lds_p4(lds, 1, lane), p2 = -lds_p4(lds, 4, lane);
            f2[0] = pair_prop(p0, p1), f2[1] = pair_prop(p0, p2), f2[2] = pair_prop(p1, p2);
        }
        static_for<3>([&](auto I) {
            constexpr int a = I == 2 ? 1 : 0, b = I == 0 ? 1 : 2;
            if constexpr (SHARED_PROPS) f2[I] = prop_lds[64 * I + lane];
            J2[I] = f2[I] * vvv_acc(zero4(), E[a], k[a], E[b], k[b], dot2(E[a], E[b]));
        });
        const P4 pt = lds_p4(lds, 2, lane), pu = lds_p4(lds, 3, lane);
        V4 U[N], S[N];
        static_for<N>([&](auto I) {
            U[I] = spinor(ext_ubar<double>(pt, mt, spin(I, 1)));
            S[I] = spinor(ext_v<double>(pu, mt, spin(I, 0)));
        });
        C J[N * N][NC];   // [quark spin, antiquark spin][flow]
        [[maybe_unused]] ChannelSums sums[N * N];
        [[maybe_unused]] const int channel = SDE && e < n_evt ? chan[e] : -1;
        const auto weigh = [&](int sp, auto I, C a) { sums[sp].add(channel_diagram[I], channel_weight[I], channel, a); };
        {   // all gluons in one current
            const V4x2 j3 = three_currents(E[0], k[0], E[1], k[1], E[2], k[2], J2[0], J2[1], J2[2]);
            static_for<N * N>([&](auto SP) {
                const V4 c = pair(U[SP / N], S[SP % N]);
                const C l0 = rc(c, j3.v[0]), l1 = rc(c, j3.v[1]), l2 = neg(l0 + l1);
                J[SP][flow(0, 1, 2)] = l0, J[SP][flow(2, 1, 0)] = l0;
                J[SP][flow(0, 2, 1)] = l1, J[SP][flow(1, 2, 0)] = l1;
                J[SP][flow(1, 0, 2)] = l2, J[SP][flow(2, 0, 1)] = l2;
                static_for<NC>([&](auto F) { pin_cx(J[SP][F]); });
            });
            if constexpr (SDE) {   // the trees and the four-gluon structures one by one
                const double f = -rcp(sq(k[0] + k[1] + k[2]));
                const V4 t[3] = {f * vvv_acc(zero4(), J2[0], k[0] + k[1], E[2], k[2], dot2(J2[0], E[2])),
                                 f * vvv_acc(zero4(), J2[1], k[0] + k[2], E[1], k[1], dot2(J2[1], E[1])),
                                 f * vvv_acc(zero4(), J2[2], k[1] + k[2], E[0], k[0], dot2(J2[2], E[0]))};
                const C d01 = times(0.5 * f, dot2(E[0], E[1])), d02 = times(0.5 * f, dot2(E[0], E[2])),
                        d12 = times(0.5 * f, dot2(E[1], E[2]));
                static_for<N * N>([&](auto SP) {
                    const V4 c = pair(U[SP / N], S[SP % N]);
                    static_for<3>([&](auto T) { weigh(SP, std::integral_constant<int, 12 + T>{}, rc(c, t[T])); });
                    const C x0 = cmul(rc(c, full(E[0])), d12), x1 = cmul(rc(c, full(E[1])), d02),
                            x2 = cmul(rc(c, full(E[2])), d01);
                    weigh(SP, std::integral_constant<int, 15>{}, x1 - x2);
                    weigh(SP, std::integral_constant<int, 16>{}, x0 - x2);
                    weigh(SP, std::integral_constant<int, 17>{}, x0 - x1);
                });
            }
        }
        V4 L[N][3];   // the quark has taken gluon a
        static_for<3>([&](auto A) {
            const Prop q = prop(P(2) - k[A], mt);
            static_for<N>([&](auto SU) { L[SU][A] = prop_row(q, row(U[SU], E[A])); });
        });
        static_for<N>([&](auto SV) {
            pin_v(S[SV]);
            V4 R[3];   // the antiquark has taken gluon c
            static_for<3>([&](auto A) { R[A] = prop_col(prop(k[A] - P(3), mt), col(E[A], S[SV])); });
            static_for<3>([&](auto A) {   // (a | b c) and (a | c b), b < c; then the pair (b c) next to the quark
                constexpr int a = A, b = a == 0 ? 1 : 0, c = a == 2 ? 1 : 2, bc = a == 0 ? 2 : a == 1 ? 1 : 0;
                const V4 y = col(J2[bc], S[SV]);
                const V4 X = col_acc(y, E[b], R[c]), Y = col_acc(-y, E[c], R[b]);
                static_for<N>([&](auto SU) {
                    C* const j = J[N * SU + SV];
                    const C t = rc(pair(U[SU], R[a]), J2[bc]);
                    j[flow(a, b, c)] = rc_acc(j[flow(a, b, c)], L[SU][a], X);
                    j[flow(a, c, b)] = rc_acc(j[flow(a, c, b)], L[SU][a], Y);
                    j[flow(b, c, a)] = j[flow(b, c, a)] + t;
                    j[flow(c, b, a)] = j[flow(c, b, a)] - t;
                    if constexpr (SDE) {
                        weigh(N * SU + SV, std::integral_constant<int, flow(a, b, c)>{}, rc(L[SU][a], col(E[b], R[c])));
                        weigh(N * SU + SV, std::integral_constant<int, flow(a, c, b)>{}, rc(L[SU][a], col(E[c], R[b])));
                        weigh(N * SU + SV, std::integral_constant<int, 6 + a>{}, rc(L[SU][a], y));
                        weigh(N * SU + SV, std::integral_constant<int, 9 + a>{}, t);
                    }
                });
            });
            static_for<N>([&](auto SU) { static_for<NC>([&](auto F) { pin_cx(J[N * SU + SV][F]); }); });
        });
        static_for<N * N>([&](auto SP) {
            const int h = row_cfg[1 + (N == 1 ? wave : (int)SP)];
            if (h < 0) return;
            if (HSUM || fc.aop) {
                double Jr[2 * NC];
                static_for<NC>([&](auto F) { Jr[2 * F] = J[SP][F].r, Jr[2 * F + 1] = J[SP][F].i; });
                const double me_h = colour_sum_regs<NC>(Jr, static_cast<const double*>(fc.aop));
                if constexpr (HSUM && SDE) {
                    sde_lds[2 * h * 64 + lane] = sums[SP].ch;
                    sde_lds[(2 * h + 1) * 64 + lane] = sums[SP].all;
                }
                if constexpr (HSUM) me_lds[h * 64 + lane] = me_h;
                else if (e < n_evt) jamp[(int64_t)h * n_evt + e] = me_h;
            } else if (e < n_evt) {
                double* const o = jamp + (int64_t)h * (2 * NC) * ld + e0;
                static_for<NC>([&](auto F) {
                    (o + (2 * F) * ld)[lane] = J[SP][F].r;
                    (o + (2 * F + 1) * ld)[lane] = J[SP][F].i;
                });
                if constexpr (SDE) {
                    double* const t = sde + (int64_t)h * 2 * ld + e0;
                    t[lane] = sums[SP].ch;
                    (t + ld)[lane] = sums[SP].all;
                }
            }
        });
    }
    if constexpr (HSUM) {
        __syncthreads();
        if (wave == 0 && e < n_evt) {   // in the groups and order of the separate helicity sum
            double s = 0.0;
            for (int h0 = 0; h0 < n_rows; h0 += fc.hel_per_group) {
                const int h1 = min(n_rows, h0 + fc.hel_per_group);
                double m = 0.0;
                for (int h = h0; h < h1; ++h) m += members_of(members, h) * me_lds[h * 64 + lane];
                s += m;
            }
            double r = s * fc.hsum_scale;
            if (SDE && chan[e] >= 0) {
                double num = 0.0, den = 0.0;
                for (int h = 0; h < n_rows; ++h) {
                    const double w = members_of(members, h);
                    num += w * sde_lds[2 * h * 64 + lane], den += w * sde_lds[(2 * h + 1) * 64 + lane];
                }
                r *= num / den;
            }
            (fc.hsum_out + e0)[lane] = r;
        }
    }
}

// Up to here one spin configuration per lane: the batch leaves SIMDs without a wave either way, and a
// wave's program is 2k instructions instead of 4.2k (64 events 12.3 us per call, 4096 14.9; with all spins in a
// lane 14.8 at any size that fits the GPU at once, where 8192 events take 18.7 with one).
constexpr int64_t ONE_SPIN = 4096;

hipError_t launch(const double* mom, int64_t n_evt, int64_t ld, const HelicityGroups& hg, double mt, double gs,
                  double* jamp, const int* chan, double* sde, const FusedColour* fc, hipStream_t st)
{
    const unsigned blocks = (unsigned)((n_evt + 63) / 64);
    if (hg.n_rows > MAX_ROWS) return hipErrorInvalidValue;
    const FusedColour f = fc ? *fc : FusedColour{nullptr, nullptr, 0, 0, nullptr, 0.0, 1};
    const auto go = [&](auto kernel, unsigned grid) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, st, mom, n_evt, ld, hg.table, hg.n, hg.members, hg.n_rows, mt, gs, jamp,
                           chan, sde, f);
    };
    const unsigned by_one = blocks * (unsigned)hg.n, by_four = blocks * (unsigned)((hg.n + 3) / 4);
    if (f.hsum_out && chan) go(amp_rec<true, 2, true>, blocks);
    else if (f.hsum_out) go(amp_rec<true, 2>, blocks);
    else if (n_evt <= ONE_SPIN && chan) go(amp_rec<false, 1, true>, by_one);
    else if (n_evt <= ONE_SPIN) go(amp_rec<false, 1>, by_one);
    else if (chan) go(amp_rec<false, 2, true>, by_four);
    else go(amp_rec<false, 2>, by_four);
    return hipGetLastError();
}
}  // namespace rec3
}  // namespace me
