// rec_gg_ttgg.hip -- FP64 colour-flow amplitudes of gg -> t t~ g g by colour-ordered recursion.
//
// A workgroup evaluates 64 events in one configuration of the four gluon helicities: its eight waves
// make the gluon currents and the strings of one gluon together, through LDS, and then each the twelve
// flows that have gluon 0 among the first two, or among the last two, for one of the four quark spin
// configurations.  Bound by FP64 issue (3.4k vector instructions per wave; the issue slots are 63 % full)
// with two waves per SIMD, for which the 158 KB of LDS leave room.  2^19 events: the diagram program
// 20.6 ms per call, 4.9 now (2 % more with four waves that made their strings themselves).  The
// kernel also gives the helicities' |M_h|^2 and the flows' weights, so neither call takes the jamps through
// memory: 20000 events with the per-helicity output 260 -> 216 us, with selection 326 -> 265 us (9973
// events 192 -> 149).
#include "colorsum.hpp"
#include "process.hpp"
#include "recursion.hpp"

namespace me {
namespace rec4 {
using namespace rec;

constexpr int NG = 4, NPAR = 6, NC = 24;
// LDS, in doubles: the momenta, the polarisation vectors, then vectors of 512 doubles: the spinors of
// either helicity, J(ij) with i < j, J of the two independent orderings (xyz), (xzy) of the gluons
// without w, and the strings of one gluon from the quark and from the antiquark end
constexpr int EPS = 4 * NPAR * 64, CUR = EPS + 5 * NG * 64;
constexpr int SU = 0, SV = 2, S2 = 4, S3 = 10, SL = 18, SR = 26, NSLOT = 34;
// once the strings are used: J(0 s) times the quark currents, |J|^2 of the flows, and the parts of the flows
// that waves exchange
constexpr int FOUR = CUR + 512 * S2, LCW = FOUR + 6 * 4 * 128, XCH = LCW + 8 * 12 * 64;
static_assert(XCH + 8 * 12 * 64 <= CUR + 512 * NSLOT, "");

__host__ __device__ constexpr int s2(int i, int j) { return S2 + i * (2 * NG - i - 1) / 2 + j - i - 1; }   // i < j
// the gluons without w in ascending order
__host__ __device__ constexpr int rest(int w, int k) { return k < w ? k : k + 1; }
// the six pairs i < j, and the pair that is left
__host__ __device__ constexpr int pair_i(int p) { return p < 3 ? 0 : p < 5 ? 1 : 2; }
__host__ __device__ constexpr int pair_j(int p) { return p < 3 ? p + 1 : p < 5 ? p - 1 : 3; }
__host__ __device__ constexpr int flow(int a, int b, int c, int d)
{
    Perm<4> x{};
    x.p[0] = a, x.p[1] = b, x.p[2] = c, x.p[3] = d;
    return perm_rank<4>(x);
}


// the flow (a b c d) belongs to half H; the number of a flow within its half
template <int H>
__host__ __device__ constexpr bool own(int a, int b)
{
    return (a == 0 || b == 0) == (H == 0);
}
__host__ __device__ constexpr int half_of(int f) { return own<0>(perm_at<4>(f).p[0], perm_at<4>(f).p[1]) ? 0 : 1; }
__host__ __device__ constexpr int in_half(int f)
{
    int n = 0;
    for (int g = 0; g < f; ++g) n += half_of(g) == half_of(f);
    return n;
}
__host__ __device__ constexpr int flow_in_half(int H, int k)
{
    for (int f = 0;; ++f)
        if (half_of(f) == H && k-- == 0) return f;
}
struct Flows {
    C v[NC / 2];
};
// J(a b c d) += SGN x, if that flow belongs to the half
template <int H, int SGN, int A, int B, int D, int E>
__device__ __forceinline__ void add(Flows& J, C x)
{
    if constexpr (own<H>(A, B)) {
        constexpr int k = in_half(flow(A, B, D, E));
        J.v[k] = SGN > 0 ? J.v[k] + x : J.v[k] - x;
    }
}
__device__ __forceinline__ void pin(Flows& J)
{
    static_for<NC / 2>([&](auto K) { pin_cx(J.v[K]); });
}

// the flows of half H without the four-gluon currents; k: momenta, su, sv: quark spins
template <int H>
__device__ __forceinline__ Flows quark_line(const double* lds, unsigned lane, int su, int sv, double mt)
{
    const double* const cur = lds + CUR;
    const auto P = [&](int i) { return lc(lds_p4(lds, i, lane)); };
    const auto kin = [&](int i) { return i < 2 ? P(i) : -P(i + 2); };
    const auto G1 = [&](int i) { return ld_e(lds + EPS, i, lane); };
    const auto G2 = [&](int i, int j) { return ld_v(cur, s2(i, j), lane); };
    const auto L = [&](int i) { return ld_v(cur, SL + 4 * su + i, lane); };
    const auto R = [&](int i) { return ld_v(cur, SR + 4 * sv + i, lane); };
    const V4 U = ld_v(cur, SU + su, lane), S = ld_v(cur, SV + sv, lane);
    Flows J;
    // two gluons on either side: the pairs (a b) with gluon 0 for half 0, without it for half 1
    static_for<3>([&](auto P_) {
        constexpr int p = H ? 5 - P_ : P_, a = pair_i(p), b = pair_j(p), c = pair_i(5 - p), d = pair_j(5 - p);
        V4 Lab, Lba;
        {
            const V4 x = row(U, G2(a, b));
            const Prop q = prop(P(2) - kin(a) - kin(b), mt);
            Lab = prop_row(q, row_acc(x, L(a), G1(b)));
            Lba = prop_row(q, row_acc(-x, L(b), G1(a)));
            pin_v(Lab), pin_v(Lba);
        }
        const V4 y = col(G2(c, d), S);
        const V4 Rcd = col_acc(y, G1(c), R(d)), Rdc = col_acc(-y, G1(d), R(c));
        J.v[in_half(flow(a, b, c, d))] = rc(Lab, Rcd);
        J.v[in_half(flow(a, b, d, c))] = rc(Lab, Rdc);
        J.v[in_half(flow(b, a, c, d))] = rc(Lba, Rcd);
        J.v[in_half(flow(b, a, d, c))] = rc(Lba, Rdc);
        pin_cx(J.v[in_half(flow(a, b, c, d))]), pin_cx(J.v[in_half(flow(a, b, d, c))]);
        pin_cx(J.v[in_half(flow(b, a, c, d))]), pin_cx(J.v[in_half(flow(b, a, d, c))]);
    });
    // a current J(cd) at the cut: (a c d b) and (a d c b)
    static_for<6>([&](auto P_) {
        constexpr int a = pair_i(P_), b = pair_j(P_), c = pair_i(5 - P_), d = pair_j(5 - P_);
        const V4 Gcd = G2(c, d);
        if constexpr (own<H>(a, c) || own<H>(a, d)) {
            const C t = rc(L(a), col(Gcd, R(b)));
            add<H, 1, a, c, d, b>(J, t);
            add<H, -1, a, d, c, b>(J, t);
        }
        if constexpr (own<H>(b, c) || own<H>(b, d)) {
            const C t = rc(L(b), col(Gcd, R(a)));
            add<H, 1, b, c, d, a>(J, t);
            add<H, -1, b, d, c, a>(J, t);
        }
        pin(J);
    });
    // J of three gluons next to the antiquark or to the quark
    static_for<4>([&](auto W_) {
        constexpr int m = W_, x = rest(m, 0), y = rest(m, 1), z = rest(m, 2);
        const V4 G0 = ld_v(cur, S3 + 2 * m, lane), G1_ = ld_v(cur, S3 + 2 * m + 1, lane);
        if constexpr (H == 0 || m != 0) {   // (m | ...): flows with m first
            const V4 cl = pair(L(m), S);
            const C l0 = rc(cl, G0), l1 = rc(cl, G1_), l2 = l0 + l1;
            add<H, 1, m, x, y, z>(J, l0), add<H, 1, m, z, y, x>(J, l0);
            add<H, 1, m, x, z, y>(J, l1), add<H, 1, m, y, z, x>(J, l1);
            add<H, -1, m, y, x, z>(J, l2), add<H, -1, m, z, x, y>(J, l2);
        }
        if constexpr (H == 1 || m != 0) {   // (... | m): flows with m last
            const V4 cr = pair(U, R(m));
            const C r0 = rc(cr, G0), r1 = rc(cr, G1_), r2 = r0 + r1;
            add<H, 1, x, y, z, m>(J, r0), add<H, 1, z, y, x, m>(J, r0);
            add<H, 1, x, z, y, m>(J, r1), add<H, 1, y, z, x, m>(J, r1);
            add<H, -1, y, x, z, m>(J, r2), add<H, -1, z, x, y, m>(J, r2);
        }
        pin(J);
    });
    return J;
}

// the rest of a wave's work, with barriers: the flows of half H of spin configuration sp, |M_h|^2 or the jamps
template <int H>
__device__ __forceinline__ void finish(double* lds, unsigned lane, int wave, int sp, const C (&four)[4], int64_t n_evt,
                                       int64_t ld, int64_t e0, int h, double mt, double* __restrict__ jamp, bool me,
                                       double members, double* __restrict__ flow_weights)
{
    const int64_t e = e0 + lane;
    Flows J = quark_line<H>(lds, lane, sp >> 1, sp & 1, mt);
    typedef double v2d __attribute__((ext_vector_type(2)));
    typedef __attribute__((address_space(3))) const volatile v2d lds_v2d;
    typedef __attribute__((address_space(3))) const volatile double lds_d;
    __syncthreads();   // currents and strings are used
    if (wave < 6)
        static_for<4>([&](auto SP) { reinterpret_cast<v2d*>(lds + FOUR)[(4 * wave + SP) * 64 + lane] = {four[SP].r, four[SP].i}; });
    __syncthreads();
    C s[6];
    static_for<6>([&](auto K) {
        const v2d t = ((lds_v2d*)(lds + FOUR))[(4 * K + sp) * 64 + lane];
        s[K] = {t.x, t.y};
    });
    static_for<NC / 2>([&](auto F_) {
        constexpr int f = flow_in_half(H, F_);
        static_for<6>([&](auto K) {
            constexpr int c = kk_table<4>.c[f][K];
            static_assert(c >= -1 && c <= 1, "");
            if constexpr (c == 1) J.v[F_] = J.v[F_] + s[K];
            if constexpr (c == -1) J.v[F_] = J.v[F_] - s[K];
        });
        pin_cx(J.v[F_]);
    });
    if (!me) {
        if (h < 0 || e >= n_evt) return;
        double* const o = jamp + (int64_t)h * (2 * NC) * ld + e0;
        static_for<NC / 2>([&](auto F_) {
            constexpr int f = flow_in_half(H, F_);
            (o + (2 * f) * ld)[lane] = J.v[F_].r;
            (o + (2 * f + 1) * ld)[lane] = J.v[F_].i;
        });
        return;
    }
    // half 0 takes the real parts of all flows through the colour sum, half 1 the imaginary parts
    static_for<NC / 2>([&](auto F_) { lds[XCH + (12 * wave + F_) * 64 + lane] = H == 0 ? J.v[F_].i : J.v[F_].r; });
    if (flow_weights)
        static_for<NC / 2>([&](auto F_) {
            lds[LCW + (12 * wave + F_) * 64 + lane] = members * fma(J.v[F_].r, J.v[F_].r, J.v[F_].i * J.v[F_].i);
        });
    __syncthreads();
    if (flow_weights && e < n_evt)   // three flows per wave, over the spin configurations
        static_for<NC>([&](auto F_) {
            if (F_ / 3 != wave) return;
            lds_d* const x = (lds_d*)(lds + LCW) + (12 * half_of(F_) + in_half(F_)) * 64 + lane;
            (flow_weights + F_ * n_evt)[e] = (x[0] + x[24 * 64]) + (x[48 * 64] + x[72 * 64]);
        });
    lds_d* const other = (lds_d*)(lds + XCH) + 12 * (wave ^ 1) * 64;
    double all[NC];
    static_for<NC>([&](auto F_) {
        constexpr int k = in_half(F_);
        if constexpr (half_of(F_) == H) all[F_] = H == 0 ? J.v[k].r : J.v[k].i;
        else all[F_] = other[k * 64 + lane];
    });
    const auto part = [&](auto F_) { return all[F_]; };
    const double q = colour_blocks_signs<NG>(part);
    double* const sum = lds + FOUR;
    if (H == 1) sum[sp * 64 + lane] = q;
    __syncthreads();
    if (H == 0 && h >= 0 && e < n_evt) jamp[(int64_t)h * n_evt + e] = colour_blocks_total(q, sum[sp * 64 + lane]);
}

__global__ __launch_bounds__(512, 2) void amp_rec(const double* __restrict__ mom, int64_t n_evt, int64_t ld,
                                                  const int* __restrict__ cfg, int n_cfg, double mt, double gs,
                                                  double* __restrict__ jamp, bool me,
                                                  const int2* __restrict__ members, double* __restrict__ flow_weights)
{
    __shared__ double lds[CUR + NSLOT * 512];
    double* const cur = lds + CUR;
    const unsigned lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t w = xcd_remap(blockIdx.x, gridDim.x);
    const int64_t e0 = (w / n_cfg) * 64;
    const int* const row_cfg = cfg + (w % n_cfg) * 5;
    const int bits = row_cfg[0];
    stage_momenta<NPAR, 8>(mom, n_evt, e0, lds, threadIdx.x);
    const auto P = [&](int i) { return lc(lds_p4(lds, i, lane)); };
    // incoming momentum of gluon i
    const auto pin = [&](int i) { return i < 2 ? lds_p4(lds, i, lane) : -lds_p4(lds, i + 2, lane); };
    const auto kin = [&](int i) { return lc(pin(i)); };
    const auto G1 = [&](int i) { return ld_e(lds + EPS, i, lane); };

    // external states, one per wave
    if (wave < 4) st_e(lds + EPS, wave, lane, gluon(lds_p4(lds, wave < 2 ? wave : wave + 2, lane), (bits >> wave) & 1 ? 1 : -1, wave >= 2, gs));
    else if (wave < 6) st_v(cur, SU + wave - 4, lane, spinor(ext_ubar<double>(lds_p4(lds, 2, lane), mt, wave == 5 ? 1 : -1)));
    else st_v(cur, SV + wave - 6, lane, spinor(ext_v<double>(lds_p4(lds, 3, lane), mt, wave == 7 ? 1 : -1)));
    __syncthreads();
    // strings of one gluon i: from the quark end (rows L) and the antiquark end (columns R)
    const auto string = [&](int k) {
        const int i = (k >> 1) & 3, sp = k & 1;
        if (k < 8)
            st_v(cur, SL + 4 * sp + i, lane, prop_row(prop(P(2) - kin(i), mt), row(ld_v(cur, SU + sp, lane), G1(i))));
        else
            st_v(cur, SR + 4 * sp + i, lane, prop_col(prop(kin(i) - P(3), mt), col(G1(i), ld_v(cur, SV + sp, lane))));
    };
    // A wave's gluons are run-time values, so that the eight waves run the same instructions (50 KB of
    // program; 97 KB with a copy for each wave, 4.96 ms)
    const auto J2 = [&](int i, int j) {
        return (i < j ? 1.0 : -1.0) * ld_v(cur, s2(min(i, j), max(i, j)), lane);
    };
    const auto J3 = [&](int x, int y, int z) {
        const int s = S3 + 2 * (6 - x - y - z);
        return three_ordered(x, y, z, [&] { return ld_v(cur, s, lane); }, [&] { return ld_v(cur, s + 1, lane); });
    };
    // two-gluon currents; the last two waves begin with the strings
    if (wave < 6) {
        const int i = pair_i(wave), j = pair_j(wave);
        const E4 A = G1(i), B = G1(j);
        const P4 pi = pin(i), pj = pin(j);
        const K4 ki = lc(pi), kj = lc(pj);
        st_v(cur, S2 + wave, lane, pair_prop(pi, pj) * vvv_acc(zero4(), A, ki, B, kj, dot2(A, B)));
    } else {
        string(wave - 6);
    }
    __syncthreads();
    // three-gluon currents, an ordering per wave
    {
        const int m = wave >> 1, x = rest(m, 0), y = rest(m, wave & 1 ? 2 : 1), z = rest(m, wave & 1 ? 1 : 2);
        const E4 X = G1(x), Y = G1(y), Z = G1(z);
        const V4 XY = J2(x, y), YZ = J2(y, z);
        const K4 kx = kin(x), ky = kin(y), kz = kin(z);
        V4 o = vvv_acc(zero4(), X, kx, YZ, ky + kz, dot2(X, YZ));
        o = vvv_acc(o, XY, kx + ky, Z, kz, dot2(XY, Z));
        st_v(cur, S3 + wave, lane, (-rcp(sq(kx + ky + kz))) * vvvv_acc(o, X, Y, Z, dot2(X, Y), dot2(Y, Z), dot2(X, Z)));
    }
    __syncthreads();
    // four-gluon currents, contracted at once with the quark currents; the last two waves make the other strings
    C four[4];
    if (wave >= 6) {
#pragma unroll 1
        for (int k = wave - 4; k < 16; k += 2) string(k);
    } else {
        const int b = (wave >> 1) + 1, lo = b == 1 ? 2 : 1, hi = b == 3 ? 2 : 3;
        const K4 k[4] = {kin(0), kin(1), kin(2), kin(3)}, kb = kin(b), kc = kin(wave & 1 ? hi : lo), kd = kin(wave & 1 ? lo : hi);
        const V4 o = (-rcp(sq((k[0] + k[1]) + (k[2] + k[3])))) *
                     four_numerator(b, wave & 1 ? hi : lo, wave & 1 ? lo : hi, G1, J2, J3, k[0], kb, kc, kd);
        static_for<4>([&](auto SP) {
            four[SP] = rc(pair(ld_v(cur, SU + SP / 2, lane), ld_v(cur, SV + SP % 2, lane)), o);
            pin_cx(four[SP]);
        });
    }
    __syncthreads();
    const int sp = wave >> 1, h = row_cfg[1 + sp];   // the row of this wave's spins, or -1
    const double count = h >= 0 ? members_of(members, h) : 0.0;
    if (flow_weights) flow_weights += (w % n_cfg) * NC * n_evt;
    if (wave & 1) finish<1>(lds, lane, wave, sp, four, n_evt, ld, e0, h, mt, jamp, me, count, flow_weights);
    else finish<0>(lds, lane, wave, sp, four, n_evt, ld, e0, h, mt, jamp, me, count, flow_weights);
}

hipError_t launch(const double* mom, int64_t n_evt, int64_t ld, const HelicityGroups& hg, double mt, double gs,
                  double* jamp, const FusedColour* fc, hipStream_t st)
{
    const int64_t blocks = ((n_evt + 63) / 64) * hg.n;
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(amp_rec, dim3((unsigned)blocks), dim3(512), 0, st, mom, n_evt, ld, hg.table, hg.n, mt, gs, jamp,
                       fc != nullptr, hg.members, fc ? fc->flow_weights : nullptr);
    return hipGetLastError();
}
}  // namespace rec4
}  // namespace me
