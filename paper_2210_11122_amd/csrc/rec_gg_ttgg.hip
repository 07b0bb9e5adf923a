// rec_gg_ttgg.hip -- FP64 colour-flow amplitudes of gg -> t t~ g g by colour-ordered recursion.
//
// Bound by FP64 issue: 6.3k FP64 instructions per (event, helicity) lane, where the diagram program
// takes 11.5k, one wave per SIMD (the vector registers and the 108 KB of currents allow no second).
// 2^19 events: 20.6 -> 5.0 ms per call (10.2 with all 64 helicities evaluated).
#include "colorsum.hpp"
#include "process.hpp"
#include "recursion.hpp"

namespace me {
namespace rec4 {
using namespace rec;

constexpr int NG = 4, NPAR = 6, NC = 24;
// LDS slots of the gluon currents: J(i), J(ij) with i < j, J of the two independent orderings
// (xyz), (xzy) of the gluons without w, and J(0 s) for the six orderings s of gluons 1, 2, 3
constexpr int S1 = 0, S2 = 4, S3 = 10, S4 = 18, NSLOT = 24;
constexpr int MOM = 4 * NPAR * 64;   // doubles of the staged momenta

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

// One workgroup: 64 events, one configuration of the four gluon helicities; its four waves are
// the four spin configurations of the quarks, which share every gluon current.
__global__ __launch_bounds__(256, 1) void amp_rec(const double* __restrict__ mom, int64_t n_evt, int64_t ld,
                                                  const int* __restrict__ cfg, int n_cfg, double mt, double gs,
                                                  double* __restrict__ jamp, FusedColour fc)
{
    __shared__ double lds[MOM + NSLOT * 512];
    double* const cur = lds + MOM;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t w = xcd_remap(blockIdx.x, gridDim.x);
    const int64_t e0 = (w / n_cfg) * 64;
    const int64_t e = e0 + lane;
    const int* const row_cfg = cfg + (w % n_cfg) * 5;
    const int bits = row_cfg[0];
    const int h = row_cfg[1 + wave];   // good helicity of this wave's spins, or -1
    stage_momenta<NPAR, 4>(mom, n_evt, e0, lds, threadIdx.x);
    const auto P = [&](int i) { return lc(lds_p4(lds, i, lane)); };
    // incoming momentum of gluon i
    const auto kin = [&](int i) { return i < 2 ? P(i) : -P(i + 2); };
    const auto ld1 = [&](int k) { return ld_v(cur, k, lane); };

    // --- gluon currents, shared out among the waves
    {
        const int p = wave < 2 ? wave : wave + 2;
        st_v(cur, S1 + wave, lane, full(gluon(lds_p4(lds, p, lane), (bits >> wave) & 1 ? 1 : -1, wave >= 2, gs)));
    }
    __syncthreads();
    static_for<6>([&](auto P_) {
        constexpr int p = P_, i = pair_i(p), j = pair_j(p);
        if ((p & 3) != wave) return;
        const V4 A = ld1(S1 + i), B = ld1(S1 + j);
        const K4 ki = kin(i), kj = kin(j);
        st_v(cur, s2(i, j), lane, (-rcp(sq(ki + kj))) * vvv_acc(zero4(), A, ki, B, kj, dot2(A, B)));
    });
    __syncthreads();
    static_for<4>([&](auto W_) {
        constexpr int m = W_, x = rest(m, 0), y = rest(m, 1), z = rest(m, 2);
        if (m != wave) return;
        const V4 X = ld1(S1 + x), Y = ld1(S1 + y), Z = ld1(S1 + z);
        const V4 XY = ld1(s2(x, y)), XZ = ld1(s2(x, z)), YZ = ld1(s2(y, z));
        const K4 kx = kin(x), ky = kin(y), kz = kin(z);
        const C xy = dot2(X, Y), yz = dot2(Y, Z), xz = dot2(X, Z);
        const double f = -rcp(sq(kx + ky + kz));
        const V4 v = vvv_acc(zero4(), X, kx, YZ, ky + kz, dot2(X, YZ));   // V(x, yz) = -V(x, zy)
        V4 o = vvv_acc(v, XY, kx + ky, Z, kz, dot2(XY, Z));
        st_v(cur, S3 + 2 * m, lane, f * vvvv_acc(o, X, Y, Z, xy, yz, xz));
        o = vvv_acc(-v, XZ, kx + kz, Y, ky, dot2(XZ, Y));
        st_v(cur, S3 + 2 * m + 1, lane, f * vvvv_acc(o, X, Z, Y, xz, yz, xy));
    });
    __syncthreads();
    static_for<6>([&](auto R_) {
        constexpr int r = R_;
        if (((r + 2) & 3) != wave) return;
        constexpr Perm<3> s = perm_at<3>(r);
        constexpr int b = s.p[0] + 1, c = s.p[1] + 1, d = s.p[2] + 1;
        const V4 A = ld1(S1), B = ld1(S1 + b), Cc = ld1(S1 + c), D = ld1(S1 + d);
        const K4 ka = kin(0), kb = kin(b), kc = kin(c), kd = kin(d);
        const V4 AB = ld1(s2(0, b));
        V4 BC = b < c ? ld1(s2(b < c ? b : c, b < c ? c : b)) : -ld1(s2(b < c ? b : c, b < c ? c : b));
        V4 CD = c < d ? ld1(s2(c < d ? c : d, c < d ? d : c)) : -ld1(s2(c < d ? c : d, c < d ? d : c));
        const V4 ABC = ld1(S3 + 2 * d + (b < c ? 0 : 1));
        constexpr int k0 = kk_table<3>.c[r][0], k1 = kk_table<3>.c[r][1];
        V4 BCD;
        if constexpr (k1 == 0) BCD = ld1(S3);
        else if constexpr (k0 == 0) BCD = ld1(S3 + 1);
        else BCD = -(ld1(S3) + ld1(S3 + 1));
        static_assert((k0 == 1 && k1 == 0) || (k0 == 0 && k1 == 1) || (k0 == -1 && k1 == -1), "");
        V4 o = vvv_acc(zero4(), A, ka, BCD, kb + kc + kd, dot2(A, BCD));
        o = vvv_acc(o, AB, ka + kb, CD, kc + kd, dot2(AB, CD));
        o = vvv_acc(o, ABC, ka + kb + kc, D, kd, dot2(ABC, D));
        o = vvvv_acc(o, A, B, CD, dot2(A, B), dot2(B, CD), dot2(A, CD));
        o = vvvv_acc(o, A, BC, D, dot2(A, BC), dot2(BC, D), dot2(A, D));
        o = vvvv_acc(o, AB, Cc, D, dot2(AB, Cc), dot2(Cc, D), dot2(AB, D));
        st_v(cur, S4 + r, lane, (-rcp(sq(ka + kb + kc + kd))) * o);
    });

    // --- the quark line of this wave's spins
    C J[NC];
    if (h >= 0) {
        const V4 U = spinor(ext_ubar<double>(lds_p4(lds, 2, lane), mt, (wave & 2) ? 1 : -1));
        const V4 S = spinor(ext_v<double>(lds_p4(lds, 3, lane), mt, (wave & 1) ? 1 : -1));
        // strings of one gluon, from the quark end (rows L) and the antiquark end (columns R)
        V4 L[NG], R[NG];
        static_for<NG>([&](auto I_) {
            constexpr int i = I_;
            const V4 G = ld1(S1 + i);
            const K4 k = kin(i);
            L[i] = prop_row(prop(P(2) - k, mt), row(U, G));
            R[i] = prop_col(prop(k - P(3), mt), col(G, S));
        });
        // the line cut in the middle: two gluons on either side, or a current J(cd) at the cut
        static_for<6>([&](auto P_) {
            constexpr int p = P_, a = pair_i(p), b = pair_j(p), c = pair_i(5 - p), d = pair_j(5 - p);
            const V4 Gab = ld1(s2(a, b)), Ga = ld1(S1 + a), Gb = ld1(S1 + b);
            const V4 x = row(U, Gab);
            const Prop q = prop(P(2) - kin(a) - kin(b), mt);
            const V4 Lab = prop_row(q, row_acc(x, L[a], Gb)), Lba = prop_row(q, row_acc(-x, L[b], Ga));
            const V4 Gcd = ld1(s2(c, d)), Gc = ld1(S1 + c), Gd = ld1(S1 + d);
            const V4 y = col(Gcd, S);
            const V4 Rcd = col_acc(y, Gc, R[d]), Rdc = col_acc(-y, Gd, R[c]);
            J[flow(a, b, c, d)] = rc(Lab, Rcd);
            J[flow(a, b, d, c)] = rc(Lab, Rdc);
            J[flow(b, a, c, d)] = rc(Lba, Rcd);
            J[flow(b, a, d, c)] = rc(Lba, Rdc);
        });
        static_for<6>([&](auto P_) {
            constexpr int p = P_, a = pair_i(p), b = pair_j(p), c = pair_i(5 - p), d = pair_j(5 - p);
            const V4 Gcd = ld1(s2(c, d));
            C t = rc(L[a], col(Gcd, R[b]));
            J[flow(a, c, d, b)] = J[flow(a, c, d, b)] + t;
            J[flow(a, d, c, b)] = J[flow(a, d, c, b)] - t;
            t = rc(L[b], col(Gcd, R[a]));
            J[flow(b, c, d, a)] = J[flow(b, c, d, a)] + t;
            J[flow(b, d, c, a)] = J[flow(b, d, c, a)] - t;
        });
        // J of three gluons next to the antiquark or to the quark
        static_for<4>([&](auto W_) {
            constexpr int m = W_, x = rest(m, 0), y = rest(m, 1), z = rest(m, 2);
            const V4 G0 = ld1(S3 + 2 * m), G1 = ld1(S3 + 2 * m + 1);
            const V4 cl = pair(L[m], S), cr = pair(U, R[m]);
            const C l0 = rc(cl, G0), l1 = rc(cl, G1), r0 = rc(cr, G0), r1 = rc(cr, G1);
            const C l2 = l0 + l1, r2 = r0 + r1;
            J[flow(m, x, y, z)] = J[flow(m, x, y, z)] + l0;
            J[flow(m, z, y, x)] = J[flow(m, z, y, x)] + l0;
            J[flow(m, x, z, y)] = J[flow(m, x, z, y)] + l1;
            J[flow(m, y, z, x)] = J[flow(m, y, z, x)] + l1;
            J[flow(m, y, x, z)] = J[flow(m, y, x, z)] - l2;
            J[flow(m, z, x, y)] = J[flow(m, z, x, y)] - l2;
            J[flow(x, y, z, m)] = J[flow(x, y, z, m)] + r0;
            J[flow(z, y, x, m)] = J[flow(z, y, x, m)] + r0;
            J[flow(x, z, y, m)] = J[flow(x, z, y, m)] + r1;
            J[flow(y, z, x, m)] = J[flow(y, z, x, m)] + r1;
            J[flow(y, x, z, m)] = J[flow(y, x, z, m)] - r2;
            J[flow(z, x, y, m)] = J[flow(z, x, y, m)] - r2;
        });
    }
    __syncthreads();   // J(0 s) written
    if (h < 0) return;
    {
        const V4 U = spinor(ext_ubar<double>(lds_p4(lds, 2, lane), mt, (wave & 2) ? 1 : -1));
        const V4 S = spinor(ext_v<double>(lds_p4(lds, 3, lane), mt, (wave & 1) ? 1 : -1));
        const V4 c4 = pair(U, S);
        C s[6];
        static_for<6>([&](auto R_) { s[R_] = rc(c4, ld1(S4 + R_)); });
        static_for<24>([&](auto F_) {
            static_for<6>([&](auto R_) {
                constexpr int k = kk_table<4>.c[F_][R_];
                static_assert(k >= -1 && k <= 1, "");
                if constexpr (k == 1) J[F_] = J[F_] + s[R_];
                if constexpr (k == -1) J[F_] = J[F_] - s[R_];
            });
        });
    }
    if (fc.aop) {
        const double me_h = colour_blocks<NG>(J);
        if (e < n_evt) jamp[(int64_t)h * n_evt + e] = me_h;
        return;
    }
    if (e < n_evt) {
        double* o = jamp + (int64_t)h * (2 * NC) * ld + e;
        static_for<NC>([&](auto F_) {
            o[(2 * F_) * ld] = J[F_].r;
            o[(2 * F_ + 1) * ld] = J[F_].i;
        });
    }
}

hipError_t launch(const double* mom, int64_t n_evt, int64_t ld, const HelicityGroups& hg, double mt, double gs,
                  double* jamp, const FusedColour* fc, hipStream_t st)
{
    const FusedColour none{nullptr, nullptr, 0, 0, nullptr, 0.0, 1};
    const int64_t blocks = ((n_evt + 63) / 64) * hg.n;
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(amp_rec, dim3((unsigned)blocks), dim3(256), 0, st, mom, n_evt, ld, hg.table, hg.n, mt, gs, jamp,
                       fc ? *fc : none);
    return hipGetLastError();
}
}  // namespace rec4
}  // namespace me
