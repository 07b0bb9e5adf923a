// recursion.hpp -- FP64 wavefunction algebra of the colour-ordered recursion.
//
// The FP64 kernels do not evaluate diagram by diagram: they build colour-ordered off-shell
// currents (Berends and Giele, Nucl. Phys. B306 (1988) 759).  For an ordering s of gluons, with P
// the sum of their incoming momenta and every current times g_s,
//   J(s) = -1/P^2 [ sum_{s = A B} V(J_A, J_B) + sum_{s = A B C} Q(J_A, J_B, J_C) ]
//   V(A, B) = (A.B)(k_A - k_B) + 2 (k_B.A) B - 2 (k_A.B) A      (currents are transverse)
//   Q(A, B, C) = A (B.C) + C (A.B) - 2 B (A.C)
// and a quark string takes gluon blocks one after the other with the propagator
//   -(qslash + m) / (q^2 - m^2).
// The sum over all blocks of an ordering is its colour-flow amplitude (jamp), up to one phase
// common to all flows, which |M|^2 and the flow weights do not see.
//
// Vectors are held in the components of gamma.G = [[0, G.sigma], [G.sigmabar, 0]]:
//   a = G0 + G3, b = G0 - G3, c = G1 + i G2, d = G1 - i G2,
// so a quark vertex needs no additions, and 2 A.B = A.a B.b + A.b B.a - A.c B.d - A.d B.c.
#pragma once
#include "flows.hpp"
#include "helas.hpp"

namespace me {
namespace rec {

typedef cx<double> C;
// a vector current (a, b, c, d) or a spinor (four components)
struct V4 {
    C a, b, c, d;
};
// A real momentum in the same components (d = conj(c)).  Momenta are also summed in them, but for P^2 of two
// gluons (pair_prop).
struct K4 {
    double a, b, x, y;
};
__device__ __forceinline__ K4 lc(const P4& p) { return {p.t + p.z, p.t - p.z, p.x, p.y}; }
__device__ __forceinline__ K4 operator+(const K4& p, const K4& q) { return {p.a + q.a, p.b + q.b, p.x + q.x, p.y + q.y}; }
__device__ __forceinline__ K4 operator-(const K4& p, const K4& q) { return {p.a - q.a, p.b - q.b, p.x - q.x, p.y - q.y}; }
__device__ __forceinline__ K4 operator-(const K4& p) { return {-p.a, -p.b, -p.x, -p.y}; }
__device__ __forceinline__ double sq(const K4& p) { return fma(p.a, p.b, -fma(p.x, p.x, p.y * p.y)); }
// The propagator of two gluons, -1/P^2, from the Cartesian sum of their momenta, rounded as in the diagram program
// (msq of helas.hpp: mixed forms, channel weights).  A gluon along a beam, or two along each other, leave few digits
// of P^2 and |M|^2 follows its rounding: with this one the FP64 values agree with the diagram program's to 1.1e-12 in
// each of 2^20 gg -> tt~g, 2^18 gg -> tt~gg and 2^17 gg -> tt~ggg events of 9 to 17 seeds.  With sq() of the K4 sum
// single events, some of nearly a batch's whole norm, were 1e-9 to 6e-8 from them.  (That form loses less: gg -> tt~gg
// p99.9 against long double 1.4e-13, this one 5.7e-13.  But such an event's momenta, rounded to 64 bits, leave as
// much open: 1.8e-8 in the event that was 1.1e-8 off, by the particle that takes up what they miss of conservation.)
__device__ __forceinline__ double pair_prop(const P4& p, const P4& q) { return -rcp(msq(p + q)); }

__device__ __forceinline__ C cmul(C a, C b) { return {fma(a.r, b.r, -a.i * b.i), fma(a.r, b.i, a.i * b.r)}; }
__device__ __forceinline__ C neg(C a) { return {-a.r, -a.i}; }
__device__ __forceinline__ V4 operator+(const V4& x, const V4& y) { return {x.a + y.a, x.b + y.b, x.c + y.c, x.d + y.d}; }
__device__ __forceinline__ V4 operator-(const V4& x, const V4& y) { return {x.a - y.a, x.b - y.b, x.c - y.c, x.d - y.d}; }
__device__ __forceinline__ V4 operator*(double f, const V4& x) { return {f * x.a, f * x.b, f * x.c, f * x.d}; }
__device__ __forceinline__ C cadd_s(C x, double s, C y) { return {fma(s, y.r, x.r), fma(s, y.i, x.i)}; }  // x + s y

// 2 A.B and 2 A.k
__device__ __forceinline__ C dot2(const V4& A, const V4& B)
{
    return cfms(A.d, B.c, cfms(A.c, B.d, cfma(A.b, B.a, cmul(A.a, B.b))));
}
__device__ __forceinline__ C dot2(const V4& A, const K4& k)
{
    C o = {fma(A.b.r, k.a, A.a.r * k.b), fma(A.b.i, k.a, A.a.i * k.b)};
    // - c conj(kc) - d kc, kc = x + i y
    o.r = fma(-A.c.r, k.x, fma(-A.c.i, k.y, o.r));
    o.i = fma(-A.c.i, k.x, fma(A.c.r, k.y, o.i));
    o.r = fma(-A.d.r, k.x, fma(A.d.i, k.y, o.r));
    o.i = fma(-A.d.i, k.x, fma(-A.d.r, k.y, o.i));
    return o;
}
// acc + s A, acc - s A
__device__ __forceinline__ V4 axpy(const V4& acc, C s, const V4& A)
{
    return {cfma(s, A.a, acc.a), cfma(s, A.b, acc.b), cfma(s, A.c, acc.c), cfma(s, A.d, acc.d)};
}
__device__ __forceinline__ V4 axmy(const V4& acc, C s, const V4& A)
{
    return {cfms(s, A.a, acc.a), cfms(s, A.b, acc.b), cfms(s, A.c, acc.c), cfms(s, A.d, acc.d)};
}
// A polarisation vector (times g): no time component, a real longitudinal one, so a = G3 is real
// and b = -a: five numbers, and products with it take three quarters of the operations.
struct E4 {
    double a;
    C c, d;
};
__device__ __forceinline__ C conj(C a) { return {a.r, -a.i}; }
// the vector of the other helicity
__device__ __forceinline__ E4 flip(const E4& e) { return {-e.a, neg(conj(e.d)), neg(conj(e.c))}; }
__device__ __forceinline__ V4 full(const E4& e) { return {{e.a, 0.0}, {-e.a, 0.0}, e.c, e.d}; }
__device__ __forceinline__ C scaled_add(C o, double f, C x) { return {fma(f, x.r, o.r), fma(f, x.i, o.i)}; }
__device__ __forceinline__ C dot2(const E4& A, const V4& B)
{
    const C t = B.b - B.a;
    return cfms(A.d, B.c, cfms(A.c, B.d, {A.a * t.r, A.a * t.i}));
}
__device__ __forceinline__ C dot2(const V4& A, const E4& B) { return dot2(B, A); }
__device__ __forceinline__ C dot2(const E4& A, const E4& B)
{
    return cfms(A.d, B.c, cfms(A.c, B.d, {-2.0 * (A.a * B.a), 0.0}));
}
__device__ __forceinline__ C dot2(const E4& A, const K4& k)
{
    C o = {A.a * (k.b - k.a), 0.0};
    o.r = fma(-A.c.r, k.x, fma(-A.c.i, k.y, o.r));
    o.i = fma(-A.c.i, k.x, A.c.r * k.y);
    o.r = fma(-A.d.r, k.x, fma(A.d.i, k.y, o.r));
    o.i = fma(-A.d.i, k.x, fma(-A.d.r, k.y, o.i));
    return o;
}
__device__ __forceinline__ V4 axpy(const V4& acc, C s, const E4& A)
{
    return {scaled_add(acc.a, A.a, s), scaled_add(acc.b, -A.a, s), cfma(s, A.c, acc.c), cfma(s, A.d, acc.d)};
}
__device__ __forceinline__ V4 axmy(const V4& acc, C s, const E4& A)
{
    return {scaled_add(acc.a, -A.a, s), scaled_add(acc.b, A.a, s), cfms(s, A.c, acc.c), cfms(s, A.d, acc.d)};
}

// k/2 + q
__device__ __forceinline__ K4 half_plus(const K4& k, const K4& q)
{
    return {fma(0.5, k.a, q.a), fma(0.5, k.b, q.b), fma(0.5, k.x, q.x), fma(0.5, k.y, q.y)};
}
// acc + V(A, B); AB = 2 A.B
template <class TA, class TB>
__device__ __forceinline__ V4 vvv_acc(const V4& acc, const TA& A, const K4& ka, const TB& B, const K4& kb, C AB)
{
    const K4 k = ka - kb;
    const C h = 0.5 * AB, s = dot2(A, half_plus(ka, kb)), t = dot2(B, half_plus(kb, ka));
    V4 o = axmy(axpy(acc, s, B), t, A);
    o.a = cadd_s(o.a, k.a, h);
    o.b = cadd_s(o.b, k.b, h);
    // c: h (x + i y), d: h (x - i y)
    o.c = {fma(-h.i, k.y, fma(h.r, k.x, o.c.r)), fma(h.r, k.y, fma(h.i, k.x, o.c.i))};
    o.d = {fma(h.i, k.y, fma(h.r, k.x, o.d.r)), fma(-h.r, k.y, fma(h.i, k.x, o.d.i))};
    return o;
}
// acc + Q(A, B, D) from AB = 2 A.B, BD = 2 B.D, AD = 2 A.D
template <class TA, class TB, class TD>
__device__ __forceinline__ V4 vvvv_acc(const V4& acc, const TA& A, const TB& B, const TD& D, C AB, C BD, C AD)
{
    return axmy(axpy(axpy(acc, 0.5 * BD, A), 0.5 * AB, D), AD, B);
}
__device__ __forceinline__ V4 operator-(const V4& x) { return {neg(x.a), neg(x.b), neg(x.c), neg(x.d)}; }
__device__ __forceinline__ V4 zero4() { return {{0, 0}, {0, 0}, {0, 0}, {0, 0}}; }

// polarisation vector of a gluon, times g
__device__ __forceinline__ E4 gluon(const P4& p, int lam, bool outgoing, double g)
{
    const W4<double> w = ext_vec<double>(p, 1, outgoing);
    const E4 e = {g * w.c[3].r,
                  {g * (w.c[1].r - w.c[2].i), g * (w.c[1].i + w.c[2].r)},
                  {g * (w.c[1].r + w.c[2].i), g * (w.c[1].i - w.c[2].r)}};
    return lam > 0 ? e : flip(e);
}
__device__ __forceinline__ V4 spinor(const W4<double>& w) { return {w.c[0], w.c[1], w.c[2], w.c[3]}; }

// acc + u gamma.G for a row spinor, acc + gamma.G s for a column spinor
__device__ __forceinline__ V4 row_acc(const V4& o, const V4& u, const V4& G)
{
    return {cfma(u.d, G.c, cfma(u.c, G.a, o.a)), cfma(u.d, G.b, cfma(u.c, G.d, o.b)),
            cfms(u.b, G.c, cfma(u.a, G.b, o.c)), cfms(u.a, G.d, cfma(u.b, G.a, o.d))};
}
__device__ __forceinline__ V4 row(const V4& u, const V4& G)
{
    return {cfma(u.d, G.c, cmul(u.c, G.a)), cfma(u.d, G.b, cmul(u.c, G.d)), cfms(u.b, G.c, cmul(u.a, G.b)),
            cfms(u.a, G.d, cmul(u.b, G.a))};
}
__device__ __forceinline__ V4 col_acc(const V4& o, const V4& G, const V4& s)
{
    return {cfms(G.d, s.d, cfma(G.b, s.c, o.a)), cfms(G.c, s.c, cfma(G.a, s.d, o.b)),
            cfma(G.d, s.b, cfma(G.a, s.a, o.c)), cfma(G.b, s.b, cfma(G.c, s.a, o.d))};
}
__device__ __forceinline__ V4 col(const V4& G, const V4& s)
{
    return {cfms(G.d, s.d, cmul(G.b, s.c)), cfms(G.c, s.c, cmul(G.a, s.d)), cfma(G.d, s.b, cmul(G.a, s.a)),
            cfma(G.b, s.b, cmul(G.c, s.a))};
}
// the same with a polarisation vector
__device__ __forceinline__ V4 row_acc(const V4& o, const V4& u, const E4& G)
{
    return {cfma(u.d, G.c, scaled_add(o.a, G.a, u.c)), cfma(u.c, G.d, scaled_add(o.b, -G.a, u.d)),
            cfms(u.b, G.c, scaled_add(o.c, -G.a, u.a)), cfms(u.a, G.d, scaled_add(o.d, G.a, u.b))};
}
__device__ __forceinline__ C times(double f, C x) { return {f * x.r, f * x.i}; }
__device__ __forceinline__ V4 row(const V4& u, const E4& G)
{
    return {cfma(u.d, G.c, times(G.a, u.c)), cfma(u.c, G.d, times(-G.a, u.d)), cfms(u.b, G.c, times(-G.a, u.a)),
            cfms(u.a, G.d, times(G.a, u.b))};
}
__device__ __forceinline__ V4 col_acc(const V4& o, const E4& G, const V4& s)
{
    return {cfms(G.d, s.d, scaled_add(o.a, -G.a, s.c)), cfms(G.c, s.c, scaled_add(o.b, G.a, s.d)),
            cfma(G.d, s.b, scaled_add(o.c, G.a, s.a)), cfma(G.c, s.a, scaled_add(o.d, -G.a, s.b))};
}
__device__ __forceinline__ V4 col(const E4& G, const V4& s)
{
    return {cfms(G.d, s.d, times(-G.a, s.c)), cfms(G.c, s.c, times(G.a, s.d)), cfma(G.d, s.b, times(G.a, s.a)),
            cfma(G.c, s.a, times(-G.a, s.b))};
}
// a quark propagator -(qslash + m) / (q^2 - m^2) in a form ready to apply
struct Prop {
    K4 q;      // q / -(q^2 - m^2)
    double m;  // m / -(q^2 - m^2)
};
__device__ __forceinline__ Prop prop(const K4& q, double m)
{
    const double f = -rcp(fma(-m, m, sq(q)));
    return {{f * q.a, f * q.b, f * q.x, f * q.y}, f * m};
}
__device__ __forceinline__ C by_c(C u, double x, double y, C o)   // o + u (x + i y)
{
    return {fma(-u.i, y, fma(u.r, x, o.r)), fma(u.r, y, fma(u.i, x, o.i))};
}
__device__ __forceinline__ C scale(double f, C u) { return {f * u.r, f * u.i}; }
__device__ __forceinline__ V4 prop_row(const Prop& p, const V4& u)
{
    return {by_c(u.d, p.q.x, p.q.y, cadd_s(scale(p.m, u.a), p.q.a, u.c)),
            by_c(u.c, p.q.x, -p.q.y, cadd_s(scale(p.m, u.b), p.q.b, u.d)),
            by_c(u.b, -p.q.x, -p.q.y, cadd_s(scale(p.m, u.c), p.q.b, u.a)),
            by_c(u.a, -p.q.x, p.q.y, cadd_s(scale(p.m, u.d), p.q.a, u.b))};
}
__device__ __forceinline__ V4 prop_col(const Prop& p, const V4& s)
{
    return {by_c(s.d, -p.q.x, p.q.y, cadd_s(scale(p.m, s.a), p.q.b, s.c)),
            by_c(s.c, -p.q.x, -p.q.y, cadd_s(scale(p.m, s.b), p.q.a, s.d)),
            by_c(s.b, p.q.x, -p.q.y, cadd_s(scale(p.m, s.c), p.q.a, s.a)),
            by_c(s.a, p.q.x, p.q.y, cadd_s(scale(p.m, s.d), p.q.b, s.b))};
}
// row . column, and acc + row . column
__device__ __forceinline__ C rc(const V4& u, const V4& s)
{
    return cfma(u.d, s.d, cfma(u.c, s.c, cfma(u.b, s.b, cmul(u.a, s.a))));
}
__device__ __forceinline__ C rc_acc(C o, const V4& u, const V4& s)
{
    return cfma(u.d, s.d, cfma(u.c, s.c, cfma(u.b, s.b, cfma(u.a, s.a, o))));
}
// the quark current of a pair: u gamma.G s = pair(u, s) . G with the plain sum of products rc()
__device__ __forceinline__ V4 pair(const V4& u, const V4& s)
{
    return {cfma(u.b, s.d, cmul(u.c, s.a)), cfma(u.a, s.c, cmul(u.d, s.b)), cfms(u.b, s.c, cmul(u.d, s.a)),
            cfms(u.a, s.d, cmul(u.c, s.b))};
}

// the two independent currents of three gluons, J(xyz) and J(xzy), x < y < z
struct V4x2 {
    V4 v[2];
};
template <class T>
__device__ __forceinline__ V4x2 three_currents(const T& X, const K4& kx, const T& Y, const K4& ky, const T& Z, const K4& kz,
                                               const V4& XY, const V4& XZ, const V4& YZ)
{
    const C xy = dot2(X, Y), yz = dot2(Y, Z), xz = dot2(X, Z);
    const double f = -rcp(sq(kx + ky + kz));
    const V4 v = vvv_acc(zero4(), X, kx, YZ, ky + kz, dot2(X, YZ));   // V(x, yz) = -V(x, zy)
    const V4 a = vvvv_acc(vvv_acc(v, XY, kx + ky, Z, kz, dot2(XY, Z)), X, Y, Z, xy, yz, xz);
    const V4 b = vvvv_acc(vvv_acc(-v, XZ, kx + kz, Y, ky, dot2(XZ, Y)), X, Z, Y, xz, yz, xy);
    return {{f * a, f * b}};
}
// J(x y z) of three gluons in any order from the two independent ones, a = J(lo mid hi), b = J(lo hi mid)
template <class FA, class FB>
__device__ __forceinline__ V4 three_ordered(int x, int y, int z, const FA& a, const FB& b)
{
    const int lo = min(x, min(y, z)), hi = max(x, max(y, z));
    if (y == lo) return -(a() + b());
    return y == hi ? b() : a();
}
// -P^2 J(0 b c d) of four gluons 0 .. 3 from the currents j1(i), j2(i, j), j3(x, y, z) in any order, and
// the momenta
template <class F1, class F2, class F3>
__device__ __forceinline__ V4 four_numerator(int b, int c, int d, const F1& j1, const F2& j2, const F3& j3, const K4& ka,
                                             const K4& kb, const K4& kc, const K4& kd)
{
    const auto A = j1(0), B = j1(b), Cc = j1(c), D = j1(d);
    const V4 AB = j2(0, b), BC = j2(b, c), CD = j2(c, d), ABC = j3(0, b, c), BCD = j3(b, c, d);
    const K4 kab = ka + kb, kcd = kc + kd;
    V4 o = vvv_acc(zero4(), A, ka, BCD, kb + kcd, dot2(A, BCD));
    o = vvv_acc(o, AB, kab, CD, kcd, dot2(AB, CD));
    o = vvv_acc(o, ABC, kab + kc, D, kd, dot2(ABC, D));
    o = vvvv_acc(o, A, B, CD, dot2(A, B), dot2(B, CD), dot2(A, CD));
    o = vvvv_acc(o, A, BC, D, dot2(A, BC), dot2(BC, D), dot2(A, D));
    return vvvv_acc(o, AB, Cc, D, dot2(AB, Cc), dot2(Cc, D), dot2(AB, D));
}

// Marks a point in the program by which v is computed.  Arithmetic that no store or volatile access
// waits for would otherwise be moved below all later loads, which then spill.
__device__ __forceinline__ void pin_v(V4& v)
{
    asm volatile("" : "+v"(v.a.r), "+v"(v.a.i), "+v"(v.b.r), "+v"(v.b.i), "+v"(v.c.r), "+v"(v.c.i), "+v"(v.d.r), "+v"(v.d.i));
}

// The channel-weight sums of one helicity: K |a|^2 of every diagram's amplitude, and of the event's
// channel.  Pinned: put off to the end of the program they would hold every amplitude until then.
struct ChannelSums {
    double ch = 0.0, all = 0.0;
    __device__ __forceinline__ void add(int diagram, double weight, int channel, C a)
    {
        const double w = weight * fma(a.r, a.r, a.i * a.i);
        all += w;
        ch += diagram == channel ? w : 0.0;
        asm volatile("" : "+v"(all), "+v"(ch));
    }
};

// vectors in LDS: slot k holds (re, im) pairs of its components at [(4 k + m) * 64 + lane]
__device__ __forceinline__ void st_v(double* base, int k, int lane, const V4& v)
{
    typedef double v2d __attribute__((ext_vector_type(2)));
    v2d* p = reinterpret_cast<v2d*>(base) + 4 * k * 64 + lane;
    p[0] = {v.a.r, v.a.i};
    p[64] = {v.b.r, v.b.i};
    p[128] = {v.c.r, v.c.i};
    p[192] = {v.d.r, v.d.i};
}

__device__ __forceinline__ V4 ld_v(const double* base, int k, int lane)
{
    typedef double v2d __attribute__((ext_vector_type(2)));
    typedef __attribute__((address_space(3))) const volatile v2d lds_v2d;
    lds_v2d* p = (lds_v2d*)base + 4 * k * 64 + lane;
    const v2d a = p[0], b = p[64], c = p[128], d = p[192];
    return {{a.x, a.y}, {b.x, b.y}, {c.x, c.y}, {d.x, d.y}};
}

// polarisation vectors in LDS: five numbers each, slot k at [5 k * 64]
__device__ __forceinline__ void st_e(double* base, int k, int lane, const E4& v)
{
    typedef double v2d __attribute__((ext_vector_type(2)));
    double* const p = base + 5 * k * 64;
    p[lane] = v.a;
    reinterpret_cast<v2d*>(p + 64)[lane] = {v.c.r, v.c.i};
    reinterpret_cast<v2d*>(p + 192)[lane] = {v.d.r, v.d.i};
}
__device__ __forceinline__ E4 ld_e(const double* base, int k, int lane)
{
    typedef double v2d __attribute__((ext_vector_type(2)));
    typedef __attribute__((address_space(3))) const volatile v2d lds_v2d;
    typedef __attribute__((address_space(3))) const volatile double lds_d;
    lds_d* const p = (lds_d*)base + 5 * k * 64;
    const double a = p[lane];
    const v2d c = ((lds_v2d*)(p + 64))[lane], d = ((lds_v2d*)(p + 192))[lane];
    return {a, {c.x, c.y}, {d.x, d.y}};
}

}  // namespace rec
}  // namespace me
