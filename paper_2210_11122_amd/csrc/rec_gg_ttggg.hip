// rec_gg_ttggg.hip -- FP64 colour-flow amplitudes of gg -> t t~ g g g by colour-ordered recursion.
//
// Five gluons have 65 independent currents per helicity configuration, and a current of k gluons
// depends on their k helicities only.  So the currents of two to four gluons and the strings of
// one and two gluons of either quark are computed once per event into memory, level by level,
// one lane per event: 737 vectors (47 KB) per event, of which each of the 64 pairs of helicity
// configurations uses about 150.  (The slots are numbered for both helicities of every gluon, 1054 of 64 B;
// the 317 with gluon 0 at helicity + are reserved and stay unused.)  Two kernels then work per (event, pair):
// five_currents contracts the 24 independent currents of all five gluons with the quark currents, and amp_rec
// forms the 120 flows, 24 at a time (those with the same last gluon), each stored once.
//
// Against the 14 diagram segments (247k flops per lane, 977 partial jamp sums through memory):
// 2^17 events, colour sum included, 208.9 -> 24.4 ms per call (43.8 with all 128 helicities
// evaluated); 1531 events 3.05 -> 0.33 ms.
#include "process.hpp"
#include "recursion.hpp"

namespace me {
namespace rec5 {
using namespace rec;

constexpr int NG = 5, NPAR = 7, NC = 120;

__host__ __device__ constexpr int pair_index(int i, int j) { return i * (2 * NG - i - 1) / 2 + j - i - 1; }   // i < j
__host__ __device__ constexpr int triple_index(int x, int y, int z)   // x < y < z
{
    int n = 0;
    for (int a = 0; a < NG; ++a)
        for (int b = a + 1; b < NG; ++b)
            for (int c = b + 1; c < NG; ++c, ++n)
                if (a == x && b == y && c == z) return n;
    return -1;
}
struct Subset {
    int g[3];
};
__host__ __device__ constexpr Subset pair_at(int p)
{
    for (int i = 0; i < NG; ++i)
        for (int j = i + 1; j < NG; ++j)
            if (p-- == 0) return {{i, j, -1}};
    return {};
}
__host__ __device__ constexpr Subset triple_at(int t)
{
    for (int a = 0; a < NG; ++a)
        for (int b = a + 1; b < NG; ++b)
            for (int c = b + 1; c < NG; ++c)
                if (t-- == 0) return {{a, b, c}};
    return {};
}
// the gluons without w in ascending order
__host__ __device__ constexpr int rest(int w, int k) { return k < w ? k : k + 1; }
// ordered pair (a, b), a != b
__host__ __device__ constexpr int ordered(int a, int b) { return a * (NG - 1) + (b < a ? b : b - 1); }

// rank of the flow (f-th order of the gluons without g, then g), and the rank among the orders of
// the gluons without f's first one of that flow's last four
__host__ __device__ constexpr int flow_with_last(int g, int f)
{
    const Perm<4> q = perm_at<4>(f);
    Perm<5> x{};
    for (int i = 0; i < 4; ++i) x.p[i] = rest(g, q.p[i]);
    x.p[4] = g;
    return perm_rank<5>(x);
}
__host__ __device__ constexpr int last_four(int g, int f)
{
    const Perm<4> q = perm_at<4>(f);
    const int v[4] = {rest(g, q.p[1]), rest(g, q.p[2]), rest(g, q.p[3]), g};
    Perm<4> x{};
    for (int i = 0; i < 4; ++i)
        for (int j = 0; j < 4; ++j) x.p[i] += v[j] < v[i];
    return perm_rank<4>(x);
}
// rank of an order of four
__host__ __device__ constexpr int rank4(int i, int j, int k, int l)
{
    Perm<4> q{};
    q.p[0] = i, q.p[1] = j, q.p[2] = k, q.p[3] = l;
    return perm_rank<4>(q);
}
// rank of the order (b, c, d) among three
__host__ __device__ constexpr int rank3(int b, int c, int d)
{
    Perm<3> x{};
    x.p[0] = (b > c) + (b > d), x.p[1] = (c > b) + (c > d), x.p[2] = (d > b) + (d > c);
    return perm_rank<3>(x);
}

// Gluon 0 has helicity - throughout (HelicityGroups): the slots of its helicity + stay unused.
// vectors in memory: per block of 64 events, slot s holds (re, im) pairs at [(4 s + m) * 64 + lane]
constexpr int M1 = 0, M2 = M1 + 2 * NG, M3 = M2 + 4 * 10, M4 = M3 + 8 * 10 * 2, MU = M4 + 16 * 5 * 6, MS = MU + 2,
              ML1 = MS + 2, MR1 = ML1 + 4 * NG, ML2 = MR1 + 4 * NG, MR2 = ML2 + 8 * 20, MEND = MR2 + 8 * 20;
// helicity bits: of gluon i at bit i of `bits`
__device__ __forceinline__ int bit(int bits, int i) { return (bits >> i) & 1; }
__device__ __forceinline__ int m1(int i, int h) { return M1 + 2 * i + h; }
__device__ __forceinline__ int m2(int p, int hi, int hj) { return M2 + 4 * p + 2 * hi + hj; }
__device__ __forceinline__ int m3(int t, int hx, int hy, int hz, int k) { return M3 + 2 * (8 * t + 4 * hx + 2 * hy + hz) + k; }
__device__ __forceinline__ int m4(int w, int h4, int r) { return M4 + 6 * (16 * w + h4) + r; }
__device__ __forceinline__ int ml1(int a, int ha, int su) { return ML1 + 4 * a + 2 * ha + su; }
__device__ __forceinline__ int mr1(int a, int ha, int sv) { return MR1 + 4 * a + 2 * ha + sv; }
__device__ __forceinline__ int ml2(int o, int ha, int hb, int su) { return ML2 + 8 * o + 4 * ha + 2 * hb + su; }
__device__ __forceinline__ int mr2(int o, int ha, int hb, int sv) { return MR2 + 8 * o + 4 * ha + 2 * hb + sv; }
// the helicity bits of the four gluons without w, the first one highest
__device__ __forceinline__ int bits_without(int bits, int w)
{
    int h = 0;
    for (int k = 0; k < 4; ++k) h = 2 * h + bit(bits, rest(w, k));
    return h;
}

// a table pointer that the compiler cannot trace back, so that loads through it are not moved above
// this point (unrolled over the last gluon, they would all be hoisted and spilled)
template <class P>
__device__ __forceinline__ P* fresh(P* p)
{
#ifdef __HIP_DEVICE_COMPILE__
    __attribute__((address_space(1))) P* g = (__attribute__((address_space(1))) P*)p;   // stays a global pointer
    __asm__ volatile("" : "+s"(g));
    p = (P*)g;
#endif
    return p;
}

typedef double v2d __attribute__((ext_vector_type(2)));
// the vectors of one block of 64 events, and access to slot s of the lane's event: the address is
// a uniform base, a 32-bit lane offset and a constant
__device__ __forceinline__ v2d* block_of(v2d* cur, int64_t e) { return cur + (e >> 6) * (int64_t)(256 * MEND); }
__device__ __forceinline__ const v2d* block_of(const v2d* cur, int64_t e) { return cur + (e >> 6) * (int64_t)(256 * MEND); }
__device__ __forceinline__ V4 ldm(const v2d* __restrict__ blk, int s, unsigned lane)
{
    const v2d* p = blk + 256 * s;
    const v2d a = p[lane], b = p[lane + 64], c = p[lane + 128], d = p[lane + 192];
    return {{a.x, a.y}, {b.x, b.y}, {c.x, c.y}, {d.x, d.y}};
}
__device__ __forceinline__ void stm(v2d* __restrict__ blk, int s, unsigned lane, const V4& v)
{
    v2d* p = blk + 256 * s;
    p[lane] = {v.a.r, v.a.i};
    p[lane + 64] = {v.b.r, v.b.i};
    p[lane + 128] = {v.c.r, v.c.i};
    p[lane + 192] = {v.d.r, v.d.i};
}
__device__ __forceinline__ P4 mom4(const double* __restrict__ mom, int64_t e, int i)
{
    const v2d* p = reinterpret_cast<const v2d*>(mom) + (e * NPAR + i) * 2;
    const v2d a = p[0], b = p[1];
    return {a.x, a.y, b.x, b.y};
}
// incoming momentum of gluon i
__device__ __forceinline__ P4 pin(const double* __restrict__ mom, int64_t e, int i)
{
    const P4 p = mom4(mom, e, i < 2 ? i : i + 2);
    return i < 2 ? p : -p;
}
__device__ __forceinline__ K4 kin(const double* __restrict__ mom, int64_t e, int i) { return lc(pin(mom, e, i)); }

// --- level 1: external states; y: gluon, or 5: quark, 6: antiquark; both helicities
__global__ __launch_bounds__(256) void level1(const double* __restrict__ mom, int64_t n_evt, double mt, double gs,
                                              v2d* __restrict__ cur_)
{
    const unsigned wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t e0 = (int64_t)blockIdx.x * 256 + 64 * wave, e = e0 + lane;
    v2d* const cur = block_of(cur_, e0);
    const int i = blockIdx.y;
    if (e >= n_evt) return;
    if (i < NG) {
        const P4 p = mom4(mom, e, i < 2 ? i : i + 2);
        for (int h = 0; h < (i ? 2 : 1); ++h) stm(cur, m1(i, h), lane, full(gluon(p, h ? 1 : -1, i >= 2, gs)));
    } else if (i == NG) {
        const P4 p = mom4(mom, e, 2);
        for (int h = 0; h < 2; ++h) stm(cur, MU + h, lane, spinor(ext_ubar<double>(p, mt, h ? 1 : -1)));
    } else {
        const P4 p = mom4(mom, e, 3);
        for (int h = 0; h < 2; ++h) stm(cur, MS + h, lane, spinor(ext_v<double>(p, mt, h ? 1 : -1)));
    }
}
// --- level 2: two-gluon currents (y < 40) and one-gluon strings (20 of the quark, 20 of the antiquark)
__global__ __launch_bounds__(256) void level2(const double* __restrict__ mom, int64_t n_evt, double mt,
                                              v2d* __restrict__ cur_)
{
    const unsigned wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t e0 = (int64_t)blockIdx.x * 256 + 64 * wave, e = e0 + lane;
    v2d* const cur = block_of(cur_, e0);
    int y = blockIdx.y;
    if (e >= n_evt) return;
    if (y < 40) {
        const Subset s = pair_at(y >> 2);
        const int i = s.g[0], j = s.g[1], hi = (y >> 1) & 1, hj = y & 1;
        if (i == 0 && hi) return;
        const V4 A = ldm(cur, m1(i, hi), lane), B = ldm(cur, m1(j, hj), lane);
        const P4 pi = pin(mom, e, i), pj = pin(mom, e, j);
        const K4 ki = lc(pi), kj = lc(pj);
        stm(cur, m2(y >> 2, hi, hj), lane, pair_prop(pi, pj) * vvv_acc(zero4(), A, ki, B, kj, dot2(A, B)));
        return;
    }
    y -= 40;
    const int right = y >= 20, a = (y % 20) >> 2, h = (y >> 1) & 1, sp = y & 1;
    if (a == 0 && h) return;
    const V4 G = ldm(cur, m1(a, h), lane);
    const K4 k = kin(mom, e, a);
    if (!right)
        stm(cur, ml1(a, h, sp), lane, prop_row(prop(lc(mom4(mom, e, 2)) - k, mt), row(ldm(cur, MU + sp, lane), G)));
    else
        stm(cur, mr1(a, h, sp), lane, prop_col(prop(k - lc(mom4(mom, e, 3)), mt), col(G, ldm(cur, MS + sp, lane))));
}
// --- level 3: three-gluon currents, both independent orderings (y < 80), and two-gluon strings
// (160 of the quark, 160 of the antiquark)
__global__ __launch_bounds__(256) void level3(const double* __restrict__ mom, int64_t n_evt, double mt,
                                              v2d* __restrict__ cur_)
{
    const unsigned wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t e0 = (int64_t)blockIdx.x * 256 + 64 * wave, e = e0 + lane;
    v2d* const cur = block_of(cur_, e0);
    int q = blockIdx.y;
    if (e >= n_evt) return;
    if (q < 80) {
        const Subset s = triple_at(q >> 3);
        const int x = s.g[0], y = s.g[1], z = s.g[2], hx = (q >> 2) & 1, hy = (q >> 1) & 1, hz = q & 1;
        if (x == 0 && hx) return;
        const V4 X = ldm(cur, m1(x, hx), lane), Y = ldm(cur, m1(y, hy), lane), Z = ldm(cur, m1(z, hz), lane);
        const V4 XY = ldm(cur, m2(pair_index(x, y), hx, hy), lane), XZ = ldm(cur, m2(pair_index(x, z), hx, hz), lane),
                 YZ = ldm(cur, m2(pair_index(y, z), hy, hz), lane);
        const K4 kx = kin(mom, e, x), ky = kin(mom, e, y), kz = kin(mom, e, z);
        const V4x2 o = three_currents(X, kx, Y, ky, Z, kz, XY, XZ, YZ);
        stm(cur, m3(q >> 3, hx, hy, hz, 0), lane, o.v[0]);
        stm(cur, m3(q >> 3, hx, hy, hz, 1), lane, o.v[1]);
        return;
    }
    q -= 80;
    const int right = q >= 160;
    q %= 160;
    const int o = q >> 3, a = o / 4, b = o % 4 < a ? o % 4 : o % 4 + 1, ha = (q >> 2) & 1, hb = (q >> 1) & 1, sp = q & 1;
    if ((a == 0 && ha) || (b == 0 && hb)) return;
    const int lo = a < b ? a : b, hi = a < b ? b : a;
    const V4 A = ldm(cur, m1(a, ha), lane), B = ldm(cur, m1(b, hb), lane);
    V4 AB = ldm(cur, m2(pair_index(lo, hi), a < b ? ha : hb, a < b ? hb : ha), lane);
    if (a > b) AB = -AB;
    const K4 k = kin(mom, e, a) + kin(mom, e, b);
    if (!right) {   // the quark, then a, then b
        const V4 t = row_acc(row(ldm(cur, MU + sp, lane), AB), ldm(cur, ml1(a, ha, sp), lane), B);
        stm(cur, ml2(o, ha, hb, sp), lane, prop_row(prop(lc(mom4(mom, e, 2)) - k, mt), t));
    } else {        // a, then b, then the antiquark
        const V4 t = col_acc(col(AB, ldm(cur, MS + sp, lane)), A, ldm(cur, mr1(b, hb, sp), lane));
        stm(cur, mr2(o, ha, hb, sp), lane, prop_col(prop(k - lc(mom4(mom, e, 3)), mt), t));
    }
}
// --- level 4: four-gluon currents; y: the missing gluon and the helicities of the others
__global__ __launch_bounds__(64, 2) void level4(const double* __restrict__ mom, int64_t n_evt,
                                                v2d* __restrict__ cur_)
{
    const unsigned lane = threadIdx.x;
    const int64_t e0 = (int64_t)blockIdx.x * 64, e = e0 + lane;
    v2d* const cur = block_of(cur_, e0);
    // gluons 1 to 4 in all helicities, then those with gluon 0 (the first of them, at -)
    const int w = blockIdx.y < 16 ? 0 : (blockIdx.y - 8) >> 3, h4 = blockIdx.y < 16 ? blockIdx.y : blockIdx.y & 7;
    if (e >= n_evt) return;
    int g[4], h[4];
    for (int k = 0; k < 4; ++k) g[k] = rest(w, k), h[k] = (h4 >> (3 - k)) & 1;
    const auto j1 = [&](int i) { return ldm(cur, m1(g[i], h[i]), lane); };
    const auto j2 = [&](int i, int j) {
        const int a = min(i, j), b = max(i, j);
        const V4 v = ldm(cur, m2(pair_index(g[a], g[b]), h[a], h[b]), lane);
        return i < j ? v : -v;
    };
    const auto j3 = [&](int x, int y, int z) {
        const int a = min(x, min(y, z)), c = max(x, max(y, z)), b = x + y + z - a - c;
        const int s = m3(triple_index(g[a], g[b], g[c]), h[a], h[b], h[c], 0);
        return three_ordered(x, y, z, [&] { return ldm(cur, s, lane); }, [&] { return ldm(cur, s + 1, lane); });
    };
    K4 k[4];
    for (int i = 0; i < 4; ++i) k[i] = kin(mom, e, g[i]);
    const double f = -rcp(sq(k[0] + k[1] + k[2] + k[3]));
    static_for<6>([&](auto R) {
        constexpr Perm<3> s = perm_at<3>(R);
        stm(cur, m4(w, h4, R), lane, f * four_numerator(s.p[0] + 1, s.p[1] + 1, s.p[2] + 1, j1, j2, j3, k[0], k[s.p[0] + 1],
                                                         k[s.p[1] + 1], k[s.p[2] + 1]));
    });
}

// the currents of one helicity configuration in LDS: one to three gluons
constexpr int S1 = 0, S2 = 5, S3 = 15, NS = 35;
__device__ __forceinline__ void stage_currents(const v2d* __restrict__ cur, int bits, double* lds, int lane, int wave)
{
    static_for<NS>([&](auto I) {
        constexpr int s = I;
        if (s % 4 != wave) return;
        if constexpr (s < S2) {
            st_v(lds, s, lane, ldm(cur, m1(s, bit(bits, s)), lane));
        } else if constexpr (s < S3) {
            constexpr Subset p = pair_at(s - S2);
            st_v(lds, s, lane, ldm(cur, m2(s - S2, bit(bits, p.g[0]), bit(bits, p.g[1])), lane));
        } else {
            constexpr int t = (s - S3) / 2;
            constexpr Subset p = triple_at(t);
            st_v(lds, s, lane, ldm(cur, m3(t, bit(bits, p.g[0]), bit(bits, p.g[1]), bit(bits, p.g[2]), (s - S3) % 2), lane));
        }
    });
    __syncthreads();
}
// J(x, y, z) of distinct gluons in any order, and J(x, y), from LDS
template <int X, int Y, int Z>
__device__ __forceinline__ V4 lds3(const double* lds, int lane)
{
    constexpr int lo = X < Y ? (X < Z ? X : Z) : (Y < Z ? Y : Z), hi = X > Y ? (X > Z ? X : Z) : (Y > Z ? Y : Z),
                  mid = X + Y + Z - lo - hi, s = S3 + 2 * triple_index(lo, mid, hi);
    if constexpr (Y == mid) return ld_v(lds, s, lane);                    // (lo mid hi) and its reverse
    else if constexpr (Y == hi) return ld_v(lds, s + 1, lane);            // (lo hi mid) and its reverse
    else return -(ld_v(lds, s, lane) + ld_v(lds, s + 1, lane));
}
template <int X, int Y>
__device__ __forceinline__ V4 lds2(const double* lds, int lane)
{
    if constexpr (X < Y) return ld_v(lds, S2 + pair_index(X, Y), lane);
    else return -ld_v(lds, S2 + pair_index(Y, X), lane);
}

// --- J(0 s) of all five gluons contracted with the quark current of each spin configuration:
// five[h][2 r + re/im][event], r the ordering s of gluons 1 .. 4.  One workgroup: 64 events, one
// gluon configuration; wave w takes the six orderings that begin with gluon w + 1.
__global__ __launch_bounds__(256, 1) void five_currents(const double* __restrict__ mom, int64_t n_evt,
                                                        const int* __restrict__ cfg, int n_cfg,
                                                        const v2d* __restrict__ cur_, int n_rows, v2d* __restrict__ five)
{
    __shared__ double lds[NS * 512];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t w = xcd_remap(blockIdx.x, gridDim.x);
    const int64_t e0 = (w / n_cfg) * 64, e = e0 + lane;
    const v2d* const cur = block_of(cur_, e0);
    const int* const rc_ = cfg + (w % n_cfg) * 5;
    const int bits = rc_[0];
    stage_currents(cur, bits, lds, lane, wave);
    const int64_t ec = e < n_evt ? e : n_evt - 1;
    K4 k[NG];
    for (int i = 0; i < NG; ++i) k[i] = kin(mom, ec, i);
    const double f = -rcp(sq(k[0] + k[1] + k[2] + k[3] + k[4]));
    V4 q[4];
    {
        const V4 U0 = ldm(cur, MU, lane), U1 = ldm(cur, MU + 1, lane), W0 = ldm(cur, MS, lane), W1 = ldm(cur, MS + 1, lane);
        q[0] = f * pair(U0, W0), q[1] = f * pair(U0, W1), q[2] = f * pair(U1, W0), q[3] = f * pair(U1, W1);
    }
    static_for<24>([&](auto R_) {
        constexpr int r = R_;
        constexpr Perm<4> s = perm_at<4>(r);
        constexpr int b = s.p[0] + 1, c = s.p[1] + 1, d = s.p[2] + 1, g = s.p[3] + 1;
        if (b - 1 != wave) return;
        // in four stages, so that few of the vectors it reads are held at a time
        const auto one = [&](auto I) { return ld_v(lds, S1 + I, lane); };
        constexpr std::integral_constant<int, 0> i0;
        constexpr std::integral_constant<int, b> ib;
        constexpr std::integral_constant<int, c> ic;
        constexpr std::integral_constant<int, d> id;
        constexpr std::integral_constant<int, g> ig;
        const K4 kab = k[0] + k[b], kdg = k[d] + k[g], kcdg = k[c] + kdg;
        V4 o;
        {   // (0 | b c d g): four gluons without 0, from the orderings that begin with 1
            V4 X = zero4();
            const int h4 = bits_without(bits, 0);
            static_for<6>([&](auto K) {
                constexpr int cf = kk_table<4>.c[r][K];
                if constexpr (cf == 1) X = X + ldm(cur, m4(0, h4, K), lane);
                if constexpr (cf == -1) X = X - ldm(cur, m4(0, h4, K), lane);
            });
            const V4 A = one(i0);
            o = vvv_acc(zero4(), A, k[0], X, k[b] + kcdg, dot2(A, X));
            pin_v(o);
        }
        {   // (0 b | c d g), (0 | b | c d g)
            const V4 A = one(i0), B = one(ib), AB = lds2<0, b>(lds, lane), X = lds3<c, d, g>(lds, lane);
            o = vvv_acc(o, AB, kab, X, kcdg, dot2(AB, X));
            o = vvvv_acc(o, A, B, X, dot2(A, B), dot2(B, X), dot2(A, X));
            pin_v(o);
        }
        {   // (0 b c | d g), (0 | b c | d g), (0 b | c | d g)
            const V4 A = one(i0), Cc = one(ic), AB = lds2<0, b>(lds, lane), BC = lds2<b, c>(lds, lane),
                     X = lds2<d, g>(lds, lane), ABC = lds3<0, b, c>(lds, lane);
            o = vvv_acc(o, ABC, kab + k[c], X, kdg, dot2(ABC, X));
            o = vvvv_acc(o, A, BC, X, dot2(A, BC), dot2(BC, X), dot2(A, X));
            o = vvvv_acc(o, AB, Cc, X, dot2(AB, Cc), dot2(Cc, X), dot2(AB, X));
            pin_v(o);
        }
        {   // (0 b c d | g), (0 | b c d | g), (0 b | c d | g), (0 b c | d | g)
            const V4 G = one(ig), ABCD = ldm(cur, m4(g, bits_without(bits, g), rank3(b, c, d)), lane);
            o = vvv_acc(o, ABCD, kab + k[c] + k[d], G, k[g], dot2(ABCD, G));
            const V4 A = one(i0), D = one(id), AB = lds2<0, b>(lds, lane), CD = lds2<c, d>(lds, lane),
                     ABC = lds3<0, b, c>(lds, lane), BCD = lds3<b, c, d>(lds, lane);
            o = vvvv_acc(o, A, BCD, G, dot2(A, BCD), dot2(BCD, G), dot2(A, G));
            o = vvvv_acc(o, AB, CD, G, dot2(AB, CD), dot2(CD, G), dot2(AB, G));
            o = vvvv_acc(o, ABC, D, G, dot2(ABC, D), dot2(D, G), dot2(ABC, G));
        }
        pin_v(o);
        static_for<4>([&](auto SP) {
            const int h = rc_[1 + SP];
            if (h < 0) return;
            const C x = rc(q[SP], o);
            (five + ((e0 >> 6) * n_rows + h) * (int64_t)(24 * 64) + 64 * r)[(unsigned)lane] = v2d{x.r, x.i};
        });
    });
}

// --- the flows.  One workgroup: 64 events, one gluon configuration, the four quark spin
// configurations in its four waves, which share the currents of up to three gluons in LDS.
__global__ __launch_bounds__(256, 1) void amp_rec(int64_t n_evt, int64_t ld, const int* __restrict__ cfg, int n_cfg,
                                                  const v2d* __restrict__ cur_, int n_rows, const v2d* __restrict__ five,
                                                  double* __restrict__ jamp)
{
    __shared__ double lds[NS * 512];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t w = xcd_remap(blockIdx.x, gridDim.x);
    const int64_t e0 = (w / n_cfg) * 64, e = e0 + lane;
    const v2d* const cur = block_of(cur_, e0);
    const int* const rc_ = cfg + (w % n_cfg) * 5;
    const int bits = rc_[0], h = rc_[1 + wave], su = wave >> 1, sv = wave & 1;
    stage_currents(cur, bits, lds, lane, wave);
    if (h < 0) return;
    const v2d* src = cur;
    const auto J1 = [&](int i) { return ld_v(lds, S1 + i, lane); };
    const auto L1 = [&](int a) { return ldm(src, ml1(a, bit(bits, a), su), lane); };
    const auto R1 = [&](int a) { return ldm(src, mr1(a, bit(bits, a), sv), lane); };
    const auto L2 = [&](int a, int b) { return ldm(src, ml2(ordered(a, b), bit(bits, a), bit(bits, b), su), lane); };
    const auto R2 = [&](int a, int b) { return ldm(src, mr2(ordered(a, b), bit(bits, a), bit(bits, b), sv), lane); };
    const V4 U = ldm(cur, MU + su, lane), S = ldm(cur, MS + sv, lane);
    // the quark takes gluon x, the antiquark the current of the other four
    C D3[NG][6];
    static_for<NG>([&](auto X) {
        src = fresh(cur);
        const V4 c = pair(L1(X), S);
        const int h4 = bits_without(bits, X);
        static_for<6>([&](auto R) { D3[X][R] = rc(c, ldm(src, m4(X, h4, R), lane)); });
        static_for<6>([&](auto R) { pin_cx(D3[X][R]); });
    });
    // per last gluon: the contractions of all five, the string R1 and the currents of the others, read
    // before the stores of the flows before, which the waits for later reads would include
    C D4[24];
    V4 Rn, q4[6];
    const auto read_ahead = [&](int g) {
        src = fresh(cur);
        const v2d* f5 = fresh(five) + ((e0 >> 6) * n_rows + h) * (int64_t)(24 * 64);
        static_for<24>([&](auto R) {
            const v2d t = (f5 + 64 * R)[(unsigned)lane];
            D4[R] = {t.x, t.y};
        });
        Rn = R1(g);
        const int h4 = bits_without(bits, g);
        static_for<6>([&](auto R) { q4[R] = ldm(src, m4(g, h4, R), lane); });
    };
    read_ahead(0);
    // the 24 flows that end with gluon g; J[rank of the others' order]
    static_for<NG>([&](auto G_) {
        constexpr int g = G_;
        C J[24];
        src = fresh(cur);
        {   // all five gluons in one current
            static_for<24>([&](auto F) {
                constexpr int r5 = flow_with_last(g, F);
                J[F] = {0.0, 0.0};
                static_for<24>([&](auto R) {
                    constexpr int c = kk_table<5>.c[r5][R];
                    if constexpr (c == 1) J[F] = J[F] + D4[R];
                    if constexpr (c == -1) J[F] = J[F] - D4[R];
                });
            });
        }
        const V4 Rg = Rn;
        V4 rn, lh[4];
        {   // four gluons next to the quark, the last one at the antiquark
            src = fresh(cur);
            rn = R2(rest(g, 0), g);
            static_for<4>([&](auto M) { lh[M] = L1(rest(g, M)); });
            const V4 c = pair(U, Rg);
            C s[6];
            static_for<6>([&](auto R) { s[R] = rc(c, q4[R]); });
            static_for<24>([&](auto F) {
                // and four next to the antiquark: (a | b c d g)
                constexpr int a = rest(g, perm_at<4>(F).p[0]), r4 = last_four(g, F);
                static_for<6>([&](auto R) {
                    constexpr int c1 = kk_table<4>.c[F][R], c2 = kk_table<4>.c[r4][R];
                    if constexpr (c1 == 1) J[F] = J[F] + s[R];
                    if constexpr (c1 == -1) J[F] = J[F] - s[R];
                    if constexpr (c2 == 1) J[F] = J[F] + D3[a][R];
                    if constexpr (c2 == -1) J[F] = J[F] - D3[a][R];
                });
                pin_cx(J[F]);
            });
        }
        // one gluon (local label m) at an end of the block, three in a current
        static_for<4>([&](auto M) {
            constexpr int m = M, x = m == 0 ? 1 : 0, y = m <= 1 ? 2 : 1, z = m <= 2 ? 3 : 2;
            constexpr int a = rest(g, m);
            constexpr int t = triple_index(rest(g, x), rest(g, y), rest(g, z));
            const V4 G0 = ld_v(lds, S3 + 2 * t, lane), G1 = ld_v(lds, S3 + 2 * t + 1, lane);
            const V4 Rag = rn;
            if constexpr (m < 3) {
                src = fresh(cur);
                rn = R2(rest(g, m < 3 ? m + 1 : 0), g);
            }
            const V4 cl = pair(lh[m], Rg), cr = pair(U, Rag);
            const C l0 = rc(cl, G0), l1 = rc(cl, G1), r0 = rc(cr, G0), r1 = rc(cr, G1), l2 = l0 + l1, r2 = r0 + r1;
            // (a | x y z | g) and (x y z | a g)
            constexpr int f0 = rank4(m, x, y, z), f1 = rank4(m, z, y, x), f2 = rank4(m, x, z, y), f3 = rank4(m, y, z, x),
                          f4 = rank4(m, y, x, z), f5_ = rank4(m, z, x, y), q0 = rank4(x, y, z, m), q1 = rank4(z, y, x, m),
                          q2 = rank4(x, z, y, m), q3 = rank4(y, z, x, m), q4 = rank4(y, x, z, m), q5 = rank4(z, x, y, m);
            J[f0] = J[f0] + l0, J[f1] = J[f1] + l0, J[f2] = J[f2] + l1, J[f3] = J[f3] + l1, J[f4] = J[f4] - l2,
            J[f5_] = J[f5_] - l2;
            J[q0] = J[q0] + r0, J[q1] = J[q1] + r0, J[q2] = J[q2] + r1, J[q3] = J[q3] + r1, J[q4] = J[q4] - r2,
            J[q5] = J[q5] - r2;
            // (i | j k | a g): the quark takes i, a two-gluon current, the antiquark the string (a g)
            static_for<3>([&](auto I_) {
                constexpr int i = I_ == 0 ? x : I_ == 1 ? y : z, j = I_ == 0 ? y : x, k = I_ == 2 ? y : z;
                const C s = rc(lh[i], col(lds2<rest(g, j), rest(g, k)>(lds, lane), Rag));
                constexpr int u0 = rank4(i, j, k, m), u1 = rank4(i, k, j, m);
                J[u0] = J[u0] + s;
                J[u1] = J[u1] - s;
            });
            static_for<24>([&](auto F) {
                constexpr Perm<4> q = perm_at<4>(F);
                if constexpr (q.p[0] == m || q.p[3] == m) pin_cx(J[F]);
            });
        });
        V4 pf[4];
        src = fresh(cur);
        pf[0] = R2(rest(g, 3), g), pf[1] = R2(rest(g, 2), g), pf[2] = L2(rest(g, 0), rest(g, 1)), pf[3] = L2(rest(g, 1), rest(g, 0));
        // two gluons at the quark, the others at the antiquark: (a b | c d g)
        static_for<6>([&](auto P_) {
            constexpr int pi[6] = {0, 0, 0, 1, 1, 2}, pj[6] = {1, 2, 3, 2, 3, 3};
            constexpr int a = pi[P_], b = pj[P_], c = pi[5 - P_], d = pj[5 - P_];
            constexpr int ga = rest(g, a), gb = rest(g, b), gc = rest(g, c), gd = rest(g, d);
            const V4 rd = pf[0], rc_ = pf[1], Lab = pf[2], Lba = pf[3];
            if constexpr (P_ < 5) {
                constexpr int n = P_ < 5 ? P_ + 1 : 0;
                src = fresh(cur);
                pf[0] = R2(rest(g, pj[5 - n]), g), pf[1] = R2(rest(g, pi[5 - n]), g);
                pf[2] = L2(rest(g, pi[n]), rest(g, pj[n])), pf[3] = L2(rest(g, pj[n]), rest(g, pi[n]));
            }
            const V4 y = col(lds2<gc, gd>(lds, lane), Rg);
            const V4 Rcd = col_acc(col_acc(y, J1(gc), rd), lds3<gc, gd, g>(lds, lane), S);
            const V4 Rdc = col_acc(col_acc(-y, J1(gd), rc_), lds3<gd, gc, g>(lds, lane), S);
            constexpr int f0 = rank4(a, b, c, d), f1 = rank4(a, b, d, c), f2 = rank4(b, a, c, d), f3 = rank4(b, a, d, c);
            J[f0] = rc_acc(J[f0], Lab, Rcd);
            J[f1] = rc_acc(J[f1], Lab, Rdc);
            J[f2] = rc_acc(J[f2], Lba, Rcd);
            J[f3] = rc_acc(J[f3], Lba, Rdc);
            pin_cx(J[f0]), pin_cx(J[f1]), pin_cx(J[f2]), pin_cx(J[f3]);
        });
        if constexpr (g + 1 < NG) read_ahead(g + 1);
        if (e < n_evt) {
            double* const o = jamp + (int64_t)h * (2 * NC) * ld + e0;
            static_for<24>([&](auto F) {
                constexpr int r5 = flow_with_last(g, F);
                __builtin_nontemporal_store(J[F].r, (o + (2 * r5) * ld) + (unsigned)lane);
                __builtin_nontemporal_store(J[F].i, (o + (2 * r5 + 1) * ld) + (unsigned)lane);
            });
        }
    });
}

int64_t aux_doubles(int n_rows) { return 8 * (int64_t)MEND + 48 * (int64_t)n_rows; }

hipError_t launch(const double* mom, int64_t n_evt, int64_t ld, const HelicityGroups& hg, double mt, double gs,
                  double* jamp, hipStream_t st)
{
    if (n_evt == 0 || hg.n == 0) return hipSuccess;
    // after the jamps: the currents and strings of the events, then the five-gluon contractions
    v2d* const cur = reinterpret_cast<v2d*>(jamp + (int64_t)hg.n_rows * 2 * NC * ld);
    v2d* const five = cur + (int64_t)4 * MEND * ld;
    const unsigned nb = (unsigned)((n_evt + 255) / 256), n64 = (unsigned)((n_evt + 63) / 64);
    hipLaunchKernelGGL(level1, dim3(nb, NG + 2), dim3(256), 0, st, mom, n_evt, mt, gs, cur);
    hipLaunchKernelGGL(level2, dim3(nb, 40 + 40), dim3(256), 0, st, mom, n_evt, mt, cur);
    hipLaunchKernelGGL(level3, dim3(nb, 80 + 320), dim3(256), 0, st, mom, n_evt, mt, cur);
    hipLaunchKernelGGL(level4, dim3(n64, 16 + 4 * 8), dim3(64), 0, st, mom, n_evt, cur);
    hipLaunchKernelGGL(five_currents, dim3(n64 * hg.n), dim3(256), 0, st, mom, n_evt, hg.table, hg.n, cur, hg.n_rows, five);
    hipLaunchKernelGGL(amp_rec, dim3(n64 * hg.n), dim3(256), 0, st, n_evt, ld, hg.table, hg.n, cur, hg.n_rows, five, jamp);
    return hipGetLastError();
}
}  // namespace rec5
}  // namespace me
