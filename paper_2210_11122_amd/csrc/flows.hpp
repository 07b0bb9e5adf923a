// flows.hpp -- compile-time tables of the colour flows of a quark line with NG gluons: the
// orderings in the order of the jamps (lexicographic), the expansion of a colour-ordered gluon
// current in a basis, and the involutions that block-diagonalise the colour matrix.
#pragma once
#include <hip/hip_runtime.h>

#include <utility>

namespace me {

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>): a loop whose index is a
// constant in every pass, so that arrays indexed by it stay in registers
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

__host__ __device__ constexpr int factorial(int n) { return n < 2 ? 1 : n * factorial(n - 1); }

// the k-th permutation of 0..N-1 in lexicographic order, and the rank of a permutation
template <int N>
struct Perm {
    int p[N] = {};
};
template <int N>
__host__ __device__ constexpr Perm<N> perm_at(int k)
{
    Perm<N> out{};
    bool used[N] = {};
    int f = factorial(N - 1);
    for (int i = 0; i < N; ++i) {
        int r = k / f;
        k %= f;
        if (i + 1 < N) f /= N - 1 - i;
        for (int v = 0; v < N; ++v) {
            if (used[v]) continue;
            if (r-- == 0) {
                out.p[i] = v;
                used[v] = true;
                break;
            }
        }
    }
    return out;
}
template <int N>
__host__ __device__ constexpr int perm_rank(const Perm<N>& x)
{
    int k = 0;
    for (int i = 0; i < N; ++i) {
        int c = 0;
        for (int j = i + 1; j < N; ++j) c += x.p[j] < x.p[i];
        k += c * factorial(N - 1 - i);
    }
    return k;
}

// Colour-ordered gluon currents obey the Kleiss-Kuijf relations
//   J(A, 0, B) = (-1)^|A| sum over the shuffles s of (A reversed) with B of J(0, s),
// so (N - 1)! of the N! orderings of N gluons are independent: those that begin with the first
// gluon.  c[r][k]: coefficient of the k-th ordering of the other N - 1 in the r-th ordering.
template <int N>
struct KK {
    int c[factorial(N)][factorial(N - 1)] = {};
};
template <int N>
__host__ __device__ constexpr KK<N> make_kk()
{
    KK<N> out{};
    for (int r = 0; r < factorial(N); ++r) {
        const Perm<N> x = perm_at<N>(r);
        int at = 0;
        while (x.p[at] != 0) ++at;
        const int na = at;
        // every subset of positions for the reversed A among the N - 1 others
        for (int mask = 0; mask < (1 << (N - 1)); ++mask) {
            int bits = 0;
            for (int i = 0; i < N - 1; ++i) bits += (mask >> i) & 1;
            if (bits != na) continue;
            Perm<N - 1> s{};
            int ia = na - 1, ib = at + 1;
            for (int i = 0; i < N - 1; ++i) s.p[i] = (((mask >> i) & 1) ? x.p[ia--] : x.p[ib++]) - 1;
            out.c[r][perm_rank<N - 1>(s)] += (na & 1) ? -1 : 1;
        }
    }
    return out;
}
template <int N>
inline constexpr KK<N> kk_table = make_kk<N>();

// The colour matrix C of the orderings is unchanged by relabelling the gluons, (01) and (23)
// among them, and by reversing all orderings at once.  These three commuting involutions split
// the space of the flows into eight blocks between which C vanishes.  For signs chi01, chi23 of
// the relabellings,
//   y(O) = sum over the four relabellings g of chi(g) J(g rep(O)),
// O an orbit of the two relabellings, rep(O) its ordering with 0 before 1 and 2 before 3.
// Reversing rep(O) gives (01)(23) rep(O'), so for the sign rho of the reversal
//   z(O, O') = y(O) + rho chi01 chi23 y(O')  for O != O',
// and an orbit with O' = O belongs to the block with rho = chi01 chi23 alone, z = y(O).
// NG = 4: blocks of 4 and 2 (24 flows); NG = 5: blocks of 16 and 14 (120 flows).
template <int NG>
struct FlowBlocks {
    static constexpr int NC = factorial(NG), NO = NC / 4;
    int member[NO][2][2] = {};  // flow of orbit o, relabelled by (01) and / or (23)
    int n_pair = 0, n_fix = 0;
    int pair[NO][2] = {};  // orbits exchanged by the reversal
    int fix[NO] = {};      // orbits it leaves alone
};
template <int NG>
__host__ __device__ constexpr FlowBlocks<NG> make_blocks()
{
    FlowBlocks<NG> b{};
    int orbit_of[factorial(NG)] = {};
    int n = 0;
    for (int k = 0; k < factorial(NG); ++k) {
        const Perm<NG> x = perm_at<NG>(k);
        int at[NG] = {};
        for (int i = 0; i < NG; ++i) at[x.p[i]] = i;
        if (at[0] > at[1] || at[2] > at[3]) continue;
        for (int s = 0; s < 2; ++s)
            for (int t = 0; t < 2; ++t) {
                Perm<NG> y = x;
                if (s) y.p[at[0]] = 1, y.p[at[1]] = 0;
                if (t) y.p[at[2]] = 3, y.p[at[3]] = 2;
                b.member[n][s][t] = perm_rank<NG>(y);
                orbit_of[b.member[n][s][t]] = n;
            }
        ++n;
    }
    for (int o = 0; o < n; ++o) {
        const Perm<NG> x = perm_at<NG>(b.member[o][0][0]);
        Perm<NG> r{};
        for (int i = 0; i < NG; ++i) r.p[i] = x.p[NG - 1 - i];
        const int q = orbit_of[perm_rank<NG>(r)];
        if (q == o) b.fix[b.n_fix++] = o;
        if (q > o) b.pair[b.n_pair][0] = o, b.pair[b.n_pair][1] = q, ++b.n_pair;
    }
    return b;
}
template <int NG>
inline constexpr FlowBlocks<NG> flow_blocks = make_blocks<NG>();

}  // namespace me
