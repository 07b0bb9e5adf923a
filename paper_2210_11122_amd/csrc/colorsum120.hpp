// colorsum120.hpp -- the FP64 colour sum of 120 flows (gg -> tt~ggg) from the jamps in memory.
#pragma once
#include "colorsum.hpp"

namespace me {

// 120 flows: bound by reading the jamps (1920 B per (event, helicity)).  One workgroup: 64 events;
// its four waves are the real and imaginary rows times the two signs chi01.  The rows are read five
// orbits (20 rows) at a time, one group ahead of its use, past the caches (each is read by two waves
// of one workgroup only): 4096 events x 128 helicities 253 us, 4.0 TB/s; 388 us where the compiler
// placed the reads, which kept few of them in flight, and 333 us with six orbits (spills).
template <int C01>
__device__ __forceinline__ double colour_sign_pair_120(const double* __restrict__ Jh, int64_t ld, unsigned col)
{
    constexpr int NO = FlowBlocks<5>::NO, STEP = 5;
    double y0[NO], y1[NO], m[2][STEP][4];
    const auto read = [&](auto G, double (&d)[STEP][4]) {
        static_for<STEP>([&](auto I) {
            static_for<4>([&](auto K) {
                constexpr int f = flow_blocks<5>.member[G * STEP + I][K % 2][K / 2];
                d[I][K] = __builtin_nontemporal_load(&(Jh + (int64_t)(2 * f) * ld)[col]);
            });
        });
    };
    read(std::integral_constant<int, 0>{}, m[0]);
    static_for<NO / STEP>([&](auto G) {
        if constexpr (G + 1 < NO / STEP) read(std::integral_constant<int, G + 1>{}, m[(G + 1) % 2]);
        static_for<STEP>([&](auto I) {
            double(&d)[4] = m[G % 2][I];
            // the group ahead is read before this one is waited for
            asm volatile("" : "+v"(d[0]), "+v"(d[1]), "+v"(d[2]), "+v"(d[3]) : : "memory");
            y0[G * STEP + I] = orbit_sum<2 * C01>(d[0], d[1], d[2], d[3]);
            y1[G * STEP + I] = orbit_sum<2 * C01 + 1>(d[0], d[1], d[2], d[3]);
        });
    });
    return sign_blocks<5, 2 * C01>(y0) + sign_blocks<5, 2 * C01 + 1>(y1);
}
static __global__ __launch_bounds__(256, 2) void colour_sum_f64_120(
    const double* __restrict__ J, int64_t ld, int n_good, int hel_per_group, int64_t n_evt, double scale_hel,
    double scale_avg, double* __restrict__ out, double* __restrict__ out_hel, double* __restrict__ part,
    const int2* __restrict__ members, int n_hel)
{
    __shared__ double red[2][3][64];
    const unsigned lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t e0 = (int64_t)blockIdx.x * 64, e = e0 + lane;
    // lanes past the batch read the last event's column
    const unsigned col = (e < n_evt ? lane : (unsigned)(n_evt - 1 - e0)) & 63;
    const int h0 = blockIdx.y * hel_per_group, h1 = min(n_good, h0 + hel_per_group);
    double me = 0.0;
    for (int h = h0; h < h1; ++h) {
        const double* Jh = J + ((int64_t)h * 240 + (wave >> 1)) * ld + e0;
        int64_t stride = ld;
        asm volatile("" : "+s"(stride));   // the row offsets are formed here, not kept over the loop (and spilled)
        const double q = wave & 1 ? colour_sign_pair_120<1>(Jh, stride, col) : colour_sign_pair_120<0>(Jh, stride, col);
        if (wave > 0) red[h & 1][wave - 1][lane] = q;
        __syncthreads();
        if (wave == 0) {   // the other buffer is free for the next helicity until the next barrier
            const double me_h = ((q + red[h & 1][0][lane]) + (red[h & 1][1][lane] + red[h & 1][2][lane])) * (1.0 / 64.0);
            if (out_hel && e < n_evt) store_hel(out_hel + e * n_hel, members, h, me_h * scale_hel);
            me += members_of(members, h) * me_h;
        }
    }
    if (wave == 0 && e < n_evt) cs_store(me, e, n_evt, scale_avg, out, part);
}

}  // namespace me
