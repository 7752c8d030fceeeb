// Which kernel of gemm_f32.hip makes a product, and in how many parts along K. Plain C++: the choice needs no device.
#pragma once
#include <cstdint>

namespace dppo {

// 128-wide and 64-wide tiles, wavefront tiles (32-wide) of 4 and of 8 wavefronts
enum F32Kernel { F32_BIG = 0, F32_MID = 1, F32_DIRECT_4 = 2, F32_DIRECT_8 = 3, F32_KERNELS = 4 };
struct F32Plan { int kernel, parts; };

constexpr int F32_EDGE[F32_KERNELS] = {128, 64, 32, 32};          // tile edge
constexpr int F32_STEP_K[F32_KERNELS] = {32, 32, 32 * 4, 32 * 8}; // k-values of a step

// Least estimated time; parts: a power of two, where the scratch holds `room` partial results. A launch takes a start plus its K
// steps, one after the other; a step takes a latency, or, with many workgroups to a compute unit, their products' time; a split
// adds a launch that sums. The constants (us) are fitted to 2700 measured combinations (all three GEMMs; 20 to 2400 tokens, D = 64 to
// 1024, V = 500 to 32000; times within 13 % rms), and what is picked is on average 1.4 % slower than the fastest (20 % at
// worst, at 10 us).
inline F32Plan plan_gemm_f32(int32_t M, int32_t N, int32_t K, int64_t room, int cus) {
    struct Cost { double start, latency, step; };
    constexpr Cost cost[F32_KERNELS] = {{6.1, 2.0, 1.37}, {4.3, 1.13, 0.51}, {3.3, 1.18, 0.80}, {2.7, 1.9, 1.9}};
    auto div_up = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
    const double out_bytes = 4.0 * M * N;
    F32Plan best{F32_BIG, 1};
    double best_t = -1.0;
    for (int c = 0; c < F32_KERNELS; ++c) {
        const int64_t tiles = div_up(M, F32_EDGE[c]) * div_up(N, F32_EDGE[c]);
        for (int q = 1; q == 1 || (q <= room && q <= 256 && 32 * (q / 2) < K); q *= 2) {
            const double steps = (double)div_up(div_up(K, q), F32_STEP_K[c]), load = (double)div_up(tiles * q, cus) * cost[c].step;
            const double t = cost[c].start + steps * (load > cost[c].latency ? load : cost[c].latency) +
                             (q > 1 ? 3.2 + q * out_bytes / 3.1e6 : 0.0);
            if (best_t < 0.0 || t < best_t) { best_t = t; best = F32Plan{c, q}; }
        }
    }
    return best;
}

// Parts that the scratch of a dH GEMM is laid out for.
inline int gemm_f32_max_parts(int64_t K) {
    const int64_t p = K / 256;
    return (int)(p < 1 ? 1 : p > 16 ? 16 : p);
}

}  // namespace dppo
