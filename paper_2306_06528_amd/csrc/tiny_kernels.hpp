// The whole step in one launch, for problems so small that three dependent launches cost more
// than the work: a single workgroup computes the pair sums, the bandwidth, K and the update
// (passes 1 to 3 of the larger path, same arithmetic) with barriers in between instead of kernel
// boundaries.  Worth it only while one compute unit can stream X and G in about the time a launch
// takes, hence the size limit.  512 threads: at most two 4-column groups per thread, and 256
// registers per lane for the accumulators.
#pragma once
#include "bandwidth_kernels.hpp"
#include "gram_kernels.hpp"

namespace svgd {

constexpr int kTinyMaxN = 8; // the direct-difference format; larger n start to spill registers
constexpr int64_t kTinyMaxElems = 16384; // n * D
constexpr int kTinyThreads = 512;

enum TinyWhat : int {
    kTinyStep = 0,     // X updated in place
    kTinyPhi = 1,      // phi written to PHI, X untouched
    kTinyBandwidth = 2 // passes 1 and 2 only: h, K and the tables (same sums, hence the same h)
};

template <int N, int WHAT>
__global__ __launch_bounds__(kTinyThreads) void step_tiny_kernel(float *__restrict__ X,
                                                               const float *__restrict__ G,
                                                               float *__restrict__ PHI, int64_t D, int64_t ld,
                                                               float eps, double h_fixed, double log_n1,
                                                               DevState *__restrict__ st,
                                                               float *__restrict__ coef)
{
    static_assert(N <= kTinyMaxN, "direct differences only");
    constexpr int P = N * (N + 1) / 2;
    __shared__ WaveShared<N> shw[kTinyThreads / 64];
    __shared__ float red[kTinyThreads / 64][P];
    const int tid = threadIdx.x;
    const int64_t ngroups = (D + 3) >> 2;

    // pass 1: pair sums over the columns in the format of gram_valu_kernel<N>, lanes = 4-column groups.  A
    // thread's first group stays in registers, its scores are fetched beside it.
    float acc[P];
#pragma unroll
    for (int p = 0; p < P; ++p) acc[p] = 0.f;
    f32x4 x[N], g[N];
    auto load = [&](f32x4 (&v)[N], const float *A, int64_t col) __attribute__((always_inline)) {
        const RaggedGroup rg(col, D);
#pragma unroll
        for (int j = 0; j < N; ++j) v[j] = D >= 4 ? rg.load<false>(A + (int64_t)j * ld) : load_narrow(A + (int64_t)j * ld, D);
    };
    auto fix = [&](f32x4 (&v)[N], int64_t col) __attribute__((always_inline)) {
        const RaggedGroup rg(col, D);
        if (rg.s) {
#pragma unroll
            for (int j = 0; j < N; ++j) v[j] = rg.fix(v[j]);
        }
    };
    if (tid < ngroups) {
        load(x, X, (int64_t)tid << 2);
        if constexpr (WHAT != kTinyBandwidth) load(g, G, (int64_t)tid << 2);
        fix(x, (int64_t)tid << 2);
        pair_accumulate<N>(x, acc);
    }
    for (int64_t grp = tid + kTinyThreads; grp < ngroups; grp += kTinyThreads) {
        f32x4 y[N];
        load(y, X, grp << 2);
        fix(y, grp << 2);
        pair_accumulate<N>(y, acc);
    }
    wave_sums<P>(acc, red[tid >> 6]);
    block_sync<true>();

    // pass 2
    WaveShared<N> &sh = shw[tid >> 6];
    const float c2h = wave_kernel_matrix<N>(sh, h_fixed, log_n1, st, coef, tid < kWave, [&](int e) __attribute__((always_inline)) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < kTinyThreads / 64; ++w) s += (double)red[w][e];
        return s;
    });

    if constexpr (WHAT == kTinyBandwidth) return;

    // pass 3: every thread updates the columns it summed, so in place is safe
    for (int64_t grp = tid; grp < ngroups; grp += kTinyThreads) {
        const int64_t col = grp << 2;
        const bool full = (col + 4 <= D);
        if (grp >= kTinyThreads) {
            load(x, X, col);
            load(g, G, col);
            fix(x, col);
        }
        fix(g, col);
        const int c0 = opaque_zero();
        f32x4 z[N];
#pragma unroll
        for (int j = 0; j < N; ++j) z[j] = g[j] - c2h * x[j];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            float C[N], rho;
            sh.row(i, c0, C, rho);
            f32x4 a = rho * x[i];
#pragma unroll
            for (int j = 0; j < N; ++j) a += C[j] * z[j];
            if constexpr (WHAT == kTinyPhi)
                store4(PHI + (int64_t)i * ld, col, D, full, a);
            else
                store4(X + (int64_t)i * ld, col, D, full, x[i] + eps * a);
        }
    }
}

} // namespace svgd
