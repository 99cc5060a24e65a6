// Multi-SWAG running moments (paper Sec. 2: SWAG keeps the first and second moments of a network's
// parameter trajectory; multi-SWAG does so for every particle).  One more iterate X is absorbed
// into the running means of all n*D parameters after `count` earlier updates:
//     mean <- (count*mean + x)/(count+1),   sq <- (count*sq + x*x)/(count+1)
// evaluated in the incremental form m += (x - m)/(count+1), which does not lose accuracy as count
// grows; the first update (count = 0) copies x and x*x, whatever the arrays held before.  A pure
// streaming kernel: 12 bytes read and 8 written per parameter.
#pragma once
#include "common.hpp"

namespace svgd {

// BIG, for arrays beyond the memory-side cache: four 4-float groups per thread and iteration, twelve
// loads in flight, all of them streaming, and one workgroup per CU.  What bounds the pass there is
// the memory system's handling of three read and two write streams, and it likes few waves with many
// loads each: 5.7 TB/s, where eight workgroups per CU with one group per thread reach 4.9 (n D =
// 64,000,048: 259 -> 225 us, 357,566,784: 1489 -> 1262) and five quarters of a workgroup per CU 4.6.
// Arrays that cache holds are read plainly by the many waves instead (n D = 4,800,112: 16.7 us, 19.8 as BIG).
template <bool BIG>
__global__ __launch_bounds__(256) void swag_moments_kernel(float *__restrict__ mean,
                                                           float *__restrict__ sq,
                                                           const float *__restrict__ X,
                                                           int64_t total, float inv, bool first)
{
    // all three arrays are only 4-byte aligned in general; 16-byte accesses need no more than that
    constexpr int U = BIG ? 4 : 1;
    const int64_t ngroups = (total + 3) >> 2;
    const int64_t nthreads = (int64_t)gridDim.x * 256;
    for (int64_t grp = (int64_t)blockIdx.x * 256 + threadIdx.x; grp < ngroups; grp += U * nthreads) {
        f32x4 x[U], m[U], s[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t e = (grp + u * nthreads) << 2; // past the end: nothing is read, nothing stored
            const bool full = (e + 4 <= total);
            x[u] = load4_stream(X, e, total, full);
            m[u] = BIG ? load4_stream(mean, e, total, full) : load4(mean, e, total, full);
            s[u] = BIG ? load4_stream(sq, e, total, full) : load4(sq, e, total, full);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t e = (grp + u * nthreads) << 2;
            const bool full = (e + 4 <= total);
            if (first) {
                m[u] = x[u];
                s[u] = x[u] * x[u];
            } else {
                m[u] += (x[u] - m[u]) * inv;
                s[u] += (x[u] * x[u] - s[u]) * inv;
            }
            store4(mean, e, total, full, m[u]);
            store4(sq, e, total, full, s[u]);
        }
    }
}

} // namespace svgd
