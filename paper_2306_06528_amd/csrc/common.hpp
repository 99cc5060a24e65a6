// Shared device-side helpers and the layout of the handle's device state.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace svgd {

constexpr int kMaxN = 64;                              // particles
constexpr int kMaxPairsFull = kMaxN * (kMaxN + 1) / 2; // upper triangle with diagonal
constexpr int kWave = 64;
// n <= kValuMaxN runs on the vector ALU (one accumulator per pair in registers); larger n on the
// matrix cores, padded to a multiple of 16 rows.  Above 12 the register budget of the vector
// kernels (pair sums carried across steps included) no longer fits without spilling.
constexpr int kValuMaxN = 12;

typedef float f32x4 __attribute__((ext_vector_type(4)));
// rows of X start at i*D floats, so a 4-column group is only 4-byte aligned in general
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// Partial-sum formats written by the Gram kernels, both indexed by tri(i, j), i <= j.
enum GramMode : int {
    kModeDiff = 0, // entry (i<j) holds sum_k (x_ik - x_jk)^2; diagonal entries are 0
    kModeGram = 1  // entry (i<=j) holds sum_k y_ik y_jk of the column-centred y = x - mean_i x
};

__host__ __device__ inline int tri(int i, int j, int n) { return i * n - (i * (i - 1)) / 2 + (j - i); }

// Partial-sum vectors lie this many floats apart, so that every one starts on 16 bytes and is read
// four entries at a time (the up to three floats after the last entry are never used).
__host__ __device__ constexpr int pair_stride(int n) { return (n * (n + 1) / 2 + 3) & ~3; }

// Everything the update kernels need from the bandwidth kernel, in device memory.
struct DevState {
    double h;
    double med;
    float two_over_h;
    int n;
};

// Particles given as n separate rows (svgd_step_rows): where row i of X and of G starts, in floats
// relative to row 0 of the same array, and the misalignment of X's row i against a 128-byte line.
// Kernels compiled with ROWS = true take row addresses from this table instead of i * ld.
struct RowTable {
    int64_t x[kMaxN];
    int64_t g[kMaxN];
    int32_t ri[kMaxN]; // (address of X row i / 4) mod 32
    int32_t aligned;   // host side: every row of X and of G starts on a 128-byte boundary
};
// The table travels as a kernel argument (by value: nothing to allocate, copy or keep alive);
// kernels compiled with ROWS = false take this stand-in instead and never read it.
struct NoRows {
    int64_t x[1];
    int64_t g[1];
    int32_t ri[1];
    int32_t aligned;
};
template <bool ROWS> struct RowArg { typedef NoRows type; };
template <> struct RowArg<true> { typedef RowTable type; };

// Offsets (in floats) into the handle's coefficient block, which lies kStateBytes behind its DevState:
// h and K are one piece of memory, so that svgd_get_last is one copy.
//   K   [n*n]   K_ij (kept for svgd_get_last)
//   C   [n*n]   C_ij = K_ij / n
//   RHO [n]     rho_i = (2/h) * (sum_j K_ij) / n
constexpr int kStateBytes = 256;
static_assert(sizeof(DevState) <= kStateBytes, "state block");
constexpr int kOffK = 0;
constexpr int kOffC = kOffK + kMaxN * kMaxN;
constexpr int kOffRho = kOffC + kMaxN * kMaxN;
constexpr int kCoefFloats = kOffRho + kMaxN;

__device__ inline f32x4 load4(const float *__restrict__ row, int64_t col, int64_t D, bool full)
{
    if (full) return *reinterpret_cast<const f32x4u *>(row + col);
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (col + 0 < D) v.x = row[col + 0];
    if (col + 1 < D) v.y = row[col + 1];
    if (col + 2 < D) v.z = row[col + 2];
    if (col + 3 < D) v.w = row[col + 3];
    return v;
}

// streaming variant for data that is read exactly once
__device__ inline f32x4 load4_stream(const float *__restrict__ row, int64_t col, int64_t D, bool full)
{
    if (full) return __builtin_nontemporal_load(reinterpret_cast<const f32x4u *>(row + col));
    return load4(row, col, D, false);
}

// A row's 4-column groups, the last of which may be ragged, without a branch around any load: the group
// at column col is loaded at min(col, D - 4), always inside the row, and `fix` then moves what was
// loaded into place and sets the columns beyond D to 0 (a group wholly beyond D becomes 0).  With
// guarded loads of single columns the one wave that has the ragged group went through 4 N loads one
// after the other and was the last of its launch to end (n = 8, D = 100,003: 20.8 thousand
// cycles, all others 15).  Rows of fewer than four columns are one group and go through load_narrow,
// outside the loop over the groups: a choice inside it makes every load wait for the one before.
struct RaggedGroup {
    int64_t at; // column to load from
    int s;      // how far that is to the left of the group
    __device__ RaggedGroup(int64_t col, int64_t D)
    {
        at = D < 4 || col < D - 4 ? col : D - 4;
        s = (int)(col - at < 4 ? col - at : 4);
    }
    template <bool STREAM>
    __device__ f32x4 load(const float *__restrict__ row) const // rows of four columns or more
    {
        if constexpr (STREAM) return __builtin_nontemporal_load(reinterpret_cast<const f32x4u *>(row + at));
        else return *reinterpret_cast<const f32x4u *>(row + at);
    }
    __device__ f32x4 fix(f32x4 v) const
    {
        if (s & 1) v = f32x4{v.y, v.z, v.w, 0.f};
        if (s & 2) v = f32x4{v.z, v.w, 0.f, 0.f};
        if (s & 4) v = f32x4{0.f, 0.f, 0.f, 0.f};
        return v;
    }
};

// A row of fewer than four columns, the rest 0.
__device__ inline f32x4 load_narrow(const float *__restrict__ row, int64_t D)
{
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        v[e] = row[e < D ? e : 0];
        if (e >= D) v[e] = 0.f;
    }
    return v;
}

// How the column groups are dealt to the threads of a grid: thread t visits the groups t + k * stride,
// k < count(t).  Quotient and remainder of the number of groups come from the host: as a 64-bit division
// in every thread they took 0.3 us of each launch.
struct GroupSplit {
    int q, r;
    __host__ GroupSplit(int64_t ngroups, int64_t stride) : q((int)(ngroups / stride)), r((int)(ngroups % stride)) {}
    __device__ int count(int t) const { return q + (t < r ? 1 : 0); }
};

// Sum of v over the four lanes l, l ^ 16, l ^ 32, l ^ 48 (the four 16-lane rows of a wave), in every
// lane, as (v[l] + v[l ^ 16]) + (the same of l ^ 32): the gfx950 row-swap instructions exchange
// whole rows between two registers in the vector ALU, where a shuffle would go through LDS and
// make the wave wait for it twice.
__device__ inline float sum_over_rows(float v)
{
    const unsigned u = __float_as_uint(v);
    const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false); // rows 1 <-> 0 and 3 <-> 2 of the two copies
    const float s = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const unsigned w = __float_as_uint(s);
    const auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false); // rows 2, 3 <-> 0, 1
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// How the matrix-core passes share the nfull = D / 64 full 64-column tiles among nwg worker
// workgroups of four waves: either every wave owns a contiguous range [t0, t1) (stride 1), or the
// workgroup owns one and its waves take every fourth tile of it, t0, t0 + 4, ... < t1 (adjacent).
// The Gram pass and the update use the same split, so that one can start on the tiles the other
// touched last.  `per`, the tiles of a range, comes from the host: a 64-bit division by a workgroup that
// has nothing else to do yet.
__host__ inline int64_t tiles_per_range(int64_t nfull, int64_t nwg, bool adjacent)
{
    const int64_t ranges = adjacent ? nwg : nwg * 4;
    return (nfull + ranges - 1) / ranges;
}
__device__ inline void tile_range(int64_t nfull, int64_t per, int64_t wg, int wave, bool adjacent, int64_t &t0,
                                  int64_t &t1)
{
    if (adjacent) {
        const int64_t b0 = (wg * per < nfull) ? wg * per : nfull;
        t1 = (b0 + per < nfull) ? b0 + per : nfull;
        t0 = (b0 + wave < t1) ? b0 + wave : t1;
    } else {
        const int64_t w = wg * 4 + wave;
        t0 = (w * per < nfull) ? w * per : nfull;
        t1 = (t0 + per < nfull) ? t0 + per : nfull;
    }
}

// keeps the compiler from turning per-row addresses into 2 x 16 loop-carried pointer pairs
// (an integer offset is laundered, not the pointer, so the accesses stay global_load/store)
__device__ inline void opaque(int64_t &v) { asm volatile("" : "+v"(v)); }

// Between LDS writes and reads by which the lanes of one wave hand values to each other.  The wave's LDS operations
// execute in program order, so this costs no instruction: it keeps the compiler to that order.
__device__ inline void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
}

// rows that all start on a 128-byte boundary
__host__ inline bool rows_aligned(const void *base, int64_t ld)
{
    return (ld & 31) == 0 && (reinterpret_cast<uintptr_t>(base) & 127) == 0;
}

__device__ inline void store4(float *__restrict__ row, int64_t col, int64_t D, bool full, f32x4 v)
{
    if (full) {
        __builtin_nontemporal_store(v, reinterpret_cast<f32x4u *>(row + col));
        return;
    }
    if (col + 0 < D) row[col + 0] = v.x;
    if (col + 1 < D) row[col + 1] = v.y;
    if (col + 2 < D) row[col + 2] = v.z;
    if (col + 3 < D) row[col + 3] = v.w;
}

// Eight fp32 values as three bf16 operands of the matrix instructions: v = h + m + l EXACTLY - h is v
// rounded to bf16's eight bits, m the (exact) rest rounded, l what then remains, at most eight bits.
// A product of two such triples is hh + (hm + mh) + (mm + hl + lh) + terms below 2^-25 of it, whose
// signs are as random as those of rounding errors (the parts are rounded to nearest, not cut off).
// A pair's rests are one instruction each: a dot product of the packed pair with (-1, 0) or (0, -1),
// exact because the rest is representable; with shifts, masks and subtractions the split takes
// 5.5 instructions per value, so 3.5.  Finite values beyond 2^64 or so can overflow in products
// of different signs (h h and h m), which fp32 products do not: the caller looks at its sums.
struct SplitConst {
    unsigned neg_lo, neg_hi; // bf16 pairs (-1, 0) and (0, -1), in registers: as literals they would be broadcast
};
__device__ __forceinline__ SplitConst split_const()
{
    SplitConst c{0x0000BF80u, 0xBF800000u};
    asm volatile("" : "+s"(c.neg_lo), "+s"(c.neg_hi));
    return c;
}
struct Split3 {
    bf16x8 h, m, l;
};
__device__ __forceinline__ Split3 split3(f32x4 a, f32x4 b, const SplitConst &sc)
{
    const bf16x2 neg_lo = __builtin_bit_cast(bf16x2, sc.neg_lo), neg_hi = __builtin_bit_cast(bf16x2, sc.neg_hi);
    Split3 r;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        f32x2 v = k < 2 ? f32x2{a[2 * k], a[2 * k + 1]} : f32x2{b[2 * k - 4], b[2 * k - 3]};
        const bf16x2 h = __builtin_convertvector(v, bf16x2);
        v = f32x2{__builtin_amdgcn_fdot2_f32_bf16(h, neg_lo, v[0], false), __builtin_amdgcn_fdot2_f32_bf16(h, neg_hi, v[1], false)};
        const bf16x2 m = __builtin_convertvector(v, bf16x2);
        v = f32x2{__builtin_amdgcn_fdot2_f32_bf16(m, neg_lo, v[0], false), __builtin_amdgcn_fdot2_f32_bf16(m, neg_hi, v[1], false)};
        const bf16x2 l = __builtin_convertvector(v, bf16x2);
        r.h[2 * k] = h[0];
        r.h[2 * k + 1] = h[1];
        r.m[2 * k] = m[0];
        r.m[2 * k + 1] = m[1];
        r.l[2 * k] = l[0];
        r.l[2 * k + 1] = l[1];
    }
    return r;
}

// Sum over the 16 lanes of each row of a wave (or over aligned groups of L = 1, 2, 4 or 8 lanes), in
// every lane: quad swap, quad-pair swap, half-row mirror, row mirror.
template <int L = 16>
__device__ inline float row_sum(float v)
{
    if constexpr (L > 1) v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, false)); // quad_perm [1,0,3,2]
    if constexpr (L > 2) v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, false)); // quad_perm [2,3,0,1]
    if constexpr (L > 4) v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xF, 0xF, false)); // row_half_mirror
    if constexpr (L > 8) v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x140, 0xF, 0xF, false)); // row_mirror
    return v;
}

// Sum over the 64 lanes of a wave, in every lane: the rows' sums from lanes 0, 16, 32, 48.
__device__ inline float wave_sum(float v)
{
    v = row_sum(v);
    const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0));
    const float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16));
    const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32));
    const float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 48));
    return (r0 + r1) + (r2 + r3);
}

// The sums of P values per lane over the 64 lanes of a wave, to out[0 .. P) (LDS).  The two
// row-swap steps each add two values at once and leave their sums in different rows of lanes, so
// the P values shrink to P / 4 registers before the four steps inside a row: about 2.5
// instructions per value, where summing one value after the other takes eleven (the reduction at the
// end of the pair-sum kernels at n = 8: 2.2 -> 0.5 us).
template <int P>
__device__ inline void wave_sums(const float (&acc)[P], float *out)
{
    constexpr int P2 = (P + 1) / 2, P4 = (P2 + 1) / 2;
    float a[2 * P4];
    a[2 * P4 - 1] = 0.f;
#pragma unroll
    for (int k = 0; k < P2; ++k) { // lanes 0..31: value 2k, lanes 32..63: value 2k + 1
        const unsigned lo = __float_as_uint(acc[2 * k]), hi = (2 * k + 1 < P) ? __float_as_uint(acc[2 * k + 1 < P ? 2 * k + 1 : 0]) : 0u;
        const auto r = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
        a[k] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    float b[P4];
#pragma unroll
    for (int k = 0; k < P4; ++k) { // rows 0..3: values 4k, 4k + 2, 4k + 1, 4k + 3
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a[2 * k]), __float_as_uint(a[2 * k + 1]), false, false);
        b[k] = row_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
    }
    const int row = (threadIdx.x & 63) >> 4;
    const int sub = ((row & 1) << 1) | (row >> 1);
    if ((threadIdx.x & 15) == 0) {
#pragma unroll
        for (int k = 0; k < P4; ++k)
            if (4 * k + 3 < P || 4 * k + sub < P) out[4 * k + sub] = b[k];
    }
}

} // namespace svgd
