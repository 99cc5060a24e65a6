// Pairwise squared distances, pass 1: per-workgroup partial sums over a split of the D columns.
//
// Paper App. B.2 computes, per ordered pair, diff = (p_j - p_i)/l and radius^2 = dot(diff, diff).
// Here all pairs are accumulated in ONE pass over X: a thread (or a wave) holds all n values of
// a few columns on chip, adds their contribution to every pair, and moves on.
#pragma once
#include <type_traits>
#include "bandwidth_kernels.hpp"
#include "common.hpp"

namespace svgd {

// ---------------------------------------------------------------------------------------------
// n <= kValuMaxN (12): vector ALU, lanes = columns.  Each thread loads 4 consecutive columns of
// every row (one 16-byte load per row, 1 KiB contiguous per row per wave) and keeps one fp32
// accumulator per pair in registers.
//   N <= 8 : direct differences (x_i - x_j)^2 - no cancellation at all.
//   N  > 8 : Gram of the column-centred y = x - mean_i(x); d2 = S_ii + S_jj - 2 S_ij later.
// Chains are short (D / (4 * threads) terms per accumulator); lanes are combined by row swaps and
// DPP adds, waves through LDS, workgroups in fp64 by the kernel that needs the sums (or, for a long list,
// by the reduce kernel).
// ---------------------------------------------------------------------------------------------

// One 4-column group's contribution to every pair sum: acc[tri(i, j, N)] += sum over the 4
// columns of (x_i - x_j)^2 (N <= 8) or of y_i y_j, y = x - column mean (N > 8; x is overwritten
// by y).
template <int N>
__device__ __forceinline__ void pair_accumulate(f32x4 (&x)[N], float (&acc)[N * (N + 1) / 2])
{
    constexpr bool kDiff = (N <= 8);
    if constexpr (kDiff) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
#pragma unroll
            for (int j = i + 1; j < N; ++j) {
                const f32x4 d = x[i] - x[j];
                float a = acc[tri(i, j, N)];
                a = fmaf(d.x, d.x, a);
                a = fmaf(d.y, d.y, a);
                a = fmaf(d.z, d.z, a);
                a = fmaf(d.w, d.w, a);
                acc[tri(i, j, N)] = a;
            }
        }
    } else {
        f32x4 m = x[0];
#pragma unroll
        for (int j = 1; j < N; ++j) m += x[j];
        m *= (1.0f / N);
#pragma unroll
        for (int j = 0; j < N; ++j) x[j] -= m; // columns beyond D were loaded as 0 -> stay 0
#pragma unroll
        for (int i = 0; i < N; ++i) {
#pragma unroll
            for (int j = i; j < N; ++j) {
                float a = acc[tri(i, j, N)];
                a = fmaf(x[i].x, x[j].x, a);
                a = fmaf(x[i].y, x[j].y, a);
                a = fmaf(x[i].z, x[j].z, a);
                a = fmaf(x[i].w, x[j].w, a);
                acc[tri(i, j, N)] = a;
            }
        }
    }
}

// Workgroups per CU, all resident at once; as registers per wave, too, so that no CU takes more of them than another.
constexpr int kGramPerCu = 3;
// Column groups per iteration: two when the registers allow, for twice the loads in flight.
template <int N> constexpr int kGramGroups = N <= 8 ? 2 : 1;

// STREAM: loads with the streaming hint, but for the `hot` iterations walked last, see gram_mfma_kernel (here also for unaligned rows: a
// wave covers 1 KiB of a row, the one line it shares with its neighbour matters little).
template <int N, bool ROWS = false, bool STREAM = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kGramPerCu, kGramPerCu))) void gram_valu_kernel(const float *__restrict__ X, int64_t D, int64_t ld,
                                                        float *__restrict__ partials, GroupSplit split, int hot,
                                                        typename RowArg<ROWS>::type rt)
{
    constexpr int P = N * (N + 1) / 2;
    float acc[P];
#pragma unroll
    for (int p = 0; p < P; ++p) acc[p] = 0.f;

    const int64_t nthreads = (int64_t)gridDim.x * 256;
    constexpr int U = kGramGroups<N>;
    // The columns are walked from the far end: the update that follows walks them from the near
    // end, so each pass starts on the part of X that the pass before it touched last and that the
    // memory-side cache still holds.
    const int grp0 = (int)(blockIdx.x * 256 + threadIdx.x);
    auto row = [&](int j) __attribute__((always_inline)) { return X + (ROWS ? rt.x[ROWS ? j : 0] : (int64_t)j * ld); };
    const int cnt = split.count(grp0);
    auto groups = [&](int k, auto stream) __attribute__((always_inline)) { // the U groups of iteration k
        const int64_t grp = grp0 + (int64_t)k * U * nthreads;
        f32x4 x[U][N];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const RaggedGroup rg((grp + u * nthreads) << 2, D);
#pragma unroll
            for (int j = 0; j < N; ++j) x[u][j] = rg.template load<decltype(stream)::value>(row(j));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const RaggedGroup rg((grp + u * nthreads) << 2, D);
            if (rg.s) { // (a group past the end becomes 0)
#pragma unroll
                for (int j = 0; j < N; ++j) x[u][j] = rg.fix(x[u][j]);
            }
            pair_accumulate<N>(x[u], acc);
        }
    };
    if (D >= 4) {
        int k = cnt - 1;
        if constexpr (STREAM) {
            for (; k >= hot; --k) groups(k, std::true_type{});
        }
        for (; k >= 0; --k) groups(k, std::false_type{});
    } else if (cnt > 0) {
        f32x4 x[N];
#pragma unroll
        for (int j = 0; j < N; ++j) x[j] = load_narrow(row(j), D);
        pair_accumulate<N>(x, acc);
    }

    __shared__ float red[4][P];
    wave_sums<P>(acc, red[threadIdx.x >> 6]);
    __syncthreads();
    for (int p = threadIdx.x; p < P; p += 256)
        partials[(int64_t)blockIdx.x * pair_stride(N) + p] = (red[0][p] + red[1][p]) + (red[2][p] + red[3][p]);
}

// ---------------------------------------------------------------------------------------------
// kValuMaxN < n <= 64: matrix cores.  The Gram S = Y Y^T of the column-centred Y is a contraction over
// columns, so the MFMA A and B operands are both "lane = (particle row, column slot)".  Loading
// that shape straight from HBM would touch 16 rows per quarter-wave, so each wave instead
//   1. loads a 16*NB-row x 64-column slab with row-contiguous 16-byte loads (256 B per row per
//      quarter-wave), rows {4i + lane/16}, columns 4*(lane%16)..+3,
//   2. centres the columns (own rows in registers, two cross-lane adds for the other rows),
//   3. writes the slab to a wave-private LDS region with a 16-byte-granule XOR swizzle,
//   4. reads it back row-wise, eight columns per lane and step - lane (q = lane/16, rr = lane%16)
//      takes row 16b+rr - and splits each value into three bf16 parts that add up to it exactly
//      (split3); v_mfma_f32_16x16x32_bf16 wants 32 columns as its k-slots, eight per lane
//      (the loads of the next slab are issued here, before the multiply phase),
//   5. issues six MFMAs per unordered block pair b <= b', fp32 accumulators in registers: lane (q, c),
//      register r of pair (b, b') holds S[16b + 4q + r][16b' + c].
// Any assignment of columns to k-slots is valid because every column is summed exactly once.
// ---------------------------------------------------------------------------------------------
// Order of the slabs.  The update re-reads X right after this pass, every wave (or workgroup) of it
// walking a contiguous range of 64-column tiles from the left (tile_range).  What the memory-side
// cache holds of X when the update starts should therefore be the first `hot` tiles of each of
// those `nranges` ranges of `per` tiles, and this pass visits them last: its index space is
//     [0, I1)        the other ("cold") tiles, range after range,
//     [I1, I1 + I2)  the hot tiles, range after range,
//     I1 + I2        the partial slab after the last full tile, if D mod 64 != 0,
// with I1 = nranges * (per - hot), I2 = nranges * hot (indices that fall beyond a short last range
// are empty slabs), and wave w of workgroup b takes the indices W (b + k * gridDim.x) + w: the
// workgroups sweep the index space together, the W waves of one on adjacent slabs.

// Waves per workgroup (template argument W): eight, one workgroup per CU and two waves per SIMD - half
// as many partial sums as with two workgroups of four -, or four for an X of fewer slabs than four
// waves per CU take, which more CUs can share then.  (From there to eight slabs per CU every wave has
// one at most as well, and some CUs have none, but the shorter list pays: us per step at D = 65,000 in
// 254 workgroups of four and D = 65,600 in 129 of eight, n = 16 15.7 and 13.5, n = 24 23.2 and 20.0, n = 32
// 24.1 and 22.0.)
constexpr int kGramWaves = 8;
constexpr int kGramWavesSmall = 4;
// With one slab per wave the shorter code of the fp32 multiply counts, up to two blocks of rows; three and four are six
// and ten pairs of blocks, 3 and 5 thousand cycles in fp32 (step at D = 1,003, n = 40 23.5 -> 21.8 us, n = 64
// 29.9 -> 27.6; D = 20,001 24.4 -> 24.3 and 30.8 -> 30.0).
constexpr int kGramF32Blocks = 2;

// (a wave's indices are `stride` = W * gridDim.x apart; its quotient and remainder by the lengths
// of a range's cold and hot parts come from the host, so that stepping from one index to the next
// needs no division; everything fits 32 bits, the host sees to that)
struct GramOrder {
    uint32_t nranges, per, hot;
    uint32_t q_cold, r_cold; // stride = q_cold * (per - hot) + r_cold   (0, 0 if per == hot)
    uint32_t q_hot, r_hot;   // stride = q_hot * hot + r_hot             (0, 0 if hot == 0)
};

// ORDER 0: plain order, index = tile (go is not looked at) - for an X that the memory-side cache
//   holds anyway, or nearly: there the bookkeeping of the order costs more than the order gains.
// ORDER 1: the order described above.
// ORDER 2: the same, and the cold tiles are loaded with the streaming hint (no allocation on the
//   way in) - for rows on 128-byte boundaries (nothing is shared between the slabs of neighbouring
//   waves).  The pass itself then runs 5 % (n = 64, D = 11.2 M) to 28 % (n = 16, same D) faster.
// ORDER 3: as 1, and the eight waves of a workgroup send off their loads together, so that the line which two slabs
//   of unaligned rows share is asked for by both at once (fetched, n = 64, D = 11.2 M: 1.25 times the bytes, 1.06 in step; reads alone
//   516 -> 466 us).  What the waves
//   then wait for each other costs as much where little bounds the pass but itself (svgd_bandwidth 563 and 573 us) or the
//   last block of rows is mostly empty; behind the writes of an update, us per dense step, ORDER 1 and 3: n = 64, D = 11,173,962
//   2340 and 2300, D = 5,324,817 1134 and 1125, D = 2,293,777 496 and 497, n = 60, D = 9,175,057 1812 and 1793, n = 48,
//   D = 7,099,750 1096 and 1079, n = 44, D = 7,745,180 1094 and 1087; n = 40 1115 and 1116, n = 33 1092 and 1120, n = 50 1787 and 1805.
// ORDER 4: plain order, and no branch around any load (WIDE, below) - for small X with columns after the last slab.
// The host takes ORDER 1, 2 or 3 when X is larger than twice the memory-side cache.
// What bounds the pass is memory, since the multiplies are in bf16: at n = 64 the matrix pipe is busy for
// 27 % of the cycles (120 instructions of 16 per slab) and the vector ALU for 32.  In fp32
// (v_mfma_f32_16x16x4_f32, 160 per slab) they took 32 cycles each during which the vector ALU stood
// still - the fp32 matrix instructions share its multipliers, measured with both in one wave and in
// two; the bf16 ones run beside the 224 instructions of the split.  Before and after, launched by itself: n = 64, D = 11,173,962, padded rows 569 -> 459 us
// (6.2 TB/s), dense ones, whose slabs share lines that are fetched twice, 587 -> 552; n = 33, D = 5 M
// 166 -> 130 (5.1 TB/s); n = 48, D = 1 M 41.5 -> 38.0; n = 16, D = 11.2 M 116 -> 111 (6.4 TB/s).  Inside
// a step, right behind the update's writes, less of it is left: 568 -> 549 and 558 -> 554 at n = 64,
// 156 -> 130 at n = 33, 43.7 -> 39.5 at n = 48.  d2 against 64 bits, n = 13..64, D = 65,536..3 M, unit
// normal values, small ones and small ones around a large common part: 9.4e-9 -> 2.7e-9 rms on
// average (slab sums instead of one long chain: 3e-8 -> 3e-9 at 3 M; up to D = 300,007 both are at
// 3e-9); inside clusters 1e-3 wide 4.1e-3 -> 1.8e-3 of the small distances.
template <int NB, int W, bool ROWS = false, int ORDER = 0>
__global__ __launch_bounds__(64 * W) void gram_mfma_kernel(const float *__restrict__ X, int n,
                                                                    int64_t D, int64_t ld, float *__restrict__ partials,
                                                                    typename RowArg<ROWS>::type rt, GramOrder go)
{
    constexpr int NROW = 16 * NB;
    constexpr int RPL = 4 * NB; // rows per lane while loading
    constexpr int NPAIR = NB * (NB + 1) / 2;
    __shared__ float lds[W][NROW * 64];

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int q = lane >> 4, c16 = lane & 15;
    float *my = lds[wave];
    const float inv_n = 1.0f / (float)n;

    f32x4 acc[NPAIR];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < NPAIR; ++p) acc[p] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    const SplitConst sc = split_const();

    constexpr bool WIDE = ORDER == 4, ORDERED = ORDER != 0 && !WIDE, STREAM = ORDER == 2, IN_STEP = ORDER == 3;
    static_assert(!WIDE || W == kGramWavesSmall, "a slab or two per wave");
    constexpr bool F32 = W == kGramWavesSmall && NB <= kGramF32Blocks;
    const int64_t nfull = D >> 6;
    const uint32_t uper = go.per, uhot = go.hot, ucold = uper - uhot, unfull = (uint32_t)nfull;
    const uint32_t I1 = ORDERED ? go.nranges * ucold : 0u, I2 = ORDERED ? go.nranges * uhot : unfull;
    const uint32_t nidx = I1 + I2 + (((nfull << 6) < D) ? 1u : 0u);
    const uint32_t first = (uint32_t)W * blockIdx.x + (uint32_t)__builtin_amdgcn_readfirstlane(wave);
    const uint32_t stride = (uint32_t)W * gridDim.x;
    // the walk: index `at` is tile r * per + o (+ hot while cold), or the partial slab (phase 2)
    uint32_t at, phase, r, o;
    auto enter = [&]() { // state at index `at`, by division: once per wave and phase
        if (at < I1) {
            phase = 0;
            r = at / ucold;
            o = at - r * ucold;
        } else if (at < I1 + I2) {
            phase = 1;
            r = (at - I1) / uhot;
            o = (at - I1) - r * uhot;
        } else {
            phase = 2;
        }
    };
    auto advance = [&]() {
        at += stride;
        if constexpr (ORDERED) {
            if (phase == 0 && at < I1) {
                o += go.r_cold;
                r += go.q_cold;
                if (o >= ucold) { o -= ucold; ++r; }
            } else if (phase == 1 && at < I1 + I2) {
                o += go.r_hot;
                r += go.q_hot;
                if (o >= uhot) { o -= uhot; ++r; }
            } else if (phase < 2) {
                enter();
            }
        }
    };
    auto start = [&]() {
        at = first;
        phase = r = o = 0;
        if constexpr (ORDERED) enter();
    };
    f32x4 x[RPL];
    // Where this lane's rows start (separate rows only): in LDS, and - RREG - in registers from there.  With four
    // blocks there are none left for them: 47 were spilled, and the pass took 304 us at n = 64, D =
    // 5,000,000 (262 in fp32, 256 now; n = 49, D = 3,000,001 146 -> 116).
    constexpr bool RREG = ROWS && (NB < 4 || F32);
    __shared__ int64_t srow[ROWS ? kMaxN : 1];
    int64_t xro[RREG ? RPL : 1];
    if constexpr (ROWS) { // from the kernel's arguments in one coalesced read (entries beyond n repeat row 0)
        if (threadIdx.x < kMaxN) srow[threadIdx.x] = rt.x[ROWS ? threadIdx.x : 0];
        __syncthreads();
    }
    if constexpr (RREG) {
#pragma unroll
        for (int i = 0; i < RPL; ++i) xro[i] = srow[4 * i + q];
    }
    // WIDE (small X, a slab per wave): rows beyond n are loaded as row n - 1 and set to 0 when the slab is used, and the
    // partial slab is loaded like the others, at min(column, D - 4), and moved into place then (RaggedGroup): no branch around
    // any load.  With guarded ones - four per slab, and 64 single columns per row and wave in the partial slab, whose
    // wave was the last of its launch to end - svgd_bandwidth takes 17.5 us at n = 64, D = 20,001, 16.2 without, n = 40 14.4 and 13.8;
    // D = 65,003 18.6 and 17.2, 15.2 and 14.5.  Without a partial slab it is the guards that are faster (n = 64, D = 20,032 16.0
    // and 16.3, n = 36 13.3 and 13.7, n = 18 10.5 and 10.9: the code is shorter), with one block, four rows per lane, always (the pass
    // alone, n = 16, D = 8,577 3.3 and 3.5), and in the loop over many slabs what is moved and set to 0 costs more
    // than the branches (n = 64, D = 1,500,003 87.8 and 101).
    int64_t last_row[WIDE && !ROWS ? 4 : 1];
    if constexpr (WIDE && !ROWS) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int row = 4 * (RPL - 4 + k) + q;
            last_row[k] = (int64_t)(row < n ? row : n - 1) * ld;
        }
    }
    // The slab at `at` (then on to the next index): where it lies and how it is to be loaded -
    // 0: plain 16-byte loads, 1: streaming ones, 2: the partial slab (WIDE: only one of fewer than four columns), 3: an
    // empty slab.  One wave-uniform decision per slab, then sixteen loads in a row: decided per row, every load
    // sat behind its own little tree of branches, a hundred branches per slab during which the
    // matrix pipe had nothing from this wave.
    int64_t col = 0;
    bool partial = false; // WIDE: the slab in x is the partial one; then how far its columns are to be moved:
    int shift = 0;
    auto next_slab = [&]() __attribute__((always_inline)) -> int {
        const bool is_cold = ORDERED && phase == 0;
        int64_t tile = ORDERED ? nfull : (int64_t)at; // ordered, phase 2: the partial slab
        if (ORDERED && phase < 2) {
            const uint32_t t = r * uper + (is_cold ? uhot : 0u) + o;
            const uint32_t end = ((uint64_t)(r + 1) * uper < unfull) ? (r + 1) * uper : unfull;
            tile = t < end ? (int64_t)t : -1; // beyond a short last range: an empty slab
        }
        advance();
        const int64_t wcol = tile << 6;
        col = wcol + 4 * c16;
        if (ORDERED && tile < 0) return 3;
        if constexpr (WIDE) {
            partial = wcol + 64 > D && D >= 4;
            int how = wcol + 64 > D && D < 4 ? 2 : 0;
            if (partial) {
                const RaggedGroup rg(col, D);
                col = rg.at;
                shift = rg.s;
            }
            return __builtin_amdgcn_readfirstlane(how);
        }
        if (wcol + 64 > D) return 2;
        return (STREAM && is_cold) ? 1 : 0;
    };
    auto rows = [&](auto how) __attribute__((always_inline)) {
        constexpr int HOW = decltype(how)::value;
        int64_t at0 = (int64_t)q * ld + col; // this lane's place in row q; row 4i + q is a uniform distance on
        opaque(at0);
        int qv = q;
        if constexpr (ROWS && !RREG) asm volatile("" : "+v"(qv)); // (or the reads would be hoisted out of the loop)
        // Row 4i + q.  (Base plus place in row q first: what is added for the others is uniform.  With the three added up before the base
        // every load has an instruction or two of its own: n = 33, D = 100,003 14.6 us, 14.4 without.  With four blocks in plain
        // order that is the faster way all the same: svgd_bandwidth at 49 to 64 particles, D = 300,007 to 1,800,007 0.3 to 1 %, a padded
        // step n = 64, D = 300,007 80.2 and 79.7; D = 70,003 to 100,003 0.7 % slower.)
        auto row_at = [&](int i) __attribute__((always_inline)) {
            if constexpr (RREG) return X + xro[i] + col;
            else if constexpr (ROWS) return X + srow[4 * i + qv] + col;
            else if constexpr (WIDE) return i < RPL - 4 ? X + at0 + (int64_t)(4 * i) * ld : X + col + last_row[i & 3];
            else if constexpr (NB == 4 && ORDER == 0 && W == kGramWaves) return X + (at0 + (int64_t)(4 * i) * ld);
            else return X + at0 + (int64_t)(4 * i) * ld;
        };
#pragma unroll
        for (int i = 0; i < RPL; ++i) {
            const int row = 4 * i + q;
            const float *xr = row_at(i);
            f32x4 v = {0.f, 0.f, 0.f, 0.f}; // rows beyond n, and empty slabs, add nothing to any sum
            // (only the last block of 16 rows can reach beyond n)
            if (HOW != 3 && (WIDE || i < RPL - 4 || row < n)) {
                if constexpr (HOW == 0) v = *reinterpret_cast<const f32x4u *>(xr);
                else if constexpr (HOW == 1) v = __builtin_nontemporal_load(reinterpret_cast<const f32x4u *>(xr));
                else if constexpr (WIDE) v = c16 == 0 ? load_narrow(xr - col, D) : v;
                else v = load4(xr - col, col, D, false);
            }
            x[i] = v;
        }
    };
    // run `f` with the load mode as a compile-time constant
    auto with_mode = [&](int how, auto f) __attribute__((always_inline)) {
        if (how == 0) f(std::integral_constant<int, 0>{});
        else if (how == 1) f(std::integral_constant<int, 1>{});
        else if (how == 2) f(std::integral_constant<int, 2>{});
        else f(std::integral_constant<int, 3>{});
    };
    auto load_slab = [&]() __attribute__((always_inline)) { with_mode(next_slab(), rows); };
    // steps 2 and 3: the slab in x, centred, into `buf`
    auto centre_and_stage = [&](float *buf) __attribute__((always_inline)) {
        if constexpr (WIDE) {
            if (partial) {
                RaggedGroup rg(0, 4);
                rg.s = shift;
#pragma unroll
                for (int i = 0; i < RPL; ++i) x[i] = rg.fix(x[i]);
            }
#pragma unroll
            for (int i = RPL - 4; i < RPL; ++i)
                if (4 * i + q >= n) x[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        f32x4 s = x[0];
#pragma unroll
        for (int i = 1; i < RPL; ++i) s += x[i];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            s[c] = sum_over_rows(s[c]) * inv_n;
        }
        // The LDS region is private to this wave and a wave's LDS operations execute in order, so
        // no barrier is needed between consuming a slab and overwriting it.
#pragma unroll
        for (int i = 0; i < RPL; ++i) {
            const int row = 4 * i + q;
            // rows >= n hold -mean here; they only reach entries with i or j >= n, never stored
            *reinterpret_cast<f32x4 *>(&buf[row * 64 + ((c16 ^ (row & 15)) << 2)]) = x[i] - s;
        }
    };
    // steps 4 and 5 on the slab in `buf`
    auto multiply = [&](const float *buf) __attribute__((always_inline)) {
        // A slab's sums start from zero and are added to the running ones in fp32 at its end.  Straight
        // into a large running sum, squares of eight-bit values leave remainders that are not evenly
        // spread - odd squares are 1 modulo 8 - and the rounding errors do not cancel (measured: d2
        // 6e-8 too large after 30 steps).
        f32x4 t[NPAIR];
#pragma unroll
        for (int p = 0; p < NPAIR; ++p) t[p] = f32x4{0.f, 0.f, 0.f, 0.f};
        // One kind of product after the other over the pairs of blocks: a dependent matrix instruction can
        // issue after some 44 cycles, an independent one after 17.  The small products come first,
        // those of the leading parts last, so that the sum is rounded at its full size twice only.
        // Every entry of the matrix takes the same products in the same order, those on the
        // diagonal too: S_ii, S_ij and S_jj of two equal particles are then equal bit for bit,
        // wherever the particles lie, and their distance is exactly 0.  (With h l and h m of a diagonal
        // block taken once and added both ways round - four products instead of six - it was
        // rounding noise, and with it the median of an ensemble most of whose particles coincide.)
        auto products = [&](auto left, auto right) __attribute__((always_inline)) {
            int p = 0;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
#pragma unroll
                for (int b2 = b; b2 < NB; ++b2) {
                    t[p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(left(b), right(b2), t[p], 0, 0, 0);
                    ++p;
                }
            }
        };
        bf16x8 h[2][NB], m[NB], l[NB];
        auto pm = [&](int b) __attribute__((always_inline)) { return m[b]; };
        auto pl = [&](int b) __attribute__((always_inline)) { return l[b]; };
#pragma unroll
        for (int st = 0; st < 2; ++st) { // 32 columns each
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const float *row = buf + (16 * b + c16) * 64; // here c16 plays the role of rr (matrix row)
                const Split3 a = split3(*reinterpret_cast<const f32x4 *>(&row[((8 * st + q) ^ c16) << 2]),
                                        *reinterpret_cast<const f32x4 *>(&row[((8 * st + 4 + q) ^ c16) << 2]), sc);
                h[st][b] = a.h;
                m[b] = a.m;
                l[b] = a.l;
            }
            auto ph = [&](int b) __attribute__((always_inline)) { return h[st][b]; };
            products(ph, pl);
            products(pl, ph);
            products(pm, pm);
            products(ph, pm);
            products(pm, ph);
        }
#pragma unroll
        for (int st = 0; st < 2; ++st) {
            auto ph = [&](int b) __attribute__((always_inline)) { return h[st][b]; };
            products(ph, ph);
        }
#pragma unroll
        for (int p = 0; p < NPAIR; ++p) acc[p] += t[p];
    };
    // the same in fp32: v_mfma_f32_16x16x4_f32, four k-slots (columns {16s + 4q + c, q = 0..3}) at a time
    auto multiply_f32 = [&](const float *buf) __attribute__((always_inline)) {
#pragma unroll
        for (int st = 0; st < 4; ++st) {
            f32x4 a[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b)
                a[b] = *reinterpret_cast<const f32x4 *>(&buf[(16 * b + c16) * 64 + (((4 * st + q) ^ c16) << 2)]);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                int p = 0;
#pragma unroll
                for (int b = 0; b < NB; ++b) {
#pragma unroll
                    for (int b2 = b; b2 < NB; ++b2) {
                        acc[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[b][c], a[b2][c], acc[p], 0, 0, 0);
                        ++p;
                    }
                }
            }
        }
    };
    // Two waves per SIMD: one's vector instructions run beside the other's matrix instructions (the
    // bf16 ones; fp32 matrix instructions and the vector ALU exclude each other).
    auto sweep = [&](auto f32) __attribute__((always_inline)) {
        clear();
        start();
        if (first < nidx) load_slab();
        if constexpr (IN_STEP && !decltype(f32)::value) {
            uint32_t idx = first; // as many rounds, and barriers, for every wave as for the workgroup's first one
            for (uint32_t idx0 = (uint32_t)W * blockIdx.x; idx0 < nidx; idx0 += stride, idx += stride) {
                if (idx < nidx) centre_and_stage(my);
                block_sync<true>();
                if (idx + stride < nidx) load_slab();
                if (idx < nidx) multiply(my);
            }
            return;
        }
        for (uint32_t idx = first; idx < nidx; idx += stride) {
            centre_and_stage(my);
            // the next slab's loads are in flight while this one is multiplied
            if (idx + stride < nidx) load_slab();
            if constexpr (decltype(f32)::value) multiply_f32(my);
            else multiply(my);
        }
    };
    if constexpr (F32) {
        sweep(std::true_type{});
    } else {
        sweep(std::false_type{});
        // Sums that are not finite - a product overflowed, or X is not finite - are taken again in fp32,
        // whose infinities and NaNs do not depend on how the values were split.
        float odd = 0.f;
#pragma unroll
        for (int p = 0; p < NPAIR; ++p)
#pragma unroll
            for (int r = 0; r < 4; ++r) odd += 0.f * acc[p][r]; // 0, or NaN
        if (__ballot(odd != 0.f) != 0) sweep(std::true_type{});
    }

    // The waves meet in LDS, each with its sums in its own region (free by now); wave w adds up and
    // stores the block pairs w, w + 8, ... of the upper triangle in tri(i, j) order.
    static_assert(NPAIR * 256 <= NROW * 64, "a wave's sums fit its region");
#pragma unroll
    for (int p = 0; p < NPAIR; ++p)
#pragma unroll
        for (int r = 0; r < 4; ++r) my[(p * 4 + r) * 64 + lane] = acc[p][r];
    __syncthreads();
    float *out = partials + (int64_t)blockIdx.x * pair_stride(n);
    int p = 0;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
#pragma unroll
        for (int b2 = b; b2 < NB; ++b2) {
            if (p % W == wave) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = 16 * b + 4 * q + r;
                    const int j = 16 * b2 + c16;
                    double v = 0.0;
#pragma unroll
                    for (int w = 0; w < W; ++w) v += (double)lds[w][(p * 4 + r) * 64 + lane];
                    if (i <= j && j < n) out[tri(i, j, n)] = (float)v;
                }
            }
            ++p;
        }
    }
}

// A list of partials from one half of the scratch to the other.
__global__ __launch_bounds__(256) void copy_list_kernel(const f32x4 *__restrict__ src, f32x4 *__restrict__ dst, int n4)
{
    const int i = (int)(blockIdx.x * 256 + threadIdx.x);
    if (i < n4) dst[i] = src[i];
}

// Sum the per-workgroup fp32 partials in fp64: sums[p] = sum_k partials[k][p].  A workgroup takes 32
// entries, eight lanes of four next to each other, and thread group g of 32 the partials g, g + 32,
// ... with sixteen 16-byte loads in flight: up to 512 partials - 256 are usual, a carried step at 21 to
// 24 particles may leave 513 - are one batch of loads and one LDS exchange, and the result is the sums themselves, not slices for the next kernel
// to add.  3.7 us at n = 20, 4.7 at n = 32 and 64 (4.9, 4.9 and 4.8 with eight slices read four
// bytes at a time): the launch, one trip to memory the partials were just written to, the exchange.
constexpr int kReduceEntries = 32;
__global__ __launch_bounds__(256) void reduce_partials_kernel(const float *__restrict__ partials, int nparts, int n,
                                                              double *__restrict__ sums)
{
    constexpr int U = 16, GROUPS = 32;
    __shared__ double red[GROUPS][kReduceEntries + 1];
    const int stride4 = pair_stride(n) / 4, P = n * (n + 1) / 2;
    const int col = threadIdx.x & 7, g = threadIdx.x >> 3;
    const int c4 = (int)blockIdx.x * (kReduceEntries / 4) + col;
    const f32x4 *src = reinterpret_cast<const f32x4 *>(partials) + (c4 < stride4 ? c4 : stride4 - 1);
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (int k0 = g; k0 < nparts; k0 += U * GROUPS) {
        f32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) { // unconditional loads (index clamped) issue together
            const int k = k0 + u * GROUPS;
            v[u] = src[(int64_t)(k < nparts ? k : nparts - 1) * stride4];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c) s[c] += (k0 + u * GROUPS < nparts) ? (double)v[u][c] : 0.0;
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) red[g][4 * col + c] = s[c];
    __syncthreads();
    // thread (e, part): four of the 32 groups' sums of entry e, then across the eight parts
    const int e = threadIdx.x >> 3, part = threadIdx.x & 7;
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < GROUPS / 8; ++k) t += red[part * (GROUPS / 8) + k][e];
    t += dpp_f64<0xB1>(t);
    t += dpp_f64<0x4E>(t);
    t += dpp_f64<0x141>(t);
    const int p = (int)blockIdx.x * kReduceEntries + e;
    if (part == 0 && p < P) sums[p] = t;
}

} // namespace svgd
