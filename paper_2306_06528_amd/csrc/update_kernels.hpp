// Pass 3: the fused all-particle update.  For every column k independently
//
//     z_jk   = g_jk - (2/h) x_jk
//     phi_ik = sum_j C_ij z_jk + rho_i x_ik,      C_ij = K_ij / n,  rho_i = (2/h) (sum_j K_ij) / n
//     x_ik  <- x_ik + eps * phi_ik
//
// which is phi_i = (1/n) sum_j [K_ij g_j + (2/h) K_ij (x_i - x_j)] with the sum over j of the
// x_j terms folded into a single n x n product (paper App. B.2, SVGD routine: per-pair kernel value,
// accumulation of the kernel-weighted gradients and of the kernel gradient, division by n, then
// the followers' parameter update; here in the score/ascent convention, x += eps * phi).
// X and G are read once and X is written once, in place: a column's outputs depend only on that
// column's inputs, and every thread/wave loads all n rows of its columns before storing any, so
// every phi_i is computed from the pre-step X.
#pragma once
#include <type_traits>

#include "bandwidth_kernels.hpp"
#include "common.hpp"

namespace svgd {

// Passes 2 and 3 in one launch: always on the vector ALU, FUSED on the matrix cores.  The kernel starts
// with pass 2 (every workgroup - kernel_matrix - or, on the vector ALU, every wave - wave_kernel_matrix - derives
// h, C and rho for itself from a short list of partials, or (21 to 48 particles) from the sums that a launch in
// between has made of a longer one; workgroup 0 records h and K) and needs no tables in device memory.  A CARRY kernel
// leaves the partials of the new X in the other half of the scratch, because workgroups still in their
// prologue read the old list.
struct UpdateArgs {
    // passes 2 and 3 in one launch only: the list of partial sums, or (21 particles and more) what it adds up to
    const float *partials;
    int nparts;
    const double *sums;
    double h_fixed, log_n1;
    // all update kernels:
    // walk the columns from the far end.  Which thread or wave owns which columns does not change, only the order in which it
    // visits them.  A caller that alternates the direction from step to step starts every pass
    // on the part of X that the previous pass touched last, i.e. on what the memory-side cache
    // still holds.
    int reverse;
    // matrix-core kernels that store from the registers: the four waves of a workgroup take adjacent tiles of
    // one range instead of a range each (see tile_range).
    int adjacent;
    int64_t per; // matrix-core kernels: tiles_per_range for the mode they take
};

// ---------------------------------------------------------------------------------------------
// n <= kValuMaxN (12): vector ALU, lanes = columns, 4 consecutive columns per thread (16-byte
// loads, 1 KiB contiguous per row per wave).  C and rho are wave-uniform: LDS broadcasts.
// ---------------------------------------------------------------------------------------------
// Workgroups per CU, all resident at once, or the prologue (and with CARRY the reduction of the pair sums at
// the end) is paid twice.  Two where that leaves each thread's rows enough registers for loads in flight: plain
// step at D = 6,000,000, one against two per CU, n = 9 182 / 168 us, n = 12 235 / 240; at D = 1,000,000
// 44 / 38 and 57 / 64.  The kernel claims the registers of that many waves, so that no CU takes more
// workgroups than another, and the host sizes the grid by it.
__host__ __device__ constexpr int update_per_cu(int n, bool carry) { return n <= (carry ? 8 : 10) ? 2 : 1; }

template <int N, bool EMIT, bool CARRY, bool ROWS = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(update_per_cu(N, CARRY), update_per_cu(N, CARRY))))
void update_valu_kernel(float *__restrict__ X,
                                                          const float *__restrict__ G,
                                                          float *__restrict__ PHI,
                                                          float *__restrict__ coef,
                                                          DevState *__restrict__ st,
                                                          int64_t D, int64_t ld, float eps,
                                                          float *__restrict__ gram_out, GroupSplit split,
                                                          typename RowArg<ROWS>::type rt, UpdateArgs ua)
{
    static_assert(!(ROWS && (EMIT || CARRY)), "separate rows: plain in-place step only");
    static_assert(!(CARRY && EMIT), "the pair sums are carried only when X is updated");
    // CARRY: the pair sums of the UPDATED columns, in the format of gram_valu_kernel<N>
    constexpr bool kDiff = (N <= 8);
    constexpr int P = N * (N + 1) / 2;
    float pacc[CARRY ? P : 1];
    if constexpr (CARRY) {
#pragma unroll
        for (int p = 0; p < P; ++p) pacc[p] = 0.f;
    }
    const int64_t nthreads = (int64_t)gridDim.x * 256;
    // PREFETCH (carried pair sums of 6 particles and more): the loads of a thread's next column group are issued as
    // soon as this group's results are stored, before its pair sums are accumulated, so that arithmetic
    // runs while the loads are in flight (88.6 instead of 94.3 us per step at n = 12, D = 3,000,000; 15.8 and
    // 15.1 at n = 7, D = 1,000,000; at n <= 5 no difference).
    constexpr bool PREFETCH = CARRY && N > 5;
    f32x4 x[N], z[N];
    // All of X first, then all of G, in that order also in the machine code: in the mixed order that the compiler chose
    // the loads of G, which come from memory, kept those of X, half of which a cache holds, waiting (carried sums,
    // n = 8, padded rows, D = 1,000,003 18.5 -> 17.8 us per step, D = 11,173,962 164.2 -> 162.9; plain, n = 12,
    // D = 1,000,003 41.4 -> 40.9).
    auto load_group = [&](int64_t g) __attribute__((always_inline)) {
        const RaggedGroup rg(g << 2, D);
#pragma unroll
        for (int j = 0; j < N; ++j) {
            x[j] = rg.load<false>(X + (ROWS ? rt.x[ROWS ? j : 0] : (int64_t)j * ld));
            asm volatile("" ::: "memory");
        }
#pragma unroll
        for (int j = 0; j < N; ++j) {
            z[j] = rg.load<true>(G + (ROWS ? rt.g[ROWS ? j : 0] : (int64_t)j * ld));
            asm volatile("" ::: "memory");
        }
    };
    // LATE_STORES: a group's results are stored together, behind the arithmetic on the last of them.  For an X beyond the
    // memory-side cache that is the better way at 8 particles (D = 11,173,962, padded 162.9 -> 162.1 us per step, dense
    // 171.6 -> 171.1; at D = 1,000,003 it loses half of what the order of the loads gained, 17.8 -> 18.2), not at 6 and 7
    // (n = 7, padded, D = 1,000,003 14.8 -> 15.2, D = 11,173,962 140.2 -> 140.5).
    constexpr bool LATE_STORES = CARRY && N == 8;
    // this thread's groups: grp0 + k * nthreads, k < cnt, visited upwards or (reverse) downwards
    const int64_t grp0 = (int)(blockIdx.x * 256 + threadIdx.x);
    const int cnt = split.count((int)grp0);
    const int64_t gstep = ua.reverse ? -nthreads : nthreads;
    int64_t grp = ua.reverse ? grp0 + (cnt - 1) * nthreads : grp0;
    // Pass 2: the list of partial sums by all waves together, everything else by every wave for itself.  C and
    // rho are wave-uniform, read back as LDS broadcasts from the wave's own copy.
    __shared__ WaveShared<N> shw[4];
    __shared__ GatherShared<N> gather;
    WaveShared<N> &sh = shw[threadIdx.x >> 6];
    gather_wave_sums<N>(gather, ua.partials, ua.nparts, [&]() __attribute__((always_inline)) {
        if (cnt > 0 && D >= 4) load_group(grp); // the first column group is on its way while h and K are computed
    });
    block_sync<true>();
    const float c2h = wave_kernel_matrix<N>(
        sh, ua.h_fixed, ua.log_n1, st, coef, blockIdx.x == 0 && threadIdx.x < kWave,
        [&](int e) __attribute__((always_inline)) { return gather.sum(e); });
    if (cnt > 0 && D < 4) {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            x[j] = load_narrow(X + (ROWS ? rt.x[ROWS ? j : 0] : (int64_t)j * ld), D);
            z[j] = load_narrow(G + (ROWS ? rt.g[ROWS ? j : 0] : (int64_t)j * ld), D);
        }
    }
    for (int k = 0; k < cnt; ++k, grp += gstep) {
        const int64_t col = grp << 2;
        const bool full = (col + 4 <= D);
        if constexpr (!PREFETCH) {
            if (k > 0) load_group(grp);
        }
        if (!full) {
            const RaggedGroup rg(col, D);
#pragma unroll
            for (int j = 0; j < N; ++j) {
                x[j] = rg.fix(x[j]);
                z[j] = rg.fix(z[j]);
            }
        }

        const int c0 = opaque_zero();
        f32x4 m = f32x4{0.f, 0.f, 0.f, 0.f};
        if constexpr (CARRY && !kDiff) { // centre by the pre-update column mean
#pragma unroll
            for (int j = 0; j < N; ++j) m += x[j];
            m *= (1.0f / N);
        }
#pragma unroll
        for (int j = 0; j < N; ++j) z[j] -= c2h * x[j];
        f32x4 y[N]; // the results; CARRY: then the centred new values
        float *__restrict__ OUT = EMIT ? PHI : X;
        auto store = [&](int i, auto whole) __attribute__((always_inline)) {
            store4(OUT + (ROWS ? rt.x[ROWS ? i : 0] : (int64_t)i * ld), col, D, decltype(whole)::value || full, y[i]);
        };
        auto rows = [&](auto whole) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                float C[N], rho;
                sh.row(i, c0, C, rho);
                f32x4 acc = rho * x[i];
#pragma unroll
                for (int j = 0; j < N; ++j) acc += C[j] * z[j];
                if constexpr (EMIT) y[i] = acc;
                else y[i] = x[i] + eps * acc;
                if constexpr (!LATE_STORES) store(i, whole);
            }
            if constexpr (LATE_STORES) {
#pragma unroll
                for (int i = 0; i < N; ++i) store(i, whole);
            }
        };
        // one decision per wave: with a branch around every row's store no row's coefficients were read ahead
        if (__ballot(!full) == 0) rows(std::true_type{});
        else rows(std::false_type{});
        if constexpr (CARRY) {
#pragma unroll
            for (int i = 0; i < N; ++i) y[i] -= m; // columns beyond D: x = g = 0 -> 0
        }
        if constexpr (CARRY) {
            if constexpr (PREFETCH) {
                if (k + 1 < cnt) load_group(grp + gstep);
            }
#pragma unroll
            for (int i = 0; i < N; ++i) {
#pragma unroll
                for (int j = kDiff ? i + 1 : i; j < N; ++j) {
                    const f32x4 u = kDiff ? y[i] - y[j] : y[i];
                    const f32x4 v = kDiff ? u : y[j];
                    float a = pacc[tri(i, j, N)];
                    a = fmaf(u.x, v.x, a);
                    a = fmaf(u.y, v.y, a);
                    a = fmaf(u.z, v.z, a);
                    a = fmaf(u.w, v.w, a);
                    pacc[tri(i, j, N)] = a;
                }
            }
        }
    }
    if constexpr (CARRY) {
        __shared__ float red[4][P];
        wave_sums<P>(pacc, red[threadIdx.x >> 6]);
        __syncthreads();
        for (int p = threadIdx.x; p < P; p += 256)
            gram_out[(int64_t)blockIdx.x * pair_stride(N) + p] = (red[0][p] + red[1][p]) + (red[2][p] + red[3][p]);
    }
}

// ---------------------------------------------------------------------------------------------
// kValuMaxN < n <= 64: matrix cores, v_mfma_f32_16x16x4_f32 with M = output particle i, K = input
// particle j, N = column.
//
// Register tile.  A wave owns 16*NB rows x 64 columns at a time: lane (q = lane/16, c = lane%16)
// loads, for b < NB and r < 4, row 16b + 4q + r at columns 4c..4c+3 of the tile (256 B contiguous
// per row per quarter-wave).  Step s = 4b + r of the contraction feeds k-slot q with row
// 16b + 4q + r; the 4 components of the 16-byte load are 4 independent N-tiles (tile t = columns
// {4c + t}).  The 16x16 result of output block bi puts row 16bi + 4q + r, column c in register r
// of lane (q, c) - exactly the rows this lane loaded, so x_old is already in place for the
// epilogue and nothing crosses lanes.  The A operands (C re-ordered into the per-lane layout by
// the prologue) sit in LDS, shared by the workgroup's 4 waves, and are re-read per output block.
//
// Stores.  A row starts at i*ld floats, so in general the rows are not 128-byte aligned and a
// store of "the tile's columns" would cut cache lines in two for almost every row; partial-line
// writes cost far more HBM time than they carry bytes.  Loads do not care.  So each wave
//   - owns a CONTIGUOUS range of tiles and walks it left to right,
//   - stages each finished 16-row output block in LDS (cur, 16 x 64 floats),
//   - and for row i stores the 64-column window that ends r_i columns before the tile does,
//     r_i = (address of row i at the tile's first column, in floats) mod 32: that window starts
//     on a 128-byte boundary, and its first r_i columns are the previous tile's last ones, kept
//     in LDS (carry, 64 x 32 floats per wave).
// Every store instruction then writes whole cache lines.  Only the two ends of a wave's range
// see partial lines: the first tile masks what lies left of the range, and the carry is flushed
// element-wise after the last tile.
// The other two modes store the tile itself, straight from the registers that computed it
// (FROM_REGS) - no staging at all unless the Gram operands need it: where every row starts on a
// 128-byte boundary (kStoreLines: r_i = 0 for all rows, the windows are the tiles), and, wherever the rows
// start, where the cut lines cost less than the staging (kStoreDirect; the host's choice, by size).
// Columns beyond the last full tile (D mod 64) are done by one extra workgroup (TailColumns).  Rows >= n (n not
// a multiple of 16) are neither loaded nor stored; their A entries are
// zero (their contraction steps still run: skipping them behind wave-uniform branches cost more
// than it saved, see below).  One to four rows beyond a multiple of 16 do not get a block of
// their own at all (REM, below).
// ---------------------------------------------------------------------------------------------
// Where pass 2 is done: before the update, in a launch of its own; or inside the update, by every workgroup, from the list
// of partial sums (up to 32 particles) or from the sums that a launch in between has made of it (21 to 48 particles).
enum Pass2 : int { kPass2Apart = 0, kPass2OnList = 1, kPass2OnSums = 2 };
enum StoreMode : int {
    kStoreStaged = 0, // re-aligned through LDS, as described above
    kStoreLines = 1,  // every row starts on a 128-byte boundary: straight from the registers, G streamed
    kStoreDirect = 2  // straight from the registers to wherever the row starts, all accesses plain: for an X
                      // that the caches hold, where lines written in two parts meet again before they leave
};
constexpr int kUpdCur = 16 * 64;    // floats per wave
constexpr int kUpdCarry = 64 * 32;  // floats per wave

// The < 64 columns after the last full tile, by one workgroup of 256 threads.  x, z and - CARRY - the centred new
// values are staged in LDS, z and C with rows padded to a multiple of four, and a thread computes 4 columns
// of every sixteenth row, four rows of z at a time: 16 RT multiply-adds for RT + 4 reads of 16 bytes.  At small
// D this workgroup is the last to finish, so its loads go out with the other workgroups' first ones, all of
// them together, and every particle count has all 256 threads at work.  (Loaded after pass 2, and with 4 x 4
// tiles that left 192 threads idle at n = 16 and took C transposed, it ended 3.3 thousand cycles after the
// others at n = 16, D = 8,577, and 5 at n = 33, D = 20,001.  As one more tile on the matrix cores it cost the loop over
// the full tiles registers: n = 14, D = 4,000,003, padded, carried sums 110 -> 126 us.)
template <int NMAX, bool EMIT, bool CARRY, bool ROWS, bool FUSED> // n <= NMAX, a multiple of 4
struct TailColumns {
    static constexpr int RT = (NMAX + 15) / 16; // rows per thread
    static constexpr int U = NMAX / 4;          // loads per array and thread
    static constexpr int UC = FUSED ? 1 : (NMAX * NMAX + 255) / 256;
    float xv[U], gv[U];

    // column tid % 64 of the rows tid / 64, + 4, + 8 ...; clamped, not guarded: all of them go out together
    __device__ __forceinline__ void load(int n, int64_t D, int64_t ld, const float *X, const float *G, const int64_t *xrow, const int64_t *grow)
    {
        const int64_t col = (D & ~(int64_t)63) + (threadIdx.x & 63), at = col < D ? col : D - 1;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = (int)(threadIdx.x >> 6) + 4 * u, j = r < n ? r : n - 1;
            xv[u] = X[(ROWS ? xrow[ROWS ? j : 0] : (int64_t)j * ld) + at];
            gv[u] = G[(ROWS ? grow[ROWS ? j : 0] : (int64_t)j * ld) + at];
        }
    }

    // Cm: rows `cs` floats apart - FUSED: in LDS, padded with zeros to a multiple of four; else in memory, n.
    __device__ __forceinline__ void run(float *__restrict__ OUT, const float *Cm, int cs, const float *rhov, float c2h, int n, int64_t D,
                                        int64_t ld, float eps, float *__restrict__ lds, float *__restrict__ gram_out, const int64_t *xrow)
    {
        const int n4 = (n + 3) & ~3, tid = threadIdx.x;
        const int64_t col0 = D & ~(int64_t)63;
        // yn: groups of four rows keep their 16-byte granules in orders of their own, so that the pair sums can
        // read different groups at the same column without meeting in the LDS banks
        auto yn_index = [](int i, int c) { return i * 64 + (c ^ (((i >> 2) & 15) << 2)); };
        float *zs = lds, *xs = zs + n4 * 64, *yn = xs + n * 64, *Cs = yn + (CARRY ? n * 64 : 0);
        __shared__ __attribute__((aligned(16))) float means[CARRY ? 4 * 64 : 4]; // the waves' shares of the column sums
        float cv[UC];
        if constexpr (!FUSED) {
#pragma unroll
            for (int u = 0; u < UC; ++u) cv[u] = Cm[tid + 256 * u < n * n ? tid + 256 * u : n * n - 1];
        }
        float rho[RT];
#pragma unroll
        for (int k = 0; k < RT; ++k) rho[k] = rhov[16 * k + (tid >> 4) < n ? 16 * k + (tid >> 4) : 0];
        {
            const int col = tid & 63;
            const bool in = col0 + col < D;
            float s = 0.f;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int r = (tid >> 6) + 4 * u;
                const float x = in ? xv[u] : 0.f, g = in ? gv[u] : 0.f;
                if (r < n) {
                    xs[r * 64 + col] = x;
                    s += x;
                }
                if (r < n4) zs[r * 64 + col] = r < n ? g - c2h * x : 0.f;
            }
            if constexpr (CARRY) means[tid] = s;
        }
        if constexpr (!FUSED) {
#pragma unroll
            for (int u = 0; u < UC; ++u) {
                const int e = tid + 256 * u, i = e / n;
                if (e < n * n) Cs[i * n4 + e - i * n] = cv[u];
            }
            if (n4 > n) // the padding
                for (int e = tid; e < n * 4; e += 256)
                    if (n4 - 4 + (e & 3) >= n) Cs[(e >> 2) * n4 + n4 - 4 + (e & 3)] = 0.f;
        }
        block_sync<true>();
        const float *C = FUSED ? Cm : Cs;
        const int st = FUSED ? cs : n4;
        const int cg = 4 * (tid & 15), i0 = tid >> 4; // 4 columns, rows i0 + 16 k
        f32x4 acc[RT];
#pragma unroll
        for (int k = 0; k < RT; ++k) acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
        for (int j = 0; j < n4; j += 4) {
            f32x4 z[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) z[r] = *reinterpret_cast<const f32x4 *>(&zs[(j + r) * 64 + cg]);
#pragma unroll
            for (int k = 0; k < RT; ++k) {
                const int i = i0 + 16 * k < n ? i0 + 16 * k : n - 1;
                const f32x4 c = *reinterpret_cast<const f32x4 *>(&C[i * st + j]);
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[k] += c[r] * z[r];
            }
        }
        f32x4 m = {0.f, 0.f, 0.f, 0.f};
        if constexpr (CARRY) {
#pragma unroll
            for (int w = 0; w < 4; ++w) m += *reinterpret_cast<const f32x4 *>(&means[64 * w + cg]);
            m *= 1.0f / (float)n;
        }
#pragma unroll
        for (int k = 0; k < RT; ++k) {
            const int i = i0 + 16 * k;
            if (i < n) {
                const f32x4 x = *reinterpret_cast<const f32x4 *>(&xs[i * 64 + cg]);
                f32x4 out;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float phi = fmaf(rho[k], x[e], acc[k][e]);
                    out[e] = EMIT ? phi : fmaf(eps, phi, x[e]);
                }
                store4(OUT + (ROWS ? xrow[ROWS ? i : 0] : (int64_t)i * ld), col0 + cg, D, col0 + cg + 4 <= D, out);
                if constexpr (CARRY) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) out[e] = col0 + cg + e < D ? out[e] - m[e] : 0.f;
                    *reinterpret_cast<f32x4 *>(&yn[yn_index(i, cg)]) = out;
                }
            }
        }
        if constexpr (CARRY) {
            // Gram of the updated, column-centred tail columns, in tri(i, j) order: a 4 x 4 tile of pairs, at
            // most 136 tiles, belongs to PARTS neighbouring threads that share its columns - as many as
            // the workgroup has for it.  (With one thread per tile ten of them walked all columns at n = 16
            // while the others waited: D = 1,003, 15.8 us per step, now 12.1.)  Every pair adds its columns
            // in the same order, so that equal particles stay at distance exactly 0.
            constexpr int kTiles = (NMAX / 4) * (NMAX / 4 + 1) / 2;
            constexpr int PARTS = kTiles * 16 <= 256 ? 16 : (kTiles * 4 <= 256 ? 4 : (kTiles * 2 <= 256 ? 2 : 1));
            block_sync<true>(); // (LDS only: nothing waits for the stores of the new columns)
            const int ng = n4 / 4, part = threadIdx.x % PARTS;
            int bi = 0, rem = threadIdx.x / PARTS;
            while (bi < ng && rem >= ng - bi) rem -= ng - bi++;
            const int bj = bi + rem;
            if (bi < ng) {
                float acc[4][4] = {};
                for (int c = 4 * part; c < 64; c += 4 * PARTS) {
                    f32x4 a[4], b[4];
    #pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        a[r] = *reinterpret_cast<const f32x4 *>(&yn[yn_index(4 * bi + r < n ? 4 * bi + r : 0, c)]);
                        b[r] = *reinterpret_cast<const f32x4 *>(&yn[yn_index(4 * bj + r < n ? 4 * bj + r : 0, c)]);
                    }
    #pragma unroll
                    for (int r = 0; r < 4; ++r)
    #pragma unroll
                        for (int t = 0; t < 4; ++t)
    #pragma unroll
                            for (int e = 0; e < 4; ++e) acc[r][t] = fmaf(a[r][e], b[t][e], acc[r][t]);
                }
    #pragma unroll
                for (int r = 0; r < 4; ++r)
    #pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const float v = row_sum<PARTS>(acc[r][t]);
                        const int i = 4 * bi + r, j = 4 * bj + t;
                        if ((4 * r + t) % PARTS == part && i <= j && j < n) gram_out[tri(i, j, n)] = v;
                    }
            }
        }
    }
};

// CARRY: additionally accumulate the Gram of the UPDATED columns, centred by the pre-update column
// mean (any per-column shift common to all particles leaves every d2 unchanged), and write one
// partial per workgroup (the last one is the tail's) to gram_out in the format of
// gram_mfma_kernel.  The next step can then skip its own pass over X.
//
// Instruction mix.  One wave per SIMD has to keep the matrix pipe, the vector ALU, LDS and the
// memory pipe busy at once, so the work of a tile is ordered as
//     M(0) | M(1)+E(0)+G(0) | M(2)+E(1)+G(1) | ... | E(NB-1)+G(NB-1)
// with M(b) = the MFMAs and epilogue of output block b, E(b) = the aligned stores of block b
// (LDS reads, address arithmetic, global stores) and G(b) = the Gram MFMAs of block b (CARRY).
// The pieces of one group are written interleaved and sit in one basic block (no branches in the
// steady-state tile), which lets the scheduler fill the MFMA shadows; a handful of wave-uniform
// branches inside the tile made it 20-30 % slower when tried.  The first tile of a range, which
// has to mask its left edge, is a separate, branchy instance of the same code.
// ROWS: the particles are n separately allocated rows; row addresses (and store alignments) come
// from a RowTable instead of i * ld (plain in-place step only, re-aligned stores).
// REM: n = 16 NB + R with 1 <= R <= 4.  A whole further block of 16 rows for those few particles
// would cost a tile the instructions of 16 more rows while it moves the bytes of R; instead the R
// remainder rows ride along in one register per array - lane (q, c) holds row 16 NB + q, columns
// 4c..4c+3, exactly one contraction step of the matrix instruction.  Their contribution to the
// other rows' phi is that one extra step per output block; their own phi, R x n x 64 products,
// is summed on the vector ALU (each lane over its own rows, then across the wave's four rows of
// lanes); they are stored as one more store group, and their pair sums (CARRY) are accumulated
// like those of a further block whose rows R..15 are zero.
template <int NB, bool EMIT, bool FULLROWS, bool CARRY, int STORE = kStoreStaged, bool ROWS = false, int PASS2 = kPass2Apart,
          bool REV = false, bool REM = false>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu((NB <= 2 && !FULLROWS) ? 2 : 1, (NB <= 2 && !FULLROWS) ? 2 : 1)))
void update_mfma_kernel(float *__restrict__ X, const float *__restrict__ G, float *__restrict__ PHI,
                        float *__restrict__ coef, DevState *__restrict__ st, int n,
                        int64_t D, int64_t ld, float eps, float *__restrict__ gram_out,
                        typename RowArg<ROWS>::type rt, UpdateArgs ua)
{
    // FROM_REGS says nothing of where rows start; what needs them on 128-byte boundaries asks for STREAM
    constexpr bool FROM_REGS = STORE != kStoreStaged, STREAM = STORE == kStoreLines;
    constexpr bool FUSED = PASS2 != kPass2Apart;
    constexpr int NMAX = 16 * NB + (REM ? 4 : 0); // particles
    static_assert(PASS2 != kPass2OnList || NMAX <= 32, "256 threads read a list of up to 32 particles");
    static_assert(PASS2 != kPass2OnSums || (NMAX <= 48 && FROM_REGS), "pass 2 on sums: problems that are never stored re-aligned");
    static_assert(!(CARRY && EMIT), "the Gram is carried only when X is updated");
    static_assert(!(ROWS && (EMIT || CARRY)), "separate rows: plain in-place step");
    static_assert(!REV || (CARRY && !FROM_REGS), "the mirrored walk exists for re-aligned stores with carried sums");
    static_assert(!REM || (FULLROWS && NB <= 3), "remainder rows come after full blocks");
    constexpr int NS = 4 * NB; // contraction steps = rows per lane
    constexpr int NBG = NB + (REM ? 1 : 0); // blocks as the pair sums see them
    constexpr int NPAIR = NBG * (NBG + 1) / 2;
    const int R = REM ? n - 16 * NB : 0; // remainder rows
    // [A operands: NB*NB*64 float4][4 waves x (cur + carry)]
    __shared__ __attribute__((aligned(16))) float lds[NB * NB * 64 * 4 + 4 * (kUpdCur + kUpdCarry)];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q = lane >> 4, c16 = lane & 15;
    float *__restrict__ OUT = EMIT ? PHI : X;
    const int64_t nfull = D >> 6; // full 64-column tiles
    // The tiles of this wave: t0, t0 + TS, ... < t1.  Re-aligned stores hand a row's tail from one
    // tile to the next through the wave's carry, so there each wave walks a contiguous range of
    // its own (TS = 1).  FROM_REGS has nothing to hand over: on request (ua.adjacent, the host's
    // choice) the workgroup owns a contiguous range and its four waves take adjacent tiles
    // (TS = 4), which makes the workgroup's accesses 1 KiB contiguous per row.
    const int64_t TS = (FROM_REGS && ua.adjacent != 0) ? 4 : 1;
    int64_t t0, t1;
    const bool has_tail = (nfull << 6) < D; // the last workgroup does the columns after the last full tile
    const int nwork = (int)gridDim.x - (has_tail ? 1 : 0);
    tile_range(nfull, ua.per, blockIdx.x, wave, TS == 4, t0, t1);
    const int64_t c_begin = t0 << 6;
    // visiting order: tiles t_first + k * t_step, k < ntiles.  FROM_REGS kernels take the direction
    // at run time; re-aligned stores hand a row's leftover from tile to tile, so their mirror
    // image, which walks right to left, is an instance of its own (REV).
    const int64_t ntiles = (t1 - t0 + TS - 1) / TS;
    const bool rev = REV || (FROM_REGS && ua.reverse != 0);
    const int64_t t_step = rev ? -TS : TS;
    const int64_t t_first = rev ? t0 + (ntiles - 1) * TS : t0;

    // lane part of every load address: row 4q, column 4c; the rest is wave-uniform
    const int64_t in_lane = ROWS ? (int64_t)(4 * c16) : (int64_t)(4 * q) * ld + 4 * c16;
    // stores: lane (rl = q, p = c16) writes row urow + q; a row's misalignment in floats is
    // (a0 + row * dm) mod 32 because every tile starts at a multiple of 32 columns
    const int64_t out_lane = ROWS ? (int64_t)(4 * c16) : (int64_t)q * ld + 4 * c16;
    const uint32_t dm = (uint32_t)ld & 31u;
    const uint32_t a0 = (uint32_t)(reinterpret_cast<uintptr_t>(OUT) >> 2) & 31u;
    // separate rows: where every row of X and of G starts, and X's alignment.  The table goes from the
    // kernel's arguments to LDS first, one coalesced read: read by every lane where it needs
    // an entry, the arguments (in host memory) took 5.5 us of each workgroup's start (n = 24, D =
    // 1,500,001: 125.8 -> 123.8 us per step; n = 13, D = 1,001: 27.3 -> 22.4 with pass 2 fused).
    int64_t xro[ROWS ? NS : 1], gro[ROWS ? NS : 1];
    __shared__ int64_t srow[ROWS ? kMaxN : 1], sgrow[ROWS ? kMaxN : 1];
    __shared__ int sri[ROWS ? kMaxN : 1];
    if constexpr (ROWS) {
        if (threadIdx.x < kMaxN) { // (entries beyond n repeat row 0)
            srow[threadIdx.x] = rt.x[ROWS ? threadIdx.x : 0];
            sgrow[threadIdx.x] = rt.g[ROWS ? threadIdx.x : 0];
            sri[threadIdx.x] = rt.ri[ROWS ? threadIdx.x : 0];
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int row = 16 * (s >> 2) + (s & 3) + 4 * q;
            xro[s] = srow[ROWS ? row : 0];
            gro[s] = sgrow[ROWS ? row : 0];
        }
    }

    // Software pipeline across tiles: the loads of tile t+1 are issued while tile t is being
    // multiplied.  Schedules chosen by measurement:
    //   XBUF (NB <= 2): the x rows of tile t+1 are loaded at the top of tile t into a second set of
    //     registers - small tiles are short, and the loads need the whole tile time to come back;
    //     otherwise into the registers of tile t as they fall free, the rows of block bi after
    //     that block's epilogue (more requests in flight only added HBM contention at n = 64);
    //   GBUF (NB <= 2, or CARRY): the same for the g rows.  Without it they are fetched as the last
    //     output block consumes them, i.e. issued last and needed first by the next tile; the
    //     longer tile of the carried sums then waits for them at every tile start (1.75 -> 1.72 ms
    //     at n = 64), while the plain update, which waits on memory anyway, is not helped.
    // The last tile of the range "prefetches" itself again (a few KB that nobody uses) so that the
    // steady-state code has no branch.
    constexpr bool XBUF = (NB <= 2);
    constexpr bool GBUF = (NB <= 2) || CARRY;
    f32x4 x[NS], z[NS], xn[XBUF ? NS : 1], gn[GBUF ? NS : 1];
    // remainder rows: this tile's x and z, and the next tile's x and g (always fetched a tile ahead)
    f32x4 xr = {0.f, 0.f, 0.f, 0.f}, zr = xr, xrn = xr, grn = xr;
    int64_t rem_x, rem_g; // row 16NB + q relative to in_lane (which has 4q ld on one array)
    if constexpr (ROWS) {
        rem_x = (REM && q < R) ? srow[ROWS ? 16 * NB + q : 0] : 0;
        rem_g = (REM && q < R) ? sgrow[ROWS ? 16 * NB + q : 0] : 0;
    } else {
        rem_x = rem_g = (int64_t)(16 * NB - 3 * q) * ld;
    }
    // G is read exactly once per step.  When no cache line is shared between tiles or rows
    // (STREAM) it is loaded with the streaming hint, which does not allocate on the way in:
    // measurably faster (a plain read-read-write stream over these buffers runs at 5.25 instead of
    // 5.08 TB/s), and it leaves the memory-side cache to X, which this kernel reads again in the
    // next step - at n = 32, D = 2,000,000 (X is 256 MB) that alone takes the update from 154 to
    // 119 us.  X itself is therefore loaded plainly.  With unaligned rows the line that a row
    // segment shares with the next tile has to stay cached, so nothing streams.
    auto load16x = [](const float *p) __attribute__((always_inline)) -> f32x4 {
        return *reinterpret_cast<const f32x4u *>(p);
    };
    auto load16g = [](const float *p) __attribute__((always_inline)) -> f32x4 {
        if constexpr (STREAM) return __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(p));
        else return *reinterpret_cast<const f32x4u *>(p);
    };
    // The rows of step s are all there and need no predicate.  Blocks before the last one never reach beyond n, but
    // only two blocks that are stored from the registers gain from knowing it (us per step, n = 24, padded, carried sums,
    // D = 300,007 31.7 -> 29.3, D = 1,000,003 66.0 -> 60.3, D = 2,000,003 112.4 -> 107.3; dense, D = 500,009, plain 51.6 -> 50.3,
    // phi, n = 28, D = 120,011 23.8 -> 22.3): with re-aligned stores and carried sums the registers do not suffice, and with three or
    // four blocks the compiler then moves the loads to where they cost 4 to 7 %.
    auto whole = [](int s) { return FULLROWS || (NB == 2 && FROM_REGS && s < NS - 4); };
    auto load_x = [&](const float *xt, int s) __attribute__((always_inline)) {
        const int urow = 16 * (s >> 2) + (s & 3); // uniform part of the row index
        if (whole(s) || urow + 4 * q < n) x[s] = load16x(xt + (ROWS ? xro[ROWS ? s : 0] : (int64_t)urow * ld));
    };
    auto load_g = [&](const float *gt, int s) __attribute__((always_inline)) {
        const int urow = 16 * (s >> 2) + (s & 3);
        if (whole(s) || urow + 4 * q < n) z[s] = load16g(gt + (ROWS ? gro[ROWS ? s : 0] : (int64_t)urow * ld));
    };
    auto load_next_rem = [&](const float *xt, const float *gt) __attribute__((always_inline)) {
        if constexpr (REM) {
            if (q < R) {
                xrn = load16x(xt + rem_x);
                grn = load16g(gt + rem_g);
            }
        }
    };
    auto load_next = [&](const float *xt, const float *gt) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int urow = 16 * (s >> 2) + (s & 3);
            if (whole(s) || urow + 4 * q < n) {
                if constexpr (XBUF) xn[s] = load16x(xt + (ROWS ? xro[ROWS ? s : 0] : (int64_t)urow * ld));
                if constexpr (GBUF) gn[s] = load16g(gt + (ROWS ? gro[ROWS ? s : 0] : (int64_t)urow * ld));
            }
        }
        load_next_rem(xt, gt);
    };
    // the extra workgroup: ragged tail only
    // (staged stores with two blocks of rows have no register to spare for loads across pass 2: three to five were
    // spilled in the loop)
    constexpr bool TAIL_EARLY = FUSED && (NB == 1 || FROM_REGS);
    const bool in_tail = has_tail && (int)blockIdx.x == nwork;
    TailColumns<NMAX, EMIT, CARRY, ROWS, FUSED> tail;
    auto first_loads = [&]() __attribute__((always_inline)) {
        if constexpr (TAIL_EARLY) {
            if (in_tail) tail.load(n, D, ld, X, G, srow, sgrow);
        }
        if (t0 < t1) {
            int64_t in_off = in_lane + (t_first << 6);
            opaque(in_off);
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                x[s] = f32x4{0.f, 0.f, 0.f, 0.f};
                z[s] = f32x4{0.f, 0.f, 0.f, 0.f};
                if constexpr (XBUF) xn[s] = f32x4{0.f, 0.f, 0.f, 0.f};
                else load_x(X + in_off, s);
                if constexpr (GBUF) gn[s] = f32x4{0.f, 0.f, 0.f, 0.f};
                else load_g(G + in_off, s);
            }
            load_next(X + in_off, G + in_off);
        }
    };

    // C (n x n) and rho (n): the handle's tables, or - FUSED - this workgroup's own copies in LDS,
    // computed by the prologue in the (still unused) staging area
    __shared__ __attribute__((aligned(16))) float cl[FUSED ? NMAX * NMAX + NMAX : 1];
    const float *Cm = coef + kOffC, *rhov = coef + kOffRho;
    const int cs = FUSED ? (n + 3) & ~3 : n; // rows of C (kernel_matrix pads its own with zeros)
    float c2h;
    if constexpr (FUSED) {
        constexpr int MAXN = NMAX <= 32 ? 32 : NMAX;
        typedef BwShared<MAXN, 256> Shared;
        static_assert(sizeof(Shared) % 16 == 0 && sizeof(Shared) + (PASS2 == kPass2OnList ? 4 * 256 * sizeof(double) : 0) <= 4 * (kUpdCur + kUpdCarry) * sizeof(float),
                      "pass 2 fits into the staging area");
        Shared &sh = *reinterpret_cast<Shared *>(lds + NB * NB * 64 * 4);
        double *red = reinterpret_cast<double *>(reinterpret_cast<char *>(&sh) + sizeof(Shared));
        kernel_matrix<256, MAXN, true>(
            sh, BwArgs{n, kModeGram, ua.h_fixed, ua.log_n1}, st, coef, cl, blockIdx.x == 0, c2h,
            [&](auto meanwhile) __attribute__((always_inline)) {
                if constexpr (PASS2 == kPass2OnList)
                    gather_sums<256, true, (NB == 1 || FULLROWS) && !ROWS ? 2 * kSumLoads : kSumLoads>(sh.S, red, ua.partials, ua.nparts, n, meanwhile, first_loads);
                else copy_sums<256, MAXN>(sh.S, ua.sums, n, meanwhile, first_loads);
            });
        // (the first tile is on its way while the list is summed and h and K are computed)
        Cm = cl;
        rhov = cl + n * cs;
    } else {
        c2h = st->two_over_h;
    }

    if (in_tail) {
        if constexpr (!TAIL_EARLY) tail.load(n, D, ld, X, G, srow, sgrow);
        float *tail_out = nullptr;
        if constexpr (CARRY) tail_out = gram_out + (int64_t)nwork * pair_stride(n); // after the workers' partials
        tail.run(OUT, Cm, cs, rhov, c2h, n, D, ld, eps, lds, tail_out, srow);
        return;
    }

    // With CARRY the staging block doubles as the Gram operand source (lane = row reads), so its
    // 16-byte granules are XOR-swizzled by the row; without it the block is plain row-major.
    auto cur_index = [](int rloc, int col) {
        return CARRY ? rloc * 64 + ((((col >> 2) ^ rloc) & 15) << 2) + (col & 3) : rloc * 64 + col;
    };
    f32x4 accg[CARRY ? NPAIR : 1];
    if constexpr (CARRY) {
#pragma unroll
        for (int p = 0; p < NPAIR; ++p) accg[p] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const float inv_n = 1.0f / (float)n;

    f32x4 *As4 = reinterpret_cast<f32x4 *>(lds);
    float *cur = lds + NB * NB * 64 * 4 + wave * (kUpdCur + kUpdCarry);
    float *carry = cur + kUpdCur;
    // A operands of v_mfma_f32_16x16x4_f32 for output block bi, steps 4sg..4sg+3, as one float4
    // per lane: for step s = 4sg + k lane (q = l/16, m = l%16) holds C[16bi + m][16sg + 4q + k]
    // (zero beyond n: rows and columns of the padding take no part)
    // FULLROWS: all loads go out before the first result is used - one trip to memory, where a loop made
    // four at n = 64 (3.4 us, now 1.1).  Padded blocks keep guarded loads: with clamped ones the
    // whole kernel came out slower (separate rows, n = 24, D = 1,500,001: 124.8 -> 132.4 us per step).
    constexpr int NA = (NB * NB * 64 + 255) / 256;
    f32x4 av[NA];
#pragma unroll
    for (int it = 0; it < NA; ++it) {
        const int e0 = (int)threadIdx.x + 256 * it, e = e0 < NB * NB * 64 ? e0 : 0;
        const int l = e & 63, sg = (e >> 6) % NB, bi = (e >> 6) / NB;
        const int i = 16 * bi + (l & 15), j0 = 16 * sg + 4 * (l >> 4);
        if constexpr (FULLROWS) {
            av[it] = *reinterpret_cast<const f32x4u *>(Cm + i * cs + j0);
        }
    }
    // rho of this lane's rows: in registers, or (RHO_LDS) in LDS, four of a block at a time, where the registers
    // do not suffice: with two waves per SIMD there are 256, and a spilled one read back in every tile
    // waits for all loads of the next tile, which are older (n = 24, D = 3,000,001, dense rows:
    // 203 us per step with three spilled, 188 now; n = 21 194 -> 172, n = 30, D = 1,000,003 88 -> 82).
    constexpr bool RHO_LDS = CARRY && !FROM_REGS && !FULLROWS && NB == 2;
    __shared__ __attribute__((aligned(16))) float rho_lds[RHO_LDS ? 16 * NB : 4];
    float rho[RHO_LDS ? 1 : NS];
    if constexpr (RHO_LDS) {
        if (threadIdx.x < 16 * NB) rho_lds[threadIdx.x] = (int)threadIdx.x < n ? rhov[threadIdx.x] : 0.f;
    } else {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int row = 16 * (s >> 2) + 4 * q + (s & 3);
            rho[s] = (FULLROWS || row < n) ? rhov[row] : 0.f;
        }
    }
#pragma unroll
    for (int it = 0; it < NA; ++it) {
        const int e = (int)threadIdx.x + 256 * it;
        if constexpr (!FULLROWS) {
            const int l = e & 63, sg = (e >> 6) % NB, bi = (e >> 6) / NB;
            const int i = 16 * bi + (l & 15), j0 = 16 * sg + 4 * (l >> 4);
            if (e < NB * NB * 64)
#pragma unroll
            for (int k = 0; k < 4; ++k) av[it][k] = (i < n && j0 + k < n) ? Cm[i * cs + j0 + k] : 0.f;
        }
        if (e < NB * NB * 64) As4[e] = av[it];
    }
    // remainder rows.  arem: the A operand of their one contraction step for output block bi -
    // lane (q, m) holds C[16bi + m][16NB + q].  crem: for remainder row r and lane row q the
    // coefficients C[16NB + r][.] of the rows that a lane of that q holds, in the order of its
    // registers (NS rows of the full blocks, then row 16NB + q), padded to a multiple of four.
    constexpr int CREM = NS + 4;
    __shared__ float arem[REM ? NB * 64 : 1];
    __shared__ __attribute__((aligned(16))) float crem[REM ? 16 * CREM : 4];
    float rho_r = 0.f;
    if constexpr (REM) {
        for (int e = threadIdx.x; e < NB * 64; e += 256) {
            const int l = e & 63, bi = e >> 6;
            arem[e] = ((l >> 4) < R) ? Cm[(16 * bi + (l & 15)) * cs + 16 * NB + (l >> 4)] : 0.f;
        }
        for (int e = threadIdx.x; e < 16 * CREM; e += 256) {
            const int s = e % CREM, rq = e / CREM, r = rq >> 2, qq = rq & 3;
            float v = 0.f;
            if (r < R) {
                if (s < NS) v = Cm[(16 * NB + r) * cs + 16 * (s >> 2) + 4 * qq + (s & 3)];
                else if (s == NS && qq < R) v = Cm[(16 * NB + r) * cs + 16 * NB + qq];
            }
            crem[e] = v;
        }
        if (q < R) rho_r = rhov[16 * NB + q];
    }
    block_sync<FUSED>(); // (does not wait for the first tile's loads)
    if constexpr (!FUSED) first_loads();

    auto process_tile = [&](auto first_tag, int64_t tile, bool last) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(first_tag)::value;
        const int64_t base = tile << 6;
        const int64_t next = last ? tile : tile + t_step;
        int64_t in_off = in_lane + (next << 6);
        int64_t out_off = out_lane + base;
        const int qv = q; // (the per-row store offsets are tile-invariant and may be hoisted)
        opaque(in_off);
        const float *xt = X + in_off, *gt = G + in_off;
        float *ot = OUT + out_off;

        if constexpr (XBUF || GBUF) { // this tile's data becomes current, the next tile's loads go out
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                if constexpr (XBUF) x[s] = xn[s];
                if constexpr (GBUF) z[s] = gn[s];
            }
            if constexpr (REM) {
                xr = xrn;
                zr = grn;
            }
            load_next(xt, gt);
        } else if constexpr (REM) {
            xr = xrn;
            zr = grn;
            load_next_rem(xt, gt);
        }
        // the lane's 16 bytes of a row: where it loaded x from
        auto store_direct = [&](int64_t row_off, f32x4 v) __attribute__((always_inline)) {
            float *dst = OUT + in_lane + base + row_off;
            if constexpr (STREAM) __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(dst));
            else *reinterpret_cast<f32x4u *>(dst) = v;
        };

        f32x4 mg[CARRY ? 4 : 1];      // pre-update column means in the Gram operand layout
        f32x4 ag[CARRY ? NBG : 1][4]; // Gram operands of the blocks finished so far
        if constexpr (CARRY) {
            f32x4 m = x[0];
#pragma unroll
            for (int s = 1; s < NS; ++s) m += x[s];
            if constexpr (REM) m += xr; // zero in the lanes without a remainder row
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                m[e] = sum_over_rows(m[e]) * inv_n;
            }
            // through the (currently idle) staging block: lane (q, c) knows columns 4c..4c+3,
            // the Gram layout wants columns 4(4st + q)..+3
            if (q == 0) *reinterpret_cast<f32x4 *>(&cur[4 * c16]) = m;
#pragma unroll
            for (int st4 = 0; st4 < 4; ++st4) mg[st4] = *reinterpret_cast<const f32x4 *>(&cur[4 * (4 * st4 + q)]);
        }
#pragma unroll
        for (int s = 0; s < NS; ++s) z[s] -= c2h * x[s];
        // phi of the remainder rows: lane (q, c) ends up with that of row 16NB + q
        f32x4 phir = {0.f, 0.f, 0.f, 0.f};
        if constexpr (REM) {
            zr -= c2h * xr;
            for (int r = 0; r < R; ++r) { // wave-uniform trip count
                const float *cr = crem + (4 * r + q) * CREM;
                f32x4 p = cr[NS] * zr;
#pragma unroll
                for (int sg = 0; sg < NB; ++sg) {
                    const f32x4 c4 = *reinterpret_cast<const f32x4 *>(cr + 4 * sg);
#pragma unroll
                    for (int k = 0; k < 4; ++k) p += c4[k] * z[4 * sg + k];
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) p[e] = sum_over_rows(p[e]);
                if (q == r) phir = p;
            }
        }

        // E(b), one of its four store groups: 4 rows x 256 B, lane (rl = q, p = c16)
        auto emit_group = [&](int b, int k) __attribute__((always_inline)) {
            const int urow = 16 * b + 4 * k;     // uniform part of the row index
            const int rloc = 4 * k + qv;         // row within the block
            const int row = urow + qv;
            const int ri = ROWS ? sri[ROWS ? row : 0] : (int)((a0 + (uint32_t)row * dm) & 31u);
            // the row's 64-float window starts on a line boundary: ri floats before the tile, or
            // (REV) 32 - ri floats into it, where it takes in the head of the tile to the right
            const int sh = REV ? ((32 - ri) & 31) : -ri;
            const int o0 = 4 * c16 + sh;         // window offset relative to the tile start
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int o = o0 + e; // one address, so nothing is read outside the arrays
                if constexpr (REV) v[e] = cur[(o >= 64) ? (kUpdCur + row * 32 + o - 64) : cur_index(rloc, o)];
                else v[e] = cur[(o < 0) ? (kUpdCur + row * 32 + 32 + o) : cur_index(rloc, o)];
            }
            if ((FULLROWS && !(REM && b == NB)) || row < n) {
                float *dst = ot + (ROWS ? srow[ROWS ? row : 0] : (int64_t)urow * ld) + sh;
                if constexpr (!FIRST) {
                    __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(dst));
                } else { // the end of the range the walk starts from: nothing beyond it is ours
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (REV ? (o0 + e < 64) : (o0 + e >= 0)) dst[e] = v[e];
                }
            }
        };
        // after E(b): the block's last (REV: first) 32 columns become the carry of its 16 rows
        auto carry_copy = [&](int b) __attribute__((always_inline)) {
            const int rloc = lane >> 2, cc = (REV ? 0 : 32) + 8 * (lane & 3);
            const f32x4 v0 = *reinterpret_cast<const f32x4 *>(&cur[cur_index(rloc, cc)]);
            const f32x4 v1 = *reinterpret_cast<const f32x4 *>(&cur[cur_index(rloc, cc + 4)]);
            float *dstc = &carry[(16 * b + rloc) * 32 + (cc & 31)];
            *reinterpret_cast<f32x4 *>(dstc) = v0;
            *reinterpret_cast<f32x4 *>(dstc + 4) = v1;
        };
        // G(b), the part that pairs block b with block b0 <= b
        auto gram_pair = [&](int b0, int b) __attribute__((always_inline)) {
            const int pidx = b0 * NBG - (b0 * (b0 - 1)) / 2 + (b - b0);
#pragma unroll
            for (int st4 = 0; st4 < 4; ++st4)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    accg[pidx] = __builtin_amdgcn_mfma_f32_16x16x4f32(ag[b0][st4][e], ag[b][st4][e], accg[pidx], 0, 0, 0);
        };

#pragma unroll
        for (int bi = 0; bi < NB; ++bi) {
            // M(bi), interleaved with E(bi-1) and G(bi-1)
            f32x4 acc[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int sg = 0; sg < NB; ++sg) {
                const f32x4 a4 = As4[(bi * NB + sg) * 64 + lane];
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a4[k], z[4 * sg + k][t], acc[t], 0, 0, 0);
                if (REM && sg == NB - 1) { // the remainder rows' contraction step
                    const float ar = arem[bi * 64 + lane];
#pragma unroll
                    for (int t = 0; t < 4; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(ar, zr[t], acc[t], 0, 0, 0);
                }
                if (!GBUF && bi == NB - 1) { // z rows 4sg..4sg+3 are dead: fetch the next tile's g
#pragma unroll
                    for (int k = 0; k < 4; ++k) load_g(gt, 4 * sg + k);
                }
                if (bi > 0) {
                    // the four store groups of the previous block are spread over the NB step groups
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (!FROM_REGS && k * NB / 4 == sg) emit_group(bi - 1, k);
                    if constexpr (CARRY) {
                        if (sg < bi) gram_pair(sg, bi - 1); // pairs (0..bi-1, bi-1): one per step group
                    }
                }
            }
            if (!FROM_REGS && bi > 0) carry_copy(bi - 1);
            // epilogue for rows 16bi + 4q + r, then stage the block in LDS
            f32x4 rho4;
            if constexpr (RHO_LDS) rho4 = *reinterpret_cast<const f32x4 *>(&rho_lds[16 * bi + 4 * q]);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int s = 4 * bi + r;
                f32x4 o;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float phi = fmaf(RHO_LDS ? rho4[r] : rho[RHO_LDS ? 0 : s], x[s][t], acc[t][r]);
                    o[t] = EMIT ? phi : fmaf(eps, phi, x[s][t]);
                }
                if constexpr (FROM_REGS) {
                    if (whole(s) || 16 * bi + 4 * q + r < n) store_direct(ROWS ? xro[ROWS ? s : 0] : (int64_t)(16 * bi + r) * ld, o);
                }
                if constexpr (!FROM_REGS || CARRY) // staged for the re-aligned stores and/or as Gram operands
                    *reinterpret_cast<f32x4 *>(&cur[cur_index(4 * q + r, 4 * c16)]) = o;
            }
            if constexpr (!XBUF) { // x rows of this block are dead: fetch the next tile's
#pragma unroll
                for (int r = 0; r < 4; ++r) load_x(xt, 4 * bi + r);
            }
            if constexpr (CARRY) {
                // lane (q, rr = c16) takes row rr of this block, columns 4(4st + q)..+3, centred
#pragma unroll
                for (int st4 = 0; st4 < 4; ++st4)
                    ag[bi][st4] = *reinterpret_cast<const f32x4 *>(&cur[cur_index(c16, 4 * (4 * st4 + q))]) - mg[st4];
            }
        }
        // E(NB-1) interleaved with G(NB-1)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if constexpr (!FROM_REGS) emit_group(NB - 1, k);
            if constexpr (CARRY) {
#pragma unroll
                for (int b0 = 0; b0 < NB; ++b0)
                    if (b0 * 4 / NB == k) gram_pair(b0, NB - 1);
            }
        }
        if constexpr (!FROM_REGS) carry_copy(NB - 1);
        if constexpr (REM) {
            // the remainder rows: epilogue, staging as rows 0..3 of a further block, one store group
            f32x4 o;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float phi = fmaf(rho_r, xr[t], phir[t]);
                o[t] = EMIT ? phi : fmaf(eps, phi, xr[t]);
            }
            if constexpr (FROM_REGS) {
                if (q < R) store_direct(rem_x, o);
            }
            if constexpr (!FROM_REGS || CARRY) *reinterpret_cast<f32x4 *>(&cur[cur_index(q, 4 * c16)]) = o;
            if constexpr (CARRY) {
#pragma unroll
                for (int st4 = 0; st4 < 4; ++st4) {
                    const f32x4 v = *reinterpret_cast<const f32x4 *>(&cur[cur_index(c16 & 3, 4 * (4 * st4 + q))]) - mg[st4];
                    ag[NB][st4] = (c16 < R) ? v : f32x4{0.f, 0.f, 0.f, 0.f};
                }
            }
            if constexpr (!FROM_REGS) emit_group(NB, 0);
            if constexpr (CARRY) {
#pragma unroll
                for (int b0 = 0; b0 <= NB; ++b0) gram_pair(b0, NB);
            }
            if constexpr (!FROM_REGS) carry_copy(NB);
        }
    };

    if constexpr (FROM_REGS) { // no left edge to mask
        int64_t tile = t_first;
        // Two waves per SIMD fetch their instructions faster or slower with the place of this loop against the 64-byte lines:
        // us per step, n = 24, padded, carried sums, with 12 instructions between a line's start and the compiler's own
        // before the loop, with 7 and where it falls: D = 300,007 29.3, 29.6 and 29.4, D = 1,000,003 60.3, 61.8 and 61.0, n = 21
        // 59.1, 59.9 and 60.1.  Other instances stay where they fall.  (What the compiler puts in between is that of ROCm 7.2; with another
        // one the number is to be found again, and one that does not fit costs those 1 to 2 %, nothing else.)
        if constexpr (STREAM && CARRY && NB == 2 && !FULLROWS) asm volatile(".p2align 6\n\t.rept 12\n\ts_nop 0\n\t.endr");
        for (int64_t k = 0; k < ntiles; ++k, tile += t_step) process_tile(std::false_type{}, tile, k + 1 == ntiles);
    } else if (t0 < t1) {
        process_tile(std::true_type{}, t_first, ntiles == 1);
        int64_t tile = t_first + t_step;
        for (int64_t k = 1; k < ntiles; ++k, tile += t_step) process_tile(std::false_type{}, tile, k + 1 == ntiles);
    }

    // flush: the last r_i columns of the range (REV: its first 32 - r_i) are still in the carry
    if (!FROM_REGS && t1 > t0) {
        const int64_t c_end = t1 << 6;
        for (int idx = lane; idx < 16 * NBG * 32; idx += 64) {
            const int row = idx >> 5, cc = idx & 31;
            const int ri = ROWS ? sri[ROWS ? row : 0] : (int)((a0 + (uint32_t)row * dm) & 31u);
            if constexpr (REV) {
                if (row < n && cc < ((32 - ri) & 31)) OUT[(int64_t)row * ld + c_begin + cc] = carry[row * 32 + cc];
            } else {
                if (row < n && cc >= 32 - ri && c_end - 32 + cc >= c_begin)
                    OUT[(ROWS ? srow[ROWS ? row : 0] : (int64_t)row * ld) + c_end - 32 + cc] = carry[row * 32 + cc];
            }
        }
    }

    if constexpr (CARRY) {
        // One partial per workgroup, upper triangle in tri(i, j) order (zeros if all four ranges
        // were empty): the waves' sums meet in their staging areas, which are free by now, and
        // wave p mod 4 adds up and writes block pair p.
        static_assert(NPAIR * 4 * 64 <= kUpdCur + kUpdCarry, "the staging area holds a wave's Gram sums");
#pragma unroll
        for (int p = 0; p < NPAIR; ++p) {
#pragma unroll
            for (int r = 0; r < 4; ++r) cur[(p * 4 + r) * 64 + lane] = accg[p][r];
        }
        __syncthreads();
        const float *all = lds + NB * NB * 64 * 4;
        float *out = gram_out + (int64_t)blockIdx.x * pair_stride(n);
        int p = 0;
#pragma unroll
        for (int b = 0; b < NBG; ++b) {
#pragma unroll
            for (int b2 = b; b2 < NBG; ++b2) {
                if ((p & 3) == wave) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int i = 16 * b + 4 * q + r;
                        const int j = 16 * b2 + c16;
                        const int e = (p * 4 + r) * 64 + lane;
                        const float v = (all[e] + all[(kUpdCur + kUpdCarry) + e]) +
                                        (all[2 * (kUpdCur + kUpdCarry) + e] + all[3 * (kUpdCur + kUpdCarry) + e]);
                        if (i <= j && j < n) out[tri(i, j, n)] = v;
                    }
                }
                ++p;
            }
        }
    }
}

} // namespace svgd
