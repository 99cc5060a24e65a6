// Pass 2: from the reduced pair sums to d2, the median-heuristic bandwidth h, the RBF kernel
// matrix K, its row sums, and the coefficient tables of the update kernels.  By one workgroup as a kernel of its
// own, by every workgroup or every wave for itself as the start of an update (two implementations: kernel_matrix,
// and wave_kernel_matrix up to 12 particles); fp64 throughout (at most 2016 pairs: the cost is nil and none
// of the 1e-5 budget on h and K is spent here).  Nothing returns to the host: the paper's routine (App. B.2) reads each kernel
// value back to the host, one synchronisation per pair; here K stays on the device.
#pragma once
#include <type_traits>

#include "common.hpp"

namespace svgd {

constexpr int kBwThreads = 1024;
// Selection among more than kCounted values: they are spread over kBuckets buckets by value, and a bucket of at
// most kSelDirect values is ranked directly.
constexpr int kSelDirect = 64;
constexpr int kBuckets = 256;

__device__ inline int pair_index(int i, int j, int n) { return i * n - (i * (i + 1)) / 2 + (j - i - 1); } // i < j

// LDS of pass 2 for at most MAXN particles and THREADS threads.
template <int MAXN, int THREADS>
struct BwShared {
    static constexpr int kPairs = MAXN * (MAXN - 1) / 2;
    static constexpr int kPr = (kPairs > 2 * kWave) ? kPairs : 2 * kWave; // (count_ranks reads that many)
    double S[MAXN * (MAXN + 1) / 2]; // reduced pair sums, later K per pair
    __attribute__((aligned(16))) double pr[kPr]; // d2 per unordered pair i < j
    double list[kSelDirect];         // the final short list
    double sel[2];
    unsigned long long mm[4];        // min / max bit patterns, two alternating slots
    __attribute__((aligned(16))) unsigned hist[kBuckets];
    unsigned counters[kSelDirect];   // partial ranks of the list elements
    unsigned misc[4];                // 0: length of the list
    __attribute__((aligned(16))) unsigned short counts[THREADS / kWave][2 * kWave]; // count_ranks
};

// A double moved across lanes by a DPP control word (both halves).
template <int CTRL>
__device__ inline double dpp_f64(double v)
{
    int lo = __double2loint(v), hi = __double2hiint(v);
    lo = __builtin_amdgcn_update_dpp(0, lo, CTRL, 0xF, 0xF, false);
    hi = __builtin_amdgcn_update_dpp(0, hi, CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

__device__ inline double readlane_f64(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Minimum and maximum over the 64 lanes of a wave, returned in every lane (four DPP steps inside
// each row of 16 lanes, then the four rows; no LDS traffic).
__device__ inline void wave_minmax(double &mn, double &mx)
{
#define SVGD_MM_STEP(C)                                                                            \
    mn = fmin(mn, dpp_f64<C>(mn));                                                                 \
    mx = fmax(mx, dpp_f64<C>(mx));
    SVGD_MM_STEP(0xB1)  // quad_perm [1,0,3,2]
    SVGD_MM_STEP(0x4E)  // quad_perm [2,3,0,1]
    SVGD_MM_STEP(0x141) // row_half_mirror
    SVGD_MM_STEP(0x140) // row_mirror
#undef SVGD_MM_STEP
    mn = fmin(fmin(readlane_f64(mn, 0), readlane_f64(mn, 16)), fmin(readlane_f64(mn, 32), readlane_f64(mn, 48)));
    mx = fmax(fmax(readlane_f64(mx, 0), readlane_f64(mx, 16)), fmax(readlane_f64(mx, 32), readlane_f64(mx, 48)));
}

// Sum over the 16 lanes of each row of a wave (or over aligned groups of L = 8 lanes), in every lane.
template <int L = 16>
__device__ inline double row_sum_f64(double v)
{
    v += dpp_f64<0xB1>(v);
    v += dpp_f64<0x4E>(v);
    v += dpp_f64<0x141>(v);
    if constexpr (L > 8) v += dpp_f64<0x140>(v);
    return v;
}

// The value of lane l ^ M, M = 16 or 32, in lane l: the row-swap instructions, no LDS.
template <int M>
__device__ inline double swap_f64(double v)
{
    static_assert(M == 16 || M == 32, "whole rows of lanes");
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    const bool upper = (threadIdx.x & M) != 0;
    unsigned l, h;
    if constexpr (M == 16) {
        const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false), b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        l = upper ? a[0] : a[1];
        h = upper ? b[0] : b[1];
    } else {
        const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false), b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        l = upper ? a[0] : a[1];
        h = upper ? b[0] : b[1];
    }
    return __hiloint2double((int)h, (int)l);
}

// Inclusive prefix sum over the 64 lanes of a wave: four DPP shift-adds inside each row of 16
// lanes, then the totals of the lower rows (read from lanes 15, 31, 47) are added to the upper ones.
__device__ inline unsigned wave_inclusive_scan(unsigned x)
{
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true); // row_shr:1, 0 shifted in
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true); // row_shr:2
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true); // row_shr:4
    x += (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true); // row_shr:8
    const unsigned t0 = (unsigned)__builtin_amdgcn_readlane((int)x, 15);
    const unsigned t1 = (unsigned)__builtin_amdgcn_readlane((int)x, 31);
    const unsigned t2 = (unsigned)__builtin_amdgcn_readlane((int)x, 47);
    const int row = (threadIdx.x & 63) >> 4;
    return x + (row >= 1 ? t0 : 0u) + (row >= 2 ? t1 : 0u) + (row >= 3 ? t2 : 0u);
}

// Non-negative doubles (and +inf) order like their bit patterns read as unsigned integers.
__device__ inline unsigned long long f64_key(double v) { return (unsigned long long)__double_as_longlong(v); }
__device__ inline double key_f64(unsigned long long k) { return __longlong_as_double((long long)k); }

// minimum and maximum of the calling waves' values into two LDS words: DPP inside the wave, one
// atomic per wave on the bit patterns (mx >= 0)
__device__ inline void minmax_to_lds(double mn, double mx, unsigned long long *slot)
{
    wave_minmax(mn, mx);
    if ((threadIdx.x & 63) == 0) {
        atomicMin(&slot[0], f64_key(mn));
        atomicMax(&slot[1], f64_key(mx));
    }
}

// Workgroup barrier.  LO ("LDS only"): for code whose barriers order nothing but LDS traffic -
// it waits for this wave's LDS operations and not for its outstanding global loads, which
// __syncthreads() would (the fused step has its first tile's loads in flight during pass 2).
template <bool LO>
__device__ inline void block_sync()
{
    if constexpr (LO) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else __syncthreads();
}

// Rank (position in sorted order, ties by index) of every element of a short list: len <=
// kSelDirect values, +inf in the entries from len to kSelDirect; the elements of the wanted ranks
// are stored to sel.  E >= len threads take an element each and THREADS / E of them share one, each
// comparing it with a slice of the list; the partial ranks meet in `counters`, which must be zero
// on entry.  E and with it the slice follow len.  A barrier lies between the writes of the list and this call.
template <int THREADS, bool LO>
__device__ inline void rank_directly(const double *list, int len, int below, int r_lo, int r_hi, double *sel,
                                     unsigned *counters)
{
    const int tid = threadIdx.x;
    const int lg = (len <= 32 && THREADS <= 256) ? 5 : 6; // the slices stay multiples of four
    const int e = tid & ((1 << lg) - 1), part = tid >> lg;
    const int slice = (1 << (2 * lg)) / THREADS, u0 = part * slice;
    const double v = list[e];
    unsigned cnt = 0;
    for (int k = u0; k < u0 + slice; k += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const double w = list[k + u];
            cnt += (w < v || (w == v && k + u < e)) ? 1u : 0u;
        }
    }
    if (cnt) atomicAdd(&counters[e], cnt);
    block_sync<LO>();
    if (tid < len && part == 0) {
        const int rank = below + (int)counters[e];
        if (rank == r_lo) sel[0] = v;
        if (rank == r_hi) sel[1] = v;
    }
}

// The values of rank r_lo and r_hi (0-based, r_hi = r_lo or r_lo + 1) among Pp values, written to
// sh.sel[0] and sh.sel[1].  Exact selection without sorting: thread t holds the values t + u *
// THREADS, which are spread over kBuckets buckets by value, bucket(v) = floor((v - a) * kBuckets /
// (b - a)) clamped, [a, b] = minimum and maximum of the set - monotone in v, so all of bucket k
// lies below all of bucket k + 1.  Every wave then scans all bucket counts by itself (four per
// lane: one LDS read and a DPP scan, where sharing the scan among the waves took two more
// barriers), and the bucket that holds the wanted ranks becomes the active set, gathered into a
// list and ranked directly once it is small.  a and b, the smallest and the largest FINITE value, fall
// into the first and the last bucket and infinities into the last, so the set shrinks at every
// level until all of it is equal; 2016 values (n = 64) take one level and a short list.  Ranks that
// fall into two different buckets are the maximum of the one and the minimum of the other.
// Contract: called by all THREADS threads with kCounted < Pp <= VPT * THREADS and values that are
// not negative and not NaN, after a barrier behind which
//   - sh.mm[0] / mm[1] hold the bit patterns of a / b, mm[2] = ~0, mm[3] = 0,
//   - sh.hist, sh.counters and sh.misc are zero, sh.list is +inf (kSelDirect entries each)
// (pass 2 prepares all of this on its way).
template <int THREADS, int VPT, bool LO, class Shared>
__device__ inline void select_two_ranks(Shared &sh, const double (&v)[VPT], int Pp, int r_lo, int r_hi)
{
    static_assert(kBuckets == 4 * kWave, "four buckets per lane");
    const int tid = threadIdx.x, lane = tid & 63;
    const unsigned long long kmax = ~0ull;
    const double inf = __builtin_huge_val();
    bool act[VPT];
#pragma unroll
    for (int u = 0; u < VPT; ++u) act[u] = tid + u * THREADS < Pp;
    int below = 0; // values known to be smaller than the whole active set
    int size = Pp; // of the active set

    for (int level = 0;; ++level) {
        const int slot = (level & 1) * 2;
        if (level > 0) {
            // refine: clear what the previous level used (its last reads lie behind the barrier at
            // its end), find the range of the narrowed set
            for (int e = tid; e < kBuckets; e += THREADS) sh.hist[e] = 0;
            if (tid == 0) { // the other slot, for the level after this one
                sh.mm[2 - slot] = kmax;
                sh.mm[3 - slot] = 0ull;
            }
            double mn = inf, mx = 0.0;
#pragma unroll
            for (int u = 0; u < VPT; ++u) {
                mn = fmin(mn, act[u] ? v[u] : inf);
                mx = fmax(mx, (act[u] && v[u] < inf) ? v[u] : 0.0);
            }
            minmax_to_lds(mn, mx, &sh.mm[slot]);
            block_sync<LO>();
        }
        const double a = key_f64(sh.mm[slot]), b = key_f64(sh.mm[slot + 1]);
        // (one finite value only: it goes to the first bucket; no finite value: all of them do)
        const double scale = a < b ? (double)kBuckets / (b - a) : 1.0;
        int k[VPT];
#pragma unroll
        for (int u = 0; u < VPT; ++u) {
            k[u] = (int)fmin(fmax((v[u] - a) * scale, 0.0), (double)(kBuckets - 1)); // (a NaN, inf - inf, becomes 0)
            if (act[u]) atomicAdd(&sh.hist[k[u]], 1u);
        }
        block_sync<LO>();
        // the buckets holding the wanted ranks (ranks relative to the active set)
        const uint4 c = *reinterpret_cast<const uint4 *>(&sh.hist[4 * lane]);
        const unsigned e1 = c.x, e2 = e1 + c.y, e3 = e2 + c.z, e4 = e3 + c.w;
        const unsigned excl = wave_inclusive_scan(e4) - e4;
        auto locate = [&](unsigned rank, int &bucket, int &before, int &count) __attribute__((always_inline)) {
            const unsigned r = rank - excl; // wraps for the lanes above the wanted one
            const int src = __ffsll(__ballot(rank >= excl && r < e4)) - 1; // the active set holds the rank: one lane
            const int sub = r < e1 ? 0 : (r < e2 ? 1 : (r < e3 ? 2 : 3));
            const unsigned lo = sub == 0 ? 0u : (sub == 1 ? e1 : (sub == 2 ? e2 : e3));
            const unsigned hi = sub == 0 ? e1 : (sub == 1 ? e2 : (sub == 2 ? e3 : e4));
            bucket = __builtin_amdgcn_readlane(4 * lane + sub, src);
            before = __builtin_amdgcn_readlane((int)(excl + lo), src);
            count = __builtin_amdgcn_readlane((int)(hi - lo), src);
        };
        int b_lo, b_hi, before, before_hi, cnt, cnt_hi;
        locate((unsigned)(r_lo - below), b_lo, before, cnt);
        locate((unsigned)(r_hi - below), b_hi, before_hi, cnt_hi);
        if (b_lo != b_hi) {
            // adjacent ranks in different buckets: the largest value of the one, the smallest of the
            // other (the other min/max slot is prepared and unused at this point)
            double mx = 0.0, mn = inf;
#pragma unroll
            for (int u = 0; u < VPT; ++u) {
                if (act[u] && k[u] == b_lo) mx = fmax(mx, v[u]);
                if (act[u] && k[u] == b_hi) mn = fmin(mn, v[u]);
            }
            minmax_to_lds(mn, mx, &sh.mm[2 - slot]);
            block_sync<LO>();
            if (tid == 0) {
                sh.sel[0] = key_f64(sh.mm[3 - slot]);
                sh.sel[1] = key_f64(sh.mm[2 - slot]);
            }
            return;
        }
        if (cnt == size) { // nothing left to tell apart
            if (tid == 0) {
                sh.sel[0] = a;
                sh.sel[1] = a;
            }
            return;
        }
        below += before;
        size = cnt;
#pragma unroll
        for (int u = 0; u < VPT; ++u) act[u] = act[u] && k[u] == b_lo;
        if (cnt <= kSelDirect) { // gather the bucket into a list and rank it
#pragma unroll
            for (int u = 0; u < VPT; ++u)
                if (act[u]) sh.list[atomicAdd(&sh.misc[0], 1u)] = v[u];
            block_sync<LO>();
            rank_directly<THREADS, LO>(sh.list, cnt, below, r_lo, r_hi, sh.sel, sh.counters);
            return;
        }
        block_sync<LO>(); // all reads of hist are done before the next level clears it
    }
}

// The same for at most kCounted values: every wave counts, for all of them (two per lane), the smaller ones in its
// share of the list; the shares meet in LDS, and behind one barrier every wave has all counts and picks the values
// by itself - one of rank r is one whose count is r, or with ties the largest count below r.  The
// buckets above take six barriers for it (120 values: 3.2 thousand cycles of a prologue of 14; us per step,
// padded, carried sums, n = 13, D = 1,003 8.7 -> 7.4, n = 16 8.4 -> 7.4, the list's loads in one trip included).  Choosing
// pivots and counting them by ballots, without LDS, took 4.4 thousand.  sh.pr holds kCounted values, +inf behind the last.
constexpr int kCounted = 2 * kWave;
template <int THREADS, bool LO, class Shared>
__device__ inline void count_ranks(Shared &sh, int Pp, int r_lo, int r_hi, double &lo, double &hi)
{
    constexpr int WAVES = THREADS / kWave, SHARE = kCounted / WAVES;
    static_assert(SHARE % 2 == 0, "two values per read");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double v[2];
    int cnt[2] = {0, 0};
#pragma unroll
    for (int u = 0; u < 2; ++u) v[u] = sh.pr[lane + kWave * u];
    if (wave * SHARE < Pp) {
#pragma unroll
        for (int k = 0; k < SHARE; k += 2) {
            const double2 w = *reinterpret_cast<const double2 *>(&sh.pr[wave * SHARE + k]);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                cnt[u] += w.x < v[u] ? 1 : 0;
                cnt[u] += w.y < v[u] ? 1 : 0;
            }
        }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) sh.counts[wave][lane + kWave * u] = (unsigned short)cnt[u];
    block_sync<LO>();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        cnt[u] = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) cnt[u] += sh.counts[w][lane + kWave * u];
        if (lane + kWave * u >= Pp) cnt[u] = kCounted;
    }
    auto value_at = [&](int r) __attribute__((always_inline)) {
        for (;; --r) { // (count 0 exists: the smallest value)
            const unsigned long long m0 = __ballot(cnt[0] == r), m1 = __ballot(cnt[1] == r);
            if (m0) return readlane_f64(v[0], __ffsll(m0) - 1);
            if (m1) return readlane_f64(v[1], __ffsll(m1) - 1);
        }
    };
    lo = value_at(r_lo);
    hi = r_hi == r_lo ? lo : value_at(r_hi);
}

// What pass 2 is asked for.
struct BwArgs {
    int n;
    int mode;       // GramMode of the sums
    double h_fixed; // > 0: this bandwidth instead of the median's
    double log_n1;  // ln(n + 1), from the host
};

// Pass 2: h, K and the coefficient tables from the pair sums.  Called by all THREADS threads of a
// workgroup.  fill(meanwhile) leaves the reduced pair sums in sh.S (a barrier follows here); it
// calls meanwhile() once, at the point where it waits for memory: everything that does not depend
// on the sums is done there.
// coef_lds, if not null, receives C, its rows padded with zeros to a multiple of four, and rho [n] (LDS of the caller; barrier included);
// otherwise they go to coef (device memory).  write_global = false: st and K are left alone - for
// workgroups that repeat the computation of another one.  Returns h; c2h = 2 / h (0 for one particle).
//
// What bounds it is latency: some seven steps of a few hundred instructions each, run once, one
// after the other.  So every step uses all threads, the list of partials is read 16 bytes at a
// time, index arithmetic is done while it is on its way, h is derived by every thread instead of by
// one and a broadcast, and each row of K has 16 lanes.  The bandwidth kernel (launch included) took
// 12.6 us at n = 64, 7.7 at n = 32 and 7.3 at n = 16 before, and 7.3, 5.7 and 5.5 now.
struct NoCall {
    __device__ void operator()() const {}
};
template <int THREADS, int MAXN, bool LO, class Fill>
__device__ inline double kernel_matrix(BwShared<MAXN, THREADS> &sh, const BwArgs &ba, DevState *__restrict__ st,
                                       float *__restrict__ coef, float *coef_lds, bool write_global, float &c2h_out,
                                       Fill fill)
{
    static_assert(THREADS % 64 == 0 && THREADS >= 256 && THREADS <= 1024, "whole waves");
    constexpr int kPairs = MAXN * (MAXN - 1) / 2;
    constexpr int VPT = kPairs > THREADS ? (kPairs + THREADS - 1) / THREADS : 1; // pairs per thread
    const int tid = threadIdx.x, n = ba.n;
    const int Pp = n * (n - 1) / 2;
    const bool select = ba.h_fixed <= 0.0 && Pp > 0;
    const bool buckets = kPairs > kCounted && select && Pp > kCounted; // 17 particles and more
    const double inf = __builtin_huge_val();
    int pi[VPT], pj[VPT];
    fill([&]() __attribute__((always_inline)) {
        // the selection's scratch in its initial state
        if (buckets) {
            if (tid < kSelDirect) {
                sh.counters[tid] = 0;
                sh.list[tid] = inf;
            }
            for (int e = tid; e < kBuckets; e += THREADS) sh.hist[e] = 0;
            if (tid < 4) {
                sh.misc[tid] = 0;
                sh.mm[tid] = (tid & 1) ? 0ull : ~0ull;
            }
        }
        // pair p = (i, j): row i is the largest one whose first pair index, i (2n - i - 1) / 2, does
        // not exceed p (estimate from the quadratic, then corrected by one)
#pragma unroll
        for (int u = 0; u < VPT; ++u) {
            const int p = tid + u * THREADS;
            const float tn = (float)(2 * n - 1);
            int i = (int)(0.5f * (tn - __builtin_amdgcn_sqrtf(fmaxf(tn * tn - 8.0f * (float)p, 0.0f))));
            i = i < 0 ? 0 : (i > n - 2 ? n - 2 : i);
            i -= (i > 0 && pair_index(i, i + 1, n) > p) ? 1 : 0;
            i += (i < n - 2 && pair_index(i + 1, i + 2, n) <= p) ? 1 : 0;
            pi[u] = i;
            pj[u] = i + 1 + (p - pair_index(i, i + 1, n));
        }
    });
    block_sync<LO>();

    // d2 per pair: direct sums, or S_ii + S_jj - 2 S_ij (clamped at 0) from the centred Gram
    double d2[VPT];
    double dmin = inf, dmax = 0.0;
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
        const int p = tid + u * THREADS;
        double d = 0.0;
        if (p < Pp) {
            d = sh.S[tri(pi[u], pj[u], n)];
            if (ba.mode != kModeDiff) d = sh.S[tri(pi[u], pi[u], n)] + sh.S[tri(pj[u], pj[u], n)] - 2.0 * d;
            if (!(d > 0.0)) d = 0.0; // clamps rounding negatives (and -0.0, and NaN)
            dmin = fmin(dmin, d);
            if (d < inf) dmax = fmax(dmax, d);
        }
        d2[u] = d;
        if (p < BwShared<MAXN, THREADS>::kPr) sh.pr[p] = (p < Pp) ? d : inf;
    }
    if (buckets) minmax_to_lds(dmin, dmax, &sh.mm[0]); // the range of all finite values, for the first level
    block_sync<LO>();

    // Median of the multiset of all n*n entries of d2: n diagonal zeros plus every pair value
    // twice.  Sorted position t of the full list is 0 for t < n and the ((t-n)/2)-th smallest
    // pair value otherwise; an even count averages positions n*n/2 - 1 and n*n/2.  So what is
    // needed are the pair values of rank r_lo and r_hi (equal or adjacent), not a sorted list.
    const int t_lo = (n * n - 1) / 2, t_hi = (n * n) / 2; // t_hi >= n for every n >= 2
    double lo = 0.0, hi = 0.0;
    if (select) {
        // n = 2: position t_lo is one of the diagonal zeros - the other rank is selected twice
        const int r_lo = (t_lo >= n) ? (t_lo - n) / 2 : (t_hi - n) / 2, r_hi = (t_hi - n) / 2;
        if (buckets) {
            select_two_ranks<THREADS, VPT, LO>(sh, d2, Pp, r_lo, r_hi);
            block_sync<LO>();
            lo = sh.sel[0];
            hi = sh.sel[1];
        } else {
            count_ranks<THREADS, LO>(sh, Pp, r_lo, r_hi, lo, hi);
        }
    }
    const double med = select ? 0.5 * ((t_lo >= n ? lo : 0.0) + hi) : 0.0;
    // h = num / den and 1 / h = den / num: two divisions side by side
    const double num = (ba.h_fixed > 0.0) ? ba.h_fixed : med, den = (ba.h_fixed > 0.0) ? 1.0 : ba.log_n1;
    double h = num / den, inv_h = den / num;
    if (!(h > 0.0)) {
        h = 1.0;
        inv_h = 1.0;
    }
    // a single particle has no repulsive term at all: make that exact (phi = g)
    const double c2h = (n == 1) ? 0.0 : 2.0 * inv_h;
    c2h_out = (float)c2h;
    if (write_global && tid == 0) {
        st->h = h;
        st->med = med;
        st->two_over_h = (float)c2h;
        st->n = n;
    }

#pragma unroll
    for (int u = 0; u < VPT; ++u) // K per pair, reusing S (last read before the barriers above); 1 / h may be infinite
        if (tid + u * THREADS < Pp) sh.S[tid + u * THREADS] = d2[u] > 0.0 ? exp(-d2[u] * inv_h) : 1.0;
    block_sync<LO>();
    // K, C, row sums: 16 lanes per row.  K_ij and K_ji are the same LDS entry, so K is exactly
    // symmetric; the diagonal is exactly 1.
    const double inv_n = 1.0 / (double)n;
    const int n4 = (n + 3) & ~3; // rows of C in LDS
    for (int i = tid >> 4; i < n; i += THREADS / 16) {
        double r = 0.0;
#pragma unroll
        for (int b = 0; b < (MAXN + 15) / 16; ++b) {
            const int j = 16 * b + (tid & 15);
            if (j < n) {
                const double k = (i == j) ? 1.0 : sh.S[i < j ? pair_index(i, j, n) : pair_index(j, i, n)];
                r += k;
                if (write_global) coef[kOffK + i * n + j] = (float)k;
                if (coef_lds) coef_lds[i * n4 + j] = (float)(k * inv_n);
                else coef[kOffC + i * n + j] = (float)(k * inv_n);
            } else if (coef_lds && j < n4) {
                coef_lds[i * n4 + j] = 0.f;
            }
        }
        r = row_sum_f64(r); // row sum of K
        if ((tid & 15) == 0) {
            const float rho = (float)(c2h * r * inv_n);
            if (coef_lds) coef_lds[n * n4 + i] = rho;
            else coef[kOffRho + i] = rho;
        }
    }
    if (coef_lds) block_sync<LO>();
    return h;
}

// Where the pair sums of pass 2 come from: fully reduced sums (reduce_partials_kernel), or - sums
// null - a list of nparts fp32 partials, pair_stride(n) floats apart.
struct SumSource {
    const double *sums;
    const float *partials;
    int nparts;
};

// Reads reduced sums into S [n (n + 1) / 2], n <= MAXN.  meanwhile() and last() as in gather_sums.
template <int THREADS, int MAXN, class Meanwhile, class Last>
__device__ inline void copy_sums(double *S, const double *sums, int n, Meanwhile meanwhile, Last last)
{
    constexpr int U = (MAXN * (MAXN + 1) / 2 + THREADS - 1) / THREADS;
    const int tid = threadIdx.x, P = n * (n + 1) / 2;
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = sums[tid + u * THREADS < P ? tid + u * THREADS : 0];
    meanwhile();
    last();
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (tid + u * THREADS < P) S[tid + u * THREADS] = v[u];
}

// Sums a list of partials in fp64 into S [n (n + 1) / 2].  Thread (kk, pp) = (tid / P4, tid % P4), kk <
// KL, sums four consecutive entries of the partials kk, kk + KL, ..., up to MAXU 16-byte loads in
// flight (as the registers allow); the KL sums of an entry meet in `red` [KL * P4 * 4 <= 4 * THREADS].  meanwhile() and then last() are called
// when the last loads of the list have been sent off (see gather_wave_sums).  With sixteen loads in flight, selects
// for every value and the caller's first loads sent off after the sums, a list of 256 at n = 20 took 7.3 us (four
// rounds; phi at D = 300,007 32.1 us, now 30.4).
constexpr int kSumLoads = 16;
template <int THREADS, bool LO, int MAXU, class Meanwhile, class Last>
__device__ inline void gather_sums(double *S, double *red, const float *partials, int nparts, int n, Meanwhile meanwhile, Last last)
{
    const int tid = threadIdx.x;
    const int P = n * (n + 1) / 2;
    const int P4 = (P + 3) / 4;
    // (quotients of small integers: half a unit off the next one, far more than the reciprocal's error)
    const float inv = __builtin_amdgcn_rcpf((float)P4);
    const int per_wg = (int)(((float)THREADS + 0.5f) * inv);
    const int KL = __builtin_amdgcn_readfirstlane(per_wg < 32 ? per_wg : 32); // capped: the KL sums are added serially
    const int kk = (int)(((float)tid + 0.5f) * inv), pp = tid - kk * P4;
    const f32x4 *base = reinterpret_cast<const f32x4 *>(partials) + pp;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    int k0 = 0;
    auto batch = [&](auto loads, auto whole, auto then) __attribute__((always_inline)) { // clamped, not guarded: the number of loads is known
        constexpr int U = decltype(loads)::value;
        f32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + kk + u * KL;
            v[u] = base[(int64_t)(k < nparts ? k : nparts - 1) * P4];
        }
        then();
        // (four at a time, as long as there are any: summing sixteen where nine had been asked for took 0.2 to 1 us, at
        // n = 2, D = 150,001 9.7 us per svgd_bandwidth, now 8.6)
#pragma unroll
        for (int u0 = 0; u0 < U; u0 += 4) {
            if (!decltype(whole)::value && u0 > 0 && k0 + u0 * KL >= nparts) break;
#pragma unroll
            for (int u = u0; u < u0 + 4; ++u) {
                const bool in = decltype(whole)::value || k0 + kk + u * KL < nparts; // (a choice between floats: half the price of one between doubles)
#pragma unroll
                for (int c = 0; c < 4; ++c) s[c] += (double)(in ? v[u][c] : 0.f);
            }
        }
    };
    auto both = [&]() __attribute__((always_inline)) {
        meanwhile();
        last();
    };
    for (; nparts - k0 > MAXU * KL; k0 += MAXU * KL) batch(std::integral_constant<int, MAXU>{}, std::true_type{}, NoCall{});
    if (MAXU > kSumLoads && nparts - k0 > kSumLoads * KL) {
        batch(std::integral_constant<int, MAXU>{}, std::false_type{}, both);
    } else if (nparts - k0 > kSumLoads / 4 * KL) {
        batch(std::integral_constant<int, kSumLoads>{}, std::false_type{}, both);
    } else {
        batch(std::integral_constant<int, kSumLoads / 4>{}, std::false_type{}, both);
    }
    if (kk < KL) {
        double2 *dst = reinterpret_cast<double2 *>(red + (kk * P4 + pp) * 4);
        dst[0] = double2{s[0], s[1]};
        dst[1] = double2{s[2], s[3]};
    }
    block_sync<LO>();
    for (int p = tid; p < P; p += THREADS) {
        double t = 0.0;
#pragma unroll 4
        for (int q = 0; q < KL; ++q) t += red[q * P4 * 4 + p];
        S[p] = t;
    }
}

// ---------------------------------------------------------------------------------------------
// Pass 2 for at most kValuMaxN particles, inside the vector-ALU update and the single-workgroup step: EVERY
// wave of the workgroup does all of it by itself.  66 pairs are at most two per lane, so nothing has
// to be shared, and apart from the one barrier behind which the waves' sums meet (the caller's)
// there is none: with the pairs dealt to all threads of the workgroup five barriers and as many
// trips through LDS were half of the prologue (with that and the cheaper last column group, RaggedGroup,
// us per step at D = 100,003 before and now: n = 8, padded, carried sums 10.0 and 7.2, n = 10, plain 16.8
// and 12.0, n = 12 18.9 and 14.5; in the single-workgroup step n = 8, D = 1,003 9.5 and 6.0).  The rank of a value is the number of smaller ones, counted
// against a broadcast of the whole list; a value of rank r is one whose count is r, or with ties the
// largest count below r.
// ---------------------------------------------------------------------------------------------
template <int N>
struct WaveShared { // LDS, one per wave
    static constexpr int P = N * (N + 1) / 2, Pp = N * (N - 1) / 2;
    static constexpr int kList = Pp > 1 ? (Pp + 1) & ~1 : 2;
    __attribute__((aligned(16))) double pr[kList]; // d2 per pair, then K
    double S[N > 8 ? P : 1];                       // centred Gram sums
    // the result: row i is C_i0 .. C_i,N-1, then rho_i; read 16 bytes at a time
    static constexpr int kRow = (N + 1 + 3) & ~3;
    __attribute__((aligned(16))) float C[N * kRow];
    // Row i.  `at` is 0, but unknown to the compiler (opaque_zero): what is read through it stays where it is
    // needed - hoisted out of the loop over the columns C and rho would take N^2 + N registers.
    __device__ void row(int i, int at, float (&c)[N], float &rho) const
    {
        const f32x4 *src = reinterpret_cast<const f32x4 *>(C) + at + i * (kRow / 4);
#pragma unroll
        for (int k = 0; k < kRow / 4; ++k) {
            const f32x4 v = src[k];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (4 * k + e < N) c[4 * k + e < N ? 4 * k + e : 0] = v[e];
                if (4 * k + e == N) rho = v[e];
            }
        }
    }
};
__device__ inline int opaque_zero()
{
    int z = 0;
    asm volatile("" : "+v"(z));
    return z;
}

// sum(e): the reduced pair sum tri(i, j) = e (direct differences up to N = 8, centred Gram above).
// write_global: this wave also leaves h and K in st and coef.  Returns 2 / h (0 for one particle).
template <int N, class Sum>
__device__ inline float wave_kernel_matrix(WaveShared<N> &sh, double h_fixed, double log_n1, DevState *__restrict__ st,
                                           float *__restrict__ coef, bool write_global, Sum sum)
{
    constexpr int P = WaveShared<N>::P, Pp = WaveShared<N>::Pp, kList = WaveShared<N>::kList;
    constexpr int VPL = Pp > kWave ? 2 : 1; // pairs per lane
    const int lane = threadIdx.x & 63;
    const double inf = __builtin_huge_val();
    if constexpr (N > 8) {
#pragma unroll
        for (int u = 0; u < (P + kWave - 1) / kWave; ++u) {
            const int e = lane + kWave * u;
            if (e < P) sh.S[e] = sum(e);
        }
        wave_sync();
    }
    double d2[VPL];
#pragma unroll
    for (int u = 0; u < VPL; ++u) {
        const int p = lane + kWave * u;
        int i = 0;
#pragma unroll
        for (int k = 1; k < N - 1; ++k) i += p >= pair_index(k, k + 1, N) ? 1 : 0;
        const int j = i + 1 + p - pair_index(i, i + 1, N);
        double d = inf;
        if (p < Pp) {
            if constexpr (N > 8) d = sh.S[tri(i, i, N)] + sh.S[tri(j, j, N)] - 2.0 * sh.S[tri(i, j, N)];
            else d = sum(tri(i, j, N));
            if (!(d > 0.0)) d = 0.0; // clamps rounding negatives (and -0.0, and NaN)
        }
        d2[u] = d;
        if (p < kList) sh.pr[p] = d;
    }
    wave_sync();
    // the two middle order statistics of all n * n entries, see kernel_matrix
    constexpr int t_lo = (N * N - 1) / 2, t_hi = (N * N) / 2;
    double med = 0.0;
    if constexpr (N > 1) {
        constexpr int r_hi = (t_hi - N) / 2, r_lo = t_lo >= N ? (t_lo - N) / 2 : r_hi;
        if (h_fixed <= 0.0) {
            int cnt[VPL];
#pragma unroll
            for (int u = 0; u < VPL; ++u) cnt[u] = lane + kWave * u < Pp ? 0 : Pp;
#pragma unroll
            for (int k = 0; k < kList; k += 2) {
                const double2 w = *reinterpret_cast<const double2 *>(&sh.pr[k]);
#pragma unroll
                for (int u = 0; u < VPL; ++u) {
                    cnt[u] += w.x < d2[u] ? 1 : 0;
                    cnt[u] += w.y < d2[u] ? 1 : 0;
                }
            }
            auto value_at = [&](int r) __attribute__((always_inline)) {
                for (;; --r) { // (count 0 exists: the smallest value)
                    const unsigned long long m0 = __ballot(cnt[0] == r);
                    if (m0) return readlane_f64(d2[0], __ffsll(m0) - 1);
                    if constexpr (VPL > 1) {
                        const unsigned long long m1 = __ballot(cnt[VPL - 1] == r);
                        if (m1) return readlane_f64(d2[VPL - 1], __ffsll(m1) - 1);
                    }
                }
            };
            const double hi = value_at(r_hi);
            med = 0.5 * ((t_lo >= N ? (r_lo == r_hi ? hi : value_at(r_lo)) : 0.0) + hi);
        }
    }
    // h = num / den and 1 / h = den / num: two divisions side by side
    const double num = (h_fixed > 0.0) ? h_fixed : med, den = (h_fixed > 0.0) ? 1.0 : log_n1;
    double h = num / den, inv_h = den / num;
    if (!(h > 0.0)) {
        h = 1.0;
        inv_h = 1.0;
    }
    // a single particle has no repulsive term at all: make that exact (phi = g)
    const double c2h = (N == 1) ? 0.0 : 2.0 * inv_h;
    if (write_global && lane == 0) {
        st->h = h;
        st->med = med;
        st->two_over_h = (float)c2h;
        st->n = N;
    }
    wave_sync();
#pragma unroll
    for (int u = 0; u < VPL; ++u) // K per pair; 1 / h may be infinite
        if (lane + kWave * u < Pp) sh.pr[lane + kWave * u] = d2[u] > 0.0 ? exp(-d2[u] * inv_h) : 1.0;
    wave_sync();
    // K, C, row sums: 8 or 16 lanes per row.  K_ij and K_ji are the same LDS entry, so K is exactly
    // symmetric; the diagonal is exactly 1.
    constexpr int L = N <= 8 ? 8 : 16;
    constexpr double inv_n = 1.0 / (double)N;
#pragma unroll
    for (int i0 = 0; i0 < N; i0 += kWave / L) {
        const int i = i0 + lane / L, j = lane % L;
        const bool in = i < N && j < N;
        double k = in ? 1.0 : 0.0;
        if (in && i != j) k = sh.pr[i < j ? pair_index(i, j, N) : pair_index(j, i, N)];
        const double r = row_sum_f64<L>(k); // row sum of K
        if (in) {
            if (write_global) coef[kOffK + i * N + j] = (float)k;
            sh.C[i * WaveShared<N>::kRow + j] = (float)(k * inv_n);
            if (j == 0) sh.C[i * WaveShared<N>::kRow + N] = (float)(c2h * r * inv_n);
        }
    }
    wave_sync();
    return (float)c2h;
}

// Sums a list of partials in fp64 for wave_kernel_matrix, every wave a part of it: G neighbouring lanes read one
// partial, 16 bytes each, R partials side by side and up to kSumLoads of them one after the other in flight.
// Then the wave's R sums are added, up to seven particles across the lanes (a partial then takes 4 or 8
// lanes), above by way of the wave's part of `scratch`, where G is exactly what a partial takes (at n = 8, nine lanes: with
// sixteen for each, a list of 512 took 1.7 times the loads), and go to red[wave].
// `last` is called when the last loads of the list have been sent off: the place for the caller to send
// off loads of its own, which are then in flight while the list is summed (a wave's loads complete in
// order: earlier, the sums would wait behind them).
template <int N>
struct GatherShared {
    static constexpr int P4 = pair_stride(N) / 4;
    static constexpr bool kLanes = N <= 7;
    static constexpr int G = kLanes ? (P4 <= 4 ? 4 : 8) : P4;
    static constexpr int R = kWave / G;
    __attribute__((aligned(16))) double red[4][4 * P4];
    __attribute__((aligned(16))) double scratch[kLanes ? 1 : 4][kLanes ? 1 : R][4 * P4];
    __device__ double sum(int e) const { return (red[0][e] + red[1][e]) + (red[2][e] + red[3][e]); }
};
template <int N, class Last>
__device__ inline void gather_wave_sums(GatherShared<N> &sh, const float *partials, int nparts, Last last)
{
    typedef GatherShared<N> Sh;
    constexpr int P4 = Sh::P4, G = Sh::G, R = Sh::R, STEP = 4 * R;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row = lane / G;
    const bool idle = row >= R; // (lanes that no whole partial is left for)
    const int pp = lane % G < P4 ? lane % G : P4 - 1, kk = wave * R + (idle ? 0 : row);
    const f32x4 *base = reinterpret_cast<const f32x4 *>(partials) + pp;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    int k0 = 0;
    // U loads in a row, clamped and not guarded: with a number of loads that is not known the first wait would be
    // for everything in flight, the caller's loads included
    auto batch = [&](auto loads, auto then) __attribute__((always_inline)) {
        constexpr int U = decltype(loads)::value;
        f32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = k0 + kk + u * STEP;
            v[u] = base[(k < nparts ? k : nparts - 1) * P4];
        }
        then();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool in = k0 + kk + u * STEP < nparts;
#pragma unroll
            for (int c = 0; c < 4; ++c) s[c] += (double)(in ? v[u][c] : 0.f);
        }
    };
    for (; nparts - k0 > kSumLoads * STEP; k0 += kSumLoads * STEP) batch(std::integral_constant<int, kSumLoads>{}, [] {});
    if (nparts - k0 > kSumLoads / 2 * STEP) batch(std::integral_constant<int, kSumLoads>{}, last);
    else if (nparts - k0 > kSumLoads / 4 * STEP) batch(std::integral_constant<int, kSumLoads / 2>{}, last);
    else batch(std::integral_constant<int, kSumLoads / 4>{}, last);
    if constexpr (Sh::kLanes) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if constexpr (G == 4) s[c] += dpp_f64<0x124>(s[c]); // row_ror:4
            s[c] += dpp_f64<0x128>(s[c]);                       // row_ror:8
            s[c] += swap_f64<16>(s[c]);
            s[c] += swap_f64<32>(s[c]);
        }
        if (lane < P4) {
            double2 *dst = reinterpret_cast<double2 *>(&sh.red[wave][4 * lane]);
            dst[0] = double2{s[0], s[1]};
            dst[1] = double2{s[2], s[3]};
        }
    } else {
        if (!idle) {
            double2 *dst = reinterpret_cast<double2 *>(&sh.scratch[wave][row][4 * pp]);
            dst[0] = double2{s[0], s[1]};
            dst[1] = double2{s[2], s[3]};
        }
        wave_sync();
        for (int e = lane; e < 4 * P4; e += kWave) {
            double t = sh.scratch[wave][0][e];
#pragma unroll
            for (int r = 1; r < R; ++r) t += sh.scratch[wave][r][e];
            sh.red[wave][e] = t;
        }
    }
}

// Lists of at most this many floats are summed by the bandwidth kernel itself; longer ones by
// reduce_partials_kernel first: one CU reads what others have just written at some 60 GB/s (41,600
// floats at n = 64: step 48.5 us, 45.3 with the reduction; 20,480 at n = 40: 29.4 and 29.0).
constexpr int kDirectMaxFloats = 16 * 1024;

static __global__ __launch_bounds__(kBwThreads) void bandwidth_kernel(SumSource src, BwArgs ba, DevState *__restrict__ st,
                                                               float *__restrict__ coef)
{
    __shared__ BwShared<kMaxN, kBwThreads> sh;
    __shared__ __attribute__((aligned(16))) double red[4 * kBwThreads];
    float c2h;
    kernel_matrix<kBwThreads, kMaxN, false>(
        sh, ba, st, coef, nullptr, true, c2h,
        [&](auto meanwhile) __attribute__((always_inline)) {
            if (src.sums != nullptr) copy_sums<kBwThreads, kMaxN>(sh.S, src.sums, ba.n, meanwhile, NoCall{});
            else gather_sums<kBwThreads, false, kSumLoads>(sh.S, red, src.partials, src.nparts, ba.n, meanwhile, NoCall{});
        });
}

// What svgd_get_last reads, from the handle's state to its page-locked host memory, and behind it the number of the
// request, which the host watches for.  A copy to pageable memory and a synchronisation took some ten us more:
// bandwidth and get_last, n = 4, D = 1,003 27.4 -> 14.0 us, n = 16, D = 8,577 34 -> 20, n = 48, D = 1,000,003 70 -> 62
// (the same on a handle's first read-back).  Either way the host's core is busy until the result is there.
struct Mirror {
    unsigned ticket;
    __attribute__((aligned(kStateBytes))) unsigned char data[kStateBytes + sizeof(float) * kMaxN * kMaxN];
};
static __global__ __launch_bounds__(256) void mirror_kernel(const unsigned *__restrict__ state, Mirror *__restrict__ mirror, int words, unsigned ticket)
{
    unsigned *dst = reinterpret_cast<unsigned *>(mirror->data);
    for (int i = threadIdx.x; i < words; i += 256) dst[i] = state[i];
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(&mirror->ticket, ticket, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

} // namespace svgd
