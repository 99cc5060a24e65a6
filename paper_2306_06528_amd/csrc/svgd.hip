// Host side of the C ABI declared in include/svgd.h: handle, argument validation, launches.
#include "../../include/svgd.h"

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>
#include <unordered_set>
#include <vector>

#include "bandwidth_kernels.hpp"
#include "common.hpp"
#include "diag_kernels.hpp"
#include "gram_kernels.hpp"
#include "swag_kernels.hpp"
#include "tiny_kernels.hpp"
#include "update_launch.hpp"

using namespace svgd;

namespace {

constexpr uint32_t kMagic = 0x53564744u; // "SVGD"
constexpr int kMaxParts = 2048;          // upper bound on Gram workgroups (= partial vectors)
constexpr int kMaxCu = 256;              // CUs of this part
constexpr int64_t kMemorySideCacheBytes = (int64_t)256 << 20; // this part's memory-side cache (between L2 and HBM)

} // namespace

struct svgd_ctx {
    uint32_t magic;
    int device;
    int max_n;
    int64_t max_D;
    int num_cu;
    uint32_t flags;
    double h_fixed;
    // Gram partials of the current X left behind by the last svgd_step (SVGD_FLAG_CARRY_GRAM)
    bool carry_valid;
    const float *carry_X;
    int carry_n;
    int64_t carry_D;
    int64_t carry_ld;
    int carry_nparts;
    int64_t carry_off;        // where in `partials` the carried list starts (floats): 0 or the upper half
    bool captured;            // a step on carried sums has been captured into a graph (svgd_step_ld):
    int64_t home;             // from then on every carried list ends up here
    hipStream_t carry_stream; // the stream the carried sums were produced on
    int64_t partials_cap;     // floats available in `partials`
    unsigned sweeps;          // in-place updates with carried sums so far: every other one walks X backwards
    int last_n; // 0 = nothing computed yet
    int last_hip_error;
    float *partials;  // [kMaxParts][pair_stride]
    double *sums;     // [P], the reduced pair sums
    DevState *state;
    float *coef;      // kCoefFloats, kStateBytes behind `state` in one allocation
    Mirror *mirror;   // page-locked host memory (read_back)
    unsigned ticket;
    // optional per-kernel timing (svgd_profile_begin/end): event pairs recorded around launches
    bool profiling;
    unsigned profile_kinds; // bit k set: kernels of kind k are timed
    std::vector<hipEvent_t> ev_pool; // 2 events per record
    std::vector<int> ev_kind;        // SVGD_KERNEL_* of each record
};

namespace {

struct DeviceGuard {
    int prev = -1;
    bool switched = false;
    explicit DeviceGuard(int dev)
    {
        if (hipGetDevice(&prev) == hipSuccess && prev != dev) switched = (hipSetDevice(dev) == hipSuccess);
    }
    ~DeviceGuard()
    {
        if (switched) (void)hipSetDevice(prev);
    }
};

int fail(svgd_ctx *c, hipError_t e)
{
    if (c) c->last_hip_error = (int)e;
    return SVGD_ERR_DEVICE;
}

// Live handles are kept in a registry so that a stale pointer (use after destroy) is rejected
// without being dereferenced.
std::mutex g_live_mutex;
std::unordered_set<svgd_ctx *> &live_handles()
{
    static std::unordered_set<svgd_ctx *> s;
    return s;
}

int check_handle(svgd_ctx *c)
{
    if (!c) return SVGD_ERR_BAD_HANDLE;
    std::lock_guard<std::mutex> lock(g_live_mutex);
    if (!live_handles().count(c) || c->magic != kMagic) return SVGD_ERR_BAD_HANDLE;
    return SVGD_OK;
}

// The page-locked buffers (Mirror) of handles that are gone are kept for the next ones: allocating one takes 27 us
// and freeing it 35, where all else in svgd_create and svgd_destroy takes 3 and 2.  At most
// kSpareMirrors of them (17 KB each) stay, until the process ends; any further one is freed.
struct SpareMirror {
    Mirror *p;
    int device;
};
constexpr int kSpareMirrors = 4;
std::mutex g_spare_mutex;
SpareMirror g_spare[kSpareMirrors];
int g_spares = 0;

Mirror *take_mirror(int device)
{
    Mirror *m = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_spare_mutex);
        for (int i = g_spares - 1; i >= 0 && !m; --i) {
            if (g_spare[i].device != device) continue;
            m = g_spare[i].p;
            g_spare[i] = g_spare[--g_spares];
        }
    }
    void *mapped;
    if (m && hipHostGetDevicePointer(&mapped, m, 0) != hipSuccess) { // (the device has been reset since)
        (void)hipGetLastError();
        m = nullptr;
    }
    if (!m && hipHostMalloc((void **)&m, sizeof(Mirror), hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess) return nullptr;
    m->ticket = 0;
    return m;
}

// idle: nothing on the device will write to it any more
hipError_t give_mirror(Mirror *m, int device, bool idle)
{
    if (idle) {
        std::lock_guard<std::mutex> lock(g_spare_mutex);
        if (g_spares < kSpareMirrors) {
            g_spare[g_spares++] = SpareMirror{m, device};
            return hipSuccess;
        }
    }
    return hipHostFree(m);
}

constexpr size_t kMaxProfileRecords = 2048;

// Records a start event on construction and a stop event on destruction when profiling is on.
// The events come from a pool that svgd_profile_begin* has created: nothing is allocated between
// the launches that are being timed.
struct KernelTimer {
    svgd_ctx *c;
    hipStream_t s;
    size_t slot = (size_t)-1;
    KernelTimer(svgd_ctx *ctx, int kind, hipStream_t stream) : c(ctx), s(stream)
    {
        if (!c->profiling || !((c->profile_kinds >> kind) & 1u)) return;
        const size_t idx = c->ev_kind.size();
        if (idx >= kMaxProfileRecords || c->ev_pool.size() < 2 * (idx + 1)) return;
        if (hipEventRecord(c->ev_pool[2 * idx], s) != hipSuccess) { (void)hipGetLastError(); return; }
        c->ev_kind.push_back(kind); // capacity reserved by svgd_profile_begin*
        slot = idx;
    }
    ~KernelTimer()
    {
        if (slot != (size_t)-1) (void)hipEventRecord(c->ev_pool[2 * slot + 1], s);
    }
};

// Whether what is launched on the stream goes into a graph.
bool is_capturing(hipStream_t s)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return st == hipStreamCaptureStatusActive;
}

// For calls that read back: nothing can be read while nothing runs.  To be asked before anything is launched or
// changed, or the graph would keep what the refused call has left in it.
int refuse_capture(svgd_ctx *c, hipStream_t s)
{
    return is_capturing(s) ? fail(c, hipErrorStreamCaptureUnsupported) : SVGD_OK;
}

// The first `bytes` bytes of the handle's state (DevState, then K) as they are when the work enqueued on the stream
// is done, in c->mirror->data.  A kernel writes them to page-locked memory and the host watches for its ticket;
// if that does not come within a few milliseconds the stream is waited for as usual - which keeps the host's core as
// busy - and that also reports what went wrong.  Not for a stream that is being captured: the caller has looked (refuse_capture).
int read_back(svgd_ctx *c, size_t bytes, hipStream_t s)
{
    const unsigned ticket = ++c->ticket;
    mirror_kernel<<<1, 256, 0, s>>>(reinterpret_cast<const unsigned *>(c->state), c->mirror, (int)((bytes + 3) / 4), ticket);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(c, e);
    const auto until = std::chrono::steady_clock::now() + std::chrono::milliseconds(5);
    for (unsigned k = 0;; ++k) {
        if (__atomic_load_n(&c->mirror->ticket, __ATOMIC_ACQUIRE) == ticket) return SVGD_OK;
        if ((k & 63) == 63 && std::chrono::steady_clock::now() > until) break;
        __builtin_ia32_pause();
    }
    e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail(c, e);
    return SVGD_OK;
}

int check_shape(svgd_ctx *c, int n, int64_t D, int64_t ld)
{
    if (n < 1 || D < 1 || ld < D) return SVGD_ERR_INVALID_ARG;
    if (n > c->max_n || D > c->max_D) return SVGD_ERR_TOO_LARGE;
    return SVGD_OK;
}

// n rows of D floats, ld floats apart: the byte ranges from the first to the last element
bool overlaps(const float *a, const float *b, int n, int64_t D, int64_t ld)
{
    const uintptr_t bytes = ((uintptr_t)(n - 1) * (uintptr_t)ld + (uintptr_t)D) * sizeof(float);
    const uintptr_t pa = (uintptr_t)a, pb = (uintptr_t)b;
    return pa < pb + bytes && pb < pa + bytes;
}

// rt != nullptr: the particles are separate rows (svgd_step_rows); the table goes along by value
template <int N>
void launch_gram_valu(const float *X, int64_t D, int64_t ld, float *partials, int grid, hipStream_t s,
                      const RowTable *rt, bool stream_x, int64_t hot_bytes)
{
    const int64_t stride = (int64_t)grid * 256 * kGramGroups<N>;
    const GroupSplit split((D + 3) / 4, stride);
    const int hot = (int)(hot_bytes / (stride * 16 * N));
    if (rt)
        gram_valu_kernel<N, true><<<grid, 256, 0, s>>>(X, D, ld, partials, split, 0, *rt);
    else if (stream_x)
        gram_valu_kernel<N, false, true><<<grid, 256, 0, s>>>(X, D, ld, partials, split, hot, NoRows{});
    else
        gram_valu_kernel<N, false><<<grid, 256, 0, s>>>(X, D, ld, partials, split, 0, NoRows{});
}

template <int N, bool EMIT, bool CARRY>
void launch_update_valu(float *X, const float *G, float *PHI, float *coef, DevState *st,
                        int64_t D, int64_t ld, float eps, float *gram_out, int grid, hipStream_t s,
                        const RowTable *rt, const UpdateArgs &ua)
{
    const GroupSplit split((D + 3) / 4, (int64_t)grid * 256);
    if constexpr (!EMIT && !CARRY) {
        if (rt) {
            update_valu_kernel<N, false, false, true><<<grid, 256, 0, s>>>(X, G, PHI, coef, st, D, ld, eps, gram_out, split, *rt, ua);
            return;
        }
    }
    update_valu_kernel<N, EMIT, CARRY, false><<<grid, 256, 0, s>>>(X, G, PHI, coef, st, D, ld, eps, gram_out, split, NoRows{}, ua);
}

#define SVGD_SWITCH_N(n, CALL)                                                                     \
    switch (n) {                                                                                   \
    case 1: CALL(1); break;                                                                        \
    case 2: CALL(2); break;                                                                        \
    case 3: CALL(3); break;                                                                        \
    case 4: CALL(4); break;                                                                        \
    case 5: CALL(5); break;                                                                        \
    case 6: CALL(6); break;                                                                        \
    case 7: CALL(7); break;                                                                        \
    case 8: CALL(8); break;                                                                        \
    case 9: CALL(9); break;                                                                        \
    case 10: CALL(10); break;                                                                      \
    case 11: CALL(11); break;                                                                      \
    default: CALL(12); break;                                                                      \
    }

int clampi(int64_t v, int lo, int hi) { return (int)(v < lo ? lo : (v > hi ? hi : v)); }
int mini(int a, int b) { return a < b ? a : b; }

// How many partial vectors of n(n+1)/2 floats the handle's scratch holds from `off` on: the upper bound on
// every grid whose workgroups write one partial each.
int max_parts(const svgd_ctx *c, int n, int64_t off)
{
    const int64_t m = (c->partials_cap - off) / pair_stride(n);
    return (int)(m < kMaxParts ? m : kMaxParts);
}

// The scratch in two halves: a list may be read while the new one is written.
int64_t half_scratch(const svgd_ctx *c) { return (c->partials_cap / 2) & ~(int64_t)63; }
int64_t other_half(const svgd_ctx *c, int64_t off) { return off == 0 ? half_scratch(c) : 0; }

// An X that the memory-side cache cannot hold (with a margin: n = 32, D = 2,000,000 just fits and
// behaves like a cached problem).
bool beyond_cache(int n, int64_t ld)
{
    return (int64_t)n * ld * (int64_t)sizeof(float) > kMemorySideCacheBytes + kMemorySideCacheBytes / 4;
}

// Whether the matrix-core update lets the waves of a workgroup share a range where its stores allow it (aligned rows; direct
// stores, see run_update).
bool adjacent_tiles(int n, int64_t ld) { return n > 48 || beyond_cache(n, ld); }

// Up to kFusedMaxN particles the update kernel does pass 2 itself, in every workgroup, if that costs
// less than the launches it saves: 256 threads hold at most 496 pairs comfortably, and every
// workgroup reads the whole list, in batches of sixteen 16-byte loads per thread, one after the
// other (gather_sums).  Up to four batches it wins; a longer list is summed by a launch of many workgroups, and the update
// does pass 2 on the sums (see kSumsMaxN).  us per step on dense rows, on the list, with pass 2 in a launch of its own and on sums:
// n = 24, D = 40,003 (4 batches) 17.1, 19.2 and -, D = 50,001 (5) 18.0, 18.2 to 19.8 and 15.9; n = 32, D = 12,289 (4) 16.6, 18.4
// and -, D = 20,001 (5) 18.0, 17.7 to 19.6 and 15.6, D = 30,001 (8) 20.1, 18.1 to 19.8 and 15.8; carried sums, padded,
// n = 24, D = 65,000 (6) 16.5, 17.0 and -, n = 31 19.3, 17.9 and -.
// On the vector-ALU path every list is that short (run_gram sees to it), and one launch wins up to the
// largest sizes (n = 8, D = 11,173,962: 281 -> 270 us; n = 10, D = 300,001: 31 -> 24).
constexpr int kFusedMaxN = 32;
constexpr int kFusedMaxBatches = 4;

constexpr int fused_max_parts(int n) // n <= kFusedMaxN
{
    const int groups = 256 / (pair_stride(n) / 4);
    return kFusedMaxBatches * kSumLoads * (groups < 32 ? groups : 32);
}
// Up to kFusedAlwaysN particles (one block of rows, remainder rows included) no list is longer: the grids whose workgroups
// leave a partial each have one per CU on the matrix-core path, the tail's workgroup included.
static_assert(fused_max_parts(kFusedAlwaysN) >= kMaxCu, "one partial per CU is a short list");

// A list of pair-sum partials in the handle's scratch.
struct PairList {
    int64_t off; // where it starts (floats)
    int nparts;
};

// Pass 1: the pair sums of X, one partial per workgroup, at the start of the scratch - or, once a step on
// carried sums has been captured, where the graph expects a list (carry_next), or out of its way.
// G_next: where the update that follows this call will read its scores (null: none, or one that writes
// phi to unaligned rows); carry_next: that update will carry pair sums.  They steer the order in
// which X is visited, so that the pass ends on the tiles the update starts with (n = 32, D = 9,000,000:
// separate rows 888 -> 865 us per step, phi on aligned rows 856 -> 836).
int run_gram(svgd_ctx *c, const float *X, int n, int64_t D, int64_t ld, hipStream_t s, PairList &list,
             const RowTable *rt = nullptr, const float *G_next = nullptr, bool carry_next = false)
{
    list.off = !c->captured ? 0 : (carry_next ? c->home : other_half(c, c->home));
    float *const partials = c->partials + list.off;
    const int cap_parts = max_parts(c, n, list.off);
    int nparts;
    // streaming loads in pass 1: X well beyond what the memory-side cache could keep for the update
    const bool big_x = (int64_t)n * ld * (int64_t)sizeof(float) > 2 * kMemorySideCacheBytes;
    const bool x_aligned = rt ? rt->aligned != 0 : rows_aligned(X, ld);
    KernelTimer t(c, SVGD_KERNEL_GRAM, s);
    if (n <= kValuMaxN) {
        const int64_t ngroups = (D + 3) / 4;
        // all resident at once; each ends with a reduction; the update sums the list (three per CU of
        // 256 are just what it takes at n = 12)
        nparts = clampi((ngroups + 255) / 256, 1, mini(mini(c->num_cu * kGramPerCu, cap_parts), mini(fused_max_parts(n), (int)(half_scratch(c) / pair_stride(n)))));
        const int64_t x_bytes = (int64_t)n * D * (int64_t)sizeof(float);
        // An X that outgrows the memory-side cache is loaded with the streaming hint, above 8 particles up to
        // the three quarters of that cache which the update reads first (walked last, loaded plainly): n = 12,
        // D = 11,173,962 432 -> 416 us per step, D = 6,000,002 235 -> 226.  At n = 8 that pass is 4 us faster, too, but
        // the update finds less of X and the step is slower by as much (271 -> 274): there, up to twice the cache all loads
        // are plain.
        const bool stream_x = x_bytes > (n > 8 ? 1 : 2) * kMemorySideCacheBytes;
        const int64_t hot_bytes = n > 8 ? 3 * kMemorySideCacheBytes / 4 : 0;
#define CALL(N) launch_gram_valu<N>(X, D, ld, partials, nparts, s, rt, stream_x, hot_bytes)
        SVGD_SWITCH_N(n, CALL)
#undef CALL
    } else {
        const int NB = (n + 15) / 16;
        const int64_t nfull = D / 64;
        const bool small = nfull < (int64_t)kGramWavesSmall * mini(c->num_cu, cap_parts); // a slab per wave, the partial one included
        const bool wide = small && NB >= 2 && (D & 63); // a partial slab: no branch around any load
        const int waves = small ? kGramWavesSmall : kGramWaves;
        nparts = clampi((D + 64 * waves - 1) / (64 * waves), 1, mini(c->num_cu, cap_parts));
        // the ranges of the update that follows (tile_range) and how many of each range's first
        // tiles three quarters of the memory-side cache can hold
        const bool aligned_next = G_next && x_aligned && (rt || rows_aligned(G_next, ld));
        const bool shared_ranges = aligned_next && adjacent_tiles(n, ld);
        int64_t nranges = (int64_t)long_list_workers(n, D, c->num_cu, carry_next ? cap_parts : kMaxParts, beyond_cache(n, ld), aligned_next, false, false, carry_next) *
                          (shared_ranges ? 1 : 4);
        int64_t per = (nfull + nranges - 1) / nranges > 0 ? (nfull + nranges - 1) / nranges : 1;
        int64_t hot = (3 * kMemorySideCacheBytes / 4) / ((int64_t)n * 256) / nranges;
        if (shared_ranges) hot &= ~(int64_t)3; // four waves share the start of a range
        if (hot > per) hot = per;
        if (per * nranges >= ((int64_t)1 << 31) - 1) { // the kernel maps 32-bit indices: one range, nothing kept
            nranges = 1;
            per = nfull > 0 ? nfull : 1;
            hot = 0;
        }
        const bool stream_x = big_x && x_aligned; // slabs of unaligned rows share lines
        // the waves in step (ORDER 3): a step on dense rows, X beyond 1 GiB, the last of three or four blocks at least three quarters full
        const bool in_step = !x_aligned && G_next && NB >= 3 && ((n & 15) == 0 || (n & 15) >= 12) &&
                             (int64_t)n * D * (int64_t)sizeof(float) > (int64_t)1 << 30;
        const uint32_t stride = (uint32_t)kGramWaves * (uint32_t)nparts, cold = (uint32_t)(per - hot);
        GramOrder go{(uint32_t)nranges, (uint32_t)per, (uint32_t)hot, 0, 0, 0, 0};
        if (cold) { go.q_cold = stride / cold; go.r_cold = stride % cold; }
        if (hot) { go.q_hot = stride / (uint32_t)hot; go.r_hot = stride % (uint32_t)hot; }
        // (the order is only worth its bookkeeping for an X well beyond the memory-side cache)
#define GRAM_W(NB, W, ROWS, ORDER, rows) gram_mfma_kernel<NB, W, ROWS, ORDER><<<nparts, 64 * W, 0, s>>>(X, n, D, ld, partials, rows, go)
#define GRAM(NB)                                                                                             \
    do {                                                                                                     \
        if (rt && wide) GRAM_W(NB, kGramWavesSmall, true, (NB >= 2 ? 4 : 0), *rt);                           \
        else if (rt && small) GRAM_W(NB, kGramWavesSmall, true, 0, *rt);                                     \
        else if (rt && stream_x) GRAM_W(NB, kGramWaves, true, 2, *rt);                                       \
        else if (rt && big_x) GRAM_W(NB, kGramWaves, true, 1, *rt);                                          \
        else if (rt) GRAM_W(NB, kGramWaves, true, 0, *rt);                                                   \
        else if (wide) GRAM_W(NB, kGramWavesSmall, false, (NB >= 2 ? 4 : 0), NoRows{});                      \
        else if (small) GRAM_W(NB, kGramWavesSmall, false, 0, NoRows{});                                     \
        else if (stream_x) GRAM_W(NB, kGramWaves, false, 2, NoRows{});                                       \
        else if (in_step) GRAM_W(NB, kGramWaves, false, (NB >= 3 ? 3 : 1), NoRows{});                        \
        else if (big_x) GRAM_W(NB, kGramWaves, false, 1, NoRows{});                                          \
        else GRAM_W(NB, kGramWaves, false, 0, NoRows{});                                                     \
    } while (0)
        if (NB == 1) GRAM(1);
        else if (NB == 2) GRAM(2);
        else if (NB == 3) GRAM(3);
        else GRAM(4);
#undef GRAM
#undef GRAM_W
    }
    list.nparts = nparts;
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(c, e);
    return SVGD_OK;
}

// The list of partial sums added up, by a launch of many workgroups.
int run_reduce(svgd_ctx *c, int n, const PairList &list, hipStream_t s)
{
    KernelTimer t(c, SVGD_KERNEL_REDUCE, s);
    reduce_partials_kernel<<<(pair_stride(n) + kReduceEntries - 1) / kReduceEntries, 256, 0, s>>>(c->partials + list.off, list.nparts, n, c->sums);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(c, e);
    return SVGD_OK;
}

// The list as the source of pass 2: as it is, or - longer than `max_floats` - reduced first.
int sum_source(svgd_ctx *c, int n, const PairList &list, int max_floats, hipStream_t s, SumSource &src)
{
    src.sums = nullptr;
    src.partials = c->partials + list.off;
    src.nparts = list.nparts;
    if ((int64_t)list.nparts * pair_stride(n) <= max_floats) return SVGD_OK;
    src.sums = c->sums;
    return run_reduce(c, n, list, s);
}

// The Gram kernels' format at this particle count (the update kernels with CARRY mirror it).
int gram_mode(int n) { return n <= 8 ? kModeDiff : kModeGram; }

// Pass 2 as a kernel of its own: list -> h, K, coefficient tables.
int run_bandwidth(svgd_ctx *c, int n, const PairList &list, hipStream_t s)
{
    SumSource src;
    int rc = sum_source(c, n, list, kDirectMaxFloats, s, src);
    if (rc) return rc;
    KernelTimer t(c, SVGD_KERNEL_BANDWIDTH, s);
    bandwidth_kernel<<<1, kBwThreads, 0, s>>>(src, BwArgs{n, gram_mode(n), c->h_fixed, std::log((double)n + 1.0)}, c->state, c->coef);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(c, e);
    c->last_n = n;
    return SVGD_OK;
}

// Rows that do not start on 128-byte boundaries: whether the update stores its tiles where they lie all the same
// (kStoreDirect).  Staged, a tile is some three thousand cycles longer, and a wave's first tile and the end of
// its range more than that; direct, a line that two tiles share is written twice, which costs little while the caches
// hold what is in use, and most where phi is a third array.  The lines lie where the two cross (MiB of X; dense rows,
// us per step staged and direct, other inputs from call to call): plain n = 13 70 68.6 / 67.5 and 172 152.6 / 154.0, n = 15
// 70 65.9 / 64.7 and 116 103.5 / 104.7, n = 16 116 103.2 / 98.9 and 140 122.9 / 125.5, n = 24 52 60.0 / 59.0 and 72
// 76.8 / 80.8, n = 47 52 69.5 / 69.1 and 72 85.8 / 91.3, n = 52 130 146.5 / 136.3, n = 60 150 161.4 / 153.7 and 180
// 187.6 / 197.6; phi n = 14 26 28.2 / 27.7 and 32 32.9 / 35.7, n = 24 20 33.9 / 31.6 and 32 44.8 / 45.9, n = 40 38
// 56.0 / 55.3 and 52 69.5 / 71.4, n = 64 77 100.2 / 93.5; carried sums n = 15 86 51.4 / 49.7 and 150 94.6 / 99.4, n = 28
// 86 67.2 / 64.1 and 150 104.2 / 112.3, n = 36 86 74.3 / 72.7 and 150 108.2 / 118.0, n = 64 256 201.3 / 186.5.  At small
// sizes: n = 33, D = 20,001 25.6 / 22.2, n = 64, D = 8,577 33.1 / 28.4.
bool store_directly(int n, int64_t D, bool emit, bool carry)
{
    const int mib = emit ? (n <= 32 ? 24 : (n <= 48 ? 40 : 76)) : (carry ? (n <= 48 ? 92 : 256) : (n < 16 ? 100 : (n == 16 ? 120 : (n <= 48 ? 56 : 144))));
    return (int64_t)n * D * (int64_t)sizeof(float) <= ((int64_t)mib << 20);
}

// Passes 2 and 3.  EMIT = false: X updated in place; EMIT = true: phi written to PHI.  CARRY (in
// place): the update also leaves the pair-sum partials of the new X in the scratch, described by
// `list` on return.
template <bool EMIT, bool CARRY>
int run_update(svgd_ctx *c, float *X, const float *G, float *PHI, int n, int64_t D, int64_t ld, float eps,
               hipStream_t s, PairList &list, const RowTable *rt = nullptr)
{
    UpdateArgs ua{};
    ua.h_fixed = c->h_fixed;
    ua.log_n1 = std::log((double)n + 1.0);
    const int64_t half = half_scratch(c);
    int out_cap = CARRY ? (int)std::min<int64_t>(half / pair_stride(n), kMaxParts) : kMaxParts;
    if (CARRY && n <= kValuMaxN) out_cap = mini(out_cap, fused_max_parts(n));
    bool fused = n <= kFusedAlwaysN || (n <= kFusedMaxN && list.nparts <= fused_max_parts(n) && (!CARRY || (int64_t)list.nparts * pair_stride(n) <= half));
    bool from_sums = false;
    int workers = 0;
    // rows that all start on a 128-byte boundary (X's and G's, and PHI's) need no re-aligned stores and
    // can be read with streaming loads
    const bool aligned = rt ? rt->aligned != 0 : rows_aligned(X, ld) && rows_aligned(G, ld) && (!EMIT || rows_aligned(PHI, ld));
    const bool direct = !rt && store_directly(n, D, EMIT, CARRY);
    if (n > kValuMaxN) {
        const int most = update_workers(n, D, c->num_cu, out_cap, beyond_cache(n, ld), aligned, EMIT, CARRY);
        const int w = fused_workers(n, D, c->num_cu, most, CARRY);
        workers = long_list_workers(n, D, c->num_cu, out_cap, beyond_cache(n, ld), aligned, direct, EMIT, CARRY);
        // CARRY: the number of workgroups, which is that of the carried partial sums, depends on the
        // problem only, not on the list that is read: a captured step reads what any other one left
        if (w > 0 && n <= kFusedMaxN && (CARRY ? w + ((D & 63) ? 1 : 0) <= fused_max_parts(n) : fused)) workers = w;
        fused = fused && workers == w;
        from_sums = !fused && sums_inside(n, most, w, aligned, direct, CARRY) && (n <= kFusedMaxN || (int64_t)list.nparts * pair_stride(n) > kDirectMaxFloats);
    }
    int64_t out_off = c->captured ? c->home : 0;
    if (from_sums) {
        int rc = run_reduce(c, n, list, s);
        if (rc) return rc;
        ua.sums = c->sums;
        c->last_n = n;
    } else if (fused) {
        ua.partials = c->partials + list.off;
        ua.nparts = list.nparts;
        if (CARRY) out_off = other_half(c, list.off);
        c->last_n = n;
    } else {
        int rc = run_bandwidth(c, n, list, s);
        if (rc) return rc;
    }
    float *gram_out = c->partials + out_off;
    KernelTimer t(c, SVGD_KERNEL_UPDATE, s);
    // With carried sums one update follows the other with nothing but tiny kernels in between:
    // every other one walks X from the far end, so that it starts on what the previous one
    // touched last (the part of X that the memory-side cache still holds).
    if (!EMIT && CARRY) ua.reverse = (int)(c->sweeps++ & 1u);
    // the four waves of a workgroup on adjacent tiles: always at n > 48; below only for an X beyond
    // the memory-side cache (n = 32, D = 2,000,000, which just fits it, ran 3 % slower that way)
    ua.adjacent = adjacent_tiles(n, ld);
    if (n <= kValuMaxN) {
        const int64_t ngroups = (D + 3) / 4;
        const int grid = clampi((ngroups + 255) / 256, 1, mini(c->num_cu * update_per_cu(n, CARRY), out_cap));
        if (CARRY) list = PairList{out_off, grid};
#define CALL(N) launch_update_valu<N, EMIT, CARRY>(X, G, PHI, c->coef, c->state, D, ld, eps, gram_out, grid, s, rt, ua)
        SVGD_SWITCH_N(n, CALL)
#undef CALL
    } else {
        // workers walk contiguous ranges of full 64-column tiles; one more workgroup does D mod 64
        const int grid = workers + ((D & 63) ? 1 : 0);
        if (CARRY) list = PairList{out_off, grid}; // one partial per workgroup, the tail's included
        if (direct && !aligned && ua.adjacent && own_ranges(tiles_per_range(D / 64, workers, true), EMIT, CARRY)) ua.adjacent = 0;
        ua.per = tiles_per_range(D / 64, workers, ua.adjacent && (aligned || direct)); // (staged stores: a range per wave)
        const UpdateCall call{X, G, PHI, c->coef, c->state, n, D, ld, eps, gram_out, rt, ua, grid, s,
                              aligned ? kStoreLines : (direct ? kStoreDirect : kStoreStaged),
                              from_sums ? kPass2OnSums : (fused ? kPass2OnList : kPass2Apart)};
        if (n <= kFusedMaxN) launch_update_low<EMIT, CARRY>(call);
        else launch_update_high<EMIT, CARRY>(call);
    }
    if (CARRY && c->captured && list.off != c->home) {
        const int n4 = list.nparts * (pair_stride(n) / 4);
        copy_list_kernel<<<(n4 + 255) / 256, 256, 0, s>>>(reinterpret_cast<const f32x4 *>(c->partials + list.off),
                                                          reinterpret_cast<f32x4 *>(c->partials + c->home), n4);
        list.off = c->home;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(c, e);
    return SVGD_OK;
}

// The single-launch path: sizes at which one workgroup does the whole step faster than three
// dependent launches.  It neither reads nor leaves carried pair sums.
bool is_tiny(int n, int64_t D) { return n <= kTinyMaxN && (int64_t)n * D <= kTinyMaxElems; }

template <int WHAT>
int run_tiny(svgd_ctx *c, float *X, const float *G, float *PHI, int n, int64_t D, int64_t ld, float eps, hipStream_t s)
{
    {
        KernelTimer t(c, WHAT == kTinyBandwidth ? SVGD_KERNEL_BANDWIDTH : SVGD_KERNEL_UPDATE, s);
#define TINY(N) step_tiny_kernel<N, WHAT><<<1, kTinyThreads, 0, s>>>(X, G, PHI, D, ld, eps, c->h_fixed, std::log(n + 1.0), c->state, c->coef)
        switch (n) {
        case 1: TINY(1); break;
        case 2: TINY(2); break;
        case 3: TINY(3); break;
        case 4: TINY(4); break;
        case 5: TINY(5); break;
        case 6: TINY(6); break;
        case 7: TINY(7); break;
        default: TINY(8); break;
        }
#undef TINY
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(c, e);
    c->last_n = n;
    return SVGD_OK;
}

// ---------------------------------------------------------------------------------------------
// The entry point that allocates nothing: its scratch is a file-scope device array, one copy per
// GPU, resolved to a device address once per device.
// ---------------------------------------------------------------------------------------------
constexpr int kStaticMaxParts = 528;                         // partial vectors of n(n+1)/2 <= 2080 floats: 2 * 256 + 1 fit
constexpr size_t kStaticPartialsBytes = (size_t)kStaticMaxParts * kMaxPairsFull * sizeof(float);
constexpr size_t kStaticSumsBytes = (size_t)kMaxPairsFull * sizeof(double);
constexpr size_t kStaticCoefBytes = (size_t)kCoefFloats * sizeof(float);
constexpr size_t kStaticBytes = kStaticPartialsBytes + kStaticSumsBytes + kStaticCoefBytes + kStateBytes;
static_assert(kStaticPartialsBytes % 256 == 0 && kStaticSumsBytes % 256 == 0 && kStaticCoefBytes % 256 == 0,
              "every part of the scratch starts on a 256-byte boundary");

// In host code this name is only a stand-in for the symbol: the memory is reached through the
// address that hipGetSymbolAddress returns for the current device (static_ctx below).
static __device__ __align__(256) unsigned char scratch[kStaticBytes];

constexpr int kMaxDevices = 64;
struct StaticCtx {
    bool ready = false;
    svgd_ctx ctx;
};
std::mutex g_static_mutex;
StaticCtx g_static[kMaxDevices];

// The per-device context of svgd_step_static, set up on the first call on that device (which must
// be the current one).  Returns nullptr and sets *rc on failure.
svgd_ctx *static_ctx(int dev, int *rc)
{
    std::lock_guard<std::mutex> lock(g_static_mutex);
    StaticCtx &sc = g_static[dev];
    if (sc.ready) return &sc.ctx;
    unsigned char *ptr = nullptr;
    hipError_t e = hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || ptr == nullptr) {
        (void)hipGetLastError();
        *rc = SVGD_ERR_DEVICE;
        return nullptr;
    }
    int cus = 0;
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess || cus < 1) {
        (void)hipGetLastError();
        *rc = SVGD_ERR_DEVICE;
        return nullptr;
    }
    svgd_ctx &c = sc.ctx;
    c.magic = kMagic;
    c.device = dev;
    c.max_n = SVGD_MAX_PARTICLES;
    c.max_D = SVGD_STATIC_MAX_D;
    c.num_cu = cus > kMaxCu ? kMaxCu : cus; // keeps the Gram grid (one workgroup per CU at n > 12) within kStaticMaxParts
    c.flags = 0;
    c.h_fixed = 0.0;
    c.carry_valid = false;
    c.carry_X = nullptr;
    c.carry_n = 0;
    c.carry_D = c.carry_ld = 0;
    c.carry_nparts = 0;
    c.carry_off = 0;
    c.captured = false;
    c.home = 0;
    c.carry_stream = nullptr;
    c.sweeps = 0;
    c.last_n = 0;
    c.last_hip_error = 0;
    c.partials = reinterpret_cast<float *>(ptr);
    c.partials_cap = (int64_t)kStaticMaxParts * kMaxPairsFull;
    c.sums = reinterpret_cast<double *>(ptr + kStaticPartialsBytes);
    c.state = reinterpret_cast<DevState *>(ptr + kStaticPartialsBytes + kStaticSumsBytes);
    c.coef = reinterpret_cast<float *>(ptr + kStaticPartialsBytes + kStaticSumsBytes + kStateBytes);
    c.profiling = false;
    c.profile_kinds = 0;
    sc.ready = true;
    return &c;
}

} // namespace

extern "C" {

int svgd_create(svgd_handle_t *out, int max_n, int64_t max_D, int device_id, uint32_t flags)
{
    if (!out) return SVGD_ERR_INVALID_ARG;
    *out = nullptr;
    if (max_n < 1 || max_D < 1 || (flags & ~(uint32_t)(SVGD_FLAG_CARRY_GRAM | SVGD_FLAG_FUSE_MFMA)) != 0 || device_id < -1)
        return SVGD_ERR_INVALID_ARG;
    if (max_n > SVGD_MAX_PARTICLES || max_D > SVGD_MAX_D) return SVGD_ERR_TOO_LARGE;

    svgd_ctx *c = new (std::nothrow) svgd_ctx();
    if (!c) return SVGD_ERR_ALLOC;
    c->magic = 0;
    c->max_n = max_n;
    c->max_D = max_D;
    c->flags = flags;
    c->h_fixed = 0.0;
    c->carry_valid = false;
    c->carry_X = nullptr;
    c->carry_n = 0;
    c->carry_D = 0;
    c->carry_ld = 0;
    c->carry_nparts = 0;
    c->carry_off = 0;
    c->captured = false;
    c->home = 0;
    c->carry_stream = nullptr;
    c->sweeps = 0;
    c->partials_cap = 0;
    c->last_n = 0;
    c->last_hip_error = 0;
    c->partials = nullptr;
    c->sums = nullptr;
    c->state = nullptr;
    c->coef = nullptr;
    c->mirror = nullptr;
    c->ticket = 0;
    c->profiling = false;
    c->profile_kinds = ~0u;

    hipError_t e;
    int dev = device_id;
    if (dev < 0) {
        e = hipGetDevice(&dev);
        if (e != hipSuccess) { delete c; return SVGD_ERR_DEVICE; }
    }
    int count = 0;
    e = hipGetDeviceCount(&count);
    if (e != hipSuccess || dev >= count) { delete c; return e != hipSuccess ? SVGD_ERR_DEVICE : SVGD_ERR_INVALID_ARG; }
    c->device = dev;
    DeviceGuard guard(dev);
    int cus = 0;
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess || cus < 1) { delete c; return SVGD_ERR_DEVICE; }
    c->num_cu = cus > kMaxCu ? kMaxCu : cus; // keeps every persistent grid within kMaxParts workgroups

    const size_t P = (size_t)pair_stride(max_n);
    bool ok = hipMalloc(&c->partials, (size_t)kMaxParts * P * sizeof(float)) == hipSuccess &&
              hipMalloc(&c->sums, P * sizeof(double)) == hipSuccess &&
              hipMalloc(&c->state, kStateBytes + (size_t)kCoefFloats * sizeof(float)) == hipSuccess &&
              (c->mirror = take_mirror(dev)) != nullptr;
    if (!ok) {
        (void)hipGetLastError();
        (void)hipFree(c->partials);
        (void)hipFree(c->sums);
        (void)hipFree(c->state);
        delete c;
        return SVGD_ERR_ALLOC;
    }
    c->coef = reinterpret_cast<float *>(reinterpret_cast<char *>(c->state) + kStateBytes);
    c->partials_cap = (int64_t)kMaxParts * (int64_t)P;
    c->magic = kMagic;
    {
        std::lock_guard<std::mutex> lock(g_live_mutex);
        live_handles().insert(c);
    }
    *out = c;
    return SVGD_OK;
}

int svgd_set_bandwidth(svgd_handle_t c, double h_fixed)
{
    int rc = check_handle(c);
    if (rc) return rc;
    if (std::isnan(h_fixed) || std::isinf(h_fixed)) return SVGD_ERR_INVALID_ARG;
    c->h_fixed = h_fixed > 0.0 ? h_fixed : 0.0;
    return SVGD_OK;
}

int svgd_forget_carry(svgd_handle_t c)
{
    int rc = check_handle(c);
    if (rc) return rc;
    c->carry_valid = false;
    return SVGD_OK;
}

int svgd_bandwidth_ld(svgd_handle_t c, const float *X, int n, int64_t D, int64_t ld, double *h_out_host,
                      void *stream)
{
    int rc = check_handle(c);
    if (rc) return rc;
    if (!X) return SVGD_ERR_INVALID_ARG;
    rc = check_shape(c, n, D, ld);
    if (rc) return rc;
    DeviceGuard guard(c->device);
    hipStream_t s = (hipStream_t)stream;
    if (h_out_host && (rc = refuse_capture(c, s))) return rc;
    if (is_tiny(n, D)) {
        rc = run_tiny<kTinyBandwidth>(c, const_cast<float *>(X), nullptr, nullptr, n, D, ld, 0.f, s);
    } else {
        c->carry_valid = false; // the partials buffer is about to be overwritten
        PairList list;
        rc = run_gram(c, X, n, D, ld, s, list);
        if (!rc) rc = run_bandwidth(c, n, list, s);
    }
    if (rc) return rc;
    if (h_out_host) {
        rc = read_back(c, sizeof(DevState), s);
        if (rc) return rc;
        *h_out_host = reinterpret_cast<const DevState *>(c->mirror->data)->h;
    }
    return SVGD_OK;
}

int svgd_bandwidth(svgd_handle_t c, const float *X, int n, int64_t D, double *h_out_host, void *stream)
{
    return svgd_bandwidth_ld(c, X, n, D, D, h_out_host, stream);
}

int svgd_step_ld(svgd_handle_t c, float *X, const float *G, int n, int64_t D, int64_t ld, float eps,
                 void *stream)
{
    int rc = check_handle(c);
    if (rc) return rc;
    if (!X || !G || !std::isfinite(eps)) return SVGD_ERR_INVALID_ARG;
    rc = check_shape(c, n, D, ld);
    if (rc) return rc;
    if (overlaps(X, G, n, D, ld)) return SVGD_ERR_INVALID_ARG;
    DeviceGuard guard(c->device);
    hipStream_t s = (hipStream_t)stream;
    const bool carry_mode = (c->flags & SVGD_FLAG_CARRY_GRAM) != 0;
    // the carried sums (and the tables derived from them) were written on carry_stream: a call
    // on another stream is not ordered after that work and recomputes from X
    const bool use_carry = carry_mode && c->carry_valid && c->carry_X == X && c->carry_n == n &&
                           c->carry_D == D && c->carry_ld == ld && c->carry_stream == s;
    c->carry_valid = false;
    if (is_tiny(n, D)) return run_tiny<kTinyStep>(c, X, G, nullptr, n, D, ld, eps, s);
    PairList list{c->carry_off, c->carry_nparts};
    // A step that reads one half of the scratch and writes the other cannot be replayed: the next replay
    // would read the old sums again.  From the first captured step on, every list on this handle
    // ends up where that step found its own.
    if (carry_mode && !c->captured && is_capturing(s)) {
        c->captured = true;
        c->home = use_carry ? list.off : 0;
    }
    if (!use_carry) {
        rc = run_gram(c, X, n, D, ld, s, list, nullptr, G, carry_mode);
        if (rc) return rc;
        c->sweeps = 0; // a Gram pass ends at the near end of X: the update starts there
    }
    if (!carry_mode) return run_update<false, false>(c, X, G, nullptr, n, D, ld, eps, s, list);
    rc = run_update<false, true>(c, X, G, nullptr, n, D, ld, eps, s, list);
    if (rc) return rc;
    c->carry_off = list.off;
    c->carry_nparts = list.nparts;
    c->carry_valid = true;
    c->carry_X = X;
    c->carry_n = n;
    c->carry_D = D;
    c->carry_ld = ld;
    c->carry_stream = s;
    return SVGD_OK;
}

int svgd_step(svgd_handle_t c, float *X, const float *G, int n, int64_t D, float eps, void *stream)
{
    return svgd_step_ld(c, X, G, n, D, D, eps, stream);
}

int svgd_step_rows(svgd_handle_t c, float *const *X_rows, const float *const *G_rows, int n, int64_t D, float eps,
                   void *stream)
{
    int rc = check_handle(c);
    if (rc) return rc;
    if (!X_rows || !G_rows || !std::isfinite(eps)) return SVGD_ERR_INVALID_ARG;
    rc = check_shape(c, n, D, D);
    if (rc) return rc;
    // every row: non-null, 4-byte aligned; no two of the 2n rows may overlap
    struct Span { uintptr_t lo, hi; };
    Span spans[2 * SVGD_MAX_PARTICLES];
    const uintptr_t bytes = (uintptr_t)D * sizeof(float);
    for (int i = 0; i < n; ++i) {
        const uintptr_t px = (uintptr_t)X_rows[i], pg = (uintptr_t)G_rows[i];
        if (!px || !pg || (px & 3) || (pg & 3)) return SVGD_ERR_INVALID_ARG;
        spans[2 * i] = {px, px + bytes};
        spans[2 * i + 1] = {pg, pg + bytes};
    }
    std::sort(spans, spans + 2 * n, [](const Span &a, const Span &b) { return a.lo < b.lo; });
    for (int i = 1; i < 2 * n; ++i)
        if (spans[i].lo < spans[i - 1].hi) return SVGD_ERR_INVALID_ARG;
    // row starts relative to row 0 (float pointers are 4-byte aligned, so the differences are whole floats)
    RowTable rt;
    rt.aligned = 1;
    for (int i = 0; i < n; ++i)
        if (((uintptr_t)X_rows[i] | (uintptr_t)G_rows[i]) & 127u) rt.aligned = 0;
    for (int i = 0; i < kMaxN; ++i) {
        const int k = i < n ? i : 0;
        rt.x[i] = (int64_t)(((intptr_t)X_rows[k] - (intptr_t)X_rows[0]) / (intptr_t)sizeof(float));
        rt.g[i] = (int64_t)(((intptr_t)G_rows[k] - (intptr_t)G_rows[0]) / (intptr_t)sizeof(float));
        rt.ri[i] = (int32_t)(((uintptr_t)X_rows[k] >> 2) & 31u);
    }
    DeviceGuard guard(c->device);
    hipStream_t s = (hipStream_t)stream;
    c->carry_valid = false; // the partials buffer is about to be overwritten; nothing is carried for separate rows
    float *X = X_rows[0];
    const float *G = G_rows[0];
    PairList list;
    rc = run_gram(c, X, n, D, D, s, list, &rt, G);
    if (rc) return rc;
    return run_update<false, false>(c, X, G, nullptr, n, D, D, eps, s, list, &rt);
}

int svgd_phi_ld(svgd_handle_t c, const float *X, const float *G, int n, int64_t D, int64_t ld, float *PHI,
                void *stream)
{
    int rc = check_handle(c);
    if (rc) return rc;
    if (!X || !G || !PHI) return SVGD_ERR_INVALID_ARG;
    rc = check_shape(c, n, D, ld);
    if (rc) return rc;
    if (overlaps(X, PHI, n, D, ld) || overlaps(G, PHI, n, D, ld)) return SVGD_ERR_INVALID_ARG;
    DeviceGuard guard(c->device);
    hipStream_t s = (hipStream_t)stream;
    if (is_tiny(n, D)) return run_tiny<kTinyPhi>(c, const_cast<float *>(X), G, PHI, n, D, ld, 0.f, s);
    c->carry_valid = false; // the partials buffer is about to be overwritten
    PairList list;
    rc = run_gram(c, X, n, D, ld, s, list, nullptr, rows_aligned(PHI, ld) ? G : nullptr);
    if (rc) return rc;
    return run_update<true, false>(c, const_cast<float *>(X), G, PHI, n, D, ld, 0.f, s, list);
}

int svgd_phi(svgd_handle_t c, const float *X, const float *G, int n, int64_t D, float *PHI, void *stream)
{
    return svgd_phi_ld(c, X, G, n, D, D, PHI, stream);
}

int svgd_step_static(float *X, const float *G, int n, int64_t D, int64_t ld, float eps, void *stream)
{
    if (!X || !G || !std::isfinite(eps) || n < 1 || D < 1 || ld < D) return SVGD_ERR_INVALID_ARG;
    if (n > SVGD_MAX_PARTICLES || D > SVGD_STATIC_MAX_D) return SVGD_ERR_TOO_LARGE;
    if (overlaps(X, G, n, D, ld)) return SVGD_ERR_INVALID_ARG;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return SVGD_ERR_DEVICE;
    }
    if (dev < 0 || dev >= kMaxDevices) return SVGD_ERR_DEVICE;
    int rc = SVGD_OK;
    svgd_ctx *c = static_ctx(dev, &rc);
    if (!c) return rc;
    // Every part of the scratch that a kernel reads has been written by an earlier kernel of the
    // same call (partials by all workgroups of the pairwise-d2 pass, their sums, the state and
    // the coefficient tables by the passes after it): nothing has to start at zero.
    hipStream_t s = (hipStream_t)stream;
    if (is_tiny(n, D)) return run_tiny<kTinyStep>(c, X, G, nullptr, n, D, ld, eps, s);
    PairList list;
    rc = run_gram(c, X, n, D, ld, s, list, nullptr, G, false);
    if (rc) return rc;
    return run_update<false, false>(c, X, G, nullptr, n, D, ld, eps, s, list);
}

int svgd_get_last(svgd_handle_t c, double *h_out, float *K_host, void *stream)
{
    int rc = check_handle(c);
    if (rc) return rc;
    if (c->last_n < 1) return SVGD_ERR_INVALID_ARG;
    DeviceGuard guard(c->device);
    hipStream_t s = (hipStream_t)stream;
    if (h_out || K_host) { // h and K lie in one piece (DevState, K)
        if ((rc = refuse_capture(c, s))) return rc;
        const size_t kbytes = K_host ? (size_t)c->last_n * c->last_n * sizeof(float) : 0;
        rc = read_back(c, kStateBytes + kbytes, s);
        if (rc) return rc;
        if (h_out) *h_out = reinterpret_cast<const DevState *>(c->mirror->data)->h;
        if (K_host) std::memcpy(K_host, c->mirror->data + kStateBytes, kbytes);
        return SVGD_OK;
    }
    hipError_t e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail(c, e);
    return SVGD_OK;
}

int svgd_diag_copy(void *dst, const void *src, int64_t nbytes, void *stream)
{
    if (!dst || !src || nbytes < 16 || (nbytes & 15) || ((uintptr_t)dst & 15) || ((uintptr_t)src & 15))
        return SVGD_ERR_INVALID_ARG;
    diag_copy_kernel<<<2048, 256, 0, (hipStream_t)stream>>>((const f32x4 *)src, (f32x4 *)dst, nbytes >> 4);
    return hipGetLastError() == hipSuccess ? SVGD_OK : SVGD_ERR_DEVICE;
}

int svgd_diag_axpy_rows(float *X, const float *G, int n, int64_t D, int64_t ld, float s, int pattern,
                        int workgroups, void *stream)
{
    const int base = pattern & 15, reverse = (pattern >> 4) & 1;
    if (!X || !G || n < 1 || D < 1 || ld < D || workgroups < 1 || workgroups > 65536 || pattern < 0 || pattern > 31 || base > 11)
        return SVGD_ERR_INVALID_ARG;
    if (overlaps(X, G, n, D, ld)) return SVGD_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
#define AXPY(PAT, U, NT) diag_axpy_rows_kernel<PAT, U, NT><<<workgroups, 256, 0, st>>>(X, G, n, D, ld, s, reverse)
    switch (base) {
    case 0: AXPY(0, 8, 0); break;
    case 1: AXPY(1, 8, 0); break;
    case 2: AXPY(0, 16, 0); break;
    case 3: AXPY(1, 16, 0); break;
    case 4: AXPY(0, 8, 1); break;
    case 5: AXPY(1, 8, 1); break;
    case 6: AXPY(0, 16, 1); break;
    case 7: AXPY(1, 16, 1); break;
    case 8: AXPY(0, 8, 2); break;
    case 9: AXPY(1, 8, 2); break;
    case 10: AXPY(0, 16, 2); break;
    default: AXPY(1, 16, 2); break;
    }
#undef AXPY
    return hipGetLastError() == hipSuccess ? SVGD_OK : SVGD_ERR_DEVICE;
}

int svgd_diag_read_rows(const float *X, int n, int64_t D, int64_t ld, float *sink, int pattern, int workgroups,
                        void *stream)
{
    if (!X || !sink || n < 1 || D < 1 || ld < D || workgroups < 1 || workgroups > 65536 || pattern < 0 || pattern > 3)
        return SVGD_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    switch (pattern) {
    case 0: diag_read_rows_kernel<0, 0><<<workgroups, 256, 0, st>>>(X, n, D, ld, sink); break;
    case 1: diag_read_rows_kernel<1, 0><<<workgroups, 256, 0, st>>>(X, n, D, ld, sink); break;
    case 2: diag_read_rows_kernel<0, 1><<<workgroups, 256, 0, st>>>(X, n, D, ld, sink); break;
    default: diag_read_rows_kernel<1, 1><<<workgroups, 256, 0, st>>>(X, n, D, ld, sink); break;
    }
    return hipGetLastError() == hipSuccess ? SVGD_OK : SVGD_ERR_DEVICE;
}

int swag_update_moments(float *mean, float *sqmean, const float *X, int n, int64_t D, int64_t count,
                        void *stream)
{
    if (!mean || !sqmean || !X || n < 1 || D < 1 || count < 0) return SVGD_ERR_INVALID_ARG;
    if (overlaps(mean, X, n, D, D) || overlaps(sqmean, X, n, D, D) || overlaps(mean, sqmean, n, D, D))
        return SVGD_ERR_INVALID_ARG;
    const int64_t total = (int64_t)n * D;
    const int64_t ngroups = (total + 3) / 4;
    int cus = 0, dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        return SVGD_ERR_DEVICE;
    // the line where the two kernels cross: n D = 9,600,112 (115 MB) 34.3 us for many waves, 35.6 for BIG,
    // 16,000,112 (192 MB) 58.6 and 57.7
    const bool big = total * 3 * (int64_t)sizeof(float) > kMemorySideCacheBytes / 8 * 5;
    const int grid = clampi((ngroups + 255) / 256, 1, cus * (big ? 1 : 8));
    const float inv = (float)(1.0 / ((double)count + 1.0));
    if (big) swag_moments_kernel<true><<<grid, 256, 0, (hipStream_t)stream>>>(mean, sqmean, X, total, inv, count == 0);
    else swag_moments_kernel<false><<<grid, 256, 0, (hipStream_t)stream>>>(mean, sqmean, X, total, inv, count == 0);
    return hipGetLastError() == hipSuccess ? SVGD_OK : SVGD_ERR_DEVICE;
}

int svgd_profile_begin_kinds(svgd_handle_t c, unsigned kinds)
{
    int rc = check_handle(c);
    if (rc) return rc;
    if ((kinds & ((1u << SVGD_KERNEL_KINDS) - 1u)) == 0) return SVGD_ERR_INVALID_ARG;
    {   // all events and the record list exist before the first timed launch
        DeviceGuard guard(c->device);
        try {
            c->ev_kind.reserve(kMaxProfileRecords);
            c->ev_pool.reserve(2 * kMaxProfileRecords);
        } catch (...) {
            return SVGD_ERR_ALLOC;
        }
        while (c->ev_pool.size() < 2 * kMaxProfileRecords) {
            hipEvent_t e;
            hipError_t rc_e = hipEventCreate(&e);
            if (rc_e != hipSuccess) return fail(c, rc_e);
            c->ev_pool.push_back(e);
        }
    }
    c->ev_kind.clear();
    c->profile_kinds = kinds;
    c->profiling = true;
    return SVGD_OK;
}

int svgd_profile_begin(svgd_handle_t c) { return svgd_profile_begin_kinds(c, ~0u); }

int svgd_profile_end_records(svgd_handle_t c, double *ms_sum, int *count, int *rec_kind, float *rec_ms,
                             int rec_cap, int *rec_count)
{
    int rc = check_handle(c);
    if (rc) return rc;
    if (!ms_sum || !count || rec_cap < 0 || (rec_cap > 0 && (!rec_kind || !rec_ms))) return SVGD_ERR_INVALID_ARG;
    c->profiling = false;
    for (int k = 0; k < SVGD_KERNEL_KINDS; ++k) { ms_sum[k] = 0.0; count[k] = 0; }
    if (rec_count) *rec_count = 0;
    DeviceGuard guard(c->device);
    for (size_t r = 0; r < c->ev_kind.size(); ++r) {
        hipError_t e = hipEventSynchronize(c->ev_pool[2 * r + 1]);
        float ms = 0.f;
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, c->ev_pool[2 * r], c->ev_pool[2 * r + 1]);
        if (e != hipSuccess) { c->ev_kind.clear(); return fail(c, e); }
        ms_sum[c->ev_kind[r]] += (double)ms;
        count[c->ev_kind[r]] += 1;
        if ((int)r < rec_cap) {
            rec_kind[r] = c->ev_kind[r];
            rec_ms[r] = ms;
            if (rec_count) *rec_count = (int)r + 1;
        }
    }
    c->ev_kind.clear();
    return SVGD_OK;
}

int svgd_profile_end(svgd_handle_t c, double *ms_sum, int *count)
{
    return svgd_profile_end_records(c, ms_sum, count, nullptr, nullptr, 0, nullptr);
}

int svgd_destroy(svgd_handle_t c)
{
    int rc = check_handle(c);
    if (rc) return rc;
    {
        std::lock_guard<std::mutex> lock(g_live_mutex);
        live_handles().erase(c);
    }
    c->magic = 0;
    hipError_t e = hipSuccess, t;
    {
        DeviceGuard guard(c->device);
        if ((t = hipFree(c->partials)) != hipSuccess) e = t;
        if ((t = hipFree(c->sums)) != hipSuccess) e = t;
        if ((t = hipFree(c->state)) != hipSuccess) e = t;
        // (a request that was never answered may still be on its way)
        if ((t = give_mirror(c->mirror, c->device, __atomic_load_n(&c->mirror->ticket, __ATOMIC_ACQUIRE) == c->ticket)) != hipSuccess) e = t;
        for (hipEvent_t ev : c->ev_pool) (void)hipEventDestroy(ev);
    }
    delete c;
    return e == hipSuccess ? SVGD_OK : SVGD_ERR_DEVICE;
}

int svgd_last_device_error(svgd_handle_t c)
{
    if (check_handle(c)) return 0;
    return c->last_hip_error;
}

const char *svgd_status_string(int status)
{
    switch (status) {
    case SVGD_OK: return "SVGD_OK";
    case SVGD_ERR_INVALID_ARG: return "SVGD_ERR_INVALID_ARG";
    case SVGD_ERR_BAD_HANDLE: return "SVGD_ERR_BAD_HANDLE";
    case SVGD_ERR_TOO_LARGE: return "SVGD_ERR_TOO_LARGE";
    case SVGD_ERR_ALLOC: return "SVGD_ERR_ALLOC";
    case SVGD_ERR_DEVICE: return "SVGD_ERR_DEVICE";
    default: return "SVGD_ERR_UNKNOWN";
    }
}

} // extern "C"
