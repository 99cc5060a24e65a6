// Launching the matrix-core update: which instance of update_mfma_kernel a call takes.  The instances are compiled in
// files of their own (update_*.hip), one per kind of call and half of the particle counts, so that
// they build side by side.
#pragma once
#include "launch_rules.hpp"
#include "update_kernels.hpp"

namespace svgd {

struct UpdateCall {
    float *X;
    const float *G;
    float *PHI;
    float *coef;
    DevState *st;
    int n;
    int64_t D, ld;
    float eps;
    float *gram_out;
    const RowTable *rt; // separate rows
    UpdateArgs ua;
    int grid;
    hipStream_t stream;
    int store;  // StoreMode
    int pass2;  // Pass2
};

template <int NB, bool EMIT, bool CARRY, bool FULL, bool REM, int P2>
void launch_update_instance(const UpdateCall &c)
{
#define UPD(STORE, ROWS, REV, rows)                                                                                   \
    update_mfma_kernel<NB, EMIT, FULL, CARRY, STORE, ROWS, P2, REV, REM><<<c.grid, 256, 0, c.stream>>>(               \
        c.X, c.G, c.PHI, c.coef, c.st, c.n, c.D, c.ld, c.eps, c.gram_out, rows, c.ua)
    constexpr bool STAGED = P2 != kPass2OnSums; // (the host sees to it)
    if constexpr (!EMIT && !CARRY) {
        if (c.rt) {
            if (c.store == kStoreLines) UPD(kStoreLines, true, false, *c.rt);
            else if constexpr (STAGED) UPD(kStoreStaged, true, false, *c.rt);
            return;
        }
    }
    if (c.store == kStoreLines) UPD(kStoreLines, false, false, NoRows{});
    else if (c.store == kStoreDirect) UPD(kStoreDirect, false, false, NoRows{});
    else if constexpr (STAGED) {
        if (CARRY && c.ua.reverse) UPD(kStoreStaged, false, CARRY, NoRows{});
        else UPD(kStoreStaged, false, false, NoRows{});
    }
#undef UPD
}

template <int NB, bool EMIT, bool CARRY, bool FULL, bool REM>
void launch_update_blocks(const UpdateCall &c)
{
    constexpr int NMAX = 16 * NB + (REM ? 4 : 0);
    if constexpr (NMAX <= 20) {
        launch_update_instance<NB, EMIT, CARRY, FULL, REM, kPass2OnList>(c); // n <= kFusedAlwaysN
    } else {
        if constexpr (NMAX <= 32) {
            if (c.pass2 == kPass2OnList) return launch_update_instance<NB, EMIT, CARRY, FULL, REM, kPass2OnList>(c);
        }
        if constexpr (NMAX <= 48) {
            if (c.pass2 == kPass2OnSums) return launch_update_instance<NB, EMIT, CARRY, FULL, REM, kPass2OnSums>(c);
        }
        launch_update_instance<NB, EMIT, CARRY, FULL, REM, kPass2Apart>(c);
    }
}

// 13 to 32 particles, and 33 to 64
template <bool EMIT, bool CARRY>
void launch_update_low(const UpdateCall &c)
{
    const int n = c.n;
    if (has_remainder_rows(n)) launch_update_blocks<1, EMIT, CARRY, true, true>(c);
    else if (n == 16) launch_update_blocks<1, EMIT, CARRY, true, false>(c);
    else if (n < 16) launch_update_blocks<1, EMIT, CARRY, false, false>(c);
    else if (n == 32) launch_update_blocks<2, EMIT, CARRY, true, false>(c);
    else launch_update_blocks<2, EMIT, CARRY, false, false>(c);
}
template <bool EMIT, bool CARRY>
void launch_update_high(const UpdateCall &c)
{
    const int n = c.n;
    if (has_remainder_rows(n) && n < 48) launch_update_blocks<2, EMIT, CARRY, true, true>(c);
    else if (has_remainder_rows(n)) launch_update_blocks<3, EMIT, CARRY, true, true>(c);
    else if (n == 48) launch_update_blocks<3, EMIT, CARRY, true, false>(c);
    else if (n == 64) launch_update_blocks<4, EMIT, CARRY, true, false>(c);
    else if (n < 48) launch_update_blocks<3, EMIT, CARRY, false, false>(c);
    else launch_update_blocks<4, EMIT, CARRY, false, false>(c);
}

#ifndef SVGD_UPDATE_INSTANCES
#define SVGD_EXTERN(EMIT, CARRY)                                                                                      \
    extern template void launch_update_low<EMIT, CARRY>(const UpdateCall &);                                          \
    extern template void launch_update_high<EMIT, CARRY>(const UpdateCall &);
SVGD_EXTERN(false, false)
SVGD_EXTERN(true, false)
SVGD_EXTERN(false, true)
#undef SVGD_EXTERN
#endif

} // namespace svgd
