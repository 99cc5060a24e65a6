// How the matrix-core update's work is split, as far as numbers decide it (host code, nothing of HIP).
#pragma once
#include <algorithm>
#include <cstdint>

namespace svgd {

// One to four particles beyond a multiple of 16 ride along as remainder rows of the kernel for that multiple.
inline bool has_remainder_rows(int n) { return n > 16 && (n & 15) >= 1 && (n & 15) <= 4; }

// The instances of the matrix-core update whose blocks of rows are full, and all above 32 particles, take the registers of a
// whole CU with one workgroup; the others leave room for a second.
inline bool takes_whole_cu(int n) { return n > 32 || (n & 15) == 0 || has_remainder_rows(n); }

// The most 64-column tiles that one of the four waves of a workgroup gets, whether they have a range each or share one.
inline int64_t tiles_per_wave(int64_t nfull, int64_t workers) { return (nfull + 4 * workers - 1) / (4 * workers); }

// Whether one worker less than there are CUs makes room for the workgroup that does D mod 64.  Where a workgroup takes all
// registers of its CU, that one otherwise starts when the first worker ends: up to kTailRoomTiles tiles per wave there is one
// worker less.  us per step with 256 and 255 workers: n = 48, D = 120,011, padded, carried sums 35.0 and 28.6, n = 64 48.0 and
// 39.7, plain, dense 51.4 and 45.8; D = 300,007 (five tiles per wave) 74.1 and 68.4, plain 91.3 and 90.2; D = 800,003 (12) 138.2
// and 137.7.  Beyond, the workgroups end so far apart that the tail is done in time, and a worker less costs its share
// (n = 64, D = 11,173,962, carried sums 1698 and 1715).
// Above 48 particles a workgroup's waves share a range, and just above a multiple of 1,024 tiles so few workgroups have one that the
// tail finds a CU all the same, up to seven eighths of them (28 of the 32 of an XCD, seven in each of its four shader engines): us with
// 256 and 255 workers, padded, seven tiles per workgroup, n = 64, 224 workgroups 45.4 and 45.4, 225 49.7 and 45.9, phi 42.7 and
// 42.7, 48.3 and 42.9; five, 218, n = 50 35.6 and 37.3, n = 56 40.1 and 41.6.  (Dense rows without carried sums, in ranges of their own at five and
// six tiles: a worker less is 1 to 2 % faster at 56 and 60 particles and up to 4 % slower at 49 to 51.)
// Just below a multiple of 1,024 tiles a worker less gives the waves a tile more.  Still the faster way, us with 256 and 255
// (tiles per wave with 255):
// - on carried sums, whose tail takes longer, up to 8 tiles at 36 particles, 5 at 48, 3 above: padded, D = 65,500 (2), n = 33
//   25.1 and 21.1, n = 48 29.0 and 25.6, n = 64 38.4 and 35.9; D = 196,100 (4), n = 48 40.9 and 39.0, n = 64 56.7 and 57.0;
//   D = 261,500 (5), n = 36 40.1 and 39.3, n = 48 46.1 and 45.0, n = 64 64.0 and 64.8; D = 785,307 (13), n = 33 66.4 and 69.1.
// - up to 48 particles, where it lets pass 2 be part of the update, from four tiles on, up to 16 at 36 particles, four or five
//   above: dense, D = 196,100 (4), n = 33 38.6 and 36.2, n = 48 52.1 and 48.6; padded, D = 391,000 (7), n = 33 51.2 and 50.6,
//   n = 44 64.8 and 66.5.  With two or three it goes one way or the other: phi, dense, D = 65,500 (2), n = 33 24.4 and 21.6,
//   n = 44 27.4 and 26.6, padded n = 44 26.7 and 25.5, but n = 48 27.8 and 29.0; D = 131,000 (3), dense n = 33 29.7 and 30.3,
//   padded 28.6 and 27.6, n = 44 37.6 and 38.4, 33.2 and 34.2.  A step with full blocks of rows, dense, D = 131,000, n = 48 42.5
//   and 39.0; other steps up to 14 % slower (D = 65,400, padded n = 33 24.3 and 25.6, n = 48 28.6 and 32.0; dense n = 44 27.5 and
//   28.7), but for exactly four tiles per CU (a workgroup of the pairwise pass and one of the update then have the same columns;
//   dense, n = 32 22.7 and 19.2, n = 44 29.4 and 27.2; padded n = 33 25.4 and 23.9, but n = 48 29.4 and 30.6).
// Otherwise a worker less costs up to a tenth there (above 48, padded, plain, D = 65,400 n = 52 33.5 and 37.4, n = 64 35.9 and
// 38.8; D = 131,000 n = 52 45.6 and 49.4).
// aligned: all rows on 128-byte boundaries; emit: phi is written out; carry: the update leaves pair sums.
constexpr int kTailRoomTiles = 16;
inline bool leaves_room_for_tail(int n, int64_t D, int num_cu, bool aligned, bool emit, bool carry)
{
    const int64_t nfull = D / 64;
    if (!takes_whole_cu(n) || (D & 63) == 0 || num_cu < 2 || nfull > (int64_t)kTailRoomTiles * 4 * num_cu) return false;
    const int64_t per = std::max<int64_t>((nfull + num_cu - 1) / num_cu, 1);
    if (n > 48 && (aligned || carry) && 8 * ((nfull + per - 1) / per) <= 7 * (int64_t)num_cu) return false;
    const int64_t tiles = tiles_per_wave(nfull, num_cu - 1);
    if (tiles == tiles_per_wave(nfull, num_cu)) return true;
    if (carry) return tiles <= (n <= 36 ? 8 : (n <= 48 ? 5 : 3));
    if (n > 48) return false;
    const bool full_dense = (n & 15) == 0 && !aligned;
    if (tiles == 2) return full_dense || ((emit || nfull == 4 * (int64_t)num_cu) && (n < 48 || !aligned));
    if (tiles == 3) return full_dense || (emit && n <= 36);
    return tiles <= (n <= 36 ? kTailRoomTiles : (full_dense ? 5 : 4));
}

// Worker workgroups of the matrix-core update (each walks ranges of 64-column tiles; one more
// workgroup does D mod 64): one per CU - the kernel overlaps its own loads with its multiplies, and
// fewer concurrent row streams keep more HBM pages open.  Exception: 21 to 24 particles, whose
// tiles cost the instructions of 32 rows but move little more than half the bytes, so that the
// fixed costs of a tile show (17 to 20 are 16 rows plus remainder rows, see has_remainder_rows).
// The kernel instances for n not a multiple of 16, n < 32, are built for two waves per SIMD, and
// for those particle counts and an X beyond the memory-side cache two workgroups per CU overlap
// one's arithmetic with the other's loads (with carried sums at D = 5,000,000: n = 24
// 258 -> 241 us; from n = 25 on the gain is below the cost of the longer list of partial sums,
// with 16 or 32 particles the second workgroup costs 2-5 %, and for an X that cache serves it
// costs 9 %).
// `cap` bounds the grid, the tail's workgroup included; beyond_cache: of an X that the memory-side cache does not hold.
// (D mod 64 = 0: no workgroup for the tail.)
// One worker less where that makes room for the tail's workgroup (leaves_room_for_tail).
inline int update_workers(int n, int64_t D, int num_cu, int cap, bool beyond_cache, bool aligned, bool emit, bool carry)
{
    const int64_t nfull = D / 64;
    const int per_cu = (n >= 17 && n <= 24 && !has_remainder_rows(n) && beyond_cache) ? 2 : 1;
    const int max_workers = std::min(num_cu * per_cu - (leaves_room_for_tail(n, D, num_cu, aligned, emit, carry) ? 1 : 0), cap - 1);
    return (int)std::max<int64_t>(std::min<int64_t>((nfull + 3) / 4, max_workers), 1);
}

// Pass 2 is part of the update only if all its workgroups are resident at once, or it is paid for twice: the instances
// whose blocks are full take a CU's registers for one workgroup, the others for half of one.  Where
// the tail's workgroup comes on top of a worker for every CU, one worker less makes room for it
// (257 and 256 workgroups: n = 16, D = 300,007 35 and 25 us per step; n = 13, D = 100,003, padded rows,
// carried sums 16.1 and 13.8).  That may give the waves a tile more, which is still the faster way
// with full blocks (n = 16, D = 131,100, two tiles per wave or three: 32 us in 257 workgroups, 22.9
// in launches of their own, 21.9) and, carrying sums, where the tail's workgroup takes longer, up to 15
// particles (n = 15, same D, padded: 17.8 and 14.2); otherwise two workgroups share a CU (n = 15,
// plain step: 17.5, 21.1 with a tile more; n = 21, carried: 23.8 and 27.3).
// Returns the number of workers, 0: not as one launch (21 particles or more only).
inline int fused_workers(int n, int64_t D, int num_cu, int workers, bool carry)
{
    const bool full_rows = takes_whole_cu(n);
    const int64_t nfull = D / 64;
    for (int per_cu = 1; per_cu <= (full_rows ? 1 : 2); ++per_cu) {
        const int room = std::max(num_cu * per_cu - ((D & 63) ? 1 : 0), 1);
        if (workers <= room) return workers;
        if (full_rows || (carry && n < 16) || tiles_per_wave(nfull, room) == tiles_per_wave(nfull, workers)) return room;
    }
    return 0;
}

// 21 to kSumsMaxN particles and a list too long to be read by every workgroup: a launch of many workgroups sums it, and
// the update's workgroups start with pass 2 on the sums - a launch less than with pass 2 in between, and the tile's first
// loads and the tables of C are no longer waited for behind it.  us per step, apart and inside: n = 24, dense, D = 50,001
// 18.2 and 15.9, D = 120,011 23.6 and 21.5, n = 28, carried, padded, D = 40,003 15.6 and 13.7, n = 32, D = 16,403 17.7 and 15.2,
// phi 17.1 and 14.9, D = 120,011 26.9 and 23.3, carried, padded 25.1 and 19.6, n = 33, D = 25,003 21.8 and 20.1, n = 40,
// D = 50,021, plain 25.6 and 23.9, n = 48 26.6 and 25.2; separate rows, n = 24, D = 1,500,001 120.9 and 118.4, padded, n = 32,
// D = 2,000,000 195.4 and 193.9.  From 49 particles on 256 threads take longer for pass 2 than the 1024 of a launch of its
// own and that launch together (n = 50, D = 50,021 30.3 and 30.1, n = 56 32.9 and 33.4, n = 64 32.4 and 34.0).
// Not with re-aligned stores (two instances per kernel instead of three or four), and only where all workgroups are resident
// without a tile more for any wave, or where leaves_room_for_tail has it so.  Above 32 particles a list that the launch of pass 2 sums by itself saves no launch.
constexpr int kFusedAlwaysN = 20; // (their lists are never that long)
constexpr int kSumsMaxN = 48;

// Whether it does: `workers` and `w` as update_workers and fused_workers have them.
inline bool sums_inside(int n, int workers, int w, bool aligned, bool direct, bool carry)
{
    return n > kFusedAlwaysN && n <= kSumsMaxN && (w == workers || (w > 0 && !takes_whole_cu(n))) && (direct || (!carry && aligned));
}

// The workers of an update that reads a long list: all resident where pass 2 is inside.  The pairwise pass orders its slabs by
// their ranges (with 256 there and 255 here, few of the tiles that it leaves in the cache are the first of a range: n = 31,
// D = 5,000,003, padded 448 us per step, 432 with the same; n = 16, D = 9,000,003 414 and 402).
inline int long_list_workers(int n, int64_t D, int num_cu, int cap, bool beyond_cache, bool aligned, bool direct, bool emit, bool carry)
{
    const int workers = update_workers(n, D, num_cu, cap, beyond_cache, aligned, emit, carry), w = fused_workers(n, D, num_cu, workers, carry);
    return w > 0 && (n <= kFusedAlwaysN || sums_inside(n, workers, w, aligned, direct, carry)) ? w : workers;
}

// Direct stores above 48 particles: whether the waves of a workgroup take ranges of their own rather than adjacent tiles of one of
// `per` tiles.  With five or six, one or two waves of each workgroup have a tile more than the others, on nearly all CUs, where
// ranges of their own give as many tiles to every wave of two thirds of them.  us, adjacent and in ranges of their own, with 255 workers
// and the tail's workgroup: a plain step with five tiles n = 52, D = 73,627 37.6 and 36.7, n = 56 41.6 and 38.9, n = 64 41.2 and
// 38.7, with six n = 52, D = 83,227 38.7 and 37.5, D = 97,627 41.3 and 40.5, n = 64 42.0 and 41.6, 45.0 and 45.9; phi with five
// n = 52 37.0 and 37.4, n = 56 41.8 and 39.6, n = 64 41.3 and 40.0, with six n = 52 38.1 and 38.7, n = 64 41.6 and 43.0.  On
// carried sums the adjacent tiles are ahead (n = 64, five 35.5 and 36.7, six 35.4 and 37.7), and with seven tiles and more
// for all (n = 64, D = 108,827, seven, 45.4 and 48.3; D = 131,163, nine, 51.6 and 53.1, phi 51.4 and 53.9; D = 146,971 54.7 and 58.2).
// With 256 workers and no tail the same: a step with five 36.5 and 34.3 (n = 52, D = 76,800), with nine 3 % the other way.
inline bool own_ranges(int64_t per, bool emit, bool carry) { return !carry && (per == 5 || (per == 6 && !emit)); }

} // namespace svgd
