// How the matrix-core update's work is split, as far as numbers decide it (host code, nothing of HIP).
#pragma once
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
    const int64_t tiles = tiles_per_wave(nfull, num_cu - 1);
    if (tiles == tiles_per_wave(nfull, num_cu)) return true;
    if (carry) return tiles <= (n <= 36 ? 8 : (n <= 48 ? 5 : 3));
    if (n > 48) return false;
    const bool full_dense = (n & 15) == 0 && !aligned;
    if (tiles == 2) return full_dense || ((emit || nfull == 4 * (int64_t)num_cu) && (n < 48 || !aligned));
    if (tiles == 3) return full_dense || (emit && n <= 36);
    return tiles <= (n <= 36 ? kTailRoomTiles : (full_dense ? 5 : 4));
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
