// Which lattices and launches take the Wilson stencil's tile form
// (wilson_tile.h), and with which tile; host arithmetic only.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

namespace ovl {

// A tile: its extents, the tiles per direction and the multipliers that divide
// by the extents (n / d = n * m >> 20, exact for n < 512 and d <= 512).  nt threads
// a block; nt = 0: no tiles.
struct Tile {
    int T[4], N[4];
    unsigned m3, m2, m1;
    int nt;
};

inline int tile_count(const Tile &t) { return t.N[0] * t.N[1] * t.N[2] * t.N[3]; }
inline int tile_sites(const Tile &t) { return t.T[0] * t.T[1] * t.T[2] * t.T[3]; }

// The tile of a lattice.  From 131072 sites on (a 512-site tile for each of 256
// CUs) every lattice measured gains with one FP64 field, below it some lose and
// there are none (one site per thread / tiles: FP64 D_W, mixed overlap apply):
//   16^4      13.7 / 16.1 us    5.80 / 6.21 ms     65536 sites
//   28x14^2x16 16.4 / 17.0      7.87 / 7.83        87808
//   24x16^3   17.6 / 19.1       7.94 / 8.15        98304
//   18^4      23.4 / 21.0       9.30 / 9.04       104976
//   28x16^3   23.5 / 20.9       8.90 / 8.73       114688
//   20x18^3   26.7 / 28.0       9.68 / 10.81      116640
//   32x16^3   32.2 / 23.1      10.56 / 9.84       131072
//   24x18^3   35.0 / 31.0      13.77 / 13.36      139968
// Rows of x3 stay whole up to 32 sites or are cut into multiples of 8 (a row is
// then whole 128-byte lines or nearly so); a lattice whose rows allow neither has
// no tiles (34x2x44x46, rows of 23: 0.96 of the one-site form's rate; 24x20x26x34,
// rows of 17: 1.00).  The other extents are divisors of the lattice's, and the
// choice follows a sweep over eight lattices of 131072 to 663552 sites: x2, whose
// neighbours are the nearest blocks, at least 2 (48x22^3: 115 us with 4x2x2x22, 137
// with 4x2x1x22), time about 4, x1 least of all; and blocks that fill the last
// round of a CU's 512 threads (40x18^3: 47 us at 2.8 rounds, 50 at 2.1).
constexpr int64_t kTileSites = 512 * 256;

inline Tile pick_tile(const int E[4], int64_t V)
{
    Tile best{};
    if (V < kTileSites) return best;
    int t3 = 0;
    for (int d = std::min(32, E[3]); d > 0 && !t3; d--)
        if (E[3] % d == 0 && (d == E[3] || d % 8 == 0)) t3 = d;
    if (!t3) return best;
    double least = 1e300;
    for (int nt : {512, 256})
        for (int t2 = 1; t2 <= std::min(8, E[2]) && t2 * t3 <= nt; t2++) {
            if (E[2] % t2) continue;
            for (int t1 = 1; t1 <= std::min(8, E[1]) && t1 * t2 * t3 <= nt; t1++) {
                if (E[1] % t1) continue;
                for (int t0 = 1; t0 <= std::min(8, E[0]) && t0 * t1 * t2 * t3 <= nt; t0++) {
                    if (E[0] % t0 || 2 * t0 * t1 * t2 * t3 <= nt) continue;
                    const Tile t{{t0, t1, t2, t3}, {E[0] / t0, E[1] / t1, E[2] / t2, E[3] / t3}, 0, 0, 0, nt};
                    const double rounds = (double)t.N[0] * t.N[1] * t.N[2] * t.N[3] * nt / (256 * 512);
                    const double cost = (3.0 + 1.5 / t0 + 0.05 * t0 + 0.7 / t1 + 2.5 / t2) *
                                        std::sqrt(std::ceil(rounds) / rounds);
                    if (cost < least) {
                        least = cost;
                        best = t;
                    }
                }
            }
        }
    auto inverse = [](int d) { return (unsigned)(((1u << 20) + d - 1) / d); };
    if (best.nt) {
        best.m3 = inverse(best.T[3]);
        best.m2 = inverse(best.T[2]);
        best.m1 = inverse(best.T[1]);
    }
    return best;
}

// Whether a launch on nrhs fields takes the lattice's tiles.  What a tile saves
// is spinor reads; it pays for that with threads that hold no site and, on
// several fields, with fewer neighbours left in L2.  Rates of the tile form over
// the one-site form on 21 lattices, by the share of a block's threads with a
// site (D_W on 1, 2, 3, 12 fields):
//   share      FP64                                     48 bits
//   0.56-0.72  1.11-1.34 1.01-1.25 0.91-1.21 0.91-1.11  0.78-1.08 0.76-0.90 0.70-0.85 0.69-0.78
//   0.77       1.22 1.15 1.05 1.10                      1.02 0.89 0.82 0.87
//   0.88       1.35 1.27 1.17 1.11                      1.27 1.06 0.97 0.91
//   0.94       1.35 1.13 1.02 1.05                      1.22 0.97 0.87 0.89
//   1          1.15-1.29 1.40-1.49 1.36 1.15-1.21       1.03-1.58 1.18-1.22 1.13-1.18 1.01-1.07
// FP64 at 0.77 and more loses nowhere on three fields or more; below it two
// fields gain up to half a million sites (48x22^3 1.01, 28x26x30^2 0.98).  48-bit
// rows of 8 sites lose on many fields (64x16x16x8, share 1: three 1.06, twelve
// 0.93).  Launches that leave partial sums, and the Lanczos passes (one form for
// both passes, which must round alike), judged by whole solves:
//   overlap apply, FP64, one field: 1.05-1.22 where the tiles carry the scalar
//   stages (carry: their sums are few enough), 0.96-1.00 below 0.88 where they do
//   not, 1.03-1.06 from 0.88 on, 1.06-1.28 at 1; three fields: 0.84-0.99 below 1,
//   1.04-1.10 at 1.  Mixed (48-bit iterations): 0.99-1.03, 0.93-0.97, 1.02-1.04,
//   1.01-1.08; three fields 0.85-0.97, 0.99-1.02 at 1.  Lanczos on three fields:
//   0.91-0.99 below 1, 1.02-1.07 at 1.
inline bool tile_pays(const Tile &t, bool f64, int nrhs, bool sums, bool carry)
{
    const int sites = tile_sites(t);
    const bool full = sites == t.nt, dense = 8 * sites >= 7 * t.nt;
    if (!t.nt) return false;
    if (sums) return full || (nrhs == 1 && (dense || carry));
    if (!f64) return (full && (nrhs <= 3 || t.T[3] >= 16)) || (dense && nrhs == 1);
    if (nrhs == 1 || 4 * sites >= 3 * t.nt) return true;
    return nrhs == 2 && (int64_t)sites * tile_count(t) <= 1 << 19;
}

}  // namespace ovl
