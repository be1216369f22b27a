// Which form of the binning a plan's atoms take (see splat.hip).  Host code
// without HIP.
#pragma once

#include <algorithm>
#include <cmath>

namespace hartree {

// The form by columns of bricks holds an atom's index in 12 bits and a
// problem's hits in LDS.
constexpr int kColAtoms = 4096;

// one problem: its bricks per axis, how many of them an atom of the largest
// width touches on average, its atoms
struct BinShape {
    int nb[3];
    double touch[3];
    int atoms;
};

// Columns win where a count, scan, fill and sort of all bricks is long, or their
// counters contended; visits where the columns are many (one returning atomic
// each on the problem's counter) or long (every brick of a column looks
// through all of the column's atoms).  Microseconds, fitted to 228 bindings of
// 1 to 5,000 atoms on 16^3 to 1024^3, 8 x 8 x 4096 and 2048 x 2048 x 8; columns / visits:
//   256^3, 4,096 atoms, 21 / 31    512^3, 4,096 29 / 40    1024^3, 4,096 72 / 140    64^3, 4,096 71 / 200
//   8 x 8 x 4096, 256 45 / 20, 4,096 553 / 42    1024 x 1024 x 8, 16 14 / 20, 256 32 / 21, 4,096 64 / 26
//   2048 x 2048 x 8, 1 27 / 23, 4,096 189 / 38 (FP64 on 8 x 8 columns: 745 / 85)
inline bool bin_by_columns(int nprob, const BinShape *shape)
{
    double claims = 0.0, walk = 0.0, cols = 0.0, bricks = 0.0, pairs = 0.0, contended = 0.0;
    for (int q = 0; q < nprob; ++q) {
        const BinShape &s = shape[q];
        if (s.atoms > kColAtoms) return false;
        const double nc = double(s.nb[0]) * s.nb[1], ab = s.touch[0] * s.touch[1];
        const double hits = s.atoms * std::min(1.0, ab / nc);      // atoms of one column
        const double entries = hits * s.touch[2];                  // slots of one column
        claims = std::max(claims, std::min(nc, s.atoms * ab));
        walk = std::max(walk, 0.065 * s.nb[2] * std::ceil(hits / 64) + entries / 64 / std::min(4, s.nb[2]));
        cols += nc;
        bricks += nc * s.nb[2];
        pairs += entries * nc;
        contended = std::max(contended, entries / s.nb[2]);
    }
    const double by_columns = 13.5 + 0.009 * claims + 0.0008 * cols + walk;
    const double by_visits =
        std::max(18.5 + 0.00035 * bricks, 14.0 + 0.00064 * bricks) + 0.0001 * pairs + 0.045 * contended;
    return by_columns <= by_visits;
}

}  // namespace hartree
