// Launch plan of the even-odd Wilson solve's vector kernels (wilson_eo.hip);
// host arithmetic only.
#pragma once

#include <algorithm>

namespace ovl {

// Blocks of a flat launch of bs threads over nc component arrays of Vh even sites
constexpr int eo_flat_blocks(int Vh, int nc, int bs) { return (nc * Vh + bs - 1) / bs; }

struct EoPlan {
    int nh;      // blocks of one thread per even site: the hops, and an element group of the vector kernels
    int parts;   // element groups of the vector kernels (grid y)
    int slots;   // partial sums reserved for a kernel: the most that any of them writes (one a block)
};

// A small lattice's vector kernels deal a site's elements to three blocks
// (12^3x16, 54 blocks otherwise: solve 2.42 -> 2.35 ms).  Below 43 even sites
// their blocks are more than those of the flat FP64 launch (12 component arrays).
inline EoPlan eo_plan(int Vh, int bs)
{
    EoPlan p;
    p.nh = eo_flat_blocks(Vh, 1, bs);
    p.parts = p.nh <= 128 ? 3 : 1;
    p.slots = std::max(eo_flat_blocks(Vh, 12, bs), p.nh * p.parts);
    return p;
}

}  // namespace ovl
