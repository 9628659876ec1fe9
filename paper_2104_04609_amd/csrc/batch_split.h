// Work split of the batch pair kernels (host).
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

namespace bem {

constexpr int BT_TILE = 32;   // trial triangles staged in LDS

// The partial rows of a launch, one set per range of trial triangles, stay with the
// mesh.  More than one range takes no more than this.
constexpr int64_t BATCH_PART_MAX = 2ll << 30;
// What all of that has to gain, as a share of the time (in proportion for less).
constexpr double BATCH_PART_WEIGHT = 0.01;

// Time of `nsplit` ranges of `len` trial triangles, in trial triangles: rounds of
// resident workgroups times a range with its prologue and output.
inline double batch_split_cost(int tiles, int slots, int nsplit, int len) {
    return std::ceil((double)tiles * nsplit / slots) * (len + 4.0);
}

// Trial-triangle ranges of a launch over `tiles` workgroups of test triangles:
// whole staged tiles, least time with the weight of the partial rows among the
// counts that BATCH_PART_MAX allows.  range_bytes: partial rows of one range.
// The least time alone took 19 to 68 ranges of large meshes for 1 to 2 % of a
// launch: 2.4 GB at 40 500 triangles and 32 vectors, now 0.1; 43 GB at 297 680, now
// 1.8.  The modelled time is at most 1.6 % above the least (0.7 % below 41 000).
inline void batch_split(int T, int tiles, int slots, int64_t range_bytes, int *nsplit, int *len) {
    const int nt = (T + BT_TILE - 1) / BT_TILE;
    double best = 1e300;
    for (int q = 1; q <= nt; q++) {   // q tiles per range
        const int ns = (nt + q - 1) / q;
        const int64_t bytes = ns * range_bytes;
        if (ns > 1 && bytes > BATCH_PART_MAX) continue;
        const double cost = batch_split_cost(tiles, slots, ns, q * BT_TILE) *
                            (1 + BATCH_PART_WEIGHT * ((double)bytes / BATCH_PART_MAX));
        if (cost < best) {
            best = cost;
            *nsplit = ns;
            *len = q * BT_TILE;
        }
    }
}

}   // namespace bem
