// Launch shapes of the tiled deep-reuse path: used by the launcher and by the host test that checks that every row number
// the gather reads has been written.
#pragma once

#include <algorithm>
#include <cstdint>

namespace ppc {

constexpr int kGatherThreads = 512;
constexpr int kGatherMaxRows = 2048;                // rows of a workgroup of the gather, at most

struct ReuseGather {
    int rpt = 4;                                    // rows per lane
    int rows = 0;                                   // rows of a workgroup
    int wgs_x = 0, blocks_y = 0;                    // workgroups over the rows, blocks of 64 columns
};

// Rows per lane: the fewest rounds of workgroups, each worth its rows and about four more for the work per segment.
inline ReuseGather reuse_gather_shape(int n, int m) {
    const int groups = kGatherThreads / (std::min(m, 64) / 4);      // row groups of a workgroup
    ReuseGather g;
    g.blocks_y = (m + 63) / 64;
    int64_t best = INT64_MAX;
    for (int rpt : {4, 8, 16}) {
        const int rows = groups * rpt;
        if (rows > kGatherMaxRows) continue;
        const int64_t wgs = (int64_t)((n + rows - 1) / rows) * g.blocks_y, cost = (wgs + 255) / 256 * (rpt + 4);
        if (cost < best) best = cost, g.rpt = rpt, g.rows = rows;
    }
    g.wgs_x = (n + g.rows - 1) / g.rows;
    return g;
}

// Rows that are numbered: all that the gather's last workgroup reads, rows per workgroup need not divide anything (544 for
// 60 columns), in whole 16-byte words of numbers.
inline int reuse_numbered_rows(const ReuseGather& g) { return (g.wgs_x * g.rows + 7) / 8 * 8; }

// Rows of a segment in the tables of signatures and numbers: holds the numbered rows of every n up to n_max.
inline int reuse_row_pitch(int n_max) { return (n_max + kGatherMaxRows - 1 + 7) / 8 * 8; }

}  // namespace ppc
