// gemm_shape.hpp -- key ranges, tile height and XCD placement of a stage-1 GEMM launch (host only).
#pragma once

#include <stdint.h>

#include <initializer_list>

#include "launch.hpp"

namespace lacache {

constexpr int kGemmMaxKB = kGemmKeyTile / 64;  // most 16-row key blocks of each of a workgroup's four waves
constexpr int kGemmMinKB = 5;                  // fewest

struct GemmShape {
    int kb;         // 16-row key blocks per wave: a tile is 64 kb keys
    int n_ktiles, n_qtiles;
    int n_ranges;   // key ranges, each walked by one workgroup per query tile; 0: the size cannot be launched
    int xq;         // XCD placement (query groups), 0: plain round-robin
};

inline GemmShape gemm_shape(int n_rows, int B, int d_pad, int num_cu) {
    const int n_qtiles = (B + kGemmQueryTile - 1) / kGemmQueryTile;
    // XCD placement: the fewest query groups (1, 2, 4 or 8) whose query tiles fit one XCD's L2 beside the key
    // stream, at most 3 MiB per XCD (a count of tiles that does not divide evenly: all in one group up to 4.5 MiB);
    // plain round-robin (0) when the counts allow none
    auto placement = [&](int ranges) {
        for (int x = 1; x <= 8; x *= 2)
            if (n_qtiles % x == 0 && ranges % (8 / x) == 0 &&
                (int64_t)(n_qtiles / x) * kGemmQueryTile * d_pad * 2 <= (int64_t(3) << 20))
                return x;
        return ranges % 8 == 0 && (int64_t)n_qtiles * kGemmQueryTile * d_pad * 2 <= (int64_t(9) << 19) ? 1 : 0;
    };
    // Key ranges and tile height, by the time of the longest workgroup in key blocks.  A CU holds one workgroup (each
    // wave has a SIMD's whole register file), so what counts is rounds of workgroups x tiles of a range x rows of a
    // tile, and:
    // - one workgroup more than the CUs costs a whole round: 2200 queries (18 query tiles) on 1M x 768 keys in 15
    //   ranges took 4.97 ms, 2.69 ms in 14; several rounds are weighed too, they fill the last one better;
    // - without a placement the workgroups of a range sit on several XCDs, each fetching its keys; with few query
    //   tiles that is slower than the contraction.  300 queries (3 tiles) on 200k x 768 keys in 86 ranges (both
    //   faults) took 200 us, 113 us in 80; 600 (5 tiles) on 500k x 768 818 and 427 us;
    // - a range of few tiles wastes much of its last one, which a lower tile avoids (64 rows per block, 8 blocks at
    //   most): 256 queries on 100k x 1024 keys, 782 rows per range, two tiles of 448 rows 60.6 us, of 512 64.3 us; on
    //   50k x 384, one of 448 rows 16.3 us, of 512 20.7 us.  A row of a lower tile takes longer (256 queries on 100k
    //   to 200k x 1024 keys, against 512-row tiles: 7 to 9 % in 448-row ones, 1 to 5 % in 384, 13 % in 320): half a
    //   block per tile for the loop and 7 % for every lower tile come within 5 % of all three;
    // - 448-row tiles, whose kernel keeps registers in scratch, gain nothing for one query tile of the widest rows, where
    //   the launch is bound by memory: 100 queries, 448 / 512 rows, 200k x 2048 keys 183-191 / 169-172 us, 220k x 2048
    //   183-191 / 174-178; but 200k x 1792 152-156 / 162-163, 210k x 1536 134-138 / 149-153.  A launch of one tile per
    //   workgroup is left to the lower one: 100k x 2048 104-106 / 106-110.
    const int scattered = n_qtiles == 1 ? 100 : n_qtiles < 12 ? 160 : n_qtiles < 24 ? 112 : 103;  // percent
    int kb = kGemmMaxKB, n_ktiles = 0, n_ranges = 0, xq = 0;
    int64_t least = INT64_MAX;
    for (int x = kGemmMaxKB; x >= kGemmMinKB; --x) {
        const int tiles = (n_rows + 64 * x - 1) / (64 * x);
        for (int rounds = 1; rounds <= 3; ++rounds) {
            const int fill = rounds * num_cu / n_qtiles, most = fill < 1 ? 1 : fill < tiles ? fill : tiles;
            for (int mask : {0, 1, 3, 7}) {
                const int ranges = most & ~mask;
                if (ranges < 1) continue;
                const int place = placement(ranges), per_range = (tiles + ranges - 1) / ranges;
                const int64_t turns = ((int64_t)ranges * n_qtiles + num_cu - 1) / num_cu;
                const bool wide_pass = x == 7 && n_qtiles == 1 && d_pad > 1792 && turns * per_range > 1;
                const int row = x == kGemmMaxKB ? 100 : wide_pass ? 114 : 107;  // percent
                const int64_t cost = turns * per_range * (2 * x + 1) * row * (place > 0 ? 100 : scattered);
                if (cost < least) kb = x, n_ktiles = tiles, n_ranges = ranges, xq = place, least = cost;
            }
        }
    }
    if (n_ranges > kMaxPartials) n_ranges = kMaxPartials, xq = placement(n_ranges);
    // the key offsets of a range stay below 2^31 bytes (its tiles plus the prefetch overrun)
    const int64_t max_tiles = ((int64_t(1) << 31) - 1) / ((int64_t)64 * kb * d_pad * 2) - 1;
    if (max_tiles < 1) return GemmShape{};
    if ((n_ktiles + n_ranges - 1) / n_ranges > max_tiles) {
        n_ranges = (int)((n_ktiles + max_tiles - 1) / max_tiles);
        xq = placement(n_ranges);
    }
    if (n_ranges > kMaxPartials) return GemmShape{};
    return GemmShape{kb, n_ktiles, n_qtiles, n_ranges, xq};
}

}  // namespace lacache
