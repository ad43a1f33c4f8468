// bsde_tiling.h -- the automatic cut of a point's M paths into tiles: groups
// workgroups of ppl blocks of kBlock paths each.
#pragma once

#include <algorithm>
#include <cmath>

namespace bsde {

constexpr int kBlock = 256; // lanes per workgroup of the path kernel

// Enough groups for 2048 tiles, and up to 16 384 of them as long as a tile
// stays long and a point has few.  About 1000 workgroups run at a time, and
// rounds of long tiles end with idle units: d = 1, n = 2048, M = 4000, N = 50 in
// FP32 takes 0.277 ms in one group a point, 0.262 in four.  Against that:
//  - A tile's start and reduction cost as much as some 8 Euler steps of a block
//    (d = 1, FP32; fewer beside more assets), so it has two blocks and 160 /
//    sqrt(d) steps or more.  Six problems of that kind in a batch, which has
//    tiles enough (n = 2048, M = 2500, N = 30): 1.34 ms in tiles of ten blocks,
//    1.49 of two; one alone, with N = 4: 0.055 ms of ten, 0.061 of two.
//  - A point's groups are combined one after the other, 0.2 us each: 32 of them
//    unless it takes more to fill the GPU (n = 9, M = 1e6, N = 1: 0.25 ms for two
//    iterations in 218 groups a point, 0.94 in 1303).
inline void auto_tiling(int n, int M, int N, int d, int &groups, int &ppl)
{
    const int blocks = (int)((M + (long)kBlock - 1) / kBlock);
    const int fill = (int)((2048L + n - 1) / n);
    const double least = std::max(2.0, 160.0 / (N * std::sqrt((double)d)));
    const int most = std::min({16384 / n, 32, (int)(blocks / least)});
    const int want = std::max(1, std::min(blocks, std::max(fill, most)));
    ppl = (blocks - 1) / want + 1;
    groups = (blocks - 1) / ppl + 1;
}

} // namespace bsde
