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
//    (d = 1, FP32), so it has two blocks and 140 asset steps a lane or more.  Six
//    problems of that kind in a batch, which has tiles enough (n = 2048, M =
//    2500, N = 30): 1.34 ms in tiles of ten blocks, 1.49 of two; one alone, with
//    N = 4: 0.055 ms of ten, 0.061 of two.
//  - A point's groups are combined one after the other, 0.2 us each, and G of
//    them shorten the launch's end by some 1000 / (n G) of it: the two balance
//    near G = sqrt(M N d / 400) in FP32, so that is the most, and 32, unless
//    it takes more to fill the GPU (d = 1, two iterations: n = 9, M = 1e6, N = 1
//    0.25 ms in 218 groups a point, 0.95 in 1303; n = 64, M = 4e6, N = 20 6.6 ms
//    in 32, 6.0 in 256).
//  - A last group with much fewer blocks than the others idles: of the numbers
//    of groups from two thirds of the 2048 tiles on, the largest that leaves less
//    than 3% of the blocks' room empty (d = 3, n = 1000, M = 4000, N = 10, 16
//    blocks: 0.126 ms in 6 + 6 + 4, 0.121 in 8 + 8).
inline void auto_tiling(int n, int M, int N, int d, int &groups, int &ppl)
{
    const int blocks = (int)((M + (long)kBlock - 1) / kBlock);
    const int fill = (int)((2048L + n - 1) / n);
    const double least = std::max(2.0, 140.0 / ((double)N * d));
    const int chain = std::max(32, (int)std::sqrt((double)M * N * d / 400.0));
    const int most = std::max(fill, std::min({16384 / n, chain, (int)(blocks / least)}));
    double best = 2.0;
    for (int g = std::min(blocks, (2 * fill + 2) / 3); g <= std::min(blocks, most); ++g) {
        const int p = (blocks - 1) / g + 1, used = (blocks - 1) / p + 1;
        const double empty = std::max(0.03, ((double)used * p - blocks) / blocks);
        if (empty > best) continue;
        best = empty;
        groups = used;
        ppl = p;
    }
}

} // namespace bsde
