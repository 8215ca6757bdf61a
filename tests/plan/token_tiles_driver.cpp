// Prints what csrc/plan.hip chooses above 128 tokens for the few-token kernel with several token tiles (test infrastructure; no GPU).  Input: lines
// "epilogue M N K"; output: one line each, rows per tile (0: not this kernel), tiles, ranges, outputs per tile, token tiles, tokens per tile.
#include "../../paper_2605_25655_amd/csrc/thi_internal.h"

#include <cstdio>

int main()
{
    int e, M, N, K;
    while (std::scanf("%d %d %d %d", &e, &M, &N, &K) == 4) {
        const thi::MidPlan p = thi::plan_mid_tiles(M, N, K, e, 256);
        std::printf("%d %d %d %d %d %d\n", p.BN, p.tiles, p.S, p.per, p.tiles_m, p.per_m);
    }
    return 0;
}
