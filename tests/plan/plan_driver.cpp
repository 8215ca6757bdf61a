// Prints what csrc/plan.hip chooses for the GEMM (test infrastructure; no GPU).  Input: lines "epilogue M N K"; output: one line each,
// configuration, tiles, workgroups, tiles cut along K, ranges per cut tile, the few-token kernel's rows per tile, ranges, outputs per tile and
// whether starts are spread over k, and the workgroups that touch the weights ahead.
#include "../../paper_2605_25655_amd/csrc/thi_internal.h"

#include <cstdio>

int main()
{
    static const char* const names[] = {"MID", "FEW64", "FEW128", "FEW256", "ONE", "BIG", "R224", "R192", "R160", "TALL", "DEEP", "SMALL"};
    int e, M, N, K;
    while (std::scanf("%d %d %d %d", &e, &M, &N, &K) == 4) {
        const thi::GemmPlan p = thi::plan_gemm(M, N, K, e, 256);
        std::printf("%s %d %d %d %d %d %d %d %d %d\n", names[p.config], p.tiles, p.grid, p.sk_tiles, p.parts, p.mid.BN, p.mid.S, p.mid.per,
                    (int)p.mid.rotate, p.helpers);
    }
    return 0;
}
