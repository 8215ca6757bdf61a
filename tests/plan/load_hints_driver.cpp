// Which loads of a k-tile the few-token kernel makes non-temporal (test infrastructure; no GPU).  Input: lines "epilogue M N K"; output: one line each,
// the loads that bring weights (0: not this kernel), token tiles, and for each of the eight waves its bits.
#include "../../paper_2605_25655_amd/csrc/thi_internal.h"

#include <cstdio>

int main()
{
    int e, M, N, K;
    while (std::scanf("%d %d %d %d", &e, &M, &N, &K) == 4) {
        const thi::GemmPlan g = thi::plan_product(M, N, K, e, 256, true);
        const bool few = g.config == thi::GEMM_MID;
        const int loads = few ? (e == thi::EPI_SWIGLU ? 2 : 1) * g.mid.per / 4 : 0;
        std::printf("%d %d", loads, g.mid.tiles_m);
        for (int w = 0; w < thi::MID_WAVES; ++w) std::printf(" %u", few ? thi::mid_streams(w, loads, g.mid.tiles_m) : 0u);
        std::printf("\n");
    }
    return 0;
}
