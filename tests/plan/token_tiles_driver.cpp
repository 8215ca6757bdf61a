// Prints what csrc/plan.hip chooses above 128 tokens for the few-token kernel with several token tiles (test infrastructure; no GPU).  Input: lines
// "epilogue M N K"; output: one line each, rows per tile (0: not this kernel), tiles, ranges, outputs per tile, token tiles, tokens per tile.
// With csrc/plan.hip built to report its functions (-finstrument-functions), a last line: how often plan_gemm was entered in all.
#include "../../paper_2605_25655_amd/csrc/thi_internal.h"

#include <cstdio>

static long gemm_plans = 0, entered = 0;
extern "C" {
__attribute__((no_instrument_function)) void __cyg_profile_func_enter(void* fn, void*)
{
    ++entered;
    gemm_plans += fn == reinterpret_cast<void*>(&thi::plan_gemm);
}
__attribute__((no_instrument_function)) void __cyg_profile_func_exit(void*, void*) {}
}

int main()
{
    int e, M, N, K;
    while (std::scanf("%d %d %d %d", &e, &M, &N, &K) == 4) {
        const thi::GemmPlan g = thi::plan_product(M, N, K, e, 256, true);
        const thi::MidPlan p = M > 128 && g.config == thi::GEMM_MID ? g.mid : thi::MidPlan{};
        std::printf("%d %d %d %d %d %d\n", p.BN, p.tiles, p.S, p.per, p.tiles_m, p.per_m);
    }
    if (entered) std::printf("%ld\n", gemm_plans);
    return 0;
}
