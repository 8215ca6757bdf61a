// Which GEMM kernel an entry point runs (test infrastructure; no GPU: nothing is launched, linked with the stand-in launchers of
// tests/sanitize/api_stubs.cpp and --wrap for launch_gemm).  Input: lines "family epilogue M N K" (thi_linear, or gate/up); output: one line each,
// configuration, tiles cut along K, workgroups that touch the weights ahead, the few-token kernel's rows per tile and token tiles; "none" where launch_gemm is not called.
#include "../../include/thi.h"
#include "../../paper_2605_25655_amd/csrc/thi_internal.h"

#include <cstdint>
#include <cstdio>

static bool planned;
static thi::GemmPlan plan;

extern "C" hipError_t __wrap__ZN3thi11launch_gemmERKNS_8GemmArgsEiiP12ihipStream_t(const thi::GemmArgs& a, int epilogue, int num_cus, hipStream_t)
{
    plan = thi::plan_product(a.M, a.N, a.K, epilogue, num_cus, a.token_tiles);
    planned = true;
    return hipSuccess;
}

int main()
{
    static const char* const names[] = {"MID", "FEW64", "FEW128", "FEW256", "ONE", "BIG", "R224", "R192", "R160", "TALL", "DEEP", "SMALL"};
    void* p = reinterpret_cast<void*>(uintptr_t(0x7f0000000000ull));      // aligned, never used
    int family, e, M, N, K;
    while (std::scanf("%d %d %d %d %d", &family, &e, &M, &N, &K) == 5) {
        thi_set_kernel_family(family);
        planned = false;
        const int rc = e == thi::EPI_SWIGLU ? thi_swiglu_gate_up(p, p, p, p, M, K, N, p, size_t(1) << 40, nullptr)
                                            : thi_linear(p, p, p, M, N, K, p, size_t(1) << 40, nullptr);
        if (rc != THI_OK || !planned) std::printf("none %d 0 0 0\n", rc);
        else std::printf("%s %d %d %d %d\n", names[plan.config], plan.sk_tiles, plan.helpers, plan.mid.BN, plan.config == thi::GEMM_MID ? plan.mid.tiles_m : 0);
    }
    return 0;
}
