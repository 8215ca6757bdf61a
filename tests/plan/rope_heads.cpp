// What thi_rmsnorm_qkv_rope returns and how many kernels it launches (test infrastructure; no GPU: nothing is launched, linked with the
// stand-in launchers of tests/sanitize/api_stubs.cpp).  Input: lines "M N K n_rot head_dim"; output: one line each.
#include "../../include/thi.h"

#include <cstdint>
#include <cstdio>

namespace thi { int stub_launch_count(); }

int main()
{
    void* p = reinterpret_cast<void*>(uintptr_t(0x7f0000000000ull));      // aligned, never used
    int M, N, K, n_rot, head_dim;
    while (std::scanf("%d %d %d %d %d", &M, &N, &K, &n_rot, &head_dim) == 5) {
        const int before = thi::stub_launch_count();
        const int rc = thi_rmsnorm_qkv_rope(p, p, 1e-6f, p, (const int*)p, (const float*)p, n_rot, head_dim, p, M, N, K, p, size_t(1) << 40, nullptr);
        std::printf("%d %d\n", rc, thi::stub_launch_count() - before);
    }
    return 0;
}
