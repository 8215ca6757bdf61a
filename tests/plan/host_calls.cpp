// Counts how often the entry points have a shared row block tried while they plan a call (test infrastructure; no GPU: nothing is launched,
// linked with the stand-in launchers of tests/sanitize/api_stubs.cpp and --wrap).  Input: lines "M H I"; output: one line each, the counts of
// the MLP, of its gate/up projection and of its down projection.
#include "../../include/thi.h"

#include <cstdint>
#include <cstdio>

static int tried = 0;
extern "C" {
bool __real__ZN3thi17rowblock_split_okEiiiii(int, int, int, int, int);
bool __wrap__ZN3thi17rowblock_split_okEiiiii(int N, int K, int epilogue, int num_cus, int split)
{
    ++tried;
    return __real__ZN3thi17rowblock_split_okEiiiii(N, K, epilogue, num_cus, split);
}
}

int main()
{
    void* p = reinterpret_cast<void*>(uintptr_t(0x7f0000000000ull));      // aligned, never used
    const size_t big = size_t(1) << 40;
    int M, H, I;
    while (std::scanf("%d %d %d", &M, &H, &I) == 3) {
        int n[3], rc = 0;
        tried = 0;
        rc |= thi_swiglu_mlp(p, p, p, p, p, M, H, I, p, big, nullptr);
        n[0] = tried;
        rc |= thi_swiglu_gate_up(p, p, p, p, M, H, I, p, big, nullptr);
        n[1] = tried - n[0];
        rc |= thi_linear(p, p, p, M, H, I, p, big, nullptr);
        n[2] = tried - n[0] - n[1];
        if (rc) return 1;
        std::printf("%d %d %d\n", n[0], n[1], n[2]);
    }
    return 0;
}
