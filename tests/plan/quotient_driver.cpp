// The few-token kernel's quotients as products, against the division (test infrastructure; no GPU): divisors up to 1024, dividends up to 2^17.
#include "../../paper_2605_25655_amd/csrc/thi_internal.h"

#include <cstdio>

int main()
{
    for (unsigned d = 1; d <= 1024; ++d)
        for (unsigned n = 0; n <= 1u << 17; ++n)
            if (thi::mid_quotient(n, d, thi::mid_divisor(d)) != n / d) return std::printf("%u / %u\n", n, d), 1;
    return 0;
}
