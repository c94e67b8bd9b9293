// The chord factor's quotient against the division, from reciprocals as far off as
// the hardware's may be (2^-24 relative, either side).
#include "quotient.h"

#include <cmath>
#include <cstdio>
#include <random>

int main()
{
    std::mt19937_64 rng(5);
    auto u = [&]() { return (double)(rng() >> 11) * 0x1p-53; };
    for (int i = 0; i < 4000000; ++i) {
        const float h = (float)std::exp2(40.0 * u() - 20.0);
        const double h2 = (double)h * (double)h;
        const double b2 = i % 16 == 0 ? 0.0 : h2 * u();
        const double off = (i & 1 ? 1.0 : -1.0) * (i % 3 ? u() : 1.0) * 0x1p-24;
        const double got = rrt::quotient_from(b2, h2, (1.0 / h2) * (1.0 + off));
        if (got == b2 / h2) continue;
        std::fprintf(stderr, "%.17g / %.17g from a reciprocal off by %.3g: %.17g, not %.17g\n", b2,
                     h2, off, got, b2 / h2);
        return 1;
    }
    std::printf("quotient checks passed\n");
    return 0;
}
