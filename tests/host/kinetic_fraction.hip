// Largest relative errors of the force model's kinetic fraction 1/2 erfc(-x) in FP64, by ranges of x,
// against the long double erfc: one line "lo hi error" a range.
#include <cmath>
#include <cstdio>

#include "gks_kernels.h"

int main()
{
    const double edge[] = {-6.5, -4.0, -2.0, -1.0, -0.5, 0.0, 1.0, 6.5};
    for (int r = 0; r < 7; r++) {
        const int n = 200000;
        double worst = 0;
        for (int i = 0; i <= n; i++) {
            const double x = edge[r] + (edge[r + 1] - edge[r]) * i / n;
            const long double want = 0.5L * erfcl(-(long double)x);
            worst = std::fmax(worst, (double)(fabsl((long double)gks::kinetic_fraction<double>(x) - want) / want));
        }
        std::printf("%g %g %.3e\n", edge[r], edge[r + 1], worst);
    }
    return 0;
}
