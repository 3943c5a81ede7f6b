// The delay tables' node count on the CPU: it meets its error bound and never
// exceeds its cap, also where the cap is the count of an argument a last place
// away (the host sizes memory by its own logarithm, the kernels use theirs).
#define __host__
#define __device__
#include "node_count.h"

#include <cmath>
#include <cstdio>

using sgwb::node_count;

int main()
{
    const int32_t big = 1 << 20;
    int jumps = 0;
    for (double h = 0.02; h < 210.0; h += 0.05) {
        const int32_t n = node_count(h, big);
        // ln(4 h^n / n!) <= ln 1e-13, and not with two nodes fewer
        auto ln_err = [&](int32_t k) { return std::log(4.0) + k * std::log(h) - std::lgamma(k + 1.0); };
        if (ln_err(n) > std::log(1e-13) || (n > 3 && ln_err(n - 2) < std::log(1e-13))) {
            std::printf("half %g: %d nodes\n", h, n);
            return 1;
        }
        // the argument at which the count rises, and its neighbours
        double lo = h, hi = h + 0.05;
        if (node_count(hi, big) == n) continue;
        for (int i = 0; i < 60; ++i) {
            const double mid = 0.5 * (lo + hi);
            (node_count(mid, big) == n ? lo : hi) = mid;
        }
        ++jumps;
        const double near[] = {hi, hi * (1 + 1e-7), hi * (1 + 1e-6), hi * (1 + 1e-5)};
        for (double x : near)
            if (node_count(x, n) > n) {
                std::printf("half %.9g: %d nodes, %d at most\n", x, node_count(x, n), n);
                return 1;
            }
    }
    if (jumps < 200 || node_count(NAN, 7) > 7 || node_count(1e30, 7) != 7) return 1;
    std::printf("all checks passed\n");
    return 0;
}
