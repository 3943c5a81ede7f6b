// Chebyshev nodes of the delay tables: one count for the host, which sizes memory
// by it, and for the two kernels that use it.
#pragma once

#include <math.h>
#include <stdint.h>

namespace sgwb {

// Nodes for a function of frequencies within F on an interval of length L, half =
// pi F L / 2: the least N with 4 half^N / N! <= 1e-13, or one more (Stirling's form
// of N!; Newton's iteration from above on a convex function stays above the root),
// and never more than `most`.  float32 will do.  The kernels' counts have to be the
// same, so nothing is contracted; the host's may differ by its logarithm's last
// place, so what it sizes is passed on as `most`.
__host__ __device__ inline int32_t node_count(double half, int32_t most)
{
#ifdef __clang__
#pragma clang fp contract(off)
#endif
    const float h = half > 1e-2 ? (float)half : 1e-2f;
    float n = 5.5f * h + 40.0f;
    for (int i = 0; i < 6; ++i) {
        const float l = logf(n / h), f = n * (l - 1.0f) + 0.5f * logf(6.2831853f * n) - 31.4f;
        n -= f / (l + 0.5f / n);
    }
    const float up = ceilf(n + 0.01f);
    return up < (float)most ? (int32_t)up : most;
}

}  // namespace sgwb
