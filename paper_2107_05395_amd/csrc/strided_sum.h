// strided_sum.h -- one thread's share of a fixed-order sum over partial sums,
// used by the kernels that fold them (band gradients, loss, statistic).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace bb {
namespace {

// sum of p[g * stride] over g = first, first + step, ... < count: four
// interleaved partial sums, so four loads are in flight, added in a fixed
// order.
__device__ __forceinline__ double strided_sum(const double *__restrict__ p, int64_t stride,
                                              int64_t first, int64_t count, int64_t step)
{
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    int64_t g = first;
    for (; g + 3 * step < count; g += 4 * step) {
        const double a = p[g * stride], b = p[(g + step) * stride];
        const double c = p[(g + 2 * step) * stride], d = p[(g + 3 * step) * stride];
        s[0] += a;
        s[1] += b;
        s[2] += c;
        s[3] += d;
    }
    for (; g < count; g += step) s[0] += p[g * stride];
    return (s[0] + s[1]) + (s[2] + s[3]);
}

}  // namespace
}  // namespace bb
