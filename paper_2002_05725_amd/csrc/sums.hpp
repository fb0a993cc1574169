// Pairwise sums of a few values.
#pragma once

#include <hip/hip_runtime.h>

namespace syk {

// v[0] + v[step] + ... + v[(N - 1) step], halved recursively: the rounding error
// grows with log2 N additions, where adding one after another grows with N - 1.
template <int N>
__host__ __device__ __forceinline__ double pairwise_sum(const double* v, int step = 1)
{
    if constexpr (N == 1) return v[0];
    else return pairwise_sum<(N + 1) / 2>(v, step) + pairwise_sum<N / 2>(v + (N + 1) / 2 * step, step);
}

}  // namespace syk
