// Sums of a thread's own values as trees.  A chain of n additions rounds n - 1 times, a tree log2(n) times: as often as the same
// sum spread over n lanes, which is what a kernel has to match when it gives a lane more columns.
#pragma once

#include <hip/hip_runtime.h>

namespace maxscore {

template <int N, int FIRST = 0, int ALL>
__device__ __forceinline__ float tree_sum(const float (&x)[ALL])
{
    static_assert((N & (N - 1)) == 0 && FIRST + N <= ALL, "a power of two");
    if constexpr (N == 1) return x[FIRST];
    else return tree_sum<N / 2, FIRST>(x) + tree_sum<N / 2, FIRST + N / 2>(x);
}

// of products; the inner one of a pair is rounded, the outer one fused with the addition
template <int N, int FIRST = 0, int ALL>
__device__ __forceinline__ float tree_dot(const float (&x)[ALL], const float *y)
{
    static_assert((N & (N - 1)) == 0 && FIRST + N <= ALL, "a power of two");
    if constexpr (N == 1) return x[FIRST] * y[FIRST];
    else return tree_dot<N / 2, FIRST>(x, y) + tree_dot<N / 2, FIRST + N / 2>(x, y);
}

}  // namespace maxscore
