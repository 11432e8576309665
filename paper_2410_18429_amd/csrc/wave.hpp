// Reductions over a 64-lane wavefront.  Device-only inline functions.
#pragma once

#include <hip/hip_runtime.h>

namespace wri {

// Wave sums of the N accumulators, exchanged by halves: the lanes of one half
// take over half of the accumulators, so N sums take about N shuffles instead of
// 6 N.  A lane ends with the sum of accumulator `id`, of `left` > 0 real ones
// (0: padding of an odd count); lanes may share one.
template <int N>
__device__ __forceinline__ double wave_sums(double (&a)[N], int off, int* id, int* left) {
  if constexpr (N == 1) {
    double v = a[0];
    for (; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
  } else {
    constexpr int H = (N + 1) / 2;
    const bool up = (threadIdx.x & off) != 0;
    double b[H];
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const double hi = (i + H < N) ? a[i + H < N ? i + H : 0] : 0.0;
      const double send = up ? a[i] : hi, keep = up ? hi : a[i];
      b[i] = keep + __shfl_xor(send, off, 64);
    }
    if (up) *id += H;
    *left = up ? max(*left - H, 0) : min(*left, H);
    return wave_sums<H>(b, off >> 1, id, left);
  }
}

}  // namespace wri
