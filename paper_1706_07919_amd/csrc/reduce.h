// Wave reductions shared by the float64 operator kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace bem {

// Wave sums of 8 values by recursive halving: lanes l and l ^ 32 trade halves
// of the values (each keeps the half picked by bit 5 of its lane), then
// quarters across 16 and pairs across 8, then the single value left is summed
// across lanes l ^ 4, l ^ 2, l ^ 1.  Afterwards every lane whose bits 3..5
// spell q holds the wave sum of value q (10 shuffles instead of 48).
__device__ inline double wave_reduce8(const double (&v)[8]) {
  const int lane = threadIdx.x & 63;
  const bool b5 = lane & 32, b4 = lane & 16, b3 = lane & 8;
  double h4[4], h2[2];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const double keep = b5 ? v[4 + m] : v[m], give = b5 ? v[m] : v[4 + m];
    h4[m] = keep + __shfl_xor(give, 32, 64);
  }
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    const double keep = b4 ? h4[2 + m] : h4[m], give = b4 ? h4[m] : h4[2 + m];
    h2[m] = keep + __shfl_xor(give, 16, 64);
  }
  double h = (b3 ? h2[1] : h2[0]) + __shfl_xor(b3 ? h2[0] : h2[1], 8, 64);
  h += __shfl_xor(h, 4, 64);
  h += __shfl_xor(h, 2, 64);
  h += __shfl_xor(h, 1, 64);
  return h;
}

}  // namespace bem
