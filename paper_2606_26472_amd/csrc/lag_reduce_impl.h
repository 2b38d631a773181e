// The KV-vector scorer's reduction: per token, the sum over the used planes
// and row segments; per channel, the range over the shares of a chunk.
#pragma once

#include "epikv_internal.h"

namespace epikv {

// q(t) = (the sum of token t's partial sums over the used planes and row
// segments) / (L*H): kLagRedParts threads each add every kLagRedParts-th
// partial in order, then the parts are added in order.
constexpr int kLagRedParts = 4;

namespace lag_reduce_impl {

__device__ __forceinline__ float part_sum(const LagReduceArgs& a, int b, int c, int part) {
  const float* p = a.partial + (int64_t)b * a.n_sums * a.C + c;
  float s = 0.f;
#pragma unroll 16
  for (int pl = part; pl < a.n_sums; pl += kLagRedParts) s += p[(int64_t)pl * a.C];
  return s;
}

// Split rows of a lag-normalised signal: channel i's range over the chunk =
// the min and max of the shares' partial ranges, in a fixed order.
__device__ __forceinline__ void chunk_range(const LagReduceArgs& a, int b, int i) {
  const int64_t half = (int64_t)a.B * a.n_chan;
  const int64_t o = (int64_t)b * a.n_chan + i;
  const int kv = (i / (a.n_chan / (2 * a.L))) & 1;
  float lo = 0.f, hi = 0.f;  // planes of an unused tensor carry no range
  if (kv == 0 ? a.use_k : a.use_v) {
    lo = a.prange[o];
    hi = a.prange[half + o];
#pragma unroll 4
    for (int sp = 1; sp < a.splits; ++sp) {
      lo = nan_min(lo, a.prange[sp * 2 * half + o]);
      hi = nan_max(hi, a.prange[sp * 2 * half + half + o]);
    }
  }
  a.range_out[o] = lo;
  a.range_out[half + o] = hi;
}

}  // namespace lag_reduce_impl
}  // namespace epikv
