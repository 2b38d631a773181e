// The smoothing kernels (zscore_impl.h, which describes the method): one
// workgroup per 64-token tile of a sequence, or per few tiles (EMA).
#include "zscore_impl.h"

namespace epikv {
namespace {

__global__ __launch_bounds__(kZscoreThreads) void k_zscore(ZscoreArgs a) {
  const int b = blockIdx.y;
  zscore_impl::zscore_tile(
      a, blockIdx.x, gridDim.x, b, [&](int l, int c) { return zscore_impl::read_sig(a, b, l, c); },
      [&](int b, int c, int N, float s) { zscore_impl::put_score(a, b, c, N, s); });
}

__global__ __launch_bounds__(kZscoreThreads) void k_ema(ZscoreArgs a, int per) {
  zscore_impl::ema_tiles(a, blockIdx.x, per, blockIdx.y, [&](int b, int c, int N, float s) {
    zscore_impl::put_score(a, b, c, N, s);
  });
}

}  // namespace

hipError_t launch_zscore(const ZscoreArgs& a, hipStream_t s) {
  const int tiles = zscore_impl::tiles_of(a);
  if (a.mode == EPIKV_SMOOTH_EMA) {
    const int per = zscore_impl::ema_per(a);
    hipLaunchKernelGGL(k_ema, dim3((tiles + per - 1) / per, a.B), dim3(kZscoreThreads), 0, s, a,
                       per);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_zscore, dim3(tiles, a.B), dim3(kZscoreThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace epikv
