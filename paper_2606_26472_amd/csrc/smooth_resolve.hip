// The smoothing of a step's chunk and the resolve stage of its out-of-place
// rebuild in a single launch, for the step whose selection is already on the
// stream (the chunk lies inside the recency window).  The two need each
// other only for the chunk's own scores, which every kept set ends with:
// their slots' copies are written by the smoothing workgroups, the others'
// by the resolve threads.  Both are latency alone: smoothing 5.9-6.7 us and
// resolve 2.7-5.8 us and a gap between two launches, together 6.9 us for one
// sequence and 8.8 us for 32 x 4096 slots.  (With the order stage in the
// launch before: one sequence's step at a budget of 256 34.8 -> 28.6 us, at
// 4096 188.5 -> 180.4 us.)
//
// Workgroups [0, smooth) have smoothing tiles, the rest 1024 slots each.
#include "compact_impl.h"
#include "zscore_impl.h"

namespace epikv {
namespace {

template <bool EMA>
__global__ __launch_bounds__(kZscoreThreads) void k_smooth_resolve(ZscoreArgs a, CompactArgs ca,
                                                                   int per, int smooth,
                                                                   int blocks_seq) {
  // (31 bits: 16 bytes of workspace for each slot, 64 tokens for each tile)
  const int blk = (int)linear_block();
  if (blk >= smooth) {
    const int x = blk - smooth;
    const int b = x / blocks_seq;
    if (b >= a.B) return;
    const int j = (x - b * blocks_seq) * kZscoreThreads + threadIdx.x;
    if (j < ca.n_pg * ca.page_size) compact_impl::resolve_slot(ca, b, j, a.n_cached[b] - a.C);
    return;
  }
  const int tiles_seq = smooth / a.B;
  const int b = blk / tiles_seq;
  const int t = blk - b * tiles_seq;
  // Where token c's score goes besides its own place: it is the (C - c)-th
  // from the end of the kept positions, too.
  auto copy_of = [&](int c) -> float* {
    const int nk = min(ca.n_keep[b], ca.K);
    const int j = nk - (a.C - c);
    if (!ca.dst_scores || nk <= 0 || j < 0 || (int64_t)j >= ca.ld_s) return nullptr;
    const compact_impl::SlotOffsets o =
        compact_impl::slot_offsets(ca, b, j, a.n_cached[b] - a.C + c);
    return o.src >= 0 && o.dst >= 0 ? ca.dst_scores + (int64_t)b * ca.ld_s + j : nullptr;
  };
  // (looked up ahead of the smoothing: behind it, its chain of loads was
  // 1.2 us more)
  const int c0 = t * kZscoreTile + threadIdx.x;
  float* const first = threadIdx.x < kZscoreTile && c0 < a.C && per == 1 ? copy_of(c0) : nullptr;
  auto put = [&](int, int c, int N, float s) {
    zscore_impl::put_score(a, b, c, N, s);
    float* const p = per == 1 ? first : copy_of(c);
    if (p) *p = s;
  };
  if (EMA)
    zscore_impl::ema_tiles(a, t, per, b, put);
  else
    zscore_impl::zscore_tile(
        a, t, tiles_seq, b, [&](int l, int c) { return zscore_impl::read_sig(a, b, l, c); }, put);
}

}  // namespace

hipError_t launch_smooth_resolve(const ZscoreArgs& a, const CompactArgs& ca, hipStream_t s) {
  const bool ema = a.mode == EPIKV_SMOOTH_EMA;
  const int per = ema ? zscore_impl::ema_per(a) : 1;
  const int smooth = (zscore_impl::tiles_of(a) + per - 1) / per * a.B;
  const int blocks_seq = (ca.n_pg * ca.page_size + kZscoreThreads - 1) / kZscoreThreads;
  const dim3 grid = linear_grid(smooth + (int64_t)blocks_seq * a.B, kZscoreThreads);
  if (ema)
    hipLaunchKernelGGL(k_smooth_resolve<true>, grid, dim3(kZscoreThreads), 0, s, a, ca, per, smooth,
                       blocks_seq);
  else
    hipLaunchKernelGGL(k_smooth_resolve<false>, grid, dim3(kZscoreThreads), 0, s, a, ca, per,
                       smooth, blocks_seq);
  return hipGetLastError();
}

}  // namespace epikv
