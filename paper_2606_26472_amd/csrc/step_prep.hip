// The small stages between a step's scoring and its selection, in a single
// launch (launch by launch each was 2-6 us of latency and a gap): the
// smoothing of the chunk, of a KV-vector signal with the reduction of its
// planes' sums, and the clearing of the split selection's scratch.  None of
// them reads what another writes: a smoothing workgroup of a KV-vector signal
// adds up the tokens of its tile and of the window before it itself (127
// tokens for 64).
//
// Workgroups of 1024 threads: [0, smooth) smoothing tiles; the scratch's
// words; the channels' ranges of split KV rows.
#include "lag_reduce_impl.h"
#include "select_impl.h"
#include "zscore_impl.h"

namespace epikv {
namespace {

constexpr int kPrepThreads = kZscoreThreads;

struct PrepArgs {
  ZscoreArgs zs;
  LagReduceArgs red;
  uint32_t* scratch;
  int64_t clear_words;
  int32_t smooth, per;     // smoothing workgroups; EMA tiles of each
  int32_t clear;           // workgroups clearing the scratch
  int32_t range_seq;       // and of one sequence's ranges
};

enum { kWindow, kWindowKv, kEma };

template <int MODE>
__device__ __forceinline__ void smooth(const PrepArgs& a, int blk) {
  const ZscoreArgs& z = a.zs;
  const int tiles_seq = a.smooth / z.B;
  const int b = blk / tiles_seq;
  const int t = blk - b * tiles_seq;
  auto put = [&](int b, int c, int N, float s) { zscore_impl::put_score(z, b, c, N, s); };
  if (MODE == kEma) {
    zscore_impl::ema_tiles(z, t, a.per, b, put);
  } else if (MODE == kWindow) {
    zscore_impl::zscore_tile(
        z, t, tiles_seq, b, [&](int l, int c) { return zscore_impl::read_sig(z, b, l, c); }, put);
  } else {
    // the signal of tokens [first, first + n) of the chunk
    constexpr int kTok = EPIKV_MAX_WINDOW - 1 + kZscoreTile;
    __shared__ float part[kLagRedParts][kTok];
    const int first = max(0, t * kZscoreTile - (z.w - 1));
    const int n = min(z.C, (t + 1) * kZscoreTile) - first;
    for (int i = threadIdx.x; i < kLagRedParts * n; i += kPrepThreads) {
      const int p = i / n;
      part[p][i - p * n] = lag_reduce_impl::part_sum(a.red, b, first + i - p * n, p);
    }
    __syncthreads();
    zscore_impl::zscore_tile(
        z, t, tiles_seq, b,
        [&](int, int c) {
          float q = part[0][c - first];
#pragma unroll
          for (int k = 1; k < kLagRedParts; ++k) q += part[k][c - first];
          return q * a.red.inv_count;
        },
        put);
  }
}

template <int MODE>
__global__ __launch_bounds__(kPrepThreads) void k_step_prep(PrepArgs a) {
  int x = (int)linear_block();  // (31 bits: 64 tokens, 1024 words or ranges each)
  if (x < a.smooth) {
    smooth<MODE>(a, x);
    return;
  }
  x -= a.smooth;
  if (x < a.clear) {
    const int64_t i = (int64_t)x * kPrepThreads + threadIdx.x;
    if (i < a.clear_words) select_impl::clear_scratch_word(a.scratch, i);
    return;
  }
  x -= a.clear;
  if (MODE == kWindowKv) {
    const int b = a.range_seq > 0 ? x / a.range_seq : a.red.B;
    if (b >= a.red.B) return;
    const int i = (x - b * a.range_seq) * kPrepThreads + threadIdx.x;
    if (i < a.red.n_chan) lag_reduce_impl::chunk_range(a.red, b, i);
  }
}

template <int MODE>
hipError_t launch(const PrepArgs& a, int64_t blocks, hipStream_t s) {
  hipLaunchKernelGGL(k_step_prep<MODE>, linear_grid(blocks, kPrepThreads), dim3(kPrepThreads), 0, s,
                     a);
  return hipGetLastError();
}

}  // namespace

// (the moving average of a long chunk reads the signal from memory)
bool step_prep_reduces(const ZscoreArgs& zs) { return zs.mode != EPIKV_SMOOTH_EMA; }

hipError_t launch_step_prep(const ZscoreArgs& zs, const LagReduceArgs* red, const SelectArgs& sel,
                            void* scratch, hipStream_t s) {
  PrepArgs a = {};
  a.zs = zs;
  a.per = zs.mode == EPIKV_SMOOTH_EMA ? zscore_impl::ema_per(zs) : 1;
  a.smooth = (zscore_impl::tiles_of(zs) + a.per - 1) / a.per * zs.B;
  a.scratch = (uint32_t*)scratch;
  a.clear_words = select_clear_words(sel, scratch);
  a.clear = (int32_t)((a.clear_words + kPrepThreads - 1) / kPrepThreads);
  int64_t blocks = (int64_t)a.smooth + a.clear;
  if (red) {
    a.red = *red;
    if (red->lag && red->splits > 1)
      a.range_seq = (red->n_chan + kPrepThreads - 1) / kPrepThreads;
    blocks += (int64_t)a.range_seq * red->B;
  }
  if (zs.mode == EPIKV_SMOOTH_EMA) return launch<kEma>(a, blocks, s);
  return red ? launch<kWindowKv>(a, blocks, s) : launch<kWindow>(a, blocks, s);
}

}  // namespace epikv
