// Causal trailing-window smoothing and band combination.
//   Eq. 3:  z(t) = (x(t) - mu(t)) / (sigma(t) + eps)     (EPIKV_SMOOTH_Z)
//   Eq. 2:  mu(t)                                          (EPIKV_SMOOTH_MEAN)
// with mu and the population sigma over the last min(w, available) samples
// up to and including t; then s(t) = mean_A - mean_B over the signal rows
// (Fig. 1; the Lag-KV signal is a single row of weight +1).  s(t) is the
// token's frozen score (Sec. 3.3).
//
// One 1024-thread workgroup scores a tile of kZscoreTile (64) tokens of one
// sequence; each of its 16 wavefronts smooths one signal row at a time (lane
// = token), so the band layers are processed in parallel.  A wavefront
// stages its row's tile plus the w-1 samples before it in its own LDS slice
// (taken from the carried ring for the chunk's first tokens) and each lane
// computes its window's mean and variance in two passes over at most w
// values (fp32; the two-pass form avoids the E[x^2] - mu^2 cancellation when
// the signal's mean is large against its spread).  The per-row values meet
// in LDS for the band combination.
#pragma once

#include "epikv_internal.h"

namespace epikv {
namespace zscore_impl {

constexpr int kWaves = kZscoreThreads / 64;
constexpr int kSlice = EPIKV_MAX_WINDOW - 1 + kZscoreTile;

// Tile `tile` of the n_tiles of sequence b.  sig(l, c): row l's signal of
// token c.  put(b, c, N, s) receives each token's score, when the sequence's
// row has room for the chunk.
template <typename Sig, typename Put>
__device__ __forceinline__ void zscore_tile(const ZscoreArgs& a, int tile, int n_tiles, int b,
                                            Sig sig, Put put) {
  __shared__ float xs[kWaves][kSlice];
  __shared__ float vals[EPIKV_MAX_BAND][kZscoreTile];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm1 = a.w - 1;
  const int c = tile * kZscoreTile + lane;
  // (both counts are read here, so that neither waits on its own)
  const int N = a.n_cached[b];
  const int n_tok = max(a.n_tok_in[b], 0);
  // The first token of a fresh hidden-state stream has no predecessor and
  // hence no sample.
  const int c0 = (a.hs && n_tok == 0) ? 1 : 0;
  const int64_t prior = a.hs ? (int64_t)max(n_tok - 1, 0) : (int64_t)n_tok;
  const int cnt = (int)min((int64_t)wm1, prior);
  // Extended index space: X[j] = ring slot j for j < w-1, X[w-1+c] = signal
  // of token c.  Valid samples are X[vstart ..].
  const int vstart = wm1 - cnt + c0;
  const bool last_tile = (tile == n_tiles - 1);
  const int base = tile * kZscoreTile;  // X index held in xs[wave][0]
  const int span = wm1 + kZscoreTile;
  const int64_t total_out = prior + (a.C - c0);
  const int cnt_out = (int)min((int64_t)wm1, total_out);
  float* x = xs[wave];

  // Every wavefront runs the same number of rounds so the barriers match.
  const int rounds = (a.n_sig + kWaves - 1) / kWaves;
  for (int rd = 0; rd < rounds; ++rd) {
    const int l = rd * kWaves + wave;
    const bool active = l < a.n_sig;
    if (active) {
      const float* ring = a.ring_in + ((int64_t)b * a.n_sig + l) * wm1;
      for (int k = lane; k < span; k += 64) {
        const int j = base + k;
        float v = 0.f;
        if (j < wm1)
          v = ring[j];
        else if (j - wm1 < a.C)
          v = sig(l, j - wm1);
        x[k] = v;
      }
    }
    __syncthreads();
    if (active) {
      float v = 0.f;
      if (c < a.C && c >= c0) {
        const int j = wm1 + c;
        v = smooth_at(x, base, max(vstart, j - wm1), j, a.mode, a.eps);
      }
      vals[l][lane] = v;
      if (a.smoothed && c < a.C) a.smoothed[((int64_t)l * a.B + b) * a.C + c] = v;
      if (last_tile) {
        // Carry the last min(w-1, samples) samples, right-aligned: slot k
        // holds X[C + k].
        float* ro = a.ring_out + ((int64_t)b * a.n_sig + l) * wm1;
        for (int k = lane; k < wm1; k += 64) {
          const bool valid = (wm1 - 1 - k) < cnt_out;
          ro[k] = valid ? x[a.C + k - base] : 0.f;
        }
      }
    }
    __syncthreads();
  }

  if (tid < kZscoreTile && c < a.C) {
    const float s = band_combine<kZscoreTile>(vals, tid, a.n_a, a.n_sig, a.n_b);
    if (N >= a.C && (int64_t)N <= a.ld_s) put(b, c, N, s);
  }
  if (last_tile && tid == 0) a.n_tok_out[b] = n_tok + a.C;
  if (last_tile && tid < a.n_sig)
    a.ema_out[(int64_t)b * a.n_sig + tid] = a.ema_in[(int64_t)b * a.n_sig + tid];
}

// EMA smoothing (App. E): y(t) = alpha*y(t-1) + (1-alpha)*x(t), y = x at the
// stream's first sample.  For each signal row a wavefront turns a 64-token
// tile into per-token affine maps y -> A*y + Bc (a token without a sample is
// the identity) and composes them with a lane-wise inclusive scan, so the
// tile's averages follow exactly from the average carried in from the
// previous tile.  The per-row values meet in LDS for the band combination.
//
// A workgroup has `per` consecutive tiles.  The average carried into the
// first of them comes from the workgroup itself, from all the samples before
// them: a tile's composed map at its last token does not need the carry, and
// only that token's is needed, so it is a tree of 63 multiply-adds (the
// scan's own at lane 63, in its order: the carry has the same bits as when
// the tiles were scanned one after the other) over the samples four to a
// lane, and the tiles' maps are applied to the carry in order.  Reading the
// samples again costs a last workgroup about 0.04 us per tile before it;
// one workgroup walking all tiles cost 1.7 us per tile, a chain of load,
// scan and barriers (15 rows; 2 x 6001 tokens 149 -> 11.5 us, 65,536 tokens
// 1704 -> 74 us, 64 x 1000 tokens 28 -> 11 us).
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

template <int CTRL>
__device__ __forceinline__ float dpp_from(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

// The carry after tiles [1, first) of row x, from the one after tile 0.
__device__ __forceinline__ float ema_carry(const float* x, int first, float al, float bl,
                                           float carry, int lane) {
  const float a1 = al * al, a2 = a1 * a1, a3 = a2 * a2, a4 = a3 * a3, a5 = a4 * a4, a6 = a5 * a5;
  constexpr int U = 4;  // loads in flight, four tiles each
  for (int q = 1; q < first; q += 4 * U) {
    f32x4u v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = q + 4 * u + (lane >> 4);  // this lane's tile
      const int tc = t < first ? t : 0;       // (tile 0 in place of one past the range)
      v[u] = *reinterpret_cast<const f32x4u*>(x + (int64_t)tc * kZscoreTile + 4 * (lane & 15));
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float b01 = fmaf(al, bl * v[u][0], bl * v[u][1]);
      const float b23 = fmaf(al, bl * v[u][2], bl * v[u][3]);
      float m = fmaf(a1, b01, b23);
      m = fmaf(a2, dpp_from<0x111>(m), m);  // row_shr:1, 2, 4, 8: lane 15 of
      m = fmaf(a3, dpp_from<0x112>(m), m);  // each row of 16 ends with its
      m = fmaf(a4, dpp_from<0x114>(m), m);  // tile's composed map
      m = fmaf(a5, dpp_from<0x118>(m), m);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float bk =
            __int_as_float(__builtin_amdgcn_readlane(__float_as_int(m), 16 * k + 15));
        if (q + 4 * u + k < first) carry = fmaf(a6, carry, bk);
      }
    }
  }
  return carry;
}

// Workgroup `blk` of sequence b, its tiles [blk * per, (blk + 1) * per).
template <typename Put>
__device__ __forceinline__ void ema_tiles(const ZscoreArgs& a, int blk, int per, int b, Put put) {
  __shared__ float vals[EPIKV_MAX_BAND][kZscoreTile];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm1 = a.w - 1;
  const int N = a.n_cached[b];
  const int n_tok = max(a.n_tok_in[b], 0);
  const int c0 = (a.hs && n_tok == 0) ? 1 : 0;
  const int64_t prior = a.hs ? (int64_t)max(n_tok - 1, 0) : (int64_t)n_tok;
  const float al = a.alpha, bl = 1.0f - a.alpha;
  const bool write_scores = N >= a.C && (int64_t)N <= a.ld_s;
  const int tiles = (a.C + kZscoreTile - 1) / kZscoreTile;
  const int first = blk * per;
  const int last = min(tiles, first + per);
  // One row's tile: each token's average given the one carried in.
  auto scan_tile = [&](const float* x, int tile, float cin, bool* has) -> float {
    const int c = tile * kZscoreTile + lane;
    *has = c < a.C && c >= c0;
    // (the stream's first sample starts the average)
    return ema_scan(*has ? x[c] : 0.f, *has, prior == 0 && c == c0, al, bl, cin, lane);
  };
  // The average carried into this workgroup's first tile; each row's stays
  // with its wavefront, in a register (through LDS and a barrier it cost 0.4 us
  // a workgroup: 4000 sequences of one tile 50.2 us, so 44.5).
  constexpr int kRows = (EPIKV_MAX_BAND + kWaves - 1) / kWaves;  // of a wavefront
  float carry[kRows];
#pragma unroll
  for (int rd = 0; rd < kRows; ++rd) {
    const int l = rd * kWaves + wave;
    if (l >= a.n_sig) break;
    const float* x = a.sig + ((int64_t)l * a.B + b) * a.C;
    float y = a.ema_in[(int64_t)b * a.n_sig + l];
    if (first > 0) {
      bool has;
      y = __shfl(scan_tile(x, 0, y, &has), 63, 64);
      y = ema_carry(x, first, al, bl, y, lane);
    }
    carry[rd] = y;
  }
  for (int tile = first; tile < last; ++tile) {
    const int c = tile * kZscoreTile + lane;
#pragma unroll
    for (int rd = 0; rd < kRows; ++rd) {
      const int l = rd * kWaves + wave;
      if (l >= a.n_sig) break;
      bool has;
      const float y = scan_tile(a.sig + ((int64_t)l * a.B + b) * a.C, tile, carry[rd], &has);
      const float v = has ? y : 0.f;
      vals[l][lane] = v;
      if (a.smoothed && c < a.C) a.smoothed[((int64_t)l * a.B + b) * a.C + c] = v;
      carry[rd] = __shfl(y, 63, 64);
    }
    __syncthreads();
    if (tid < kZscoreTile && c < a.C && write_scores)
      put(b, c, N, band_combine<kZscoreTile>(vals, tid, a.n_a, a.n_sig, a.n_b));
    __syncthreads();
  }
  if (last < tiles) return;
  // carried state: averages, sample ring, token count
#pragma unroll
  for (int rd = 0; rd < kRows; ++rd) {
    const int l = rd * kWaves + wave;
    if (l < a.n_sig && lane == 0) a.ema_out[(int64_t)b * a.n_sig + l] = carry[rd];
  }
  const int64_t total_out = prior + (a.C - c0);
  const int cnt_out = (int)min((int64_t)wm1, total_out);
  for (int i = tid; i < a.n_sig * wm1; i += kZscoreThreads) {
    const int l = i / wm1;
    const int k = i - l * wm1;
    const int j = a.C + k;  // index in [ring | chunk signal]
    float v = 0.f;
    if ((wm1 - 1 - k) < cnt_out)
      v = j < wm1 ? a.ring_in[((int64_t)b * a.n_sig + l) * wm1 + j]
                  : a.sig[((int64_t)l * a.B + b) * a.C + (j - wm1)];
    a.ring_out[((int64_t)b * a.n_sig + l) * wm1 + k] = v;
  }
  if (tid == 0) a.n_tok_out[b] = n_tok + a.C;
}

// The signal [n_sig][B][C] in memory.
__device__ __forceinline__ float read_sig(const ZscoreArgs& a, int b, int l, int c) {
  return a.sig[((int64_t)l * a.B + b) * a.C + c];
}

// The scores' row of the sequence.
__device__ __forceinline__ void put_score(const ZscoreArgs& a, int b, int c, int N, float s) {
  a.scores[(int64_t)b * a.ld_s + (N - a.C) + c] = s;
}

// EMA tiles per workgroup: one until there are kEmaWg workgroups, about one
// per compute unit; from there on more, since a further workgroup reads all
// the samples before it again.
constexpr int kEmaWg = 256;
inline int tiles_of(const ZscoreArgs& a) { return (a.C + kZscoreTile - 1) / kZscoreTile; }
inline int ema_per(const ZscoreArgs& a) {
  return (int)(((int64_t)tiles_of(a) * a.B + kEmaWg - 1) / kEmaWg);
}

}  // namespace zscore_impl
}  // namespace epikv
