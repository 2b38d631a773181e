// Per-token scoring in one launch: for chunks of up to 64 new tokens (a
// decoder scoring each token as it is generated, Sec. 3.3) the hidden-state
// change of Eq. 1, the trailing-window smoothing of Eqs. 2-3 (or raw, or
// EMA, App. E) and the band combination of Fig. 1 run in a single
// workgroup per sequence, with the signal kept in LDS.
//
// The arithmetic is the separate kernels' own, in the same order: per band
// row a wavefront accumulates the squared differences of its 16-byte columns
// lane by lane and reduces them with the same butterfly as the score kernel,
// then smooths the row with the same window statistics as the zscore
// kernel, and the rows meet for the same band combination.  So this launch
// gives bit for bit the scores and carried state of epikv_score followed by
// epikv_zscore.
#include "epikv_internal.h"

namespace epikv {
namespace {

constexpr int kWaves = kZscoreThreads / 64;
constexpr int kSlice = EPIKV_MAX_WINDOW - 1 + kZscoreTile;
constexpr int kRing = (EPIKV_MAX_WINDOW - 1 + 63) / 64;  // carried samples per lane

// How a wavefront walks the chunk's rows.
enum { kOneToken, kRowByRow, kPipelined };

// Bound by latency: at one token per call a workgroup reads 15 rows of 8 KiB
// and their predecessors, and every load is issued before the first wait, none
// behind another's value (a fresh stream's predecessor is loaded and dropped,
// as its count comes with the rows).  A wavefront works on its own rows alone
// until the bands meet.  Against a chain of count, carried samples, rows and
// window sums that waited on one another, one token of 1 and 32 sequences (15
// rows of 4096): launch 10.3 -> 6.7 us and 12.0 -> 8.7 us.
// Of more tokens (launch_score_tokens), kRowByRow compares each row with the
// one before it in registers and then loads the next; kPipelined keeps R - 1
// rows in flight, in R buffers that take turns: the waits are exact because
// every load is issued, past the chunk an empty one.
// (The widest pipeline has 12 registers in scratch: values of the smoothing,
// which the loop over the rows does not touch.)
template <int VPW, int WALK>
__global__ __launch_bounds__(kZscoreThreads) void k_score_tokens(ScoreTokArgs a) {
  constexpr int R = WALK != kPipelined ? 2 : VPW >= 4 ? 3 : 4;
  __shared__ float xs[kWaves][kSlice];
  __shared__ float vals[EPIKV_MAX_BAND][kZscoreTile];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.x;
  const int wm1 = a.w - 1;
  const int N = a.n_cached[b];
  const int n_tok = max(a.n_tok_in[b], 0);
  // The first token of a fresh stream has no predecessor and no sample.
  const bool fresh = n_tok == 0;
  const int c0 = fresh ? 1 : 0;
  const int64_t prior = (int64_t)max(n_tok - 1, 0);
  const int cnt = (int)min((int64_t)wm1, prior);
  const int vstart = wm1 - cnt + c0;
  const int64_t total_out = prior + (a.C - c0);
  const int cnt_out = (int)min((int64_t)wm1, total_out);
  const float al = a.alpha, bl = 1.0f - a.alpha;
  float* x = xs[wave];

  for (int l = wave; l < a.n_band; l += kWaves) {
    const int64_t row = (int64_t)b * a.n_band + l;
    const uint16_t* rows = a.hidden[l] + (int64_t)b * a.ld_seq;
    // buffer 0 starts with the row before the chunk, buffer u with row u - 1
    u32x4 buf[R][VPW];
    auto load = [&](const uint16_t* p, bool ok, u32x4 (&v)[VPW]) {
#pragma unroll
      for (int i = 0; i < VPW; ++i) v[i] = ld_row_nt(p, 16 * (lane + 64 * i), ok ? 2 * a.D : 0);
    };
    auto load_row = [&](int c, u32x4 (&v)[VPW]) {
      load(rows + (c < a.C ? (int64_t)c * a.ld_tok : 0), c < a.C, v);
    };
    load(a.h_prev_in + row * a.D, true, buf[0]);
#pragma unroll
    for (int u = 1; u < R; ++u) load_row(u - 1, buf[u]);
    const float* ring_in = a.ring_in + row * wm1;
    float ring[kRing];
#pragma unroll
    for (int k = 0; k < kRing; ++k) ring[k] = ring_in[min(lane + 64 * k, max(wm1 - 1, 0))];
    const float ema_c = a.ema_in[row];
    // Eq. 1 over the chunk's rows
    auto change = [&](int c, const u32x4 (&prev)[VPW], const u32x4 (&cur)[VPW]) {
      float acc = 0.f;
#pragma unroll
      for (int i = 0; i < VPW; ++i) {
        acc = sqdiff8(cur[i], prev[i], acc);
        // (few unpacked values at a time)
        if (WALK == kPipelined) __builtin_amdgcn_sched_barrier(0);
      }
      const float g2 = wave_sum(acc);
      if (lane == 0) x[wm1 + c] = (fresh && c == 0) ? 0.f : sqrtf(g2);
    };
    // the chunk's last row is the next call's predecessor
    auto carry_row = [&](const u32x4 (&v)[VPW]) {
      const __amdgpu_buffer_rsrc_t hout = __builtin_amdgcn_make_buffer_rsrc(
          a.h_prev_out + row * a.D, (short)0, 2 * a.D, kBufferRsrcWord3);
#pragma unroll
      for (int i = 0; i < VPW; ++i)
        __builtin_amdgcn_raw_buffer_store_b128(v[i], hout, 16 * (lane + 64 * i), 0, 0);
    };
    if (WALK == kOneToken) {
      change(0, buf[0], buf[1]);
      carry_row(buf[1]);
    } else if (WALK == kRowByRow) {
#pragma unroll 1
      for (int c = 0; c < a.C; ++c) {
        if (c > 0) {
#pragma unroll
          for (int i = 0; i < VPW; ++i) {
            const int v = lane + 64 * i;
            buf[1][i] = v < a.D / 8 ? ld_stream(rows + (int64_t)c * a.ld_tok + v * 8)
                                    : u32x4{0u, 0u, 0u, 0u};
          }
        }
        change(c, buf[0], buf[1]);
#pragma unroll
        for (int i = 0; i < VPW; ++i) buf[0][i] = buf[1][i];
      }
      carry_row(buf[0]);
    } else {
#pragma unroll 1
      for (int cb = 0; cb < a.C; cb += R) {
#pragma unroll
        for (int u = 0; u < R; ++u) {
          const int c = cb + u;
          if (c < a.C) {
            change(c, buf[u], buf[(u + 1) % R]);
            if (c == a.C - 1) carry_row(buf[(u + 1) % R]);
          }
          // (the row is unpacked again as the next one's predecessor: its
          // 8 * VPW values kept instead would spill)
#pragma unroll
          for (int i = 0; i < VPW; ++i) asm volatile("" : "+v"(buf[(u + 1) % R][i]));
          // (not before the rows are used: there are no registers for it)
          __builtin_amdgcn_sched_barrier(0);
          load_row(c + R - 1, buf[u]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
#pragma unroll
    for (int k = 0; k < kRing; ++k)
      if (lane + 64 * k < wm1) x[lane + 64 * k] = ring[k];
    wave_sync();

    const int c = lane;
    const bool has = c < a.C && c >= c0;
    float v = 0.f;
    float ema = ema_c;
    if (a.mode == EPIKV_SMOOTH_EMA) {
      const float y = ema_scan(has ? x[wm1 + c] : 0.f, has, prior == 0 && c == c0, al, bl, ema_c,
                               lane);
      v = has ? y : 0.f;
      ema = __shfl(y, 63, 64);
    } else if (has) {
      const int j = wm1 + c;
      v = smooth_at(x, 0, max(vstart, j - wm1), j, a.mode, a.eps);
    }
    if (lane == 0) a.ema_out[row] = ema;
    vals[l][lane] = v;
    // carried samples: the last min(w-1, samples), right-aligned
    for (int k = lane; k < wm1; k += 64)
      a.ring_out[row * wm1 + k] = ((wm1 - 1 - k) < cnt_out) ? x[a.C + k] : 0.f;
    wave_sync();  // (x is rewritten)
  }
  __syncthreads();
  if (tid < a.C) {
    const float s = band_combine<kZscoreTile>(vals, tid, a.n_a, a.n_band, a.n_b);
    if (N >= a.C && (int64_t)N <= a.ld_s) a.scores[(int64_t)b * a.ld_s + (N - a.C) + tid] = s;
  }
  if (tid == 0) a.n_tok_out[b] = n_tok + a.C;
}

template <int VPW, int WALK>
hipError_t launch_walk(const ScoreTokArgs& a, hipStream_t s) {
  hipLaunchKernelGGL((k_score_tokens<VPW, WALK>), dim3(a.B), dim3(kZscoreThreads), 0, s, a);
  return hipGetLastError();
}

// Short chunks go row by row: what a pipeline of empty loads costs at its end
// is more than it hides (4 tokens of 16 sequences, rows of 2048: 9.8 us against
// 10.7; 8 tokens 15.2 against 15.4).  So do rows of more than 2048 with many
// sequences: 16 KiB in flight for each of 480 wavefronts on an XCD's compute
// units are more than its L2 holds (16 tokens of 256 sequences 97 us against
// 110, of 64 sequences 48.5 against 49.5; 64 tokens of 64 sequences 170 against
// 162).  Narrower rows gain at any number (16 tokens of 256 sequences, rows of
// 2048 and 1024: 50.2 -> 49.0 us and 26.7 -> 24.2 us against two rows at a time
// with their loads behind one another).
template <int VPW>
hipError_t launch(const ScoreTokArgs& a, hipStream_t s) {
  if (a.C == 1) return launch_walk<VPW, kOneToken>(a, s);
  if (a.C <= 8 || (VPW == 8 && a.B > 64)) return launch_walk<VPW, kRowByRow>(a, s);
  return launch_walk<VPW, kPipelined>(a, s);
}

}  // namespace

hipError_t launch_score_tokens(const ScoreTokArgs& a, hipStream_t s) {
  const int nvec = a.D / 8;
  if (nvec <= 64) return launch<1>(a, s);
  if (nvec <= 128) return launch<2>(a, s);
  if (nvec <= 256) return launch<4>(a, s);
  if (nvec <= 512) return launch<8>(a, s);
  return hipErrorInvalidValue;
}

}  // namespace epikv
