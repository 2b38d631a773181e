// The ordering and resolving stages of the out-of-place rebuild (described in
// compact.hip), shared by its own kernels and the eviction step's merged
// launches.
#pragma once

#include "epikv_internal.h"

namespace epikv {
namespace compact_impl {

constexpr int kOrderThreads = 1024;
constexpr int kOrderWords = 16384;  // bitmap words: page ids spanning up to 512 Ki

// Exclusive prefix sum of one value per thread over the workgroup, in
// thread order; *total gets the sum.  (wsum: kOrderThreads / 64 words.)
__device__ __forceinline__ uint32_t block_exclusive_sum(uint32_t v, uint32_t* wsum, uint32_t* total) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t t = __shfl_up(x, off, 64);
    if (lane >= off) x += t;
  }
  __syncthreads();
  if (lane == 63) wsum[wave] = x;
  __syncthreads();
  uint32_t base = 0, tot = 0;
  for (int w = 0; w < kOrderThreads / 64; ++w) {
    base += w < wave ? wsum[w] : 0u;
    tot += wsum[w];
  }
  *total = tot;
  return base + x - v;
}

// The order stage, on one workgroup of kOrderThreads threads.  n_keep(b):
// rows kept of sequence b, or negative.  Any value of it gives ranks that are
// a permutation, so a wrong one would cost speed only -- but it has to be the
// same each time: it is asked once for the counts and again for the ranks.
template <typename NKeep>
__device__ __forceinline__ void order_pages(const CompactArgs& a, NKeep n_keep) {
  __shared__ uint32_t bits[kOrderWords];
  __shared__ uint32_t pre[kOrderThreads];  // per-thread prefix of the bitmap chunks
  __shared__ uint32_t wsum[kOrderThreads / 64];
  __shared__ int s_lo, s_hi, s_logical, s_unsorted;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int n_pg = a.n_pg;
  const int64_t N = (int64_t)a.B * n_pg;
  int32_t* rank = a.rank;

  // Destination page of entry e = b * n_pg + m, or -1 if the page is not
  // used (past n_keep, a refused sequence) or out of range.
  auto page_of = [&](int64_t e) -> int {
    const int b = (int)(e / n_pg);
    const int m = (int)(e - (int64_t)b * n_pg);
    const int nk = min(n_keep(b), a.K);
    if (nk <= 0 || (int64_t)m * a.page_size >= nk || m >= a.ld_dst_pt) return -1;
    const int pg = a.dst_pt[(int64_t)b * a.ld_dst_pt + m];
    return (pg >= 0 && pg < a.d_npages) ? pg : -1;
  };

  // Each thread takes a contiguous range of entries: its used and unused
  // counts, and whether its used page ids rise strictly.
  const int64_t per = (N + kOrderThreads - 1) / kOrderThreads;
  const int64_t e0 = (int64_t)tid * per;
  const int64_t e1 = min(N, e0 + per);
  uint32_t n_use = 0, n_bad = 0;
  int first = -1, last = -1;
  bool rising = true;
  for (int64_t e = e0; e < e1; ++e) {
    const int pg = page_of(e);
    if (pg < 0) {
      ++n_bad;
    } else {
      if (last >= 0 && pg <= last) rising = false;
      if (first < 0) first = pg;
      last = pg;
      ++n_use;
    }
  }
  if (tid == 0) {
    s_lo = INT32_MAX;
    s_hi = -1;
    s_logical = 0;
    s_unsorted = 0;
  }
  uint32_t n_used, n_unused;
  uint32_t used_before = block_exclusive_sum(n_use, wsum, &n_used);
  uint32_t bad_before = block_exclusive_sum(n_bad, wsum, &n_unused);
  // The used page ids rise strictly over all entries iff every thread's do
  // and each thread's first exceeds the last of the threads before it.
  {
    int mx = last;  // inclusive prefix maximum of the threads' last ids
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int t = __shfl_up(mx, off, 64);
      if (lane >= off) mx = max(mx, t);
    }
    __syncthreads();
    if (lane == 63) wsum[tid >> 6] = (uint32_t)(mx + 1);
    __syncthreads();
    int before = __shfl_up(mx, 1, 64);
    if (lane == 0) before = -1;
    for (int w = 0; w < (tid >> 6); ++w) before = max(before, (int)wsum[w] - 1);
    if (!rising || (first >= 0 && first <= before)) atomicOr(&s_unsorted, 1);
    __syncthreads();
  }

  // Rising: a used page's rank (the number of used ids below it) is the
  // number of used entries before it; the unused entries follow, in
  // logical order.
  if (!s_unsorted) {
    for (int64_t e = e0; e < e1; ++e)
      rank[e] = page_of(e) >= 0 ? (int32_t)used_before++ : (int32_t)(n_used + bad_before++);
    return;
  }

  // Otherwise the ranks come from a bitmap of the used ids over their range.
  // 1. the range of the used page ids
  int lo = INT32_MAX, hi = -1;
  for (int64_t e = tid; e < N; e += kOrderThreads) {
    const int pg = page_of(e);
    if (pg >= 0) {
      lo = min(lo, pg);
      hi = max(hi, pg);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    lo = min(lo, __shfl_xor(lo, off, 64));
    hi = max(hi, __shfl_xor(hi, off, 64));
  }
  if (lane == 0) {
    atomicMin(&s_lo, lo);
    atomicMax(&s_hi, hi);
  }
  __syncthreads();
  lo = s_lo;
  hi = s_hi;
  const int64_t span = hi >= lo ? (int64_t)hi - lo + 1 : 0;
  const int words = (int)((span + 31) / 32);
  bool logical = span == 0 || words > kOrderWords;

  // 2. mark the used page ids (a page used twice keeps the logical order)
  if (!logical) {
    for (int w = tid; w < words; w += kOrderThreads) bits[w] = 0u;
    __syncthreads();
    for (int64_t e = tid; e < N; e += kOrderThreads) {
      const int pg = page_of(e);
      if (pg >= 0) {
        const uint32_t bit = 1u << ((pg - lo) & 31);
        if (atomicOr(&bits[(pg - lo) >> 5], bit) & bit) s_logical = 1;
      }
    }
    __syncthreads();
    logical = s_logical != 0;
  }

  // 3. ranks: a used page's is the number of used ids below it; the
  //    unused entries follow, in logical order
  const int chunk = (words + kOrderThreads - 1) / kOrderThreads;  // bitmap words per thread
  if (!logical) {
    uint32_t c = 0;
    for (int k = 0; k < chunk; ++k) {
      const int w = tid * chunk + k;
      if (w < words) c += __popc(bits[w]);
    }
    uint32_t tot;
    pre[tid] = block_exclusive_sum(c, wsum, &tot);
    __syncthreads();
  }
  for (int64_t e = e0; e < e1; ++e) {
    int32_t r;
    if (logical) {
      r = (int32_t)e;
    } else {
      const int pg = page_of(e);
      if (pg >= 0) {
        const int i = pg - lo;
        const int w = i >> 5;
        const int owner = w / chunk;
        uint32_t below = pre[owner];
        for (int k = owner * chunk; k < w; ++k) below += __popc(bits[k]);
        below += __popc(bits[w] & ((1u << (i & 31)) - 1u));
        r = (int32_t)below;
      } else {
        r = (int32_t)(n_used + bad_before++);
      }
    }
    rank[e] = r;
  }
}

// The resolve stage for slot j of sequence b (j < n_pg * page_size).  The
// scores of positions from `own_scores` on are left to another writer.
struct SlotOffsets {
  int64_t src, dst;  // byte offsets in a plane; negative: out of range
};

__device__ __forceinline__ SlotOffsets slot_offsets(const CompactArgs& a, int b, int j, int idx) {
  SlotOffsets o = {-1, -1};
  const int m = j / a.page_size;
  const int slot_in = j - m * a.page_size;
  if (idx >= 0) {
    const int sp = idx / a.page_size;
    const int slot = idx - sp * a.page_size;
    if ((int64_t)sp < a.ld_src_pt) {
      const int pg = a.src_pt[(int64_t)b * a.ld_src_pt + sp];
      if (pg >= 0 && pg < a.s_npages) o.src = (int64_t)pg * a.s_page + (int64_t)slot * a.row_bytes;
    }
  }
  if ((int64_t)m < a.ld_dst_pt) {
    const int pg = a.dst_pt[(int64_t)b * a.ld_dst_pt + m];
    if (pg >= 0 && pg < a.d_npages) o.dst = (int64_t)pg * a.d_page + (int64_t)slot_in * a.row_bytes;
  }
  return o;
}

__device__ __forceinline__ void resolve_slot(const CompactArgs& a, int b, int j,
                                             int64_t own_scores) {
  const int m = j / a.page_size;
  const int slot_in = j - m * a.page_size;
  // A caller's n_keep above K is clamped so keep_idx is never read past the
  // sequence's row; n_keep < 0: sequence untouched.
  const int nk = min(a.n_keep[b], a.K);
  SlotOffsets o = {-1, -1};
  int idx = -1;
  bool bad = false;
  if (j < nk) {
    idx = a.keep_idx[(int64_t)b * a.K + j];
    o = slot_offsets(a, b, j, idx);
    bad = o.src < 0 || o.dst < 0;
  }
  const bool ok = j < nk && !bad;
  const int64_t pos = (int64_t)a.rank[(int64_t)b * a.n_pg + m] * a.page_size + slot_in;
  int64_t* rec = a.offsets + 2 * pos;
  rec[0] = ok ? o.src : -1;
  rec[1] = ok ? o.dst : -1;
  if (bad) {
    if (a.seq_status) a.seq_status[b] = EPIKV_SEQ_RANGE;
    return;
  }
  if (ok && (int64_t)idx < a.ld_s && (int64_t)j < a.ld_s) {
    const int64_t si = (int64_t)b * a.ld_s + idx;
    const int64_t di = (int64_t)b * a.ld_s + j;
    if (a.dst_scores && idx < own_scores) a.dst_scores[di] = a.src_scores[si];
    if (a.dst_pos) a.dst_pos[di] = a.src_pos[si];
  }
}

}  // namespace compact_impl
}  // namespace epikv
