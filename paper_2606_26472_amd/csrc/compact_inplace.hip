// Order-preserving rebuild of the cache inside the sequence's own pages: the
// move-minimising form of the App. H rebuild.  Slot j of sequence b receives
// the row of position keep_idx[b][j]; keep_idx is strictly ascending, so
// keep_idx[j] >= j and every row only moves towards the front.  Slots in
// front of the first hole (keep_idx[j] == j) already hold their row and are
// not touched, nor is anything at or past n_keep.
//
// Two kernels:
//   check  one 1024-thread workgroup per sequence verifies that keep_idx is
//          strictly ascending and that every page it reaches exists, writes
//          the byte offsets of each moved row (source and destination, inside
//          a plane) to the workspace together with the first hole, and moves
//          the scores and positions.  A sequence that fails the check is left
//          untouched and flagged RANGE.
//   move   one workgroup per (sequence, plane, column slice) walks the moved
//          slots in ascending order, a tile of rows at a time: it loads the tile's
//          source rows, waits until every load has returned, then stores
//          them.  A store to slot j can only overwrite a row that a slot <= j
//          reads; slots of this tile have read theirs, and slots of later
//          tiles read rows past the end of this tile (their sources are >=
//          their own slots).  So a walk moves its bytes without a second copy, and
//          different slices, planes and sequences touch disjoint bytes.  The
//          walk is pipelined: the next tile's loads are in flight while this
//          tile is stored (they read past every slot written so far).
//
// With page remapping (epikv_compact_remap) the check kernel also rewrites
// the page table so that whole retained pages change places instead of being
// copied; the walk then skips their slots, and the ordering argument above
// still holds for every row that moves (see remap_pages).
#include "epikv_internal.h"

namespace epikv {
namespace {

// Every memory operation issued so far has completed: loaded values are in
// registers and earlier stores are done.  The builtin (rather than inline
// assembly) lets the compiler see that nothing is outstanding afterwards, so
// it adds no waits of its own between the stores that follow; the empty asm
// statements keep the compiler from moving memory accesses across it.
__device__ __forceinline__ void wait_vmem() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0);
  asm volatile("" ::: "memory");
}

// Exclusive rank of this thread's flag among the workgroup's set flags (in
// thread order), and the workgroup total.
__device__ __forceinline__ int flag_rank(bool flag, int* wsum, int* total) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const uint64_t m = __ballot(flag);
  if (lane == 0) wsum[wave] = __popcll(m);
  __syncthreads();
  int pre = 0, tot = 0;
  for (int w = 0; w < kInplaceThreads / 64; ++w) {
    const int x = wsum[w];
    pre += (w < wave) ? x : 0;
    tot += x;
  }
  __syncthreads();
  *total = tot;
  return pre + __popcll(m & ((1ull << lane) - 1ull));
}

// Index of `v` in the strictly ascending keep[0, n), or -1.
__device__ __forceinline__ int find_kept(const int32_t* keep, int n, int64_t v) {
  int lo = 0, hi = n;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (keep[mid] < v) lo = mid + 1; else hi = mid;
  }
  return (lo < n && keep[lo] == v) ? lo : -1;
}

// Whole-page retention.  A destination page m (a full page of the rebuilt
// sequence) whose slots receive, in order, all rows of one source page p > m
// is not copied: the table entry m takes p's page.  The pages of such
// destinations that are not themselves such sources are released and go,
// k-th to k-th in ascending order, to the sources that are not themselves
// destinations, so the row stays a permutation of the sequence's pages.  A
// released page (that of m) then only receives rows at slots of a later
// page than m, after every slot that reads it in the front-to-back walk.
//
// Runs inside the check kernel once keep_idx is known to be valid: rewrites
// the destination half of the offset records of the moved slots, drops the
// records of remapped pages (their rows do not move) and then rewrites the
// table.  Per sequence, in the workspace, indexed by destination page:
//   src[m]  p if m is remapped, else -1
//   npg[m]  the page slot m*page_size.. writes to (remapped: the table value)
//   give[m] the rank, then the page, handed to position src[m] when that
//           position is not a destination itself, else -1
// and by rank: rel[k] the k-th released page.
__device__ void remap_pages(const InplaceArgs& a, int b, const int32_t* keep, const int32_t* pt,
                            int nk, int hole, int64_t* rec) {
  __shared__ int s_sum[kInplaceThreads / 64];
  const int tid = threadIdx.x;
  const int ps = a.page_size;
  const int npd = nk / ps;                // full destination pages
  const int ndp = (nk + ps - 1) / ps;     // destination pages
  const int m0 = hole / ps;               // the leading run's pages stay
  int32_t* src = a.remap_ws + (int64_t)b * 4 * a.n_pg;
  int32_t* npg = src + a.n_pg;
  int32_t* give = npg + a.n_pg;
  int32_t* rel = give + a.n_pg;

  for (int m = m0 + tid; m < ndp; m += kInplaceThreads) {
    int p = -1;
    if (m < npd) {
      const int k0 = keep[m * ps];
      const int k1 = keep[m * ps + ps - 1];
      // keep is strictly ascending, so a span of ps - 1 means consecutive
      if (k0 % ps == 0 && k0 > m * ps && k1 - k0 == ps - 1) p = k0 / ps;
    }
    src[m] = p;
    npg[m] = pt[p >= 0 ? p : m];
    give[m] = -1;
  }
  wait_vmem();
  __syncthreads();

  int n_rel = 0, n_give = 0;
  for (int t0 = m0; t0 < npd; t0 += kInplaceThreads) {
    const int m = t0 + tid;
    const int p = m < npd ? src[m] : -1;
    bool released = false, gives = false;
    if (p >= 0) {
      // m is itself a source if some remapped destination takes page m
      const int j = find_kept(keep, nk, (int64_t)m * ps);
      const bool is_src = j >= 0 && j % ps == 0 && j / ps >= m0 && j / ps < npd && src[j / ps] == m;
      released = !is_src;
      gives = !(p < npd && src[p] >= 0);
    }
    int tot_rel, tot_give;
    const int r_rel = n_rel + flag_rank(released, s_sum, &tot_rel);
    const int r_give = n_give + flag_rank(gives, s_sum, &tot_give);
    if (released) rel[r_rel] = pt[m];
    if (gives) give[m] = r_give;
    n_rel += tot_rel;
    n_give += tot_give;
  }
  // The two counts agree for every strictly ascending keep_idx; should they
  // not, the sequence is rebuilt without remapping rather than with a page
  // nobody handed over.
  if (n_rel != n_give) return;
  wait_vmem();
  __syncthreads();

  for (int m = m0 + tid; m < npd; m += kInplaceThreads) {
    const int r = give[m];
    if (r >= 0) {
      const int page = rel[r];
      give[m] = page;
      const int p = src[m];
      if (p < ndp) npg[p] = page;
    }
  }
  wait_vmem();
  __syncthreads();

  // The records of the rows that still move, packed in ascending slot order
  // from index `hole` on (the walk needs only their order), tile by tile:
  // every record of a tile is read before any is written, and a row's
  // packed index never exceeds its slot.
  int n_mv = 0;
  for (int j0 = hole; j0 < nk; j0 += kInplaceThreads) {
    const int j = j0 + tid;
    bool mv = false;
    int64_t so = -1, dso = -1;
    if (j < nk) {
      const int d = j / ps;
      mv = !(d < npd && src[d] >= 0);
      if (mv) {
        so = rec[2 * j];
        dso = (int64_t)npg[d] * a.s_page + (int64_t)(j - d * ps) * a.row_bytes;
      }
    }
    wait_vmem();
    int tot;
    const int k = hole + n_mv + flag_rank(mv, s_sum, &tot);
    if (mv) {
      rec[2 * k] = so;
      rec[2 * k + 1] = dso;
    }
    n_mv += tot;
  }
  if (tid == 0) a.info[2 * b + 1] = hole + n_mv;
  // every read of the old table is behind this barrier
  wait_vmem();
  __syncthreads();

  int32_t* out = a.pt_out + (int64_t)b * a.ld_pt;
  for (int m = m0 + tid; m < npd; m += kInplaceThreads) {
    const int p = src[m];
    if (p >= 0) {
      out[m] = npg[m];
      const int page = give[m];
      if (page >= 0) out[p] = page;
    }
  }
}

__global__ __launch_bounds__(kInplaceThreads) void k_inplace_check(InplaceArgs a) {
  __shared__ int s_bad[kInplaceThreads / 64];
  __shared__ int s_hole[kInplaceThreads / 64];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int b = blockIdx.x;
  int32_t* info = a.info + 2 * b;
  int nk = a.n_keep[b];
  if (nk <= 0) {  // nothing kept, or a sequence select already refused
    if (tid == 0) info[0] = info[1] = 0;
    return;
  }
  nk = min(nk, a.K);
  const int32_t* keep = a.keep_idx + (int64_t)b * a.K;
  const int32_t* pt = a.pt + (int64_t)b * a.ld_pt;
  int64_t* rec = a.offsets + 2 * (int64_t)b * a.K;
  const bool side = a.scores || a.pos;
  int bad = 0, hole = nk;
  for (int j = tid; j < nk; j += kInplaceThreads) {
    const int idx = keep[j];
    const int prev = j > 0 ? keep[j - 1] : -1;
    int64_t so = -1, dso = -1;
    if (idx > prev && !(side && (int64_t)idx >= a.ld_s)) {
      const int sp = idx / a.page_size;
      const int dp = j / a.page_size;
      if ((int64_t)sp < a.ld_pt) {  // dp <= sp since j <= idx
        const int ps = pt[sp];
        const int pd = pt[dp];
        if (ps >= 0 && ps < a.n_pages && pd >= 0 && pd < a.n_pages) {
          so = (int64_t)ps * a.s_page + (int64_t)(idx - sp * a.page_size) * a.row_bytes;
          dso = (int64_t)pd * a.s_page + (int64_t)(j - dp * a.page_size) * a.row_bytes;
        }
      }
    }
    if (so < 0) bad = 1;
    if (idx != j) hole = min(hole, j);
    rec[2 * j] = so;
    rec[2 * j + 1] = dso;
  }
  // block-wide "any bad" and "first hole"
  bad = __any(bad);
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) hole = min(hole, __shfl_xor(hole, m));
  if (lane == 0) {
    s_bad[wave] = bad;
    s_hole[wave] = hole;
  }
  __syncthreads();
  bad = 0;
  hole = nk;
  for (int w = 0; w < kInplaceThreads / 64; ++w) {
    bad |= s_bad[w];
    hole = min(hole, s_hole[w]);
  }
  if (bad) {
    if (tid == 0) {
      info[0] = info[1] = 0;
      if (a.seq_status) a.seq_status[b] = EPIKV_SEQ_RANGE;
    }
    return;
  }
  if (tid == 0) {
    info[0] = hole;
    info[1] = nk;
  }
  if (a.remap) {
    remap_pages(a, b, keep, pt, nk, hole, rec);
    wait_vmem();
    __syncthreads();
  }
  if (!side) return;
  // Scores and positions follow their rows, in ascending tiles (the same
  // argument as the row move, with the workgroup barrier as the wait).
  float* sc = a.scores ? a.scores + (int64_t)b * a.ld_s : nullptr;
  int32_t* ps = a.pos ? a.pos + (int64_t)b * a.ld_s : nullptr;
  for (int j0 = hole; j0 < nk; j0 += kInplaceThreads) {
    const int j = j0 + tid;
    float v = 0.f;
    int32_t p = 0;
    if (j < nk) {
      const int idx = keep[j];
      if (sc) v = sc[idx];
      if (ps) p = ps[idx];
    }
    wait_vmem();
    __syncthreads();
    if (j < nk) {
      if (sc) sc[j] = v;
      if (ps) ps[j] = p;
    }
  }
}

// The move: one 1024-thread workgroup per walk, a thread per 16-byte column of
// a row of the slice (inplace_slices), tiles of T rows (eight loads per thread:
// 64 rows of 2 KiB), software pipelined: tile k + 1's loads are issued before
// tile k's stores.  This keeps the ordering argument: a tile's stores follow a
// barrier behind which all of its loads have returned, and tile k + 1 reads
// positions at or past its own slots, which lie past every slot that tile k (or
// an earlier one) writes.  One barrier per tile: the records of four tiles are
// in LDS, written two tiles ahead.
//
// Bound by HBM as a walk sees it.  Every load and every store of a full tile
// is issued on every path, so that a wait is exactly for the tile it needs and
// never for the stores in between (only the last tile's stores are conditional,
// and without ALL, where the slice's columns do not divide 1024, those of the
// threads left over).
// Measured, K + 128 -> K and rows of 2 KiB in 64 planes, a wavefront per walk of
// 1 KiB or 256-byte slices -> this, in turn on the same buffers: 16 x 4096 rows
// 3354 -> 3350 us (5.1 TB/s), 1 x 2000 120 -> 106 us, 1 x 300 22.3 -> 18.2 us,
// 3 x 700 115.5 -> 111.6 us; rows of 256 bytes (16 x 4096) 441 -> 434 us; of
// 1536, 768 and 1280 bytes (1 x 2000, 2 x 1000, 4 x 600 rows) 111 -> 82, 57 ->
// 37 and 95 -> 81 us.  Large batches stay at 5.1 TB/s with either: a plain copy
// with its destination 256 KiB ahead of its source in the same buffer runs at
// 4.7 to 5.9 TB/s with the distance between the two, and here that distance
// grows along the walk.
constexpr int kTileThreads = 1024;
constexpr int kTileLoads = 8;
typedef int64_t i64x2 __attribute__((ext_vector_type(2)));

template <bool ALL>
__global__ __launch_bounds__(kTileThreads) void k_inplace_tile(InplaceArgs a) {
  extern __shared__ __align__(16) i64x2 recs[];  // [4][T] (src, dst)
  const int tid = threadIdx.x;
  const int rpi = kTileThreads / a.slice_vec;  // rows per load
  const int T = rpi * kTileLoads;              // (at most kTileThreads)
  const int per_seq = a.n_lk * a.n_slices;
  const uint32_t walk = (uint32_t)linear_block();  // (2^27 planes of 4 slices at most)
  const int b = walk / per_seq;
  if (b >= a.B) return;
  const int rem = walk - b * per_seq;
  const int pl = rem / a.n_slices;
  const int sl = rem - pl * a.n_slices;
  const int h = a.info[2 * b];
  const int n = a.info[2 * b + 1] - h;
  if (n <= 0) return;
  int sub = tid / a.slice_vec;
  const int col = sl * a.slice_vec + tid - sub * a.slice_vec;
  const bool act = ALL || sub < rpi;
  if (!act) sub = 0;
  char* base = a.pool + (int64_t)(pl >> 1) * a.s_layer + (int64_t)(pl & 1) * a.s_kv +
               (int64_t)col * 16;
  const i64x2* rec = reinterpret_cast<const i64x2*>(a.offsets) + (int64_t)b * a.K + h;
  // record `tid` of tile k (past the last: the walk's first, never used)
  auto load_rec = [&](int k) -> i64x2 {
    const int64_t j = (int64_t)k * T + tid;
    return rec[tid < T && j < n ? j : 0];
  };
  auto put_rec = [&](int k, i64x2 r) {
    if (tid < T) recs[(k & 3) * T + tid] = r;
  };
  auto load_tile = [&](int k, u32x4 (&v)[kTileLoads]) {
#pragma unroll
    for (int i = 0; i < kTileLoads; ++i) {
      const int64_t off = recs[(k & 3) * T + i * rpi + sub].x;
      v[i] = ld_stream(base + (act ? off : 0));  // (left over: the plane's first row)
    }
  };
  // every wavefront's loads of this tile have returned
  auto tile_loaded = [&](u32x4 (&v)[kTileLoads]) {
#pragma unroll
    for (int i = 0; i < kTileLoads; ++i) asm volatile("" : "+v"(v[i]));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the records written are in LDS
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  put_rec(0, load_rec(0));
  put_rec(1, load_rec(1));
  i64x2 next = load_rec(2);
  __syncthreads();
  u32x4 va[kTileLoads], vb[kTileLoads];
  load_tile(0, va);
  // tile k is in `cur`; returns false after the last
  auto step = [&](int k, u32x4 (&cur)[kTileLoads], u32x4 (&nxt)[kTileLoads]) -> bool {
    const int64_t left = n - (int64_t)k * T;
    if (left <= T) {
      tile_loaded(cur);
#pragma unroll
      for (int i = 0; i < kTileLoads; ++i) {
        const int row = i * rpi + sub;
        if (act && row < left) st_stream(base + recs[(k & 3) * T + row].y, cur[i]);
      }
      return false;
    }
    load_tile(k + 1, nxt);
    put_rec(k + 2, next);  // (over tile k - 2's, last read before two barriers)
    next = load_rec(k + 3);
    tile_loaded(cur);
#pragma unroll
    for (int i = 0; i < kTileLoads; ++i)
      if (act) st_stream(base + recs[(k & 3) * T + i * rpi + sub].y, cur[i]);
    return true;
  };
  for (int k = 0;; k += 2) {
    if (!step(k, va, vb)) break;
    if (!step(k + 1, vb, va)) break;
  }
}

}  // namespace

hipError_t launch_compact_inplace(const InplaceArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_inplace_check, dim3(a.B), dim3(kInplaceThreads), 0, s, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 grid = linear_grid((int64_t)a.B * a.n_lk * a.n_slices, kTileThreads);
  const size_t lds = 4 * (kTileThreads / a.slice_vec * kTileLoads) * sizeof(i64x2);
  if (kTileThreads % a.slice_vec == 0)
    hipLaunchKernelGGL(k_inplace_tile<true>, grid, dim3(kTileThreads), lds, s, a);
  else
    hipLaunchKernelGGL(k_inplace_tile<false>, grid, dim3(kTileThreads), lds, s, a);
  return hipGetLastError();
}

}  // namespace epikv
