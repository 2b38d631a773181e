// Order-preserving rebuild of the paged cache (App. H): for every kept slot
// j of sequence b, copy the K and V rows of position keep_idx[b][j] at every
// layer into slot j of the destination pages.  A token's row at one
// (layer, K|V) holds all KV heads (n_kv_heads * head_dim bf16, 2 KiB for
// 8 x 128), so the copy is a gather of 2 KiB rows: pure HBM streaming.
//
// Three stages, a kernel each (order and resolve: compact_impl.h; the eviction
// step runs them inside its own merged launches where it can):
//   order    one workgroup ranks every (sequence, destination page) by its
//            page id, i.e. by physical address: the used pages first, in
//            ascending page id, then the unused ones.  Writing the rebuilt
//            cache in that order streams the writes through memory the way
//            a plain copy does even when the allocator scattered the
//            destination pages (measured on MI355X: 5.2 -> 6.2 TB/s for
//            randomly placed pages; a cache rebuilt into one run of pages
//            per sequence is already in that order).  When the used ids
//            already rise in logical order the ranks follow from two prefix
//            counts; otherwise the used ids are marked in an LDS bitmap over
//            their range, and a page's rank is the number of marked ids
//            below it.  A range too wide for the bitmap, or a page id used
//            twice, keeps the logical order (sequence, page).
//   resolve  one thread per slot of the budget's pages turns keep_idx and
//            the two page tables into the byte offsets of the source and
//            destination rows inside a plane, a 16-byte record written at
//            position rank(sequence, page) * page_size + slot (slots past
//            n_keep, and rows out of range, get an empty record), and copies
//            the slot's score and position;
//   gather   a 64-thread workgroup copies 64 16-byte columns (1 KiB) in one
//            (layer, K|V) plane: half a 2 KiB row of one record, or several
//            narrow rows' (k_compact_rows, k_compact_vecs), one load and
//            one store per lane, non-temporal (each byte is touched once).
//            Workgroups walk the records in order, so consecutive
//            workgroups write consecutive addresses.  (Measured on the
//            32 x 4096-row rebuild: 1 KiB workgroups 2% faster than four
//            2 KiB rows per 256-thread workgroup.)
#include "compact_impl.h"

namespace epikv {
namespace {

__global__ __launch_bounds__(compact_impl::kOrderThreads) void k_compact_order(CompactArgs a) {
  compact_impl::order_pages(a, [&](int b) { return a.n_keep[b]; });
}

__global__ __launch_bounds__(kCompactThreads) void k_compact_resolve(CompactArgs a) {
  const int j = blockIdx.x * kCompactThreads + threadIdx.x;
  if (j >= a.n_pg * a.page_size) return;
  compact_impl::resolve_slot(a, blockIdx.y, j, INT64_MAX);
}

// Rows of whole KiB (1024, 2048, ... bytes).  Workgroup x (linear_block):
// record x / units, its columns [64 u, 64 u + 64) with u = x % units, in
// plane blockIdx.y.  The record is wave-uniform (a
// scalar load).
__global__ __launch_bounds__(64) void k_compact(CompactArgs a, int64_t total) {
  const int lane = threadIdx.x;
  const int64_t x = linear_block();
  if (x >= total) return;
  const int64_t r = x / a.units;
  const int u = (int)(x - r * a.units);
  const int64_t* rec = a.offsets + 2 * r;
  const int64_t s0 = rec[0];
  const int64_t d0 = rec[1];
  if (s0 < 0) return;
  const int c = u * 64 + lane;
  const int pl = blockIdx.y;
  const char* sb = a.src + (int64_t)(pl >> 1) * a.s_layer + (int64_t)(pl & 1) * a.s_kv + s0;
  char* db = a.dst + (int64_t)(pl >> 1) * a.d_layer + (int64_t)(pl & 1) * a.d_kv + d0;
  st_stream(db + (int64_t)c * 16, ld_stream(sb + (int64_t)c * 16));
}

// Rows of 128, 256 or 512 bytes (one rank's KV heads under tensor
// parallelism): RPW = 8, 4 or 2 consecutive records per workgroup, 64 / RPW
// lanes each, so that a workgroup still moves 1 KiB.  One record per
// workgroup left 48 of 64 lanes idle on 256-byte rows and was bound by the
// rate at which workgroups start (about 4.7 per ns), not by bytes: 32 x
// 4096 rows of 256 bytes in 64 planes 1771 us (2.4 TB/s) with one record,
// 715 us (6.0 TB/s) with four; 512-byte rows 1838 -> 1419 us, 128-byte rows
// 1770 -> 361 us.  The records come in scalar loads; loaded per lane as
// below they cost 3 % (736, 1463, 369 us).
template <int RPW>
__global__ __launch_bounds__(64) void k_compact_rows(CompactArgs a, int64_t total) {
  constexpr int LPR = 64 / RPW;
  const int lane = threadIdx.x;
  const int64_t r0 = linear_block() * RPW;
  const int sub = lane / LPR;
  int64_t s0 = -1, d0 = -1;
#pragma unroll
  for (int i = 0; i < RPW; ++i) {
    if (r0 + i < total) {
      const int64_t* rec = a.offsets + 2 * (r0 + i);
      const int64_t si = rec[0], di = rec[1];
      if (sub == i) {
        s0 = si;
        d0 = di;
      }
    }
  }
  if (s0 < 0) return;
  const int c = lane % LPR;
  const int pl = blockIdx.y;
  const char* sb = a.src + (int64_t)(pl >> 1) * a.s_layer + (int64_t)(pl & 1) * a.s_kv + s0;
  char* db = a.dst + (int64_t)(pl >> 1) * a.d_layer + (int64_t)(pl & 1) * a.d_kv + d0;
  st_stream(db + c * 16, ld_stream(sb + c * 16));
}

// Rows of any other length (3, 5, 6, ... heads): the records' 16-byte
// vectors in one sequence, 64 to a workgroup, each lane finding its record
// by division.  Against one workgroup per started KiB of a row: 384-byte
// rows 450 -> 255 us, 768-byte rows 542 -> 514 us, 1536-byte rows 1156 ->
// 1039 us (8 x 4096 rows, 64 planes; 6.2-6.3 TB/s).
__global__ __launch_bounds__(64) void k_compact_vecs(CompactArgs a, int64_t total) {
  const int row_vec = a.row_bytes >> 4;
  const int64_t v0 = linear_block() * 64;
  const int64_t q = v0 / row_vec;  // (wave-uniform)
  const int t = (int)(v0 - q * row_vec) + (int)threadIdx.x;
  const int64_t r = q + t / row_vec;
  if (r >= total) return;
  const int c = t % row_vec;
  const int64_t s0 = a.offsets[2 * r];
  const int64_t d0 = a.offsets[2 * r + 1];
  if (s0 < 0) return;
  const int pl = blockIdx.y;
  const char* sb = a.src + (int64_t)(pl >> 1) * a.s_layer + (int64_t)(pl & 1) * a.s_kv + s0;
  char* db = a.dst + (int64_t)(pl >> 1) * a.d_layer + (int64_t)(pl & 1) * a.d_kv + d0;
  st_stream(db + c * 16, ld_stream(sb + c * 16));
}

// `n` workgroups in order for each plane.
dim3 gather_grid(int64_t n, int planes) { return linear_grid(n, 64, planes); }

}  // namespace

hipError_t launch_compact_order(const CompactArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_compact_order, dim3(1), dim3(compact_impl::kOrderThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_compact_resolve(const CompactArgs& a, hipStream_t s) {
  const int slots = a.n_pg * a.page_size;
  hipLaunchKernelGGL(k_compact_resolve, dim3((slots + kCompactThreads - 1) / kCompactThreads, a.B),
                     dim3(kCompactThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_compact_gather(const CompactArgs& args, hipStream_t s) {
  CompactArgs a = args;
  a.units = (a.row_bytes >> 4) / 64;  // (rows of whole KiB)
  const int64_t records = (int64_t)a.B * a.n_pg * a.page_size;
  const int row_vec = a.row_bytes >> 4;
  if (row_vec % 64 == 0) {
    const int64_t total = records * a.units;
    hipLaunchKernelGGL(k_compact, gather_grid(total, a.n_lk), dim3(64), 0, s, a, total);
  } else if (row_vec == 32) {
    hipLaunchKernelGGL(k_compact_rows<2>, gather_grid((records + 1) / 2, a.n_lk), dim3(64), 0, s, a,
                       records);
  } else if (row_vec == 16) {
    hipLaunchKernelGGL(k_compact_rows<4>, gather_grid((records + 3) / 4, a.n_lk), dim3(64), 0, s, a,
                       records);
  } else if (row_vec == 8) {
    hipLaunchKernelGGL(k_compact_rows<8>, gather_grid((records + 7) / 8, a.n_lk), dim3(64), 0, s, a,
                       records);
  } else {
    hipLaunchKernelGGL(k_compact_vecs, gather_grid((records * row_vec + 63) / 64, a.n_lk), dim3(64),
                       0, s, a, records);
  }
  return hipGetLastError();
}

hipError_t launch_compact(const CompactArgs& a, hipStream_t s) {
  hipError_t e = launch_compact_order(a, s);
  if (e == hipSuccess) e = launch_compact_resolve(a, s);
  if (e == hipSuccess) e = launch_compact_gather(a, s);
  return e;
}

}  // namespace epikv
