// The selection and the hidden-state scoring of one eviction step in a
// single launch, for chunks no longer than the recency window (C <= R).
// Then every new token lies in the protected window [N-R, N), so which of
// the older positions survive depends only on their frozen scores (Sec. 3.3)
// and not on the chunk being scored: the two are independent and can run
// side by side instead of one after the other.
//
// Workgroups [0, B) are the select kernel's (one sequence each); with ORDER
// the next one ranks the destination pages of an out-of-place rebuild, which
// needs the number of rows kept (known from the counts alone) but not which;
// the rest carry up to 16 score wavefronts each (each wavefront one (sequence, layer,
// segment) unit, barrier-free).  Both run the very code of their own
// kernels (select_impl.h, score_hs_impl.h), so the results are those of the
// separate launches bit for bit.
#include <algorithm>

#include "compact_impl.h"
#include "score_hs_impl.h"
#include "select_impl.h"

namespace epikv {
namespace {

constexpr int kMaxUnits = kSelectThreads / 64;  // score units per workgroup, at most

template <int KPT, int VPW, int U, bool ORDER>
__global__ __launch_bounds__(kSelectThreads) void k_select_score(SelectArgs sel, ScoreHsArgs sc,
                                                                 int units, CompactArgs ca) {
  if ((int)blockIdx.x < sel.B) {
    select_impl::select_seq<KPT>(sel, blockIdx.x);
    return;
  }
  if (ORDER && (int)blockIdx.x == sel.B) {
    compact_impl::order_pages(ca, [&](int b) { return select_impl::expected_keep(sel, b); });
    return;
  }
  const int wave = threadIdx.x >> 6;
  if (wave >= units) return;
  const int64_t unit = (int64_t)(blockIdx.x - sel.B - ORDER) * units + wave;
  if (unit >= score_impl::wave_units(sc)) return;
  score_impl::score_hs_unit<VPW, U>(sc, (int)unit, threadIdx.x & 63);
}

template <int KPT, int VPW, int U>
hipError_t launch(const SelectArgs& sel, const ScoreHsArgs& sc, const CompactArgs* ca,
                  hipStream_t s) {
  const int64_t total = score_impl::wave_units(sc);
  // As few units per workgroup as put all of them on the compute units that
  // the selection leaves free: with 16 each, a batch of 32 x 128 tokens had
  // its 1,920 units on 120 of 256 compute units.  16 -> as few (launch of
  // the selection of ragged 8k-32k caches and 15 layers of 4096): 12
  // sequences 53.7 -> 38.0 us, 32 sequences 112.7 -> 87.6 us; 16 sequences
  // at 4224 cached 62.4 -> 48.2 us, 1 sequence 16.5 -> 12.6 us (now the
  // selection's time).  Two rows in flight per wavefront spill 11 registers
  // (47 and 103 us for the first two).
  const int64_t free_cus = std::max(1, device_cus() - sel.B - (ca ? 1 : 0));
  const int64_t units = std::min<int64_t>(kMaxUnits, (total + free_cus - 1) / free_cus);
  const int64_t blocks = sel.B + (ca ? 1 : 0) + (total + units - 1) / units;
  if (ca)
    hipLaunchKernelGGL((k_select_score<KPT, VPW, U, true>), dim3((unsigned)blocks),
                       dim3(kSelectThreads), 0, s, sel, sc, (int)units, *ca);
  else
    hipLaunchKernelGGL((k_select_score<KPT, VPW, U, false>), dim3((unsigned)blocks),
                       dim3(kSelectThreads), 0, s, sel, sc, (int)units, CompactArgs());
  return hipGetLastError();
}

template <int KPT>
hipError_t launch_vpw(const SelectArgs& sel, const ScoreHsArgs& sc, const CompactArgs* ca,
                      hipStream_t s) {
  // rows in flight chosen to stay within 128 registers (1024-thread blocks)
  const int nvec = sc.D / 8;
  if (nvec <= 64) return launch<KPT, 1, 8>(sel, sc, ca, s);
  if (nvec <= 128) return launch<KPT, 2, 4>(sel, sc, ca, s);
  if (nvec <= 256) return launch<KPT, 4, 2>(sel, sc, ca, s);
  return launch<KPT, 8, 1>(sel, sc, ca, s);
}

}  // namespace

bool select_score_fusable(const SelectArgs& sel, const ScoreHsArgs& sc) {
  return sc.C <= sel.R && sc.D / 8 <= 64 * 8;
}

hipError_t launch_select_score(const SelectArgs& sel, const ScoreHsArgs& score,
                               const CompactArgs* ca, hipStream_t s) {
  ScoreHsArgs sc = score;
  sc.seg_len = score_impl::wave_seg_len(sc);
  const int64_t per = (sel.ld_s + kSelectThreads - 1) / kSelectThreads;
  if (per <= 1) return launch_vpw<1>(sel, sc, ca, s);
  if (per <= 2) return launch_vpw<2>(sel, sc, ca, s);
  if (per <= 4) return launch_vpw<4>(sel, sc, ca, s);
  if (per <= 8) return launch_vpw<8>(sel, sc, ca, s);
  if (per <= 16) return launch_vpw<16>(sel, sc, ca, s);
  if (per <= 32) return launch_vpw<32>(sel, sc, ca, s);
  return launch_vpw<0>(sel, sc, ca, s);
}

}  // namespace epikv
