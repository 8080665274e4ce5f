// The whole decode step of Loki (Algorithm 1 lines 3 and 5-9 of arXiv 2406.02542) for one
// (batch, KV head) unit whose G > 1 query heads share ONE selection (one index set per KV head,
// ranked by the maximum of the group's approximate scores), in ONE block, bf16 cache:
//   rotate the G queries; score the low-rank slab on the matrix cores (score_mfma_impl.h) and
//   keep the group maximum of every row in LDS; select the top-k in LDS (select_impl.h); attend
//   over the selected rows for all G heads on the matrix cores (attend_mfma_impl.h).
// No score, index list or partial result leaves the CU and there is no launch boundary, so the
// select stage of one block overlaps the memory stages of the block it shares the CU with.
// The stages use LDS one after the other: the rotation's partial sums, then the scores, then
// the value tiles of the attention stage and finally the merge of the waves share one region.
#include "fused_gqa_impl.h"

namespace loki {

#ifdef LOKI_PHASE_TIMING
extern "C" int loki_debug_read_gqa_ts(unsigned long long* host_dst, size_t count) {
  return (int)hipMemcpyFromSymbol(host_dst, HIP_SYMBOL(loki::g_phase_ts), count * sizeof(unsigned long long));
}
#endif

// ---- host side ---------------------------------------------------------------------------------
bool fused_gqa_eligible(const Shape& s, int select_mode) {
  if (s.dtype != 1 || select_mode != 1) return false;
  if (s.G != 2 && s.G != 4 && s.G != 8) return false;
  if (s.rg.queries > 1) return false;
  const int nch = s.d / 8;
  if (s.d % 8 != 0 || (nch & (nch - 1)) != 0 || nch < 2 || s.d >= kD) return false;
  static_assert(16384 / 256 <= kGqaMaxPages, "the pages of every row fit the list in LDS");
  return s.S <= 16384 && s.k <= kGqaMaxK;
}

// One block per unit: worth it from a quarter of the CUs on (three eighths beyond 8192 rows); below
// that the split path's many blocks per unit win.  From half the CUs on with 2 query heads per KV
// head, three eighths with 4 and five sixteenths with 8 it is so whatever a row costs.  Below that
// line a block's time grows with the bytes of slab and list a row costs its unit, 2 (d + (256 - d)
// k / S), the split path's selection with the rows alone: it is so under 150 bytes at the line (160
// with 8 heads, 250 with 2 beyond 4096 rows, where the split path's selection has 16 keys a
// thread), less in proportion with fewer units, 20 more on a paged cache (the split path's kernels
// look pages up more often), 10 less for lengths that may differ (the longest sequence's block ends
// the step), and never from 140 bytes on.  (266 such shapes, mean time above the better of the two:
// 0.7 %, without the 20 and the 10 1.0 %, with 140 bytes for any number of units 2.9 %.)  Below
// 2048 rows, where every kernel is short, all but the 64-byte slab rows that the split path rotates
// and scores fastest.
// Measured at 64 to 176 units, S = 1024 to 12000, contiguous, paged, appended, ragged, us (one
// launch / split):
//   2 heads: 96 units S = 5125, k = 320, d = 32 23.4 / 28.4, 120 units S = 8192, k = 512 27.9 /
//     33.2, 104 units S = 12000, k = 750, d = 16 31.7 / 50.5, 80 units S = 4096, k = 512, d = 16
//     22.4 / 25.3; 64 units S = 4096, k = 512, d = 32, ragged 23.0 / 19.1, S = 3000, k = 375 21.0 /
//     17.9, 80 units S = 8192, k = 1024, ragged 32.8 / 27.9; 64 units S = 4096, k = 512, d = 64
//     33.1 / 25.8; 64 units, appended, S = 4096, k = 512, d = 32 20.6 / 19.5, S = 6000, k = 750
//     23.0 / 26.0, S = 8192, k = 1024 28.0 / 29.0; 120 units k = 1024 39.4 / 35.3, 64 units S =
//     1024, k = 256, d = 32 18.2 / 15.8, 128 units S = 8192 42.5 / 42.8
//   4 heads: 64 units S = 8192, k = 1024, d = 16 32.2 / 37.9, 80 units S = 4096, k = 256 20.0 /
//     25.3; 64 units S = 4096, k = 512, d = 32 24.7 / 21.8; 72 units S = 4096, k = 1024, d = 64
//     41.1 / 32.8; 96 units S = 4096 26.1 / 25.9
//   8 heads: 80 units S = 8192, k = 512, d = 32 29.5 / 35.1, 64 units S = 4096, k = 256, d = 16
//     21.2 / 28.1, k = 512, d = 64 36.1 / 28.6; 64 units, appended, k = S / 8, d = 32, S = 4096
//     23.3 / 25.4, S = 8192 30.0 / 31.8
bool fused_gqa_preferred(const Shape& s, int select_mode) {
  if (!fused_gqa_eligible(s, select_mode)) return false;
  const long long units = (long long)s.B * s.Hkv, cus = device_cus();
  if (s.S > 8192) return 8 * units >= 3 * cus;
  if (4 * units < cus) return false;
  const long long line = s.G == 2 ? 8 : s.G == 4 ? 6 : 5;  // sixteenths of the CUs
  if (16 * units >= line * cus) return true;
  if (s.S < 2048) return s.G == 8 || s.d != 32;
  const long long bytes = 2 * ((long long)s.S * s.d + (long long)s.k * (2 * kD - s.d));
  long long limit = (s.G == 8 ? 160 : s.G == 2 && s.S > 4096 ? 250 : 150) * 16 * units / (line * cus);
  if (s.pg.table != nullptr) limit += 20;
  if (s.rg.seq_lens != nullptr) limit -= 10;
  return bytes < (limit < 140 ? limit : 140) * s.S;
}

template <int THREADS, int NCH, int G, int KPT, bool PAGED>
static hipError_t launch_fused_gqa_k(const Shape& s, const void* q, const float* P, const void* klo,
                                     const void* khi, const void* v, void* out, int32_t* out_idx,
                                     hipStream_t st) {
  auto kern = fused_gqa_kernel<THREADS, NCH, G, KPT, PAGED>;
  const size_t lds = GqaLds<THREADS, G>::total_bytes(s.S, s.k);
  static std::atomic<unsigned long long> lds_allowed{0};  // per instantiation: devices already set up
  const hipError_t e = allow_dynamic_lds(
      reinterpret_cast<const void*>(kern),
      (int)GqaLds<THREADS, G>::total_bytes(THREADS == 256 ? 8192 : 16384, kGqaMaxK), lds_allowed);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(s.B * s.Hkv), dim3(THREADS), lds, st,
                     static_cast<const uint16_t*>(klo), static_cast<const uint16_t*>(khi),
                     static_cast<const uint16_t*>(v), static_cast<const uint16_t*>(q), P,
                     static_cast<uint16_t*>(out), out_idx, s.Hkv, s.S, s.S_cap, s.k, with_loads(s, kGroupLaunch), s.ap, s.pg,
                     ClusterArgs{});
  return hipGetLastError();
}

template <int NCH, int G>
static hipError_t launch_fused_gqa_g(const Shape& s, const void* q, const float* P, const void* klo,
                                     const void* khi, const void* v, void* out, int32_t* out_idx,
                                     hipStream_t st) {
  // 256 threads when two blocks have to share a CU; 512 when a block has a CU to itself anyway
  // (a unit's time is set by the instructions its waves issue, so twice the waves per unit are
  // faster: 8 query heads, S = 8192, 128 units: 45 -> 39 us)
  const bool alone = s.B * s.Hkv <= device_cus();
  if (s.pg.table != nullptr) {  // (a paged cache: two block shapes)
    if (s.S > 256 * 32 || alone)
      return launch_fused_gqa_k<512, NCH, G, 32, true>(s, q, P, klo, khi, v, out, out_idx, st);
    return launch_fused_gqa_k<256, NCH, G, 32, true>(s, q, P, klo, khi, v, out, out_idx, st);
  }
  if (s.S > 256 * 32 || alone) return launch_fused_gqa_k<512, NCH, G, 32, false>(s, q, P, klo, khi, v, out, out_idx, st);
  if (s.S <= 256 * 16) return launch_fused_gqa_k<256, NCH, G, 16, false>(s, q, P, klo, khi, v, out, out_idx, st);
  return launch_fused_gqa_k<256, NCH, G, 32, false>(s, q, P, klo, khi, v, out, out_idx, st);
}

template <int NCH>
static hipError_t launch_fused_gqa_n(const Shape& s, const void* q, const float* P, const void* klo,
                                     const void* khi, const void* v, void* out, int32_t* out_idx,
                                     hipStream_t st) {
  switch (s.G) {
    case 2: return launch_fused_gqa_g<NCH, 2>(s, q, P, klo, khi, v, out, out_idx, st);
    case 4: return launch_fused_gqa_g<NCH, 4>(s, q, P, klo, khi, v, out, out_idx, st);
    case 8: return launch_fused_gqa_g<NCH, 8>(s, q, P, klo, khi, v, out, out_idx, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_fused_gqa(const Shape& s, const void* q, const float* P, const void* klo,
                            const void* khi, const void* v, void* out, int32_t* out_idx,
                            hipStream_t st) {
  if (!fused_gqa_eligible(s, 1)) return hipErrorInvalidValue;
  switch (s.d / 8) {
    case 2: return launch_fused_gqa_n<2>(s, q, P, klo, khi, v, out, out_idx, st);
    case 4: return launch_fused_gqa_n<4>(s, q, P, klo, khi, v, out, out_idx, st);
    case 8: return launch_fused_gqa_n<8>(s, q, P, klo, khi, v, out, out_idx, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace loki
