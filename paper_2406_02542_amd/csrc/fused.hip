// The single-launch decode step of one block per query head (fused_impl.h): which calls it takes, and
// its bf16 form.
#include "fused_impl.h"

namespace loki {

#ifdef LOKI_PHASE_TIMING
extern "C" int loki_debug_read_phase_ts(unsigned long long* host_dst, size_t count) {
  return (int)hipMemcpyFromSymbol(host_dst, HIP_SYMBOL(loki::g_phase_ts), count * sizeof(unsigned long long));
}
#endif

// The static arrays of a block of grouped heads: the query before and after its rotation, the
// selection, the page list.
static size_t fused_static_lds(const Shape& s) {
  const size_t select = (sizeof(ResidentSelectSmem<kFusedThreads>) + 15) / 16 * 16;
  return select + 2 * kD * sizeof(float) + (s.pg.table != nullptr ? kFusedMaxPages * sizeof(int32_t) : 0);
}

static bool fused_two_per_cu(const Shape& s) {
  return 2 * (fused_dynamic_lds(s) + fused_static_lds(s)) <= 160 * 1024;
}

bool fused_eligible(const Shape& s) {
  // several new tokens per sequence: a block would read rows appended by other blocks of the launch
  if (s.rg.queries > 1) return false;
  return s.S <= kFusedMaxS && s.k <= kFusedMaxK;
}

bool fused_pinnable(const Shape& s) {
  return fused_eligible(s) && s.G == 1 && s.S <= 8192 && (s.pg.table == nullptr || s.pg.pages_per_seq <= 32);
}

// One block per query head, or the heads' rows spread over the chip by the split path's two launches?
// A block's time grows with what its head has to read, the split path's hardly as long as the chip is
// not full.  Measured at 8 to 1024 heads, S = 512 to 16384, both types, us (one launch / split):
//   one query head per KV head: 0.36 MB a head (S = 2048, k = 512) 8 heads 13.8 / 15.0; 0.72 MB 32
//     heads 21.5 / 19.2, 64 21.8 / 22.1; 1.4 MB 64 heads 45.5 / 36.0, 96 48.7 / 47.5, 128 50.8 /
//     56.8. Below half the CUs the MB at which the two meet grow with the heads and, up to 8192
//     rows, with S (a long row's selection costs the split path more than its bytes): 56 heads, S =
//     8192, k = 512, d = 16 on pages 20.9 / 31.0, 56 fp32, S = 2500, k = 625 22.5 / 17.4, 48 fp32,
//     S = 4096, k = 1024, d = 64 42.7 / 28.1; 112 heads, S = 8192, k = 1024, d = 32 29.2 / 37.2, 96
//     fp32, S = 8192, k = 512, d = 32 34.5 / 41.5, k = 2048 61.6 / 47.5
//   groups: 0.49 MB 32 heads 16.6 / 16.8; 0.74 MB 64 heads 22.2 / 22.7; 0.98 MB 64 heads 26.9 /
//     24.0, 128 29.5 / 29.5; 1.5 MB 128 heads 49.2 / 48.1, 256 59.1 / 70.6, 512 88.8 / 115.6
// With groups every head's block rotates its query from P_h again: 1024 heads of 0.12 MB 29.4 /
// 25.0, of 0.25 MB 38.8 / 39.3.  Past the length at which two blocks share a CU's LDS
// (fused_two_per_cu) a second round of blocks costs groups of 8 more than the split path and leaves
// groups of 4 level: 1024 heads in groups of 8, S = 13800, k = 1725 156 / 179, S = 14300, k = 893
// 124 / 141, k = 1787, one block per CU, 198 / 184, on pages S = 14000, k = 700 118 / 132, S =
// 13000, k = 1300 177 / 162; 512 heads in groups of 4, S = 13800, k = 1725 91.9 / 114, S = 14800, k
// = 462 53.9 / 67.4, k = 925 88.7 / 88.3; but S = 16384, k = 2048, 256 heads 71.6 / 76.4, 512 139 /
// 132.  A group's appended row needs a launch of its own in front (about 4 us): groups of 4, 0.49
// MB, 512 heads 38.6 / 42.2, 0.98 MB 256 heads 43.8 / 44.2; groups of 8, 0.49 MB 512 heads 35.5 /
// 32.2, 0.98 MB 256 heads 38.6 / 37.3, 512 56.7 / 60.3.
// The G heads of a unit each stream the slab, which the scoring of the split path reads once, and
// pay for it in L2 once the chip is full several times over, the more the wider the rows.  Every
// figure one launch / split as it is now / as the step was in four launches, a rotation of its own,
// selection and attention apart:
//   rows of over 256 bytes (fp32, d > 64; the kernel spills too), more heads than CUs: groups of 4,
//     S = 4096, k = 512, d = 128, 512 heads 206 / 87 / 95, 2048 heads 763 / 315 / 325; groups of 2,
//     d = 96, S = 1740, 2560 heads 512 / 298 / 325
//   groups of 8, rows of over 64 bytes, more than two heads per CU: S = 8192, d = 64, 4096 heads k
//     = 512 391 / 317 / 328, k = 1024 469 / 380 / 407, k = 2048 605 / 488 / 528; 1024 heads k = 512
//     100 / 85 / 87, 512 heads k = 1024 66.6 / 71 / 71; 64-byte rows stay: k = 512 300 / 296 / 306,
//     k = 2048 521 / 487 / 539, d = 16, k = 512 252 / 295 / 295
//   groups of 4, rows of over 192 bytes, more than two heads per CU: S = 4096, k = 512, d = 128,
//     1024 heads 106 / 99 / 101, 2048 heads 202 / 178 / 190; rows of over 64 bytes, more than six:
//     S = 4096, k = 256, d = 64, 2048 heads 117 / 103 / 105
// Many heads of little work pay more for their own rotations: from six per CU on 0.3 MB a head and
// not 0.2 (2048 heads, groups of 4, S = 1000, d = 64, 0.22 MB 64.6 / 56.1 / 62.3; 4032, groups of
// 8, S = 2383, 0.22 MB 146 / 129 / 131).
bool fused_preferred(const Shape& s) {
  if (!fused_eligible(s)) return false;
  const long long heads = (long long)s.B * s.Hq, cus = device_cus();
  const double mb = ((double)s.S * s.d + (double)s.k * (2 * kD - s.d)) * s.elem_bytes * 1e-6;
  if (s.G == 1) {
    const double spare = heads > cus / 8 ? 6.4 * (double)(heads - cus / 8) / (double)cus : 0.0;
    return 2 * heads >= cus || mb <= 0.5 + spare * (s.S < 8192 ? s.S / 8192.0 : 1.0);
  }
  if (heads > cus && s.G > 2 && !fused_two_per_cu(s)) return false;
  const int row_bytes = s.d * s.elem_bytes;
  if (heads > cus && row_bytes > 256) return false;
  if (heads > 2 * cus && (s.G == 8 ? row_bytes > 64 : s.G == 4 && row_bytes > 192)) return false;
  if (heads > 6 * cus && s.G == 4 && row_bytes > 64) return false;
  const double least = heads > 6 * cus ? 0.3 : 0.2;
  if (s.ap.k_new != nullptr) {
    if (s.G == 8) return (heads >= 2 * cus && mb >= 0.9) || (heads >= cus && mb >= 1.2);
    return (heads >= 2 * cus && mb >= least) || (heads >= cus && mb >= 0.9);
  }
  if (heads >= 2 * cus) return mb >= least;
  return mb <= 0.5 || heads >= cus || (2 * heads >= cus && mb <= 1.15) || (4 * heads >= cus && mb <= 0.75);
}

hipError_t launch_fused(const Shape& s, const void* q, const float* P, void* klo, void* khi,
                        void* v, void* out, int32_t* out_idx, hipStream_t st) {
  if (!fused_eligible(s)) return hipErrorInvalidValue;
  return s.dtype == 0 ? launch_fused_f32(s, q, P, klo, khi, v, out, out_idx, st)
                      : launch_fused_t<BF16>(s, q, P, klo, khi, v, out, out_idx, st);
}

}  // namespace loki
