// The single-launch grouped-query decode step (fused_gqa_impl.h) for launches with fewer
// (batch, KV head) units than the chip has compute units: C = 2, 4 or 8 blocks share a unit,
// each on a slice of its rows, so that the launch covers the chip.  The blocks of a unit find
// the top-k threshold together (cluster_impl.h: Algorithm 1 line 6 of arXiv 2406.02542 over
// rows that live in different blocks) and the last one to finish merges the attention partials
// (lines 7-9).
#include "fused_gqa_impl.h"

namespace loki {

constexpr int kClusterThreads = 512;
constexpr int kClusterKpt = 32;
constexpr int kClusterMaxSlice = kClusterThreads * kClusterKpt;  // rows whose keys fit the block's LDS
constexpr int kClusterMaxList = 8192;                            // selected rows one block may end up with
static_assert(kClusterMax * kClusterMaxSlice / 256 <= kClusterMaxPages, "the pages of every row fit the list in LDS");

#ifdef LOKI_PHASE_TIMING
extern "C" int loki_debug_read_cluster_ts(unsigned long long* host_dst, size_t count) {
  return (int)hipMemcpyFromSymbol(host_dst, HIP_SYMBOL(loki::g_phase_ts), count * sizeof(unsigned long long));
}
#endif

// Clears the control words that must start at zero: every block's arrival flag and the ticket
// of every unit (one word in each kClusterFlagStride words), and the error word behind the
// last unit a launch can have.
__global__ void cluster_reset_kernel(uint32_t* counters, int units) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int n = units * (kClusterMax + 1);
  if (i < n) counters[(size_t)i * kClusterFlagStride] = 0u;
  if (i == n) counters[(size_t)kClusterMaxUnits * kClusterCounterStride] = 0u;
}

static inline int cluster_padded_units(const Shape& s) { return (s.B * s.Hkv + 7) / 8 * 8; }

int fused_gqa_cluster_blocks(const Shape& s, int select_mode) {
  if (s.dtype != 1 || select_mode != 1) return 0;
  if (s.G != 2 && s.G != 4 && s.G != 8) return 0;
  const int nch = s.d / 8;
  if (s.d % 8 != 0 || (nch & (nch - 1)) != 0 || nch < 2 || s.d >= kD) return 0;
  // every block of the launch must be resident at once (the blocks of a unit wait for each
  // other): one block per compute unit at most
  const int padded = cluster_padded_units(s), cus = device_cus();
  if (s.B * s.Hkv > kClusterMaxUnits) return 0;
  int C = 1;
  while (2 * C <= kClusterMax && padded * 2 * C <= cus) C *= 2;
  if (C < 2) return 0;
  const int L = gqa_slice_rows(s.S, C);
  if (L > kClusterMaxSlice || (s.k < L ? s.k : L) > kClusterMaxList) return 0;
  return C;
}

// (A paged cache's page list fits LDS at any length, 2 KB at 131072 rows; with a limit of 64 pages, lists
// of more went to the split path's six launches: us, split / here, 32 groups of 4, S = 131072, k = 8192
// 145.6 / 69.1, 8 of 4, S = 20185, k = 2523 54.5 / 28.4, 64 of 4, S = 20433 of unequal lengths 72.8 / 39.4.)
bool fused_gqa_cluster_eligible(const Shape& s, int select_mode) {
  if (s.rg.queries > 1) return false;
  return fused_gqa_cluster_blocks(s, select_mode) > 0;
}

bool fused_gqa_cluster_preferred(const Shape& s, int select_mode) {
  if (!fused_gqa_cluster_eligible(s, select_mode)) return false;
  // An exchange between a unit's blocks and the wait for the slowest of them cost 5 to 8 us, which
  // many rows, wide slab rows or a long list pay for.  Measured at 8 to 128 units of 2, 4 and 8
  // heads, S = 2500 to 14000, appended, us (cluster / the better of one block per unit and the
  // split path):
  //   up to 64 units (four or eight blocks): S = 9500, d = 16, k = 1187 21.8 / 24.6 to 28.3 / 31.3
  //     (2 heads), 26.8 / 31.2 to 32.6 / 34.3 (8 heads; beyond 8192 rows a thread of the split
  //     path's selection holds 32 keys), S = 11000, d = 32, k = 687 24.7 / 25.3 to 30.3 / 30.4; but
  //     S = 8192, k = 1024 22.7 / 20.8 to 28.5 / 28.0, k = 2048 25.4 / 22.9 (8 units) to 33.8 /
  //     33.8 (64); 64-column rows there 25.0 / 23.4 (8 units), 27.8 / 29.4 (32), 32.7 / 36.0 (64),
  //     S = 6000 29.9 / 34.8
  //   65 to 128 units (two blocks): 64-column rows, S = 6000, k = 750 37.9 / 41.4, S = 8192 43.8 /
  //     47.6; else, where one block per unit applies, S = 8192, k = 2048 46.6 / 44.9, S = 11000
  //     40.1 / 39.1, 45.5 / 43.0, S = 14000 48.4 / 48.2, 53.5 / 53.1 (k = S / 8), 43.1 / 38.9 (k =
  //     S / 16), S = 16384, k = 2048 51.1 / 55.5, 59.1 / 63.2, k = 1024 48.9 / 44.4
  const long long units = (long long)s.B * s.Hkv, cus = device_cus();
  const long long unit_bytes = (long long)s.S * s.d * 2 + (long long)s.k * kD * 4;
  if (4 * units <= cus) {
    if (s.S > 8192 || unit_bytes >= 1800000) return true;
    return s.d >= 64 && s.S > 4096 && 8 * units >= cus && unit_bytes >= (4 * units >= cus ? 1000000 : 1310720);
  }
  if (s.d >= 64) return s.S >= 12288 || (s.S > 4096 && unit_bytes >= 1000000);
  const bool one_block = fused_gqa_preferred(s, select_mode);
  if (s.S >= 12288) return !(one_block && 12LL * s.k < s.S);
  return unit_bytes >= 1310720 && !one_block;
}

// Up to how many candidates of a unit one wave of every block ranks while the others attend over
// the certain rows; more are told apart by another histogram exchange first (4 to 5 us).  1024 fit
// that wave's registers; a list in LDS costs it about 3 us per thousand, which the other waves are
// busy for where the rows of all units' lists, 512 bytes each, take as long: one candidate for every
// 32 KB of them (7 ns at 5 TB/s).  us per step, 1024 / this rule / 8192 / all of them ranked by
// the whole block, with an exchange from 4096 on: 24 units of 8 heads, S = 45686, k = 1427, d = 64
// 47.8 / 47.8 / 59.4 / 49.7; S = 24908, k = 3113 35.8 / 35.8 / 44.9 / 39.1; 32 units of 8, S = 39386,
// k = 4923 48.5 / 48.5 / 62.3 / 54.6; 8 of 4, S = 49409, k = 6176 37.3 / 37.3 / 47.8 / 47.7; but 128
// of 4, S = 16384, k = 2048 58.8 / 56.6 / 56.6 / 62.3; 32 of 4, S = 19531, k = 6510 43.7 / 40.3 / 40.3 /
// 47.6; 64 of 2, S = 64325, k = 8192 89.4 / 85.0 / 85.0 / 95.7.  350 shapes of 4 to 128 units: never
// above the whole block's ranking, 11 % below it on average; 4.6 % below 8192, four shapes 3 to 4.5 % above.
static int cluster_rank_cap(const Shape& s) {
  const long long cap = (long long)s.B * s.Hkv * s.k * (2 * kD * 2) / 32768;
  return (int)(cap < 1024 ? 1024 : cap > kClusterCandCap ? kClusterCandCap : cap);
}

static std::atomic<uint32_t> g_spin_limit{kClusterSpinLimit};
void set_cluster_spin_limit(uint32_t polls) { g_spin_limit.store(polls, std::memory_order_relaxed); }
static std::atomic<bool> g_give_up_at_list{false};
void set_cluster_give_up_at_list(bool on) { g_give_up_at_list.store(on, std::memory_order_relaxed); }

namespace {
struct ClusterPlan {
  size_t xhist, xcand, partial, total;  // byte offsets
};
ClusterPlan cluster_plan(const Shape& s, int C) {
  const size_t units = (size_t)s.B * s.Hkv;
  auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  ClusterPlan p;
  size_t off = 0;
  p.xhist = off;
  off += up(units * kClusterRounds * C * kClusterThreads * kClusterSlotBytes);
  p.xcand = off;
  off += up(units * (size_t)kClusterCandCap * 4);
  p.partial = off;
  off += up(units * s.G * C * (size_t)kPartialStride * 4);
  p.total = off;
  return p;
}
}  // namespace

size_t fused_gqa_cluster_bytes(const Shape& s, int select_mode) {
  const int C = fused_gqa_cluster_blocks(s, select_mode);
  return C ? cluster_plan(s, C).total : 0;
}

template <int NCH, int G, bool PAGED>
static hipError_t launch_cluster_k(const Shape& s, int C, const void* q, const float* P, const void* klo,
                                   const void* khi, const void* v, void* out, int32_t* out_idx,
                                   uint32_t* ctl, bool ctl_clean, void* region, uint32_t spin_limit,
                                   hipStream_t st) {
  using Lds = GqaLds<kClusterThreads, G, true>;
  auto kern = fused_gqa_kernel<kClusterThreads, NCH, G, kClusterKpt, PAGED, true>;
  const int L = gqa_slice_rows(s.S, C);
  const size_t lds = Lds::total_bytes(L, s.k < L ? s.k : L);
  static std::atomic<unsigned long long> lds_allowed{0};  // per instantiation: devices already set up
  const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(kern),
                                         (int)Lds::total_bytes(kClusterMaxSlice, kClusterMaxList), lds_allowed);
  if (e != hipSuccess) return e;
  const ClusterPlan p = cluster_plan(s, C);
  char* base = static_cast<char*>(region);
  ClusterArgs cl;
  cl.counters = ctl;
  cl.error = ctl + (size_t)kClusterMaxUnits * kClusterCounterStride;
  cl.xhist = reinterpret_cast<uint32_t*>(base + p.xhist);
  cl.xhist_bytes = p.xcand - p.xhist;
  cl.xcand = reinterpret_cast<uint32_t*>(base + p.xcand);
  cl.xcand_bytes = p.partial - p.xcand;
  cl.partial = reinterpret_cast<float*>(base + p.partial);
  cl.C = C;
  cl.units = s.B * s.Hkv;
  cl.spin_limit = spin_limit;
  cl.rank_cap = cluster_rank_cap(s);
  cl.give_up_at_list = g_give_up_at_list.load(std::memory_order_relaxed);
  // the arrival flags and tickets start at zero: unless the caller vouches for the workspace,
  // clear them (with a kernel, not a memset: a caller may be capturing the stream into a graph)
  if (!ctl_clean) {
    const int n_zero = cl.units * (kClusterMax + 1) + 1;
    hipLaunchKernelGGL(cluster_reset_kernel, dim3((n_zero + 255) / 256), dim3(256), 0, st, cl.counters, cl.units);
  }
  hipLaunchKernelGGL(kern, dim3(cluster_padded_units(s) * C), dim3(kClusterThreads), lds, st,
                     static_cast<const uint16_t*>(klo), static_cast<const uint16_t*>(khi),
                     static_cast<const uint16_t*>(v), static_cast<const uint16_t*>(q), P,
                     static_cast<uint16_t*>(out), out_idx, s.Hkv, s.S, s.S_cap, s.k, with_loads(s, kGroupLaunch), s.ap, s.pg, cl);
  return hipGetLastError();
}

template <int NCH>
static hipError_t launch_cluster_n(const Shape& s, int C, const void* q, const float* P, const void* klo,
                                   const void* khi, const void* v, void* out, int32_t* out_idx,
                                   uint32_t* ctl, bool ctl_clean, void* region, uint32_t spin_limit,
                                   hipStream_t st) {
#define LOKI_CLUSTER_G(Gn)                                                                              \
  case Gn:                                                                                              \
    return s.pg.table != nullptr                                                                        \
               ? launch_cluster_k<NCH, Gn, true>(s, C, q, P, klo, khi, v, out, out_idx, ctl, ctl_clean, region, \
                                                 spin_limit, st)                                        \
               : launch_cluster_k<NCH, Gn, false>(s, C, q, P, klo, khi, v, out, out_idx, ctl, ctl_clean, region, \
                                                  spin_limit, st)
  switch (s.G) {
    LOKI_CLUSTER_G(2);
    LOKI_CLUSTER_G(4);
    LOKI_CLUSTER_G(8);
    default: return hipErrorInvalidValue;
  }
#undef LOKI_CLUSTER_G
}

hipError_t launch_fused_gqa_cluster(const Shape& s, const void* q, const float* P, const void* klo,
                                    const void* khi, const void* v, void* out, int32_t* out_idx,
                                    uint32_t* ctl, bool ctl_clean, void* region, hipStream_t st) {
  if (!fused_gqa_cluster_eligible(s, 1) || region == nullptr || ctl == nullptr) return hipErrorInvalidValue;
  const int C = fused_gqa_cluster_blocks(s, 1);
  const uint32_t spin_limit = g_spin_limit.load(std::memory_order_relaxed);
  switch (s.d / 8) {
    case 2: return launch_cluster_n<2>(s, C, q, P, klo, khi, v, out, out_idx, ctl, ctl_clean, region, spin_limit, st);
    case 4: return launch_cluster_n<4>(s, C, q, P, klo, khi, v, out, out_idx, ctl, ctl_clean, region, spin_limit, st);
    case 8: return launch_cluster_n<8>(s, C, q, P, klo, khi, v, out, out_idx, ctl, ctl_clean, region, spin_limit, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace loki
