// Exact softmax attention over a list of cache rows with an online softmax in the log2
// domain and scale 1/sqrt(D) (Algorithm 1 lines 7-9 of arXiv 2406.02542 for the selected set,
// Section 2 Eq. 1 for every row).  Shared by the stand-alone attention kernels and the fused
// decode kernel.
//
// A row of K (128 logical columns, possibly split between the low-rank slab and the residual
// slab) and the matching row of V are each read by LPRV consecutive lanes with one 16-byte
// load per lane; the K.q dot product is finished with DPP inside the lane group; every lane
// keeps the running output for its EPC columns of V.
//
// REUSE_LO: the low-rank part of the exact logit, sum_{j<d} qhat_j Khat[s,j], is exactly the
// approximate score the ranking stage already computed, so the lanes that would read the
// low-rank slab read nothing and the saved score is added instead.
#pragma once

#include "common.h"

namespace loki {

#ifndef LOKI_ROWS_IN_FLIGHT
#define LOKI_ROWS_IN_FLIGHT 4
#endif
constexpr int kRowsInFlight = LOKI_ROWS_IN_FLIGHT;  // rows per lane group per loop trip
constexpr int kPartialStride = kD + 2;  // o[128], m, l
constexpr float kSoftmaxScaleLog2 = kLog2e * 0.08838834764831845f;  // log2(e) / sqrt(128)

template <typename T, int NH>
struct AttendAcc {
  float m[NH], l[NH], o[NH][T::EPC];
  __device__ __forceinline__ void init() {
#pragma unroll
    for (int g = 0; g < NH; ++g) {
      m[g] = kNegBig;
      l[g] = 0.f;
#pragma unroll
      for (int e = 0; e < T::EPC; ++e) o[g][e] = 0.f;
    }
  }
};

struct RowAddr {
  const char* k_base;   // this lane's 16-byte chunk of K row 0 of the unit
  size_t k_row_bytes;
  const char* v_base;   // this lane's 16-byte chunk of V row 0 of the unit
  size_t v_row_bytes;
  bool k_load;          // false: this lane's K chunk is covered by the reused score
};

// c = lane's chunk index inside a row (0 .. 128/EPC-1).  k_a holds the first d columns
// (d = 128: the whole row), k_b the rest.  LO_ONLY: the logit uses the first d columns only
// (Algorithm 2, PCAAttn); lanes past them read no key at all.
template <typename T, bool REUSE_LO, bool LO_ONLY = false>
__device__ __forceinline__ RowAddr make_row_addr(const void* k_a, const void* k_b, const void* v,
                                                 size_t kv_unit, int S_cap, int d, int c) {
  const int nlo = d / T::EPC;
  const bool in_lo = c < nlo;
  RowAddr ra;
  ra.k_load = LO_ONLY ? in_lo : !(REUSE_LO && in_lo);
  ra.k_row_bytes = (in_lo || LO_ONLY) ? (size_t)d * T::kBytes : (size_t)(kD - d) * T::kBytes;
  const char* kb = (in_lo || LO_ONLY) ? static_cast<const char*>(k_a) + (size_t)(in_lo ? c : 0) * 16
                                      : static_cast<const char*>(k_b) + (size_t)(c - nlo) * 16;
  ra.k_base = kb + kv_unit * S_cap * ra.k_row_bytes;
  ra.v_row_bytes = (size_t)kD * T::kBytes;
  ra.v_base = static_cast<const char*>(v) + kv_unit * S_cap * ra.v_row_bytes + (size_t)c * 16;
  return ra;
}

// One trip: R rows of this lane group (ok: the row exists), their chunks and saved scores loaded.
template <typename T, int NH, int R, bool REUSE_LO>
__device__ __forceinline__ void attend_trip(AttendAcc<T, NH>& acc, const float (&qr)[NH][T::EPC], const uint4 (&kraw)[R],
                                            const uint4 (&vraw)[R], const float (&alo)[R], const bool (&ok)[R]) {
  constexpr int EPC = T::EPC;
  constexpr int LPRV = kD / EPC;
  float logit[NH][R];
#pragma unroll
  for (int j = 0; j < R; ++j) {
    float kf[EPC];
    T::unpack(kraw[j], kf);
#pragma unroll
    for (int g = 0; g < NH; ++g) {
      float p = 0.f;
#pragma unroll
      for (int e = 0; e < EPC; ++e) p = fmaf(kf[e], qr[g][e], p);
      p = group_allreduce_sum<LPRV>(p);
      if constexpr (REUSE_LO) p += alo[j];
      logit[g][j] = ok[j] ? p * kSoftmaxScaleLog2 : kNegBig;
    }
  }
  float vf[R][EPC];
#pragma unroll
  for (int j = 0; j < R; ++j) T::unpack(vraw[j], vf[j]);
#pragma unroll
  for (int g = 0; g < NH; ++g) {
    float mn = acc.m[g];
#pragma unroll
    for (int j = 0; j < R; ++j) mn = fmaxf(mn, logit[g][j]);
    const float corr = fast_exp2(acc.m[g] - mn);
    acc.m[g] = mn;
    float pj[R], ps = 0.f;
#pragma unroll
    for (int j = 0; j < R; ++j) {
      pj[j] = ok[j] ? fast_exp2(logit[g][j] - mn) : 0.f;
      ps += pj[j];
    }
    acc.l[g] = fmaf(acc.l[g], corr, ps);
#pragma unroll
    for (int e = 0; e < EPC; ++e) {
      float a = acc.o[g][e] * corr;
#pragma unroll
      for (int j = 0; j < R; ++j) a = fmaf(pj[j], vf[j][e], a);
      acc.o[g][e] = a;
    }
  }
}

// Processes list entries r in [r0, r1): cache row = GATHER ? s_idx[r - r0] : r.  NGROUPS lane
// groups of the block share the entries round-robin; `gid` is this lane's group.
// s_a: REUSE_LO: the saved score of entry r at r - r0 (SCORE_BY_ROW: the key of cache row `row`, at
// its padded position).
// APART: the arithmetic of a trip is attend_trip's, else it stands here once more: the compiler
// then loads a trip's rows earlier (fp32, 4 heads, 94 registers for 88).  apart / here, us: dense
// attention over 2 sequences of 990 rows, 32/8 fp32 heads, 20.4 / 18.3, 2 to 7 of 546 to 2310 rows
// 4 to 13 % more, large ones 0.6 %; but one block per head beyond 8192 rows, 512 heads in groups of
// 4, S = 12800, k = 400 46.4 / 47.3, S = 13300, k = 831 62.7 / 64.0.
// STREAM: rows are loaded past the caches (row_loads).  ROWS: rows per lane group and trip.
template <typename T, int NH, int NGROUPS, bool GATHER, bool REUSE_LO, bool SCORE_BY_ROW = false, bool APART = false, bool STREAM = false,
          int ROWS = kRowsInFlight>
__device__ __forceinline__ void attend_rows(AttendAcc<T, NH>& acc, const float (&qr)[NH][T::EPC],
                                            const RowAddr& ra, const int32_t* s_idx,
                                            const float* s_a, int gid, int r0, int r1) {
  constexpr int EPC = T::EPC;
  constexpr int LPRV = kD / EPC;
  constexpr int R = ROWS;
  static_assert(!REUSE_LO || NH == 1, "score reuse needs one query head per selection");
  for (int t0 = r0; t0 < r1; t0 += NGROUPS * R) {
    bool ok[R];
    uint4 kraw[R], vraw[R];
    float alo[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const int r = t0 + j * NGROUPS + gid;
      ok[j] = r < r1;
      int row = 0;
      alo[j] = 0.f;
      if (ok[j]) {
        row = GATHER ? s_idx[r - r0] : r;
        if constexpr (REUSE_LO && SCORE_BY_ROW)
          alo[j] = key_to_float(reinterpret_cast<const uint32_t*>(s_a)[row + (row >> 5)]);
        else if constexpr (REUSE_LO)
          alo[j] = s_a[r - r0];
      }
      kraw[j] = (ok[j] && ra.k_load) ? load16_hint<STREAM>(ra.k_base + (size_t)row * ra.k_row_bytes)
                                     : make_uint4(0, 0, 0, 0);
      vraw[j] = ok[j] ? load16_hint<STREAM>(ra.v_base + (size_t)row * ra.v_row_bytes) : make_uint4(0, 0, 0, 0);
    }
    if constexpr (APART) {
      attend_trip<T, NH, R, REUSE_LO>(acc, qr, kraw, vraw, alo, ok);
    } else {
      float logit[NH][R];
#pragma unroll
      for (int j = 0; j < R; ++j) {
        float kf[EPC];
        T::unpack(kraw[j], kf);
#pragma unroll
        for (int g = 0; g < NH; ++g) {
          float p = 0.f;
#pragma unroll
          for (int e = 0; e < EPC; ++e) p = fmaf(kf[e], qr[g][e], p);
          p = group_allreduce_sum<LPRV>(p);
          if constexpr (REUSE_LO) p += alo[j];
          logit[g][j] = ok[j] ? p * kSoftmaxScaleLog2 : kNegBig;
        }
      }
      float vf[R][EPC];
#pragma unroll
      for (int j = 0; j < R; ++j) T::unpack(vraw[j], vf[j]);
#pragma unroll
      for (int g = 0; g < NH; ++g) {
        float mn = acc.m[g];
#pragma unroll
        for (int j = 0; j < R; ++j) mn = fmaxf(mn, logit[g][j]);
        const float corr = fast_exp2(acc.m[g] - mn);
        acc.m[g] = mn;
        float pj[R], ps = 0.f;
#pragma unroll
        for (int j = 0; j < R; ++j) {
          pj[j] = ok[j] ? fast_exp2(logit[g][j] - mn) : 0.f;
          ps += pj[j];
        }
        acc.l[g] = fmaf(acc.l[g], corr, ps);
#pragma unroll
        for (int e = 0; e < EPC; ++e) {
          float a = acc.o[g][e] * corr;
#pragma unroll
          for (int j = 0; j < R; ++j) a = fmaf(pj[j], vf[j][e], a);
          acc.o[g][e] = a;
        }
      }
    }
  }
}

// The same over a list that is still growing: entries below `there` exist when the call begins, and
// those of the first trip are loaded before complete(), which completes the list (every wave calls
// it once).  The form of the loads is chosen around each trip's: around the whole, complete() would be there twice
// (64 heads, S = 8192, k = 2048 34.1 us, 32.7 so).
template <typename T, int NH, int NGROUPS, bool REUSE_LO, typename Complete>
__device__ __forceinline__ void attend_growing(AttendAcc<T, NH>& acc, const float (&qr)[NH][T::EPC],
                                               const RowAddr& ra, const int32_t* s_idx, const float* s_a, int gid,
                                               int r0, int r1, int there, int form_now, Complete complete) {
  constexpr int R = kRowsInFlight;
  uint4 kraw[R], vraw[R];
  float alo[R];
  auto clear = [&]() {
#pragma unroll
    for (int j = 0; j < R; ++j) {
      kraw[j] = vraw[j] = make_uint4(0, 0, 0, 0);
      alo[j] = 0.f;
    }
  };
  auto load = [&](int t0, int lo, int hi) __attribute__((always_inline)) {  // the trip's entries in [lo, hi)
    with_form<kPastCaches>(form_now, [&](auto form) __attribute__((always_inline)) {
      constexpr bool kPast = decltype(form)::value != kThroughCaches;
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const int r = t0 + j * NGROUPS + gid;
        if (r >= lo && r < hi) {
          const int row = s_idx[r - r0];
          if constexpr (REUSE_LO) alo[j] = s_a[r - r0];
          if (ra.k_load) kraw[j] = load16_hint<kPast>(ra.k_base + (size_t)row * ra.k_row_bytes);
          vraw[j] = load16_hint<kPast>(ra.v_base + (size_t)row * ra.v_row_bytes);
        }
      }
    });
  };
  clear();
  if (there > r0) load(r0, r0, min(r1, there));
  complete();
  if (there < r1) load(r0, max(r0, there), r1);
  for (int t0 = r0; t0 < r1; t0 += NGROUPS * R) {
    if (t0 > r0) {
      clear();
      load(t0, r0, r1);
    }
    bool ok[R];
#pragma unroll
    for (int j = 0; j < R; ++j) ok[j] = t0 + j * NGROUPS + gid < r1;
    attend_trip<T, NH, R, REUSE_LO>(acc, qr, kraw, vraw, alo, ok);
  }
}

// ---- dense attention over sequences of unequal length --------------------------------------------
// The X = nsplit B blocks that a launch has for every KV head are dealt out by length: sequence b is
// cut into n_b = ceil(len_b / R) equal runs with the smallest R at which all runs fit X, so every block
// has about the same rows and the chip is full for one round.  (Cut at the longest sequence's run
// length instead, a batch of lengths uniform in [S/4, S] leaves a third of the blocks without rows and
// the others with a last round that is half empty: 16 sequences of 32/8 heads,
// S = 16384, 144 us with two blocks per CU, 134 dealt out.)  Every wave works it out for itself, lane b
// for sequence b; the parts of the result lie at [query head][base_b + run].
constexpr int kDenseMinRun = 128;
// This lane's sequence: its rows, its runs, the runs of it and the sequences before it; total: rows of the batch, which
// also say how they are loaded (us, with a sum of its own for that and the dealing out behind it / so: 3 sequences of
// 32/16 heads, S = 9880 33.4 / 33.1, 12 of 32/8, S = 5000 31.9 / 31.8).
struct DenseRuns {
  int len = 0, runs = 0, incl = 0, total = 0;
};
__device__ __forceinline__ DenseRuns dense_runs(const Ragged& rg, int B, int S_max, int nsplit) {
  const int lane = threadIdx.x & 63;
  const int len = lane < B ? seq_rows(rg, lane, S_max) : 0;
  const int total = __builtin_amdgcn_readlane((int)wave_inclusive_scan_u32((uint32_t)len), 63);
  const int X = nsplit * B;
  int runs;
  // equal lengths: nothing to deal out (440 units of 8 heads, S = 3440, eight blocks per CU: 161 us
  // with the search below)
  const int first = __builtin_amdgcn_readlane(len, 0);
  if (first >= nsplit * kDenseMinRun && __ballot(lane < B && len != first) == 0ull) {
    return {len, lane < B ? nsplit : 0, nsplit * min(lane + 1, B), total};
  }
  // R lies between total / X and total / (X - B); each lane tries one length of that range
  const int lo = max((total + X - 1) / X, kDenseMinRun), hi = max((total + X - B - 1) / (X - B), lo);
  const float inv = 1.0f / (float)(lo + ((hi - lo) * lane + 62) / 63);
  int sum = 0;
  for (int b = 0; b < B; ++b) sum += max(1, (int)ceilf((float)__builtin_amdgcn_readlane(len, b) * inv));
  const unsigned long long fits = __ballot(sum <= X);
  if (fits != 0ull) {
    const float chosen = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(inv), __ffsll((long long)fits) - 1));
    runs = max(1, (int)ceilf((float)len * chosen));
  } else {
    runs = nsplit;  // (rounding at the far end of the range)
  }
  if (lane >= B) runs = 0;
  return {len, runs, (int)wave_inclusive_scan_u32((uint32_t)runs), total};
}

__device__ __forceinline__ int dense_form(const RowLoads& l, const DenseRuns& deal) {
  return l.form != kByLengths ? l.form : form_of(l, {(float)deal.total, 0.f});
}

template <int WAVES, int NH>
struct MergeSmem {
  float m[WAVES][NH], l[WAVES][NH];
  float o[WAVES][NH][kD];
};

// Merges the lane groups of each wave in registers, then publishes one (m, l, o[128]) per
// wave and head in LDS.  Ends with a barrier.
template <typename T, int NH, int WAVES>
__device__ __forceinline__ void attend_publish(AttendAcc<T, NH>& acc, MergeSmem<WAVES, NH>& sm) {
  constexpr int EPC = T::EPC;
  constexpr int LPRV = kD / EPC;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c = lane % LPRV, rg = lane / LPRV;
#pragma unroll
  for (int off = LPRV; off < 64; off <<= 1) {
#pragma unroll
    for (int g = 0; g < NH; ++g) {
      const float m2 = __shfl_xor(acc.m[g], off);
      const float l2 = __shfl_xor(acc.l[g], off);
      const float mn = fmaxf(acc.m[g], m2);
      const float a = fast_exp2(acc.m[g] - mn), b2 = fast_exp2(m2 - mn);
      acc.l[g] = acc.l[g] * a + l2 * b2;
#pragma unroll
      for (int e = 0; e < EPC; ++e) {
        const float o2 = __shfl_xor(acc.o[g][e], off);
        acc.o[g][e] = acc.o[g][e] * a + o2 * b2;
      }
      acc.m[g] = mn;
    }
  }
  if (rg == 0) {
#pragma unroll
    for (int g = 0; g < NH; ++g) {
      if (c == 0) {
        sm.m[wave][g] = acc.m[g];
        sm.l[wave][g] = acc.l[g];
      }
#pragma unroll
      for (int e = 0; e < EPC; ++e) sm.o[wave][g][c * EPC + e] = acc.o[g][e];
    }
  }
  __syncthreads();
}

// Partial results that another block of the same launch will read (the merge by the last
// block, below) are stored and loaded as device-scope relaxed atomics: such a store is written
// through to the level all XCDs share and such a load is served from there, so no block has to
// write back or invalidate a whole L2 (a device-scope fence per block costs tens of
// microseconds on this part: measured 33 -> 144 us on a 512-block gather).
__device__ __forceinline__ void store_shared_f32(float* p, float v, bool device_scope) {
  if (device_scope) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *p = v;
}
template <bool DEVICE_SCOPE>
__device__ __forceinline__ float load_shared_f32(const float* p) {
  if constexpr (DEVICE_SCOPE) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else return *p;
}

// Merge of the nsplit partial results of one query head, column col:
// sum_i o_i 2^(m_i - M) / sum_i l_i 2^(m_i - M).  Loads are issued in independent batches of 8
// splits so that the merge costs a few memory round trips, not one per split.
template <bool DEVICE_SCOPE>
__device__ __forceinline__ float combine_splits(const float* pr, int nsplit, int col) {
  constexpr int B8 = 8;
  float mn = kNegBig;
  for (int i0 = 0; i0 < nsplit; i0 += B8) {
    float mi[B8];
#pragma unroll
    for (int u = 0; u < B8; ++u)
      mi[u] = (i0 + u < nsplit) ? load_shared_f32<DEVICE_SCOPE>(pr + (i0 + u) * kPartialStride + kD) : kNegBig;
#pragma unroll
    for (int u = 0; u < B8; ++u) mn = fmaxf(mn, mi[u]);
  }
  float ls = 0.f, os = 0.f;
  for (int i0 = 0; i0 < nsplit; i0 += B8) {
    float mi[B8], li[B8], oi[B8];
#pragma unroll
    for (int u = 0; u < B8; ++u) {
      const bool ok = i0 + u < nsplit;
      const float* p = pr + (ok ? (i0 + u) : 0) * kPartialStride;
      const float m_ = load_shared_f32<DEVICE_SCOPE>(p + kD), l_ = load_shared_f32<DEVICE_SCOPE>(p + kD + 1);
      const float o_ = load_shared_f32<DEVICE_SCOPE>(p + col);
      mi[u] = ok ? m_ : kNegBig;
      li[u] = ok ? l_ : 0.f;
      oi[u] = ok ? o_ : 0.f;
    }
#pragma unroll
    for (int u = 0; u < B8; ++u) {
      const float f = fast_exp2(mi[u] - mn);
      ls = fmaf(li[u], f, ls);
      os = fmaf(oi[u], f, os);
    }
  }
  return os / ls;
}

// The row splits of a head group are merged by whichever of its blocks finishes last, so the
// merge needs no launch of its own.  Call after the block's partials are stored (with
// store_shared_f32 at device scope), by every thread of the block; `ticket` counts the group's
// finished blocks and is zero when the launch starts.  Every thread waits until its own stores
// are acknowledged (vmcnt(0)), the barrier collects the block, and only then one thread takes
// the ticket with a device-scope atomic; the block that draws the last one reads the others'
// partials with device-scope loads issued after that atomic has returned.  No block waits for
// another.
__device__ __forceinline__ bool splits_all_done(int32_t* ticket, int nsplit) {
  __shared__ int s_last_block;
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0); expcnt and lgkmcnt left alone
  __syncthreads();
  if (threadIdx.x == 0) s_last_block = (atomicAdd(ticket, 1) == nsplit - 1) ? 1 : 0;
  __syncthreads();
  return s_last_block != 0;
}

// Merged (max, sum, output) of head g, column col over the block's waves.
template <int WAVES, int NH>
__device__ __forceinline__ void attend_merged(const MergeSmem<WAVES, NH>& sm, int g, int col,
                                              float& mn, float& ls, float& os) {
  mn = sm.m[0][g];
#pragma unroll
  for (int w = 1; w < WAVES; ++w) mn = fmaxf(mn, sm.m[w][g]);
  ls = 0.f;
  os = 0.f;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) {
    const float f = fast_exp2(sm.m[w][g] - mn);
    ls = fmaf(sm.l[w][g], f, ls);
    os = fmaf(sm.o[w][g][col], f, os);
  }
}

}  // namespace loki
