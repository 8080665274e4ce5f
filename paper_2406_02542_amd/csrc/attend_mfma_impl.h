// Attention over a list of cache rows for SEVERAL query heads that share those rows (grouped
// queries; Section 2 Eq. 1 for the dense baseline, Algorithm 1 lines 7-9 of arXiv 2406.02542
// for a selection shared by a KV group), bf16 caches, on the matrix cores.  Device functions
// shared by the stand-alone kernels (attend_mfma.hip) and the single-launch grouped-query
// kernel (fused_gqa.hip).
//
// A wave works on steps of 32 rows:
//   S[row, head] = K[row, :] . q[head, :]      v_mfma_f32_16x16x32_bf16, A = the 16-byte-per-lane
//                                              load of a 16-row tile of K, B = q^T (16 heads)
//   softmax scalars per head                   lane (head, k-group) sees 8 of the 32 rows; the
//                                              step maximum is shared with two cross-row moves
//   O[head, col] += P[head, row] V[row, col]   A = P straight from the accumulator layout of the
//                                              first product (two bf16 terms), B = V^T, which
//                                              needs rows contiguous per lane: lane (m, k-group)
//                                              loads 16 bytes, columns 8 m .. 8 m + 7, of each of
//                                              its k-group's 8 rows (a load instruction covers four
//                                              whole rows) and pairs the rows up with v_perm_b32, one
//                                              instruction per operand register; the second product's
//                                              column m of tile c is then column 8 m + c of V
// The next step's keys are loaded as soon as the first product has read the current ones, its
// values as soon as the second product has, so loads are in flight all the time. What bounds it is
// memory once the chip is full, the chain of a step's instructions when it is not. Against V tiles
// transposed through LDS (16 writes and 64 two-byte reads a step, 67 KB a block, 60 registers
// more): one sequence of 32/8 heads, S = 8192, k = 1024, 22.4 -> 20.9 us per step; dense attention
// over 1 to 64 sequences of 500 to 20000 rows, 4 heads 12 % less on average, 8 heads 17 %, where
// memory bounds it 1 to 4 %.
#pragma once

#include "attend_impl.h"

namespace loki {

typedef __bf16 am_bf16x8_t __attribute__((ext_vector_type(8)));
typedef float am_f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kAmRows = 32;  // rows per wave step

__device__ __forceinline__ uint32_t am_word(const uint4& x, int i) { return i == 0 ? x.x : i == 1 ? x.y : i == 2 ? x.z : x.w; }

// B operand of the first product from an fp32 (rotated) query: head r16's values at `qh`
// (global or LDS), columns 32*step + 8*kgrp .. +7, as QT bf16 terms.  Columns at or past
// `d_limit` and lanes without a head get zeros.
template <int KSTEPS, int QT>
__device__ __forceinline__ void am_query_operands(const float* qh, bool head_ok, int d_limit,
                                                  am_bf16x8_t (&bq)[KSTEPS][QT]) {
  const int kgrp = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int step = 0; step < KSTEPS; ++step) {
    const int col = 32 * step + 8 * kgrp;
    const bool col_ok = head_ok && col < d_limit;
    uint32_t w[QT][4];
#pragma unroll
    for (int e2 = 0; e2 < 4; ++e2) {
      float rest0 = col_ok ? qh[col + 2 * e2] : 0.f, rest1 = col_ok ? qh[col + 2 * e2 + 1] : 0.f;
#pragma unroll
      for (int t = 0; t < QT; ++t) {
        const uint32_t pk = BF16::round2(rest0, rest1);
        rest0 -= __uint_as_float(pk << 16);            // exact in fp32
        rest1 -= __uint_as_float(pk & 0xffff0000u);
        w[t][e2] = pk;
      }
    }
#pragma unroll
    for (int t = 0; t < QT; ++t)
      bq[step][t] = __builtin_bit_cast(am_bf16x8_t, make_uint4(w[t][0], w[t][1], w[t][2], w[t][3]));
  }
}

// Where this lane's 16-byte chunks of a K row and of a V row live: chunk 4*step + kgrp of the
// logical key row (k_a holds the first d_a columns with row pitch d_a, k_b the rest), chunk
// r16 of the value row.
template <int KSTEPS>
struct AmAddr {
  const char* kptr[KSTEPS];
  size_t kpitch[KSTEPS];
  const char* vptr;
};

// LO_ONLY: every chunk comes from k_a (the logits use its columns only).
template <int KSTEPS, bool LO_ONLY>
__device__ __forceinline__ AmAddr<KSTEPS> am_make_addr(const void* k_a, const void* k_b, const void* v,
                                                       size_t addr_unit, int S_cap, int d_a) {
  const int r16 = threadIdx.x & 15, kgrp = (threadIdx.x & 63) >> 4;
  const int nlo = d_a / 8;  // chunks held by k_a
  AmAddr<KSTEPS> ad;
#pragma unroll
  for (int step = 0; step < KSTEPS; ++step) {
    const int c = 4 * step + kgrp;
    const bool in_lo = c < nlo;
    ad.kpitch[step] = (in_lo || LO_ONLY) ? (size_t)d_a * 2 : (size_t)(kD - d_a) * 2;
    const char* base = (in_lo || LO_ONLY) ? static_cast<const char*>(k_a) + (size_t)(in_lo ? c : 0) * 16
                                          : static_cast<const char*>(k_b) + (size_t)(c - nlo) * 16;
    ad.kptr[step] = base + addr_unit * S_cap * ad.kpitch[step];
  }
  ad.vptr = static_cast<const char*>(v) + addr_unit * S_cap * (kD * 2) + (size_t)r16 * 16;
  return ad;
}

// Running state of one wave: head r16's maximum and sum over this lane's share of the rows,
// and the output accumulators o[c][i] = column 8*r16 + c of head 4*kgrp + i.
struct AmState {
  float m_run, l_run;
  am_f32x4_t o[8];
  __device__ __forceinline__ void init() {
    m_run = kNegBig;
    l_run = 0.f;
#pragma unroll
    for (int c = 0; c < 8; ++c) o[c] = am_f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
};

// Which steps a wave takes.  next(base, end): the wave's next step, entries [base, base + 32) of
// which those below `end` exist; false: no more, base = end (uniform for the wave).  early():
// whether the first step may be asked for, and its rows loaded, before the list is complete. The
// block's WAVES waves take the steps of entries [r0, r1) round-robin; entries below `there` are
// there early.
template <int WAVES>
struct AmRoundRobin {
  int at, r1, there;
  __device__ __forceinline__ AmRoundRobin(int r0, int r1_, int there_ = 0)
      : at(r0 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) * kAmRows), r1(r1_), there(there_) {}
  // (a wave without a step has nothing to load)
  __device__ __forceinline__ bool early() const { return at < r1 && at + kAmRows <= there; }
  __device__ __forceinline__ bool next(int& base, int& end) {
    base = min(at, r1);
    end = r1;
    at += WAVES * kAmRows;
    return base < r1;
  }
};

// Cache row of list entry r = GATHER ? s_idx[r - r0] : r.  s_idx: 16-byte aligned.  complete():
// called once by every wave, completes the list; the loads of a first step that may be asked for
// early are in flight meanwhile.  STREAM_V: values are loaded past the caches (row_loads); keys are
// not, of which an instruction takes 64 bytes of 16 rows, half lines: 16 sequences of 32/8 heads, S =
// 16384, dense, neither 129.6 us, values 116.7, both 118.3; one selection per group, 96 units, S =
// 6073, d = 16 39.2, 36.4, 44.6.
template <bool GATHER, int KSTEPS, int QT, bool STREAM_V, typename Steps, typename Complete>
__device__ __forceinline__ void am_attend_rows(const AmAddr<KSTEPS>& ad,
                                               const am_bf16x8_t (&bq)[KSTEPS][QT],
                                               const int32_t* s_idx, int r0, Steps steps, AmState& st, Complete complete) {
  const int lane = threadIdx.x & 63;
  const int r16 = lane & 15, kgrp = lane >> 4;
  int base, end;

  uint4 kraw[2][KSTEPS], vraw[8];
  // two 16-row tiles of K (A operands); rows past the end re-read the last one
  auto issue_k = [&](int b, int r1) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int r = min(b + 16 * t + r16, r1 - 1);
      const int row = GATHER ? s_idx[r - r0] : r;
#pragma unroll
      for (int step = 0; step < KSTEPS; ++step) kraw[t][step] = load16(ad.kptr[step] + (size_t)row * ad.kpitch[step]);
    }
  };
  // this k-group's rows of V: e = 4 t + i is row 16 t + 4 kgrp + i of the step
  auto issue_v = [&](int b, int r1) {
    int row[8];
    if (GATHER && b + kAmRows <= r1) {  // (uniform)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int4 x = *reinterpret_cast<const int4*>(s_idx + (b - r0 + 16 * t + 4 * kgrp));
        row[4 * t] = x.x;
        row[4 * t + 1] = x.y;
        row[4 * t + 2] = x.z;
        row[4 * t + 3] = x.w;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int r = min(b + 16 * (e / 4) + 4 * kgrp + e % 4, r1 - 1);
        row[e] = GATHER ? s_idx[r - r0] : r;
      }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) vraw[e] = load16_hint<STREAM_V>(ad.vptr + (size_t)row[e] * (kD * 2));
  };
  const bool early = steps.early();
  if (early) {
    steps.next(base, end);
    issue_k(base, end);
    issue_v(base, end);
  }
  complete();
  if (!early) {
    if (!steps.next(base, end)) return;
    issue_k(base, end);
    issue_v(base, end);
  }
  for (bool more = true; more;) {
    // ---- S = K q^T: acc[t][i] = logit of entry base + 16 t + 4 kgrp + i for head r16 -----------
    am_f32x4_t s_acc[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      s_acc[t] = am_f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int qt = QT - 1; qt >= 0; --qt)
#pragma unroll
        for (int step = 0; step < KSTEPS; ++step)
          s_acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              __builtin_bit_cast(am_bf16x8_t, kraw[t][step]), bq[step][qt], s_acc[t], 0, 0, 0);
    }
    const int b0 = base, r1 = end;
    more = steps.next(base, end);  // (no more: the loads below re-read the last row)
    issue_k(base, end);
    // ---- softmax scalars of head r16 -----------------------------------------------------------
    float logit[2][4];
    float smax = kNegBig;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool ok = b0 + 16 * t + 4 * kgrp + i < r1;
        logit[t][i] = ok ? s_acc[t][i] * kSoftmaxScaleLog2 : kNegBig;
        smax = fmaxf(smax, logit[t][i]);
      }
    smax = fmaxf(smax, __shfl_xor(smax, 16));
    smax = fmaxf(smax, __shfl_xor(smax, 32));
    const float m_new = fmaxf(st.m_run, smax);
    const float corr = fast_exp2(st.m_run - m_new);
    st.m_run = m_new;
    float p[8], psum = 0.f;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool ok = b0 + 16 * t + 4 * kgrp + i < r1;
        p[4 * t + i] = ok ? fast_exp2(logit[t][i] - m_new) : 0.f;
        psum += p[4 * t + i];
      }
    st.l_run = fmaf(st.l_run, corr, psum);
    // A operand of the second product: P[head r16][k = 8 kgrp + e], two bf16 terms
    uint32_t ph[4], pl[4];
#pragma unroll
    for (int e2 = 0; e2 < 4; ++e2) {
      ph[e2] = BF16::round2(p[2 * e2], p[2 * e2 + 1]);
      pl[e2] = BF16::round2(p[2 * e2] - __uint_as_float(ph[e2] << 16),
                            p[2 * e2 + 1] - __uint_as_float(ph[e2] & 0xffff0000u));
    }
    const am_bf16x8_t a_hi = __builtin_bit_cast(am_bf16x8_t, make_uint4(ph[0], ph[1], ph[2], ph[3]));
    const am_bf16x8_t a_lo = __builtin_bit_cast(am_bf16x8_t, make_uint4(pl[0], pl[1], pl[2], pl[3]));
    // ---- rescale the running output when some head's maximum moved ---------------------------
    if (__ballot(corr != 1.0f) != 0ull) {
      float c4[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) c4[i] = __shfl(corr, 4 * kgrp + i);  // lane of head 4 kgrp + i
#pragma unroll
      for (int c = 0; c < 8; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) st.o[c][i] *= c4[i];
    }
    // ---- O += P V: B operand c = column 8 r16 + c of this k-group's rows, two to a register ----
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      uint32_t w[4];
#pragma unroll
      for (int e2 = 0; e2 < 4; ++e2)
        w[e2] = __builtin_amdgcn_perm(am_word(vraw[2 * e2 + 1], c / 2), am_word(vraw[2 * e2], c / 2),
                                      c % 2 ? 0x07060302u : 0x05040100u);
      const am_bf16x8_t bv = __builtin_bit_cast(am_bf16x8_t, make_uint4(w[0], w[1], w[2], w[3]));
      st.o[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a_lo, bv, st.o[c], 0, 0, 0);
      st.o[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a_hi, bv, st.o[c], 0, 0, 0);
    }
    issue_v(base, end);
  }
}

// Wave totals (sum over the four k-groups) into LDS, one (m, l, o[128]) per wave and head.
// Ends with a barrier.
template <int NH, int WAVES>
__device__ __forceinline__ void am_publish(AmState& st, MergeSmem<WAVES, NH>& sm) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r16 = lane & 15, kgrp = lane >> 4;
  st.l_run += __shfl_xor(st.l_run, 16);
  st.l_run += __shfl_xor(st.l_run, 32);
  if (kgrp == 0 && r16 < NH) {
    sm.m[wave][r16] = st.m_run;
    sm.l[wave][r16] = st.l_run;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int head = 4 * kgrp + i;
    if (head < NH) {
      float4* dst = reinterpret_cast<float4*>(&sm.o[wave][head][8 * r16]);
      dst[0] = make_float4(st.o[0][i], st.o[1][i], st.o[2][i], st.o[3][i]);
      dst[1] = make_float4(st.o[4][i], st.o[5][i], st.o[6][i], st.o[7][i]);
    }
  }
  __syncthreads();
}

}  // namespace loki
