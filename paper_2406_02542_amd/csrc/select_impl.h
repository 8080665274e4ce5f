// Block-wide exact top-k selection over a score array (global memory or LDS), shared by the
// stand-alone select kernel and the fused decode kernel.
//
// Scores are mapped to order-preserving 32-bit keys.  Three histogram passes (11 + 11 + 10
// bits, most significant first) find the key T of the k-th largest score and how many rows
// equal to T are still needed; one ordered compaction pass (wave ballot + prefix popcount)
// then emits every position with key > T plus the first `need_eq` positions with key == T,
// in ascending position order.  Lowest position wins among equal scores; no sort anywhere.
#pragma once

#include "common.h"

namespace loki {

constexpr int kSelMaxCand = 1024;  // candidates of the threshold bin ranked directly (<= 2048 / 2)

template <int THREADS>
struct SelectSmem {
  static constexpr int kWaves = THREADS / 64;
  uint32_t hist[2048];  // digit histogram; its first kSelMaxCand words later hold the candidates
  uint32_t wave[kWaves];
  uint32_t out[2];
  uint32_t ncand;
  uint32_t cnt[2][kWaves][2];
};

// Scanning bins from the highest down, finds the bin holding the rem-th largest key and how
// many keys are still needed from inside it: sm.out[0] = bin, sm.out[1] = remainder.
// Thread t owns the BPT consecutive bins ending at nbins-1-BPT*t.  Ends with a barrier.
template <int THREADS>
__device__ __forceinline__ void find_threshold_bin(SelectSmem<THREADS>& sm, int nbins,
                                                   uint32_t rem) {
  constexpr int BPT = 2048 / THREADS > 1 ? 2048 / THREADS : 1;  // bins per thread (nbins <= 2048)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int top = nbins - 1 - BPT * tid;
  uint32_t cbin[BPT];
  uint32_t c = 0;
#pragma unroll
  for (int i = 0; i < BPT; ++i) {
    const int b = top - i;
    cbin[i] = b >= 0 ? sm.hist[b] : 0u;
    c += cbin[i];
  }
  uint32_t incl = wave_inclusive_scan_u32(c);
  if (lane == 63) sm.wave[wave] = incl;
  __syncthreads();
  uint32_t off = 0;
  for (int w = 0; w < wave; ++w) off += sm.wave[w];
  incl += off;
  uint32_t excl = incl - c;
  if (excl < rem && rem <= incl) {
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      if (excl < rem && rem <= excl + cbin[i]) {
        sm.out[0] = (uint32_t)(top - i);
        sm.out[1] = rem - excl;
      }
      excl += cbin[i];
    }
  }
  __syncthreads();
}

// a[0..S) must be visible to the whole block on entry.  emit(rank, pos) is called exactly k
// times over the block, rank in [0, k) ascending with pos.
template <int THREADS, typename Emit>
__device__ __forceinline__ void block_select_topk(const float* a, int S, int k,
                                                  SelectSmem<THREADS>& sm, Emit emit) {
  constexpr int kWaves = THREADS / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

  uint32_t prefix = 0;  // the bits of T fixed so far, right-aligned
  uint32_t rem = (uint32_t)k;
  int fixed = 0;
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    const int bits = p < 2 ? 11 : 10;
    const int nbins = 1 << bits;
    const int shift = 32 - fixed - bits;
    for (int i = tid; i < nbins; i += THREADS) sm.hist[i] = 0u;
    __syncthreads();
    for (int pos = tid; pos < S; pos += THREADS) {
      const uint32_t key = float_to_key(a[pos]);
      const bool match = (fixed == 0) || ((key >> (32 - fixed)) == prefix);
      if (match) atomicAdd(&sm.hist[(key >> shift) & (uint32_t)(nbins - 1)], 1u);
    }
    __syncthreads();
    find_threshold_bin<THREADS>(sm, nbins, rem);
    prefix = (prefix << bits) | sm.out[0];
    rem = sm.out[1];
    fixed += bits;
    __syncthreads();
  }
  const uint32_t T = prefix;
  const uint32_t need_eq = rem;  // 1 <= need_eq <= count(key == T)

  uint32_t base_gt = 0, base_eq = 0;
  int buf = 0;
  for (int tile = 0; tile < S; tile += THREADS, buf ^= 1) {
    const int pos = tile + tid;
    const bool valid = pos < S;
    const uint32_t key = valid ? float_to_key(a[pos]) : 0u;
    const bool gt = valid && key > T;
    const bool eq = valid && key == T;
    const unsigned long long mgt = __ballot(gt);
    const unsigned long long meq = __ballot(eq);
    const unsigned long long below = (1ull << lane) - 1ull;
    const uint32_t lgt = __popcll(mgt & below), leq = __popcll(meq & below);
    if (lane == 0) {
      sm.cnt[buf][wave][0] = __popcll(mgt);
      sm.cnt[buf][wave][1] = __popcll(meq);
    }
    __syncthreads();
    uint32_t wgt = 0, weq = 0, tgt = 0, teq = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const uint32_t cg = sm.cnt[buf][w][0], ce = sm.cnt[buf][w][1];
      if (w < wave) {
        wgt += cg;
        weq += ce;
      }
      tgt += cg;
      teq += ce;
    }
    const uint32_t gt_before = base_gt + wgt + lgt;
    const uint32_t eq_before = base_eq + weq + leq;
    if (gt || (eq && eq_before < need_eq)) emit((int)(gt_before + min(eq_before, need_eq)), pos);
    base_gt += tgt;
    base_eq += teq;
  }
}

// Same selection for a score array (LDS or global) small enough for every thread to keep its
// keys in registers: C = per_thread <= KPT keys each, C a multiple of 4, THREADS*C >= S
// (nothing at or past S is read).  Two histogram passes (11 + 11 bits) run on the register
// keys, the second one only over the keys of the first pass's threshold bin; the handful of
// keys that still share all 22 leading bits with the threshold are ranked against each other
// directly (a third, 10-bit pass replaces the ranking if there are more than kSelMaxRank of
// them, e.g. many equal scores).  The compaction is one block-wide exclusive scan of
// per-thread counts.  emit(rank, pos, score) is called exactly k times,
// rank in [0, k) ascending with pos.
//
// resident_select_clear() zeroes both histograms; the caller runs it any time before the
// call (with a barrier in between), e.g. ahead of the scoring loop whose closing barrier
// then covers it.
constexpr int kSelMaxRank = 64;

template <int THREADS>
struct ResidentSelectSmem {
  static constexpr int kWaves = THREADS / 64;
  uint32_t hist[2][2048];
  uint32_t wave[2][kWaves];
  uint32_t out[2][2];
  uint32_t ncand;
  uint32_t cand[kSelMaxRank];
};

template <int THREADS>
__device__ __forceinline__ void resident_select_clear(ResidentSelectSmem<THREADS>& sm) {
  for (int i = threadIdx.x; i < 2 * 2048; i += THREADS) (&sm.hist[0][0])[i] = 0u;
  if (threadIdx.x == 0) sm.ncand = 0u;
}

// As find_threshold_bin, on histogram `which` (2048 bins).  One barrier inside, one at the end.
template <int THREADS>
__device__ __forceinline__ void resident_find_bin(ResidentSelectSmem<THREADS>& sm, int which,
                                                  uint32_t rem) {
  constexpr int kWaves = THREADS / 64;
  constexpr int BPT = 2048 / THREADS;
  static_assert(BPT >= 1, "at most 2048 threads");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int top = 2047 - BPT * tid;
  uint32_t cbin[BPT];
  uint32_t c = 0;
#pragma unroll
  for (int i = 0; i < BPT; ++i) {
    cbin[i] = sm.hist[which][top - i];
    c += cbin[i];
  }
  uint32_t incl = wave_inclusive_scan_u32(c);
  if (lane == 63) sm.wave[which][wave] = incl;
  __syncthreads();
  uint32_t off = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const uint32_t t = sm.wave[which][w];
    off += (w < wave) ? t : 0u;
  }
  incl += off;
  uint32_t excl = incl - c;
  if (excl < rem && rem <= incl) {
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      if (excl < rem && rem <= excl + cbin[i]) {
        sm.out[which][0] = (uint32_t)(top - i);
        sm.out[which][1] = rem - excl;
      }
      excl += cbin[i];
    }
  }
  __syncthreads();
}

#define LOKI_SEL_VALID(i) ((valid_mask >> (i)) & 1u)
// resident_threshold (below) from its second pass on: sm.out[0] as resident_find_bin left it for the leading
// 11 bits, histogram 1 and sm.ncand clear.
template <int THREADS, int KPT>
__device__ __forceinline__ void resident_threshold_in_bin(const uint32_t (&key)[KPT], uint32_t valid_mask,
                                                          ResidentSelectSmem<THREADS>& sm, uint32_t& T,
                                                          uint32_t& need_eq) {
  const int tid = threadIdx.x;
  const uint32_t bin1 = sm.out[0][0];
  // pass 2: bits 20..10 of the keys inside the threshold bin
#pragma unroll
  for (int i = 0; i < KPT; ++i)
    if (LOKI_SEL_VALID(i) && (key[i] >> 21) == bin1) atomicAdd(&sm.hist[1][(key[i] >> 10) & 2047u], 1u);
  __syncthreads();
  resident_find_bin<THREADS>(sm, 1, sm.out[0][1]);
  const uint32_t top22 = (bin1 << 11) | sm.out[1][0];
  const uint32_t rem = sm.out[1][1];
  LOKI_STAMP(14);

  // the keys that share all 22 leading bits with the threshold
#pragma unroll
  for (int i = 0; i < KPT; ++i)
    if (LOKI_SEL_VALID(i) && (key[i] >> 10) == top22) {
      const uint32_t slot = atomicAdd(&sm.ncand, 1u);
      if (slot < (uint32_t)kSelMaxRank) sm.cand[slot] = key[i];
    }
  __syncthreads();
  const uint32_t ncand = sm.ncand;
  if (ncand <= (uint32_t)kSelMaxRank) {
    // T is the candidate with (#greater < rem <= #greater + #equal) among the candidates
    if (tid < (int)ncand) {
      const uint32_t ki = sm.cand[tid];
      uint32_t gt = 0, eq = 0;
      for (uint32_t j = 0; j < ncand; ++j) {
        const uint32_t kj = sm.cand[j];
        gt += kj > ki;
        eq += kj == ki;
      }
      if (gt < rem && rem <= gt + eq) {
        sm.out[0][0] = ki;
        sm.out[0][1] = rem - gt;
      }
    }
    __syncthreads();
    T = sm.out[0][0];
    need_eq = sm.out[0][1];
  } else {
    // many keys agree on 22 bits (e.g. equal scores): resolve bits 9..0 with a third pass,
    // reusing histogram 0 (everyone is past its last read: two barriers ago)
    for (int i = tid; i < 2048; i += THREADS) sm.hist[0][i] = 0u;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < KPT; ++i)
      if (LOKI_SEL_VALID(i) && (key[i] >> 10) == top22) atomicAdd(&sm.hist[0][1024u + (key[i] & 1023u)], 1u);
    __syncthreads();
    resident_find_bin<THREADS>(sm, 0, rem);   // bins 1024..2047 hold the 10-bit digit
    T = (top22 << 10) | (sm.out[0][0] - 1024u);
    need_eq = sm.out[0][1];
  }
}

// Exact threshold of the rem-th largest of the block's register-resident keys: returns the
// key T and how many keys equal to T are needed (need_eq >= 1).  valid_mask bit i says whether
// key[i] takes part.  Both histograms and sm.ncand must be clear on entry (see
// resident_select_clear) and every thread must be past any earlier use of sm.
template <int THREADS, int KPT>
__device__ __forceinline__ void resident_threshold(const uint32_t (&key)[KPT], uint32_t valid_mask,
                                                   uint32_t rem_in, ResidentSelectSmem<THREADS>& sm,
                                                   uint32_t& T, uint32_t& need_eq) {
  // pass 1: bits 31..21 of every key
#pragma unroll
  for (int i = 0; i < KPT; ++i)
    if (LOKI_SEL_VALID(i)) atomicAdd(&sm.hist[0][key[i] >> 21], 1u);
  __syncthreads();
  resident_find_bin<THREADS>(sm, 0, rem_in);
  LOKI_STAMP(13);
  resident_threshold_in_bin<THREADS, KPT>(key, valid_mask, sm, T, need_eq);
}
#undef LOKI_SEL_VALID

// The block's positions are laid out wave by wave: wave w owns the 64*C consecutive positions
// from w*64*C in tiles of 256, and inside a tile lane l holds the 4 positions from 4l — one
// coalesced 16-byte load per lane and tile, and a position order (wave, tile, lane, element)
// that the compaction can follow with per-tile DPP scans and a single barrier.
//
// resident_load_keys: reads a[0..n) in that layout; key[4j + e] is position
// resident_pos0(C) + 256 j + e.
__device__ __forceinline__ int resident_pos0(int C) {
  return (int)(threadIdx.x >> 6) * 64 * C + (int)(threadIdx.x & 63) * 4;
}

// The same for an array that already holds keys (16-byte aligned).
template <int KPT>
__device__ __forceinline__ void resident_load_keys(const uint32_t* a, int n, int C, uint32_t (&key)[KPT],
                                                   uint32_t& valid_mask) {
  constexpr int kTiles = KPT / 4;
  const int wbase = resident_pos0(C);
  valid_mask = 0;
#pragma unroll
  for (int j = 0; j < kTiles; ++j) {
    const int i = 4 * j;
    const int p = wbase + 256 * j;
    key[i + 0] = key[i + 1] = key[i + 2] = key[i + 3] = 0u;
    if (i < C) {
      if (p + 3 < n) {
        const uint4 f = *reinterpret_cast<const uint4*>(a + p);
        key[i + 0] = f.x;
        key[i + 1] = f.y;
        key[i + 2] = f.z;
        key[i + 3] = f.w;
        valid_mask |= 0xfu << i;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (p + e < n) {
            key[i + e] = a[p + e];
            valid_mask |= 1u << (i + e);
          }
      }
    }
  }
}

template <int KPT>
__device__ __forceinline__ void resident_load_keys(const float* a, int n, int C, uint32_t (&key)[KPT],
                                                   uint32_t& valid_mask) {
  constexpr int kTiles = KPT / 4;
  const int wbase = resident_pos0(C);
  const bool aligned = (reinterpret_cast<uintptr_t>(a) & 15u) == 0;
  valid_mask = 0;
#pragma unroll
  for (int j = 0; j < kTiles; ++j) {
    const int i = 4 * j;
    const int p = wbase + 256 * j;
    key[i + 0] = key[i + 1] = key[i + 2] = key[i + 3] = 0u;
    if (i < C) {
      if (aligned && p + 3 < n) {
        const float4 f = *reinterpret_cast<const float4*>(a + p);
        key[i + 0] = float_to_key(f.x);
        key[i + 1] = float_to_key(f.y);
        key[i + 2] = float_to_key(f.z);
        key[i + 3] = float_to_key(f.w);
        valid_mask |= 0xfu << i;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (p + e < n) {
            key[i + e] = float_to_key(a[p + e]);
            valid_mask |= 1u << (i + e);
          }
      }
    }
  }
}

// Ordered emission of the keys > T and of the first need_eq keys == T (counted from
// eq_base equal keys already seen at lower positions); ranks start at gt_base +
// min(eq_base, need_eq).  Per tile a DPP exclusive scan over the lanes (greater in the low
// half-word, equal in the high half-word: a wave holds at most 64*KPT <= 65535 keys), then one
// barrier to learn how many selected rows the earlier waves hold.  wave_g / wave_e are two
// LDS arrays of THREADS/64 words that nobody else touches until the next barrier.
// emit(rank, local position, score).
template <int THREADS, int KPT, typename Emit>
__device__ __forceinline__ void resident_compact(const uint32_t (&key)[KPT], uint32_t valid_mask,
                                                 int C, uint32_t T, uint32_t need_eq,
                                                 uint32_t gt_base, uint32_t eq_base,
                                                 uint32_t* wave_g_tot, uint32_t* wave_e_tot,
                                                 Emit emit) {
  constexpr int kWaves = THREADS / 64;
  constexpr int kTiles = KPT / 4;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wbase = resident_pos0(C);
  uint32_t excl[kTiles];
  uint32_t wave_g = 0, wave_e = 0;
#pragma unroll
  for (int j = 0; j < kTiles; ++j) {
    uint32_t mine = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if ((valid_mask >> (4 * j + e)) & 1u)
        mine += (key[4 * j + e] > T ? 1u : 0u) + (key[4 * j + e] == T ? 0x10000u : 0u);
    const uint32_t incl = wave_inclusive_scan_u32(mine);
    const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    excl[j] = (wave_g + ((incl - mine) & 0xffffu)) | ((wave_e + ((incl - mine) >> 16)) << 16);
    wave_g += tot & 0xffffu;
    wave_e += tot >> 16;
  }
  if (lane == 0) {
    wave_g_tot[wave] = wave_g;
    wave_e_tot[wave] = wave_e;
  }
  __syncthreads();
  uint32_t before_g = gt_base, before_e = eq_base;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const uint32_t tg = wave_g_tot[w], te = wave_e_tot[w];
    before_g += (w < wave) ? tg : 0u;
    before_e += (w < wave) ? te : 0u;
  }
#pragma unroll
  for (int j = 0; j < kTiles; ++j) {
    uint32_t g_before = before_g + (excl[j] & 0xffffu), e_before = before_e + (excl[j] >> 16);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if ((valid_mask >> (4 * j + e)) & 1u) {
        const uint32_t kk = key[4 * j + e];
        const bool gt = kk > T, eq = kk == T;
        if (gt || (eq && e_before < need_eq))
          emit((int)(g_before + min(e_before, need_eq)), wbase + 256 * j + e, key_to_float(kk));
        g_before += gt;
        e_before += eq;
      }
  }
}

// Ordered split of the register-resident keys by their leading 11 bits against the threshold
// bin: keys in a higher bin are certain to be selected, keys inside the bin are the candidates
// among which the exact threshold lies.  emit_gt(rank, pos) sees every key above the bin with
// its rank among those (ascending with pos) and its key; emit_eq(rank, pos, key) every key inside the bin
// likewise.  Same layout, scans and single barrier as resident_compact.
template <int THREADS, int KPT, typename EmitGt, typename EmitEq>
__device__ __forceinline__ void resident_partition(const uint32_t (&key)[KPT], uint32_t valid_mask,
                                                   int C, uint32_t bin, uint32_t* wave_g_tot,
                                                   uint32_t* wave_e_tot, EmitGt emit_gt,
                                                   EmitEq emit_eq) {
  constexpr int kWaves = THREADS / 64;
  constexpr int kTiles = KPT / 4;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wbase = resident_pos0(C);
  uint32_t excl[kTiles];
  uint32_t wave_g = 0, wave_e = 0;
#pragma unroll
  for (int j = 0; j < kTiles; ++j) {
    uint32_t mine = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if ((valid_mask >> (4 * j + e)) & 1u) {
        const uint32_t b = key[4 * j + e] >> 21;
        mine += (b > bin ? 1u : 0u) + (b == bin ? 0x10000u : 0u);
      }
    const uint32_t incl = wave_inclusive_scan_u32(mine);
    const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    excl[j] = (wave_g + ((incl - mine) & 0xffffu)) | ((wave_e + ((incl - mine) >> 16)) << 16);
    wave_g += tot & 0xffffu;
    wave_e += tot >> 16;
  }
  if (lane == 0) {
    wave_g_tot[wave] = wave_g;
    wave_e_tot[wave] = wave_e;
  }
  __syncthreads();
  uint32_t before_g = 0, before_e = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const uint32_t tg = wave_g_tot[w], te = wave_e_tot[w];
    before_g += (w < wave) ? tg : 0u;
    before_e += (w < wave) ? te : 0u;
  }
#pragma unroll
  for (int j = 0; j < kTiles; ++j) {
    uint32_t g_before = before_g + (excl[j] & 0xffffu), e_before = before_e + (excl[j] >> 16);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if ((valid_mask >> (4 * j + e)) & 1u) {
        const uint32_t kk = key[4 * j + e];
        const uint32_t b = kk >> 21;
        if (b > bin) emit_gt((int)g_before, wbase + 256 * j + e, kk);
        if (b == bin) emit_eq((int)e_before, wbase + 256 * j + e, kk);
        g_before += b > bin;
        e_before += b == bin;
      }
  }
}

// ---- keys in LDS, every thread owning C consecutive positions ------------------------------------
// The array is padded by one word per 32 (position r lives at r + r / 32), so that the lanes of a
// wave, whose runs start C words apart, read different banks.  C is a power of two of at most 32,
// so a run never crosses a multiple of 32 and lies in consecutive words.  Thread t owns positions
// [t C, (t + 1) C); ranks follow the thread order, so everything emitted is ascending in position.
// All reads are unconditional (a run past the end of the data is read and masked out): guarded
// reads cost a branch per key.
__device__ __forceinline__ int padded_pos(int r) { return r + (r >> 5); }
__host__ __device__ inline size_t padded_words(size_t n) { return n + (n >> 5) + 33; }

// bit e set: position t C + e is inside the thread's run and below n
__device__ __forceinline__ uint32_t contiguous_valid_mask(int n, int C) {
  const int nv = max(0, min(C, n - (int)threadIdx.x * C));
  return nv >= 32 ? 0xffffffffu : ((1u << nv) - 1u);
}

template <int KPT>
__device__ __forceinline__ void contiguous_load_keys(const uint32_t* s_key, int n, int C,
                                                     uint32_t (&key)[KPT], uint32_t& valid_mask) {
  const uint32_t* run = s_key + padded_pos((int)threadIdx.x * C);
  valid_mask = contiguous_valid_mask(n, C);
#pragma unroll
  for (int e = 0; e < KPT; ++e) {
    const uint32_t x = run[e];  // (inside the array's slack when e >= C)
    key[e] = ((valid_mask >> e) & 1u) ? x : 0u;
  }
}

// One pass over the block's keys: emit_gt(rank, pos) for every key whose leading bits
// (key >> shift) exceed thr, emit_eq(rank, pos, key) for every key whose leading bits equal it,
// ranks counted separately and ascending with pos.  A thread first builds two bit masks over
// its run, the ranks come from one wave scan and one barrier (wave_tot: a word per wave), and the
// emission loops run once per set bit, not once per key.
template <int THREADS, int KPT, typename EmitGt, typename EmitEq>
__device__ __forceinline__ void contiguous_partition(const uint32_t* s_key, int n, int C, int shift,
                                                     uint32_t thr, uint32_t* wave_tot, EmitGt emit_gt,
                                                     EmitEq emit_eq) {
  constexpr int kWaves = THREADS / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r0 = (int)threadIdx.x * C;
  const uint32_t* run = s_key + padded_pos(r0);
  uint32_t gt = 0, eq = 0;
#pragma unroll
  for (int e = 0; e < KPT; ++e) {
    const uint32_t b = run[e] >> shift;
    gt |= (b > thr ? 1u : 0u) << e;
    eq |= (b == thr ? 1u : 0u) << e;
  }
  const uint32_t vm = contiguous_valid_mask(n, C);
  gt &= vm;
  eq &= vm;
  LOKI_STAMP(3);
  const uint32_t mine = (uint32_t)__popc(gt) | ((uint32_t)__popc(eq) << 16);
  const uint32_t incl = wave_inclusive_scan_u32(mine);
  if (lane == 63) wave_tot[wave] = incl;
  __syncthreads();
  LOKI_STAMP(5);
  uint32_t before = incl - mine;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) before += (w < wave) ? wave_tot[w] : 0u;
  int g_rank = (int)(before & 0xffffu), e_rank = (int)(before >> 16);
  while (gt) {
    const int e = __ffs((int)gt) - 1;
    gt &= gt - 1;
    emit_gt(g_rank++, r0 + e);
  }
  while (eq) {
    const int e = __ffs((int)eq) - 1;
    eq &= eq - 1;
    emit_eq(e_rank++, r0 + e, run[e]);
  }
}

// ---- a candidate list ranked by one wave, without a barrier ---------------------------------------
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// What is chosen: keys above T and the first need_eq of those equal to it.
struct WaveThreshold {
  uint32_t T, need_eq;
};

// Sum over the wave, uniform.
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan_u32(x), 63);
}

// The rem largest (1 <= rem <= n) of n keys of at most `bits` bits: a search on the number of keys
// at or above a trial value, by interpolation first (the keys of one histogram bin lie almost
// evenly: about five trials for a thousand of them) and by halves after that, until a trial has
// exactly rem of them or the threshold is known to the last bit.  count(x): keys >= x, x >= 1,
// uniform.
template <typename Count>
__device__ __forceinline__ WaveThreshold wave_search(int n, int bits, uint32_t rem, Count count) {
  if (rem >= (uint32_t)n) return {0u, (uint32_t)n};
  uint32_t lo = 0, hi = 1u << bits, n_lo = (uint32_t)n, n_hi = 0;  // keys >= lo: n_lo > rem; keys >= hi: n_hi < rem
  for (int trial = 0; hi - lo > 1; ++trial) {
    uint32_t mid = (lo + hi) >> 1;
    if (trial < 12 && (trial & 3) != 3) {
      const float at = (float)(hi - lo) * ((float)(n_lo - rem) * __builtin_amdgcn_rcpf((float)(n_lo - n_hi)));
      mid = min(max(lo + (uint32_t)at, lo + 1u), hi - 1u);
    }
    mid = (uint32_t)__builtin_amdgcn_readfirstlane((int)mid);
    const uint32_t c = count(mid);
    if (c == rem) return {mid - 1u, 0u};
    if (c > rem) {
      lo = mid;
      n_lo = c;
    } else {
      hi = mid;
      n_hi = c;
    }
  }
  return {lo, rem - n_hi};
}

// Up to 64 KPT keys in registers (one wave alone issues an instruction every five cycles or so: two a key
// and trial, and a scan).
template <int KPT>
__device__ __forceinline__ WaveThreshold wave_search_regs(const uint32_t* a, int n, int bits, uint32_t rem) {
  const int lane = threadIdx.x & 63;
  uint32_t key[KPT];
#pragma unroll
  for (int j = 0; j < KPT; ++j) {
    const uint32_t x = a[min(lane + 64 * j, n - 1)];
    key[j] = lane + 64 * j < n ? x : 0u;
  }
  return wave_search(n, bits, rem, [&](uint32_t x) {
    uint32_t c = 0;
#pragma unroll
    for (int j = 0; j < KPT; ++j) c += key[j] >= x ? 1u : 0u;
    return wave_sum_u32(c);
  });
}

// a: LDS, 16-byte aligned, with room up to the next multiple of 256 keys, which is overwritten.
__device__ __forceinline__ WaveThreshold wave_threshold(uint32_t* a, int n, int bits, uint32_t rem) {
  const int lane = threadIdx.x & 63;
  n = __builtin_amdgcn_readfirstlane(n);  // (uniform, and so told to the compiler)
  rem = (uint32_t)__builtin_amdgcn_readfirstlane((int)rem);
  bits = __builtin_amdgcn_readfirstlane(bits);
  if (n <= 256) return wave_search_regs<4>(a, n, bits, rem);
  if (n <= 1024) return wave_search_regs<16>(a, n, bits, rem);
  const int padded = (n + 255) & ~255;
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (n + 64 * j + lane < padded) a[n + 64 * j + lane] = 0u;
  wave_lds_fence();
  return wave_search(n, bits, rem, [&](uint32_t x) {
    uint32_t c = 0;
#pragma unroll 4
    for (int i = 4 * lane; i < padded; i += 256) {
      const uint4 w = *reinterpret_cast<const uint4*>(a + i);
      c += (w.x >= x ? 1u : 0u) + (w.y >= x ? 1u : 0u) + (w.z >= x ? 1u : 0u) + (w.w >= x ? 1u : 0u);
    }
    return wave_sum_u32(c);
  });
}

// Keys of a[0, n) above T, and equal to it.
__device__ __forceinline__ void wave_count(const uint32_t* a, int n, uint32_t T, uint32_t& gt, uint32_t& eq) {
  const int lane = threadIdx.x & 63;
  n = __builtin_amdgcn_readfirstlane(n);
  uint32_t c = 0, e = 0;
#pragma unroll 8
  for (int i = lane; i < n; i += 64) {
    const uint32_t x = a[i];
    c += x > T ? 1u : 0u;
    e += x == T ? 1u : 0u;
  }
  gt = wave_sum_u32(c);
  eq = wave_sum_u32(e);
}

// The wave emits the chosen of a[0, n) in order: emit(rank, i) for every key above T and for the
// first need_eq equal to it, eq_before equal ones having been seen before.  Returns how many.
template <typename Emit>
__device__ __forceinline__ int wave_choose(const uint32_t* a, int n, const WaveThreshold& t, uint32_t eq_before, Emit emit) {
  const int lane = threadIdx.x & 63;
  const unsigned long long below = (1ull << lane) - 1ull;
  constexpr int kBatch = 4;
  int rank = 0;
  n = __builtin_amdgcn_readfirstlane(n);
  for (int i0 = 0; i0 < n; i0 += 64 * kBatch) {
    uint32_t x[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) x[j] = a[min(i0 + 64 * j + lane, n - 1)];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int i = i0 + 64 * j + lane;
      bool take = i < n && x[j] > t.T;
      if (t.need_eq > 0) {  // (uniform; else nothing that equals T is chosen)
        const unsigned long long meq = __ballot(i < n && x[j] == t.T);
        take = take || (i < n && x[j] == t.T && eq_before + (uint32_t)__popcll(meq & below) < t.need_eq);
        eq_before += (uint32_t)__popcll(meq);
      }
      const unsigned long long m = __ballot(take);
      if (take) emit(rank + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u)), i);
      rank += (int)__popcll(m);
    }
  }
  return rank;
}

// Whole selection of keys in LDS (padded as above) whose leading 11 bits are counted in sm.hist[0],
// the rest of sm being clear: emit(rank, pos, key) is called exactly k times, rank in [0, k)
// ascending with pos.  Every thread looks at its run once: the rows above the threshold's bin and
// the rows inside it, the candidates, become two bit masks.  The candidates' keys are collected in
// any order, the first wave finds the exact threshold among them (wave_threshold), and every thread
// then looks at its own candidates again.  More candidates than hist[1] holds (long runs of equal
// scores): the further digit passes of resident_threshold over all keys.
template <int THREADS, int KPT, typename Emit>
__device__ __forceinline__ void contiguous_select(const uint32_t* s_key, int n, int C, int k, ResidentSelectSmem<THREADS>& sm,
                                                  Emit emit) {
  constexpr int kWaves = THREADS / 64, kCap = 2048;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r0 = tid * C;
  const uint32_t* run = s_key + padded_pos(r0 < n ? r0 : 0);  // (threads without rows read the first run and mask it out)
  const uint32_t vm = contiguous_valid_mask(n, C);
  resident_find_bin<THREADS>(sm, 0, (uint32_t)k);
  const uint32_t bin = sm.out[0][0], rem = sm.out[0][1];
  const int n_cand = __builtin_amdgcn_readfirstlane((int)sm.hist[0][bin]);
  LOKI_STAMP(13);
  uint32_t gt = 0, eq = 0, T, need_eq;
  if (n_cand <= kCap) {
#pragma unroll
    for (int e = 0; e < KPT; ++e) {
      const uint32_t b = run[e] >> 21;
      gt |= (b > bin ? 1u : 0u) << e;
      eq |= (b == bin ? 1u : 0u) << e;
    }
    gt &= vm;
    eq &= vm;
    if (eq) {
      uint32_t slot = atomicAdd(&sm.ncand, (uint32_t)__popc(eq));
      for (uint32_t m = eq; m; m &= m - 1) sm.hist[1][slot++] = run[__ffs((int)m) - 1] & ((1u << 21) - 1u);
    }
    __syncthreads();
    LOKI_STAMP(14);
    if (wave == 0) {
      const WaveThreshold t = wave_threshold(sm.hist[1], n_cand, 21, rem);
      if (lane == 0) {
        sm.out[1][0] = (bin << 21) + t.T;
        sm.out[1][1] = t.need_eq;
      }
    }
    __syncthreads();
    T = sm.out[1][0];
    need_eq = sm.out[1][1];
    uint32_t m = eq;
    eq = 0;
    for (; m; m &= m - 1) {
      const uint32_t x = run[__ffs((int)m) - 1], bit = m & (0u - m);
      gt |= x > T ? bit : 0u;
      eq |= x == T ? bit : 0u;
    }
  } else {
    uint32_t key[KPT];
#pragma unroll
    for (int e = 0; e < KPT; ++e) key[e] = run[e];
    resident_threshold_in_bin<THREADS, KPT>(key, vm, sm, T, need_eq);
#pragma unroll
    for (int e = 0; e < KPT; ++e) {
      gt |= (key[e] > T ? 1u : 0u) << e;
      eq |= (key[e] == T ? 1u : 0u) << e;
    }
    gt &= vm;
    eq &= vm;
  }
  LOKI_STAMP(4);
  const uint32_t mine = (uint32_t)__popc(gt) | ((uint32_t)__popc(eq) << 16);
  const uint32_t incl = wave_inclusive_scan_u32(mine);
  if (lane == 63) sm.wave[0][wave] = incl;  // (last read several barriers ago)
  __syncthreads();
  uint32_t before = incl - mine;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) before += (w < wave) ? sm.wave[0][w] : 0u;
  int g_rank = (int)(before & 0xffffu), e_rank = (int)(before >> 16);
  for (uint32_t m = gt | eq; m; m &= m - 1) {
    const int e = __ffs((int)m) - 1;
    const bool is_eq = (eq >> e) & 1u;
    if (!is_eq || e_rank < (int)need_eq) emit(g_rank + min(e_rank, (int)need_eq), r0 + e, run[e]);
    g_rank += is_eq ? 0 : 1;
    e_rank += is_eq ? 1 : 0;
  }
  LOKI_STAMP(12);
}

// ---- selection of keys that the block's threads hold, in two parts --------------------------------
// Thread t holds positions [t C, (t + 1) C) (C <= KPT, a multiple of 4), so ranks follow the thread order.
//   run_select_certain  one digit histogram: the rows above the threshold's bin are certain; the
//                       bin's rows, the candidates, go to a list of their own.  Three barriers, and
//                       one at the end
//   run_threshold       the exact threshold among the candidates, by one wave, without a barrier, so that a caller can
//                       have the certain rows' loads in flight
// A bin of more than kRunCand rows (a quarter of a long sequence kept, or long runs of nearly equal
// scores) makes run_select_certain find the exact threshold with resident_threshold's further
// passes.
constexpr int kRunCand = 1024;

template <int KPT>
struct RunKeys {
  uint32_t key[KPT];
  uint32_t valid;  // bit i: key[i] exists
  int pos0;
};

struct RunSelect {
  int n_def;          // certain rows
  int n_cand;         // candidates listed (0: the threshold is known)
  uint32_t bin, rem;  // the threshold's bin; rows needed from it
  WaveThreshold t;    // on whole keys, once known
};

template <int KPT>
__device__ __forceinline__ void run_load_keys(const float* a, int n, int C, RunKeys<KPT>& rk) {
  const int p0 = (int)threadIdx.x * C;
  const bool aligned = (reinterpret_cast<uintptr_t>(a) & 15u) == 0;  // (uniform)
  rk.pos0 = p0;
  const int nv = max(0, min(C, n - p0));
  rk.valid = nv >= 32 ? 0xffffffffu : ((1u << nv) - 1u);
#pragma unroll
  for (int i = 0; i < KPT; i += 4) {
    float4 f = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < C) {
      if (aligned && p0 + i + 3 < n) {
        f = *reinterpret_cast<const float4*>(a + p0 + i);
      } else {
        if (p0 + i < n) f.x = a[p0 + i];
        if (p0 + i + 1 < n) f.y = a[p0 + i + 1];
        if (p0 + i + 2 < n) f.z = a[p0 + i + 2];
        if (p0 + i + 3 < n) f.w = a[p0 + i + 3];
      }
    }
    rk.key[i] = float_to_key(f.x);
    rk.key[i + 1] = float_to_key(f.y);
    rk.key[i + 2] = float_to_key(f.z);
    rk.key[i + 3] = float_to_key(f.w);
  }
}

// Keys whose leading bits exceed thr / equal it, and the block-wide ranks of this thread's first ones (one
// barrier; wave_tot: a word per wave that nobody else touches until the next barrier).
template <int THREADS, int KPT>
__device__ __forceinline__ void run_partition(const RunKeys<KPT>& rk, int shift, uint32_t thr, uint32_t* wave_tot,
                                              uint32_t& gt, uint32_t& eq, int& g_rank, int& e_rank) {
  constexpr int kWaves = THREADS / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  gt = eq = 0;
#pragma unroll
  for (int i = 0; i < KPT; ++i) {
    const uint32_t b = rk.key[i] >> shift;
    gt |= (b > thr ? 1u : 0u) << i;
    eq |= (b == thr ? 1u : 0u) << i;
  }
  gt &= rk.valid;
  eq &= rk.valid;
  const uint32_t mine = (uint32_t)__popc(gt) | ((uint32_t)__popc(eq) << 16);
  const uint32_t incl = wave_inclusive_scan_u32(mine);
  if (lane == 63) wave_tot[wave] = incl;
  __syncthreads();
  uint32_t before = incl - mine;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) before += (w < wave) ? wave_tot[w] : 0u;
  g_rank = (int)(before & 0xffffu);
  e_rank = (int)(before >> 16);
}

// emit(rank, pos, key) for every certain row, ranks ascending with the position, unless the
// threshold has been found instead.  sm.hist clear and rk loaded by every thread; sm.hist[1] holds
// the candidates afterwards.
template <int THREADS, int KPT, typename Emit>
__device__ __forceinline__ RunSelect run_select_certain(const RunKeys<KPT>& rk, int k, ResidentSelectSmem<THREADS>& sm,
                                                        Emit emit) {
#pragma unroll
  for (int i = 0; i < KPT; ++i)
    if ((rk.valid >> i) & 1u) atomicAdd(&sm.hist[0][rk.key[i] >> 21], 1u);
  __syncthreads();
  resident_find_bin<THREADS>(sm, 0, (uint32_t)k);
  LOKI_STAMP(13);
  RunSelect rs;
  rs.bin = sm.out[0][0];
  rs.rem = sm.out[0][1];
  rs.n_def = k - (int)rs.rem;
  rs.n_cand = (int)sm.hist[0][rs.bin];
  rs.t = WaveThreshold{0u, 0u};
  if (rs.n_cand <= kRunCand) {
    uint32_t gt, eq;
    int g_rank, e_rank;
    run_partition<THREADS, KPT>(rk, 21, rs.bin, sm.wave[1], gt, eq, g_rank, e_rank);
#pragma unroll
    for (int i = 0; i < KPT; ++i) {
      if ((eq >> i) & 1u) {
        sm.hist[1][e_rank] = rk.key[i] & ((1u << 21) - 1u);
        sm.hist[1][kRunCand + e_rank] = (uint32_t)(rk.pos0 + i);
        ++e_rank;
      }
      if ((gt >> i) & 1u) emit(g_rank++, rk.pos0 + i, rk.key[i]);
    }
  } else {
    resident_threshold_in_bin<THREADS, KPT>(rk.key, rk.valid, sm, rs.t.T, rs.t.need_eq);
    rs.n_cand = 0;
  }
  __syncthreads();
  return rs;
}

template <int THREADS>
__device__ __forceinline__ WaveThreshold run_threshold(const RunSelect& rs, ResidentSelectSmem<THREADS>& sm) {
  if (rs.n_cand == 0) return rs.t;
  const WaveThreshold t = wave_threshold(sm.hist[1], rs.n_cand, 21, rs.rem);
  return {(rs.bin << 21) + t.T, t.need_eq};
}

// emit(rank, pos, key) for every selected row, ranks ascending with the position.  One barrier.
template <int THREADS, int KPT, typename Emit>
__device__ __forceinline__ void run_emit(const RunKeys<KPT>& rk, const WaveThreshold& t, ResidentSelectSmem<THREADS>& sm, Emit emit) {
  uint32_t gt, eq;
  int g_rank, e_rank;
  run_partition<THREADS, KPT>(rk, 0, t.T, sm.wave[0], gt, eq, g_rank, e_rank);
#pragma unroll
  for (int i = 0; i < KPT; ++i) {
    const bool is_eq = (eq >> i) & 1u, is_gt = (gt >> i) & 1u;
    if (is_gt || (is_eq && (uint32_t)e_rank < t.need_eq)) emit(g_rank + min(e_rank, (int)t.need_eq), rk.pos0 + i, rk.key[i]);
    g_rank += is_gt ? 1 : 0;
    e_rank += is_eq ? 1 : 0;
  }
}

// Whole selection for S <= THREADS*C: emit(rank, pos, score) is called exactly k times, rank
// in [0, k) ascending with pos.
template <int THREADS, int KPT, typename Emit>
__device__ __forceinline__ void block_select_topk_resident(const float* a, int S, int k,
                                                           int per_thread,
                                                           ResidentSelectSmem<THREADS>& sm,
                                                           Emit emit) {
  uint32_t key[KPT];
  uint32_t valid_mask;
  resident_load_keys<KPT>(a, S, per_thread, key, valid_mask);
  LOKI_STAMP(11);
  uint32_t T, need_eq;
  resident_threshold<THREADS, KPT>(key, valid_mask, (uint32_t)k, sm, T, need_eq);
  LOKI_STAMP(4);
  // sm.wave[0] / sm.wave[1] were last read two or more barriers ago
  resident_compact<THREADS, KPT>(key, valid_mask, per_thread, T, need_eq, 0u, 0u, sm.wave[0],
                                 sm.wave[1], emit);
  LOKI_STAMP(12);
}

}  // namespace loki
