// Query rotation and low-rank scoring (Algorithm 1 lines 3 and 5 of arXiv 2406.02542) as
// stand-alone kernels for the split path, where the rows of a unit are spread over many
// blocks: the low-rank slab is streamed, one block scoring a run of rows of one (batch, KV head)
// unit for all G query heads of the group, so the slab is read once per unit.  The rotated
// queries (qhat = q P_h, fp32) also go to the workspace for the attention stage.  Two forms:
//
//   one launch (ROT)   one token per sequence: every score block rotates the d columns it needs for
//                      itself while its first slab rows are on their way (d / 128 of P_h: 16 KB at
//                      d = 32), and four blocks of each unit do the rest, the whole qhat and the
//                      appended row.  Against a rotation launch in front of it, us per step: one
//                      sequence of 32 heads, S = 4096, 20.4 -> 19.4; of 32/8 heads, S = 8192,
//                      25.0 -> 22.3; 16 of 32/8 heads, S = 12345, per-head selection 118.3 -> 115.0
//   qrot_kernel first  everything else: with many blocks their own rotations cost more than the
//                      launch (rotate_score_applies), with several tokens per sequence a block
//                      reads rows that another one appends, and the histograms of a long sequence's
//                      selection have to be clear before the scoring begins.  A score block then
//                      needs no LDS and no barrier: its slice of qhat goes straight to registers
//                      while the first slab loads are already in flight.
#include "score_impl.h"
#include "score_mfma_impl.h"

namespace loki {

// Block (unit, quarter) computes 32 columns of qhat for the unit's G query heads: thread
// (column j, part p) accumulates the 16 terms of part p, then the 8 parts are added in order —
// the same association as the fused decode kernel, so every path sees bit-identical qhat.
constexpr int kQrotCols = 32;
constexpr int kQrotBlocks = kD / kQrotCols;

// What the rotation reads and writes.  With ap.k_new the unit's new key is rotated as one more
// vector beside the G queries and written, with the new value, into row seq_len-1 of the unit's cache.
struct RotArgs {
  const void* q;
  const float* P;
  float* qhat;
  void* klo;
  void* khi;
  void* v;
  Append ap;
  uint32_t* zero_words;  // n_zero words to clear (tickets, histograms), or null
  size_t n_zero;
};

template <typename T, int G>
struct RotSmem {
  float q[G + 1][kD];                     // the queries, the new key
  float part[G + 1][kRotParts][kQrotCols];
};

// Partial sums of 32 columns for vectors 0 .. NV-1 of sm.q, the last one only if `last`; pv: this
// thread's 16 entries of its column of P_h.  Needs a barrier behind it.
template <typename T, int G>
__device__ __forceinline__ void rot_partial(RotSmem<T, G>& sm, const float (&pv)[kRotPartLen], bool last) {
  const int jl = threadIdx.x % kQrotCols, part = threadIdx.x / kQrotCols;
#pragma unroll
  for (int g = 0; g < G + 1; ++g)
    if (g < G || last) {  // (uniform)
      float acc = 0.f;
#pragma unroll
      for (int i4 = 0; i4 < kRotPartLen; i4 += 4) {
        const float4 qq = *reinterpret_cast<const float4*>(&sm.q[g][part * kRotPartLen + i4]);
        acc = fmaf(qq.x, pv[i4 + 0], acc);
        acc = fmaf(qq.y, pv[i4 + 1], acc);
        acc = fmaf(qq.z, pv[i4 + 2], acc);
        acc = fmaf(qq.w, pv[i4 + 3], acc);
      }
      sm.part[g][part][jl] = acc;
    }
}

// Columns 32 quarter .. of qhat for one unit, and the appended row's columns there except those
// below write_from (another block writes them) and its value row (quarter 0).
template <typename T, int G, bool APPEND>
__device__ __forceinline__ void qrot_block(RotSmem<T, G>& sm, const RotArgs& ra, int unit, int quarter, int Hkv, int S_max,
                                           int S_cap, int d, const Ragged& rg, const Paging& pg, int write_from) {
  using ST = typename T::store_t;
  const int tid = threadIdx.x, h = unit % Hkv;
  const size_t head0 = (size_t)unit * G;
  const int jl = tid % kQrotCols, part = tid / kQrotCols;  // 8 parts of 16 terms
  const float* Ph = ra.P + (size_t)h * kD * kD + quarter * kQrotCols + jl;
  float pv[kRotPartLen];
#pragma unroll
  for (int ii = 0; ii < kRotPartLen; ++ii) pv[ii] = Ph[(size_t)(part * kRotPartLen + ii) * kD];
  const ST* q = static_cast<const ST*>(ra.q);
  for (int i = tid; i < G * kD; i += 256) sm.q[i / kD][i % kD] = T::load1(q + head0 * kD + i);
  size_t row = 0;
  if constexpr (APPEND) {
    if (tid < kD) sm.q[G][tid] = T::load1(static_cast<const ST*>(ra.ap.k_new) + (size_t)unit * kD + tid);
    row = (size_t)cache_row(pg, unit / Hkv / max(rg.queries, 1), h, Hkv, S_cap,
                            seq_rows(rg, unit / Hkv, S_max) - 1);
    if (quarter == 0 && tid >= kD)  // the value row is copied once per unit
      static_cast<ST*>(ra.v)[row * kD + (tid - kD)] = static_cast<const ST*>(ra.ap.v_new)[(size_t)unit * kD + (tid - kD)];
  }
  __syncthreads();
  rot_partial<T, G>(sm, pv, APPEND);
  __syncthreads();
  for (int i = tid; i < (G + (APPEND ? 1 : 0)) * kQrotCols; i += 256) {
    const int g = i / kQrotCols, jj = i % kQrotCols;
    float sum = 0.f;
#pragma unroll
    for (int pp = 0; pp < kRotParts; ++pp) sum += sm.part[g][pp][jj];
    const int col = quarter * kQrotCols + jj;
    if (g < G) {
      ra.qhat[(head0 + g) * kD + col] = sum;
    } else if (col >= write_from) {
      ST* dst = col < d ? static_cast<ST*>(ra.klo) + row * d + col
                        : static_cast<ST*>(ra.khi) + row * (kD - d) + (col - d);
      T::store1(dst, sum);
    }
  }
}

template <typename T, int G, bool APPEND>
__global__ __launch_bounds__(256) void qrot_kernel(RotArgs ra, int Hkv, int S_max, int S_cap, int d, Ragged rg,
                                                   Paging pg) {
  __shared__ __align__(16) RotSmem<T, G> sm;
  // the chunk histograms the score kernel adds into (long sequences) start from zero
  if (ra.zero_words != nullptr) {
    const size_t nthreads = (size_t)gridDim.x * gridDim.y * 256;
    for (size_t i = ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * 256 + threadIdx.x; i < ra.n_zero; i += nthreads)
      ra.zero_words[i] = 0u;
  }
  qrot_block<T, G, APPEND>(sm, ra, blockIdx.x, blockIdx.y, Hkv, S_max, S_cap, d, rg, pg, 0);
}

// A score block's own rotation (ROT): columns 0 .. d-1 of its G queries into s_qhat [G][kPasses * 32],
// and, in the block whose rows end with the appended one, that row's low-rank part into the slab.  d_max =
// 32 kPasses >= d.  `prefetch` is called once the rotation's own loads are issued.  Ends with a barrier;
// returns whether the block has written the row (its earlier loads may have missed it).
template <typename T, int G, int kPasses, typename Prefetch>
__device__ __forceinline__ bool score_block_rotate(RotSmem<T, G>& sm, float (&s_qhat)[G][kPasses * kQrotCols], const RotArgs& ra,
                                                   int unit, int Hkv, int S, int S_cap, int d, int row0, int row_end,
                                                   const Paging& pg, Prefetch prefetch) {
  using ST = typename T::store_t;
  constexpr int kCols = kPasses * kQrotCols;
  const int tid = threadIdx.x, h = unit % Hkv;
  const size_t head0 = (size_t)unit * G;
  const int jl = tid % kQrotCols, part = tid / kQrotCols;
  const bool append = ra.ap.k_new != nullptr && S - 1 >= row0 && S - 1 < row_end;  // (uniform)
  const float* Ph = ra.P + (size_t)h * kD * kD + jl;
  constexpr int kQPerThread = (G * kD + 255) / 256;
  float qv[kQPerThread];
  const ST* q = static_cast<const ST*>(ra.q) + head0 * kD;
#pragma unroll
  for (int j = 0; j < kQPerThread; ++j) qv[j] = T::load1(q + min(tid + 256 * j, G * kD - 1));
  const ST* kn = append ? static_cast<const ST*>(ra.ap.k_new) + (size_t)unit * kD : q;
  const float kn_mine = T::load1(kn + (tid & (kD - 1)));
  float pv[kPasses][kRotPartLen];
#pragma unroll
  for (int ps = 0; ps < kPasses; ++ps)
#pragma unroll
    for (int ii = 0; ii < kRotPartLen; ++ii) pv[ps][ii] = Ph[(size_t)(part * kRotPartLen + ii) * kD + ps * kQrotCols];
  __builtin_amdgcn_sched_barrier(0);
  prefetch();
#pragma unroll
  for (int j = 0; j < kQPerThread; ++j)
    if (tid + 256 * j < G * kD) sm.q[(tid + 256 * j) / kD][(tid + 256 * j) % kD] = qv[j];
  if (tid < kD) sm.q[G][tid] = kn_mine;
  __syncthreads();
#pragma unroll
  for (int ps = 0; ps < kPasses; ++ps) {
    if (ps > 0) __syncthreads();  // the sums of the columns before have been read
    rot_partial<T, G>(sm, pv[ps], append);
    __syncthreads();
    for (int i = tid; i < (G + (append ? 1 : 0)) * kQrotCols; i += 256) {
      const int g = i / kQrotCols, col = ps * kQrotCols + i % kQrotCols;
      float sum = 0.f;
#pragma unroll
      for (int pp = 0; pp < kRotParts; ++pp) sum += sm.part[g][pp][i % kQrotCols];
      if (g < G) {
        s_qhat[g][col] = sum;
      } else if (col < d) {
        const size_t row = (size_t)cache_row(pg, unit / Hkv, h, Hkv, S_cap, S - 1);
        T::store1(static_cast<ST*>(ra.klo) + row * d + col, sum);
      }
    }
  }
  __syncthreads();
  static_assert(kCols <= kD, "columns of P_h");
  return append;
}

// Tickets of the attention stage, cleared by the rotating blocks of a ROT launch.
__device__ __forceinline__ void zero_tickets(const RotArgs& ra) {
  const size_t nthreads = (size_t)kQrotBlocks * gridDim.y * 256;
  for (size_t i = ((size_t)blockIdx.y * kQrotBlocks + blockIdx.x) * 256 + threadIdx.x; i < ra.n_zero; i += nthreads)
    ra.zero_words[i] = 0u;
}

// Long sequences (hist_part != nullptr): the first counting pass of the selection rides along.
// The block counts the leading 11 bits of the key of every score it writes in LDS (16-bit
// counters, two bins per word: a block scores at most kHistChunk rows) and adds the counts into
// the histogram of the select chunk its rows belong to, hist_part[selecting head][chunk][2048];
// the host keeps a block inside one chunk.  The dynamic LDS holds kHistWords words per
// selecting head of the block (none without hist_part).
constexpr int kHistChunk = 16384;  // rows per select chunk (select.hip: kMbChunk)
constexpr int kHistWords = 1024;

__device__ __forceinline__ void hist_count(uint32_t* s_hist, float score) {
  const uint32_t bin = float_to_key(score) >> 21;
  atomicAdd(&s_hist[bin >> 1], 1u << ((bin & 1u) * 16));
}

template <int THREADS>
__device__ __forceinline__ void hist_flush(const uint32_t* s_hist, uint32_t* __restrict__ dst) {
  for (int i = threadIdx.x; i < kHistWords; i += THREADS) {
    const uint32_t w = s_hist[i];
    if (w & 0xffffu) atomicAdd(&dst[2 * i], w & 0xffffu);
    if (w >> 16) atomicAdd(&dst[2 * i + 1], w >> 16);
  }
}

// ROT: blocks 0 .. kQrotBlocks-1 of a unit rotate its queries and append its new row, the others
// score; no histograms.  (klo: the block that scores the appended row writes it first.)
template <typename T, int LPR, int G, bool GROUP_MAX, bool ROT>
__global__ __launch_bounds__(256) void score_kernel(
    const typename T::store_t* klo, const float* __restrict__ qhat,
    float* __restrict__ scores, int Hkv, int S_max, int S_cap, int d, int rows_per_block,
    Ragged rg, Paging pg, uint32_t* __restrict__ hist_part, int hist_chunks, RotArgs ra) {
  constexpr int EPC = T::EPC;
  constexpr int kPasses = (LPR * EPC < kD ? LPR * EPC + kQrotCols - 1 : kD) / kQrotCols;  // of 32 columns
  __shared__ __align__(16) RotSmem<T, ROT ? G : 1> s_rot;
  __shared__ __align__(16) float s_qhat[ROT ? G : 1][ROT ? kPasses * kQrotCols : 1];
  int chunk = blockIdx.x;
  if constexpr (ROT) {
    if (blockIdx.x < kQrotBlocks) {
      zero_tickets(ra);
      if (ra.ap.k_new != nullptr) qrot_block<T, G, true>(s_rot, ra, blockIdx.y, blockIdx.x, Hkv, S_max, S_cap, d, rg, pg, d);
      else qrot_block<T, G, false>(s_rot, ra, blockIdx.y, blockIdx.x, Hkv, S_max, S_cap, d, rg, pg, d);
      return;
    }
    chunk -= kQrotBlocks;
  }
  constexpr int kSelHeads = GROUP_MAX ? 1 : G;  // selecting heads whose scores the block writes
  extern __shared__ uint32_t s_hist[];          // [kSelHeads][kHistWords] when hist_part is given
  const int tid = threadIdx.x;
  const int unit = blockIdx.y;
  const int S = seq_rows(rg, unit / Hkv, S_max);  // the score buffer keeps the stride S_max
  if (chunk * rows_per_block >= S) return;
  const int head0 = unit * G;  // first query head of the group, flattened over batch
  const bool hist = !ROT && hist_part != nullptr;
  if (hist) {
    for (int i = tid; i < kSelHeads * kHistWords; i += 256) s_hist[i] = 0u;
    __syncthreads();
  }

  const int lane = tid & 63;
  const int c = lane % LPR;
  const int nch = d / EPC;  // 16-byte chunks per slab row, <= LPR
  const bool cact = c < nch;
  const size_t row_bytes = (size_t)d * T::kBytes;
  const int row0 = chunk * rows_per_block;
  const int row_end = min(S, row0 + rows_per_block);
  // the block's rows are consecutive in memory (a paged cache: the host keeps a block inside a page)
  const long long row_shift =
      cache_row(pg, unit / Hkv / max(rg.queries, 1), unit % Hkv, Hkv, S_cap, row0) - row0;
  const char* base = reinterpret_cast<const char*>(klo) + row_shift * (long long)row_bytes +
                     (size_t)(cact ? c : 0) * 16;
  const ContiguousRows rows{base, row_bytes};
  // two trips of eight loads per lane in flight (LPR <= 8), refilled as they are consumed
  constexpr bool kPipelined = LPR <= 8;
  ScoreTrip<kPipelined ? LPR : 8> t0, t1;
  auto prefetch = [&]() {
    if constexpr (kPipelined) {
      const int tile0 = row0 + (tid >> 6) * 64;
      score_load_trip<LPR, 4>(rows, tile0, row_end, t0);
      score_load_trip<LPR, 4>(rows, tile0 + 4 * 64 * ScoreTrip<LPR>::TPI, row_end, t1);
    }
  };
  float qr[G][EPC];
  if constexpr (ROT) {
    if (score_block_rotate<T, G, kPasses>(s_rot, s_qhat, ra, unit, Hkv, S, S_cap, d, row0, row_end, pg, prefetch))
      prefetch();  // the block has just written row S - 1
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int e = 0; e < EPC; ++e) qr[g][e] = cact ? s_qhat[g][c * EPC + e] : 0.f;
  } else {
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int e = 0; e < EPC; ++e)
        qr[g][e] = cact ? qhat[(size_t)(head0 + g) * kD + c * EPC + e] : 0.f;
    prefetch();
  }
  auto emit = [&](int row, const float (&sc)[G]) {
    if constexpr (GROUP_MAX) {
      float m = sc[0];
#pragma unroll
      for (int g = 1; g < G; ++g) m = fmaxf(m, sc[g]);
      scores[(size_t)unit * S_max + row] = m;
      if (hist) hist_count(s_hist, m);
    } else {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        scores[(size_t)(head0 + g) * S_max + row] = sc[g];
        if (hist) hist_count(s_hist + g * kHistWords, sc[g]);
      }
    }
  };
  if constexpr (kPipelined)
    score_rows_pipelined<T, LPR, G, 4>(rows, qr, row0, row_end, t0, t1, emit);
  else
    score_rows<T, LPR, G, 4>(rows, cact, qr, row0, row_end, emit);
  if (hist) {
    __syncthreads();
    const size_t sel0 = GROUP_MAX ? (size_t)unit : (size_t)head0;
#pragma unroll
    for (int g = 0; g < kSelHeads; ++g)
      hist_flush<256>(s_hist + g * kHistWords,
                      hist_part + ((sel0 + g) * hist_chunks + row0 / kHistChunk) * 2048);
  }
}

// ---- matrix-core variant for grouped queries on a bf16 cache ----------------------------------
// With G > 1 query heads per KV head the scoring step is a small dense contraction per row tile,
// scores[s, g] = sum_j Klo[s, j] qhat[g, j], and the per-byte vector work of the kernel above
// grows with G until it, not HBM, sets the pace.  The tile loop is score_mfma_rows
// (score_mfma_impl.h); this kernel decides which heads form the 16 columns and where their
// scores go.
//
// NCH = 16-byte chunks per slab row (d = 8 * NCH).
// TILE: several new tokens per sequence (rg.queries = m > 1).  The m G query heads that read one
// KV head's slab form the 16 columns of the B operand, 16 / G tokens per block (blockIdx.z picks
// the tile of tokens, blockIdx.y the sequence and KV head), so the slab is read once per tile
// instead of once per token: [m G, d] x [d, S] as one contraction.  Token j only has scores for
// the rows of its own causal length; the block covers the longest length of its tile.
// ROT: as in score_kernel.
template <int NCH, int G, bool GROUP_MAX, bool TILE, bool ROT>
__global__ __launch_bounds__(256) void score_mfma_kernel(
    const uint16_t* klo, const float* __restrict__ qhat, float* __restrict__ scores,
    int Hkv, int S_max, int S_cap, int rows_per_block, Ragged rg, Paging pg,
    uint32_t* __restrict__ hist_part, int hist_chunks, RotArgs ra) {
  static_assert(!(TILE && ROT), "several tokens per sequence append in a launch of their own");
  constexpr int kPasses = (8 * NCH + kQrotCols - 1) / kQrotCols;
  __shared__ __align__(16) RotSmem<BF16, ROT ? G : 1> s_rot;
  __shared__ __align__(16) float s_qhat[ROT ? G : 1][ROT ? kPasses * kQrotCols : 1];
  int chunk = blockIdx.x;
  if constexpr (ROT) {
    if (blockIdx.x < kQrotBlocks) {
      zero_tickets(ra);
      if (ra.ap.k_new != nullptr)
        qrot_block<BF16, G, true>(s_rot, ra, blockIdx.y, blockIdx.x, Hkv, S_max, S_cap, 8 * NCH, rg, pg, 8 * NCH);
      else
        qrot_block<BF16, G, false>(s_rot, ra, blockIdx.y, blockIdx.x, Hkv, S_max, S_cap, 8 * NCH, rg, pg, 8 * NCH);
      return;
    }
    chunk -= kQrotBlocks;
  }
  constexpr int kSelHeads = GROUP_MAX ? 1 : G;  // (histograms: one token per sequence only)
  extern __shared__ uint32_t s_hist[];          // [kSelHeads][kHistWords] when hist_part is given
  const int lane = threadIdx.x & 63;
  const int r16 = lane & 15;

  // column r16 of the tile: which query head it is, where its scores go, how many rows it sees
  int S;            // rows the block scores up to (uniform)
  int S_lane;       // rows head r16 has scores for
  bool head_ok;
  size_t head;      // row of qhat
  size_t score_row; // row of the score buffer
  int cache_b, hkv;
  if constexpr (TILE) {
    constexpr int QPT = 16 / G;  // tokens per tile
    const int m = rg.queries;
    const int bs = (int)blockIdx.y / Hkv, j0 = (int)blockIdx.z * QPT;
    hkv = (int)blockIdx.y % Hkv;
    cache_b = bs;
    const int j = j0 + r16 / G;
    head_ok = j < m;
    const int entry = bs * m + min(j, m - 1);
    head = ((size_t)entry * Hkv + hkv) * G + r16 % G;
    score_row = GROUP_MAX ? (size_t)entry * Hkv + hkv : head;
    S_lane = seq_rows(rg, entry, S_max);
    S = 0;
    for (int jj = j0; jj < min(j0 + QPT, m); ++jj) S = max(S, seq_rows(rg, bs * m + jj, S_max));
  } else {
    const int unit = blockIdx.y;
    hkv = unit % Hkv;
    cache_b = unit / Hkv;
    head_ok = r16 < G;
    head = (size_t)unit * G + (head_ok ? r16 : 0);
    score_row = GROUP_MAX ? (size_t)unit : head;
    S = S_lane = seq_rows(rg, cache_b, S_max);  // the score buffer keeps the stride S_max
  }
  if (chunk * rows_per_block >= S) return;
  const bool hist = !TILE && !ROT && hist_part != nullptr;
  if (hist) {
    for (int i = threadIdx.x; i < kSelHeads * kHistWords; i += 256) s_hist[i] = 0u;
    __syncthreads();
  }

  // (ahead of the slab addresses: behind them the kernel holds 100 registers in place of 96 at NCH
  // = 16, four waves per SIMD in place of five: 64 sequences of 8 KV heads, S = 8192, 207 / 198 us)
  bf16x8_t bq[ScoreMfmaGeom<NCH>::NB][3];
  if constexpr (!ROT) score_mfma_operands<NCH>(qhat + head * kD, head_ok, bq);

  const int row0 = chunk * rows_per_block;
  const int row_end = min(S, row0 + rows_per_block);
  // the block's rows are consecutive in memory (a paged cache: the host keeps a block inside a page)
  const long long row_shift = cache_row(pg, cache_b, hkv, Hkv, S_cap, row0) - row0;
  const int lane_end = min(row_end, S_lane);
  const char* slab = reinterpret_cast<const char*>(klo) + row_shift * (long long)(NCH * 16);
  const bool vec_ok = (S_max & 3) == 0;
  ScoreMfmaBufs<NCH, 8> bufs;
  const ContiguousRows slab_rows = score_mfma_contiguous<NCH>(slab);
  auto prefetch = [&]() { score_mfma_prefetch<NCH, 4, 8>(slab_rows, row0, row_end, bufs); };
  if constexpr (ROT) {
    if (score_block_rotate<BF16, G, kPasses>(s_rot, s_qhat, ra, blockIdx.y, Hkv, S, S_cap, 8 * NCH, row0, row_end, pg,
                                             prefetch))
      prefetch();  // the block has just written row S - 1
    score_mfma_operands<NCH>(s_qhat[head_ok ? r16 : 0], head_ok, bq);
  } else {
    prefetch();
  }
  if constexpr (GROUP_MAX && !TILE) {
    // One score per row, the maximum over the group: qhat is the A operand and the row tile the
    // B operand, so a lane holds one row and four heads in its registers and the maximum needs
    // no exchange between lanes but one, which also puts the results of two tiles side by side:
    // thirty-two lanes store the rows of two tiles.
    const int kgrp = lane >> 4;
    score_mfma_rows<NCH, 4, 8, true>(
        slab_rows, row0, row_end, bq, bufs,
        [&](int rowbase_a, const f32x4_t& acc_a, int rowbase_b, const f32x4_t& acc_b) {
          // lanes 0-15: the group maximum of tile a's rows, lanes 16-31: of tile b's
          const float m = group_max_pair<G>(acc_a, acc_b);
          const int row = (kgrp == 0 ? rowbase_a : rowbase_b) + r16;
          if (kgrp < 2 && row < lane_end) {
            scores[score_row * S_max + row] = m;
            if (hist) hist_count(s_hist, m);
          }
        });
  } else {
  score_mfma_rows<NCH, 4, 8>(slab_rows, row0, row_end, bq, bufs, [&](int rowbase, const f32x4_t& acc) {
    float v[4] = {acc[0], acc[1], acc[2], acc[3]};
    bool writer = head_ok;
    if constexpr (GROUP_MAX) {
      // the G heads of one token sit in G consecutive lanes
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = group_allreduce_max<G>(head_ok ? v[i] : -3.0e38f);
      writer = head_ok && (r16 % G == 0);
    }
    float* dst = scores + score_row * S_max + rowbase;
    if (writer && rowbase < lane_end) {
      if (vec_ok && rowbase + 3 < lane_end) {
        *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (rowbase + i < lane_end) dst[i] = v[i];
      }
      if (hist) {
        uint32_t* mine = s_hist + (GROUP_MAX ? 0 : r16) * kHistWords;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (rowbase + i < lane_end) hist_count(mine, v[i]);
      }
    }
  });
  }
  if (hist) {
    __syncthreads();
    const size_t sel0 = GROUP_MAX ? (size_t)blockIdx.y : (size_t)blockIdx.y * G;
#pragma unroll
    for (int g = 0; g < kSelHeads; ++g)
      hist_flush<256>(s_hist + g * kHistWords,
                      hist_part + ((sel0 + g) * hist_chunks + row0 / kHistChunk) * 2048);
  }
}

// tokens of one sequence that share a score block (TILE), and the blocks along z that takes
static int score_tile_tokens(const Shape& s) { return 16 / s.G; }

// rot: the launch rotates the queries too (ROT); null: qhat is there.
template <int NCH, int G, bool TILE, bool ROT>
static hipError_t launch_score_mfma_r(const Shape& s, int select_mode, const void* klo, float* scores,
                                      const float* qhat, uint32_t* hist_part, int hist_chunks, const RotArgs& rot,
                                      hipStream_t st) {
  const int m = TILE ? s.rg.queries : 1;
  const int nz = TILE ? (m + score_tile_tokens(s) - 1) / score_tile_tokens(s) : 1;
  Shape blocks = s;  // the grid's y*z extent stands in for the batch when the row block is sized
  blocks.B = s.B / m * nz;
  const int rpb = score_rows_per_block(blocks);
  dim3 grid((s.S + rpb - 1) / rpb + (ROT ? kQrotBlocks : 0), s.B / m * s.Hkv, nz);
  if (TILE) hist_part = nullptr;  // (several tokens per sequence keep the separate counting pass)
  if (select_mode == 1 && G > 1) {
    hipLaunchKernelGGL((score_mfma_kernel<NCH, G, (G > 1), TILE, ROT>), grid, dim3(256),
                       hist_part ? kHistWords * 4 : 0, st, static_cast<const uint16_t*>(klo), qhat,
                       scores, s.Hkv, s.S, s.S_cap, rpb, s.rg, s.pg, hist_part, hist_chunks, rot);
  } else {
    hipLaunchKernelGGL((score_mfma_kernel<NCH, G, false, TILE, ROT>), grid, dim3(256),
                       hist_part ? G * kHistWords * 4 : 0, st, static_cast<const uint16_t*>(klo), qhat,
                       scores, s.Hkv, s.S, s.S_cap, rpb, s.rg, s.pg, hist_part, hist_chunks, rot);
  }
  return hipGetLastError();
}

template <int NCH, int G, bool TILE>
static hipError_t launch_score_mfma_g(const Shape& s, int select_mode, const void* klo, float* scores,
                                      const float* qhat, uint32_t* hist_part, int hist_chunks, const RotArgs* rot,
                                      hipStream_t st) {
  if constexpr (!TILE)
    if (rot != nullptr)
      return launch_score_mfma_r<NCH, G, false, true>(s, select_mode, klo, scores, qhat, nullptr, 0, *rot, st);
  return launch_score_mfma_r<NCH, G, TILE, false>(s, select_mode, klo, scores, qhat, hist_part, hist_chunks, RotArgs{}, st);
}

template <int NCH>
static hipError_t launch_score_mfma_n(const Shape& s, int select_mode, const void* klo, float* scores,
                                      const float* qhat, uint32_t* hist_part, int hist_chunks, const RotArgs* rot,
                                      hipStream_t st) {
  if (s.rg.queries > 1) {
    switch (s.G) {
      case 1: return launch_score_mfma_g<NCH, 1, true>(s, select_mode, klo, scores, qhat, hist_part, hist_chunks, rot, st);
      case 2: return launch_score_mfma_g<NCH, 2, true>(s, select_mode, klo, scores, qhat, hist_part, hist_chunks, rot, st);
      case 4: return launch_score_mfma_g<NCH, 4, true>(s, select_mode, klo, scores, qhat, hist_part, hist_chunks, rot, st);
      case 8: return launch_score_mfma_g<NCH, 8, true>(s, select_mode, klo, scores, qhat, hist_part, hist_chunks, rot, st);
      default: return hipErrorInvalidValue;
    }
  }
  switch (s.G) {
    case 2: return launch_score_mfma_g<NCH, 2, false>(s, select_mode, klo, scores, qhat, hist_part, hist_chunks, rot, st);
    case 4: return launch_score_mfma_g<NCH, 4, false>(s, select_mode, klo, scores, qhat, hist_part, hist_chunks, rot, st);
    case 8: return launch_score_mfma_g<NCH, 8, false>(s, select_mode, klo, scores, qhat, hist_part, hist_chunks, rot, st);
    default: return hipErrorInvalidValue;
  }
}

// bf16 cache, a power-of-two number of chunks per slab row, and at least two query heads that
// share a slab: 2..8 per KV head, or several new tokens per sequence.  With rows of 16 or 32
// bytes (d <= 16) a matrix instruction is spent on very few bytes and the vector kernel is the
// faster one when every head's score is written (d = 16, 4 heads per KV head, S = 131072: 39
// against 44 us; d = 8: 12 against 33 us); with one selection per group, where the tiles are
// finished in pairs in registers, 32-byte rows are level or slightly ahead (35 against 36 us).
static bool score_mfma_applies(const Shape& s, int select_mode) {
  const int nch = s.d / 8;
  const bool tile = s.rg.queries > 1;
  const bool shared = (s.G >= 2 || tile) && s.G <= 8;
  const bool wide_enough = nch > 2 || tile || (nch == 2 && select_mode == 1);
  return s.dtype == 1 && shared && s.d % 8 == 0 && (nch & (nch - 1)) == 0 && wide_enough;
}

static hipError_t launch_score_mfma(const Shape& s, int select_mode, const void* klo, float* scores,
                                    const float* qhat, uint32_t* hist_part, int hist_chunks, const RotArgs* rot,
                                    hipStream_t st) {
  switch (s.d / 8) {
    case 1: return launch_score_mfma_n<1>(s, select_mode, klo, scores, qhat, hist_part, hist_chunks, rot, st);
    case 2: return launch_score_mfma_n<2>(s, select_mode, klo, scores, qhat, hist_part, hist_chunks, rot, st);
    case 4: return launch_score_mfma_n<4>(s, select_mode, klo, scores, qhat, hist_part, hist_chunks, rot, st);
    case 8: return launch_score_mfma_n<8>(s, select_mode, klo, scores, qhat, hist_part, hist_chunks, rot, st);
    case 16: return launch_score_mfma_n<16>(s, select_mode, klo, scores, qhat, hist_part, hist_chunks, rot, st);
    default: return hipErrorInvalidValue;
  }
}

template <typename T, int LPR, int G, bool GM>
static hipError_t launch_score_r(const Shape& s, const void* klo, float* scores, const float* qhat, uint32_t* hist_part,
                                 int hist_chunks, const RotArgs* rot, hipStream_t st) {
  using ST = typename T::store_t;
  const int rpb = score_rows_per_block(s);
  const int chunks = (s.S + rpb - 1) / rpb, units = s.B * s.Hkv;
  if (rot != nullptr) {
    if constexpr (LPR <= 16)  // (rotate_score_applies)
      hipLaunchKernelGGL((score_kernel<T, LPR, G, GM, true>), dim3(chunks + kQrotBlocks, units), dim3(256), 0, st,
                         static_cast<const ST*>(klo), qhat, scores, s.Hkv, s.S, s.S_cap, s.d, rpb, s.rg, s.pg, nullptr, 0, *rot);
    else
      return hipErrorInvalidValue;
  } else {
    if (s.rg.queries > 1) hist_part = nullptr;  // (several tokens per sequence keep the separate counting pass)
    hipLaunchKernelGGL((score_kernel<T, LPR, G, GM, false>), dim3(chunks, units), dim3(256),
                       hist_part ? (GM ? 1 : G) * kHistWords * 4 : 0, st, static_cast<const ST*>(klo), qhat, scores,
                       s.Hkv, s.S, s.S_cap, s.d, rpb, s.rg, s.pg, hist_part, hist_chunks, RotArgs{});
  }
  return hipGetLastError();
}

template <typename T, int LPR, int G>
static hipError_t launch_score_g(const Shape& s, int select_mode, const void* klo, float* scores, const float* qhat,
                                 uint32_t* hist_part, int hist_chunks, const RotArgs* rot, hipStream_t st) {
  if (select_mode == 1 && G > 1)
    return launch_score_r<T, LPR, G, (G > 1)>(s, klo, scores, qhat, hist_part, hist_chunks, rot, st);
  return launch_score_r<T, LPR, G, false>(s, klo, scores, qhat, hist_part, hist_chunks, rot, st);
}

template <typename T, int LPR>
static hipError_t launch_score_l(const Shape& s, int select_mode, const void* klo, float* scores, const float* qhat,
                                 uint32_t* hist_part, int hist_chunks, const RotArgs* rot, hipStream_t st) {
  switch (s.G) {
    case 1: return launch_score_g<T, LPR, 1>(s, select_mode, klo, scores, qhat, hist_part, hist_chunks, rot, st);
    case 2: return launch_score_g<T, LPR, 2>(s, select_mode, klo, scores, qhat, hist_part, hist_chunks, rot, st);
    case 4: return launch_score_g<T, LPR, 4>(s, select_mode, klo, scores, qhat, hist_part, hist_chunks, rot, st);
    case 8: return launch_score_g<T, LPR, 8>(s, select_mode, klo, scores, qhat, hist_part, hist_chunks, rot, st);
    default: return hipErrorInvalidValue;
  }
}

template <typename T>
static hipError_t launch_score_t(const Shape& s, int select_mode, const void* klo, float* scores, const float* qhat,
                                 uint32_t* hist_part, int hist_chunks, const RotArgs* rot, hipStream_t st) {
  const int nch = s.d / T::EPC;
  int lpr = 1;
  while (lpr < nch) lpr <<= 1;
#define LOKI_SCORE(L) return launch_score_l<T, L>(s, select_mode, klo, scores, qhat, hist_part, hist_chunks, rot, st)
  switch (lpr) {
    case 1: LOKI_SCORE(1);
    case 2: LOKI_SCORE(2);
    case 4: LOKI_SCORE(4);
    case 8: LOKI_SCORE(8);
    case 16: LOKI_SCORE(16);
    case 32:
      if constexpr (T::EPC == 4) LOKI_SCORE(32);
      return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
#undef LOKI_SCORE
}

template <typename T, bool APPEND>
static hipError_t launch_qrot_t(const Shape& s, const RotArgs& ra, hipStream_t st) {
  const dim3 grid(s.B * s.Hkv, kQrotBlocks), block(256);
#define LOKI_QROT(GV)                                                                                      \
  hipLaunchKernelGGL((qrot_kernel<T, GV, APPEND>), grid, block, 0, st, ra, s.Hkv, s.S, s.S_cap, s.d, s.rg, s.pg); \
  break
  switch (s.G) {
    case 1: LOKI_QROT(1);
    case 2: LOKI_QROT(2);
    case 4: LOKI_QROT(4);
    case 8: LOKI_QROT(8);
    default: return hipErrorInvalidValue;
  }
#undef LOKI_QROT
  return hipGetLastError();
}

hipError_t launch_qrot(const Shape& s, const void* q, const float* P, float* qhat, void* klo,
                       void* khi, void* v, uint32_t* zero_words, size_t n_zero, hipStream_t st) {
  const RotArgs ra{q, P, qhat, klo, khi, v, s.ap, zero_words, n_zero};
  if (s.ap.k_new != nullptr) return s.dtype == 0 ? launch_qrot_t<F32, true>(s, ra, st) : launch_qrot_t<BF16, true>(s, ra, st);
  return s.dtype == 0 ? launch_qrot_t<F32, false>(s, ra, st) : launch_qrot_t<BF16, false>(s, ra, st);
}

static hipError_t launch_score_any(const Shape& s, int select_mode, const void* klo, float* scores, const float* qhat,
                                   uint32_t* hist_part, int hist_chunks, const RotArgs* rot, hipStream_t st) {
  if (score_mfma_applies(s, select_mode))
    return launch_score_mfma(s, select_mode, klo, scores, qhat, hist_part, hist_chunks, rot, st);
  return s.dtype == 0 ? launch_score_t<F32>(s, select_mode, klo, scores, qhat, hist_part, hist_chunks, rot, st)
                      : launch_score_t<BF16>(s, select_mode, klo, scores, qhat, hist_part, hist_chunks, rot, st);
}

hipError_t launch_score(const Shape& s, int select_mode, const void* klo, float* scores, const float* qhat,
                        uint32_t* hist_part, int hist_chunks, hipStream_t st) {
  return launch_score_any(s, select_mode, klo, scores, qhat, hist_part, hist_chunks, nullptr, st);
}

// Rotation inside the scoring, or a launch in front of it?  It saves that launch, about 3 us, and
// costs every score block a rotation of its own, of all G heads of the group, and the score kernel
// the registers that hold a pass's P_h across the first slab loads (matrix cores, waves per SIMD
// without / with: d = 32 7 / 4, d = 64 6 / 3, d = 128 4 / 2).  So it is taken while all blocks are
// soon resident: at most 18 per CU, where a unit's four rotating blocks count as eight (each reads
// a quarter of P_h and stores qhat), and everything counts twice at 64 columns (two passes) and
// eight times beyond; on the vector units twice again with several heads per KV head, but no more
// than twice for bf16 rows of over 64 columns, which hold no slab loads in flight.  fp32 rows of
// over 64 columns spill in this form: never.
// One launch / two, us per step, both with the same stages behind them (1287 shapes, 8 to 4096
// heads, S = 500 to 131072): 32 units, S = 4096, k = 512, d = 32 18.4 / 20.2 (fp32, contiguous),
// 19.6 / 20.5 (bf16, paged); 4 sequences of 32/8 heads, S = 131072, d = 16 206.9 / 210.0; 512
// units, S = 12000, d = 32 271 / 247; 64 sequences of 64/8 heads, S = 8192, d = 64, every head
// selecting for itself, k = 512 377 / 317, k = 1024 438 / 380, k = 2048 545 / 488 (the scoring
// alone 209 / 142); of 32/8 heads, S = 4096, d = 48, one selection per group 149 / 115; 16 of 32/8,
// S = 4096, fp32, d = 128 99 / 87.
bool rotate_score_applies(const Shape& s, int select_mode) {
  if (s.rg.queries > 1) return false;
  const int rpb = score_rows_per_block(s), passes = (s.d + kQrotCols - 1) / kQrotCols;
  const long long units = (long long)s.B * s.Hkv, blocks = (long long)((s.S + rpb - 1) / rpb) * units;
  int weight = passes > 2 ? 8 : passes;
  if (!score_mfma_applies(s, select_mode)) {
    if (s.d * s.elem_bytes > 256) return false;
    if (s.dtype == 1 && passes > 2) weight = 2;
    else if (s.G > 1) weight *= 2;
  }
  return (blocks + 8 * units) * weight <= 18LL * device_cus();
}

hipError_t launch_rotate_score(const Shape& s, int select_mode, const void* q, const float* P, void* klo, void* khi, void* v,
                               float* scores, float* qhat, uint32_t* zero_words, size_t n_zero, hipStream_t st) {
  if (!rotate_score_applies(s, select_mode)) return hipErrorInvalidValue;
  const RotArgs ra{q, P, qhat, klo, khi, v, s.ap, zero_words, n_zero};
  return launch_score_any(s, select_mode, klo, scores, qhat, nullptr, 0, &ra, st);
}

}  // namespace loki
