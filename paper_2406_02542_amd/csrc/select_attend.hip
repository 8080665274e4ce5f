// Top-k selection and exact attention over the selected rows in one launch (Algorithm 1 lines 6-9
// of arXiv 2406.02542), for score rows short enough to be selected by one block (S <= 16384): the
// last kernel of the split path, behind the query rotation and the scoring, where its blocks are not too
// many (select_attend_applies); else select.hip and attend.hip follow each other.
//
// Block (split, head): the block makes the whole selection of its head for itself, from the scores
// the launch before left in L2, and attends over its share of the list, which never leaves LDS.
// With several splits per head the selection is repeated by each of their blocks: it is a chain of
// barriers and LDS round trips that costs a head the same few microseconds whoever runs it, while
// a launch of its own costs those and a launch, and the list written and read back.  Against the two
// launches, us per step: one sequence of 32 heads, S = 4096, k = 1024, 23.1 -> 20.4; of 32/8 heads,
// S = 8192, k = 1024, 26.7 -> 25.0; 16 of 32/8 heads, S = 12345, per-head selection 123.8 -> 118.3 (there
// a block's selection also runs beside its neighbour's row loads).
#include "attend_mfma_impl.h"
#include "select_impl.h"

namespace loki {

constexpr int kSaThreads = 512;
constexpr int kSaWaves = kSaThreads / 64;

// What both kernels are given beside their operands.
struct SelectAttendArgs {
  const float* scores;   // [selecting heads][S_max]
  int32_t* user_idx;     // [selecting heads][k_max] or null: the caller's copy of the lists
  float* partial;        // [B*Hq][nsplit][130] when nsplit > 1
  int32_t* tickets;      // [selecting heads], zeroed
  int Hkv, G, S_max, S_cap, d, k_max, nsplit, per_thread;
  int xcd_group_blocks, xcd_sets;  // see attend.hip (0: launch order as is)
  Ragged rg;
  Paging pg;
};

// The selection of score row `sel` for batch entry b, entries [r0, r1) of it into s_idx (as rows of
// the cache unit, or of the pool when the cache is paged) and, with s_a, their scores.  Ends with a
// barrier.
template <int KPT>
__device__ __forceinline__ void select_share(const SelectAttendArgs& a, int sel, int b, int hkv, int S, int k, int r0,
                                             int r1, bool write_user, ResidentSelectSmem<kSaThreads>& sm,
                                             int32_t* s_idx, float* s_a) {
  int32_t* user = write_user && a.user_idx != nullptr ? a.user_idx + (size_t)sel * a.k_max : nullptr;
  if (user)
    for (int i = k + (int)threadIdx.x; i < a.k_max; i += kSaThreads) user[i] = -1;  // a sequence keeping fewer rows
  // a paged cache: the pages of the sequence's rows, clamped into the pool
  __shared__ int32_t s_pages[kSaThreads * KPT / 256];
  const bool paged = a.pg.table != nullptr;
  if (paged && (int)threadIdx.x <= (S - 1) >> a.pg.lg_rows) {
    const int32_t* table = a.pg.table + (size_t)(b / max(a.rg.queries, 1)) * a.pg.pages_per_seq;
    s_pages[threadIdx.x] = min(max(table[threadIdx.x], 0), a.pg.n_pages - 1);
  }
  resident_select_clear<kSaThreads>(sm);
  __syncthreads();
  block_select_topk_resident<kSaThreads, KPT>(
      a.scores + (size_t)sel * a.S_max, S, k, a.per_thread, sm, [&](int rank, int pos, float score) {
        if (user) user[rank] = pos;
        if (rank >= r0 && rank < r1) {
          const int lg = a.pg.lg_rows;
          s_idx[rank - r0] = paged ? ((s_pages[pos >> lg] * a.Hkv + hkv) << lg) | (pos & ((1 << lg) - 1)) : pos;
          if (s_a) s_a[rank - r0] = score;
        }
      });
  __syncthreads();
}

// The same selection in two parts, so that the attention can begin in between (GROWING): begin()
// leaves the entries that are certain, below the value returned; complete() appends the chosen
// candidates, ranked by the first wave while every wave has its first rows' loads in flight, and
// writes the caller's ascending copy.  The list is two ascending runs, or one where the bin held
// too many candidates.
template <int KPT>
struct SelectShare {
  RunKeys<KPT> keys;
  RunSelect rs;
  int32_t* user;
  bool ordered;

  __device__ __forceinline__ int32_t row_of(const SelectAttendArgs& a, int hkv, const int32_t* s_pages, int pos) const {
    const int lg = a.pg.lg_rows;
    return a.pg.table != nullptr ? ((s_pages[pos >> lg] * a.Hkv + hkv) << lg) | (pos & ((1 << lg) - 1)) : pos;
  }

  __device__ __forceinline__ int begin(const SelectAttendArgs& a, int sel, int b, int hkv, int S, int k, int r0, int r1,
                                       bool write_user, ResidentSelectSmem<kSaThreads>& sm, int32_t* s_pages, int32_t* s_idx,
                                       float* s_a) {
    run_load_keys<KPT>(a.scores + (size_t)sel * a.S_max, S, a.per_thread, keys);
    user = write_user && a.user_idx != nullptr ? a.user_idx + (size_t)sel * a.k_max : nullptr;
    if (user)
      for (int i = k + (int)threadIdx.x; i < a.k_max; i += kSaThreads) user[i] = -1;  // a sequence keeping fewer rows
    // a paged cache: the pages of the sequence's rows, clamped into the pool
    if (a.pg.table != nullptr && (int)threadIdx.x <= (S - 1) >> a.pg.lg_rows) {
      const int32_t* table = a.pg.table + (size_t)(b / max(a.rg.queries, 1)) * a.pg.pages_per_seq;
      s_pages[threadIdx.x] = min(max(table[threadIdx.x], 0), a.pg.n_pages - 1);
    }
    resident_select_clear<kSaThreads>(sm);
    __syncthreads();
    LOKI_STAMP(1);
    rs = run_select_certain<kSaThreads, KPT>(keys, k, sm, [&](int rank, int pos, uint32_t key) {
      if (rank >= r0 && rank < r1) {
        s_idx[rank - r0] = row_of(a, hkv, s_pages, pos);
        if (s_a) s_a[rank - r0] = key_to_float(key);
      }
    });
    LOKI_STAMP(12);
    ordered = rs.n_cand == 0;
    return ordered ? 0 : rs.n_def;
  }

  __device__ __forceinline__ void complete(const SelectAttendArgs& a, int hkv, int r0, int r1, ResidentSelectSmem<kSaThreads>& sm,
                                           const int32_t* s_pages, int32_t* s_idx, float* s_a) {
    __shared__ WaveThreshold s_t;
    auto put = [&](int rank, int pos, uint32_t key) {
      if (rank >= r0 && rank < r1) {
        s_idx[rank - r0] = row_of(a, hkv, s_pages, pos);
        if (s_a) s_a[rank - r0] = key_to_float(key);
      }
    };
    if (threadIdx.x < 64) {
      const WaveThreshold t = run_threshold<kSaThreads>(rs, sm);
      if (threadIdx.x == 0) s_t = t;
      if (!ordered)
        wave_choose(sm.hist[1], rs.n_cand, WaveThreshold{t.T - (rs.bin << 21), t.need_eq}, 0u, [&](int rank, int i) {
          put(rs.n_def + rank, (int)sm.hist[1][kRunCand + i], (rs.bin << 21) | sm.hist[1][i]);
        });
    }
    __syncthreads();
    if (ordered || user) {  // (uniform)
      run_emit<kSaThreads, KPT>(keys, s_t, sm, [&](int rank, int pos, uint32_t key) {
        if (user) user[rank] = pos;
        if (ordered) put(rank, pos, key);
      });
      __syncthreads();
    }
    LOKI_STAMP(6);
  }
};

// The block's merged (max, sum, output) of NH heads: the result, or its part of it, merged by the
// block of the head group that finishes last (see splits_all_done).
template <typename T, int NH>
__device__ __forceinline__ void finish_share(const SelectAttendArgs& a, const MergeSmem<kSaWaves, NH>& sm, size_t head0,
                                             int sel, int split, typename T::store_t* out) {
  for (int i = threadIdx.x; i < NH * kD; i += kSaThreads) {
    const int g = i / kD, col = i % kD;
    float mn, ls, os;
    attend_merged<kSaWaves, NH>(sm, g, col, mn, ls, os);
    if (a.nsplit == 1) {
      T::store1(out + (head0 + g) * kD + col, os / ls);
    } else {
      float* pr = a.partial + ((head0 + g) * a.nsplit + split) * kPartialStride;
      store_shared_f32(pr + col, os, true);
      if (col == 0) {
        store_shared_f32(pr + kD, mn, true);
        store_shared_f32(pr + kD + 1, ls, true);
      }
    }
  }
  if (a.nsplit > 1 && splits_all_done(a.tickets + sel, a.nsplit))
    for (int i = threadIdx.x; i < NH * kD; i += kSaThreads) {
      const size_t head = head0 + i / kD;
      T::store1(out + head * kD + i % kD,
                combine_splits<true>(a.partial + head * a.nsplit * kPartialStride, a.nsplit, i % kD));
    }
}

// List entries of a block: equal shares of what the sequence keeps.
__device__ __forceinline__ void share_of(int k, int nsplit, int split, int& r0, int& r1) {
  const int n = (k + nsplit - 1) / nsplit;
  r0 = min(k, split * n);
  r1 = min(k, r0 + n);
}

// Vector form.  NH = query heads that share a selection; with one, the ranking score is the
// low-rank part of the logit and the slab is not read again (REUSE_LO).
// (Whether the rows are loaded past the caches, see row_loads, is known when the list is.)
template <typename T, int NH, int KPT, bool GROWING>
__global__ __launch_bounds__(kSaThreads, NH == 1 ? 4 : 2) void select_attend_kernel(
    const void* __restrict__ klo, const void* __restrict__ khi, const void* __restrict__ v,
    const float* __restrict__ qhat, typename T::store_t* __restrict__ out, SelectAttendArgs a) {
  constexpr bool REUSE_LO = NH == 1;
  constexpr int EPC = T::EPC;
  constexpr int LPRV = kD / EPC;
  constexpr int RPW = 64 / LPRV;
  __shared__ ResidentSelectSmem<kSaThreads> s_sel;
  __shared__ int32_t s_idx[kMaxGatherChunk];
  __shared__ float s_a[REUSE_LO ? kMaxGatherChunk : 1];
  __shared__ MergeSmem<kSaWaves, NH> s_merge;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = lane % LPRV, rg = lane / LPRV;
  // query heads that read the same cached KV head stay on one XCD, next to each other (attend.hip)
  int split = blockIdx.x, sel = blockIdx.y;
  if (a.xcd_group_blocks > 0) {
    const int n = sel * a.nsplit + split;
    const int j = n >> 3, set = (j / a.xcd_group_blocks) * 8 + (n & 7), m = j % a.xcd_group_blocks;
    if (set >= a.xcd_sets) return;  // uniform for the block, before any barrier
    const int member = m / a.nsplit;  // (token, head of the group)
    const int seq = set / a.Hkv, tokens = max(a.rg.queries, 1);
    sel = ((seq * tokens + member / a.G) * a.Hkv + set % a.Hkv) * a.G + member % a.G;
    split = m % a.nsplit;
  }
  const size_t head0 = (size_t)sel * NH;
  const int Hq = a.Hkv * a.G;
  const int b = (int)(head0 / Hq), hkv = (int)(head0 % Hq) / a.G;
  const int S = seq_rows(a.rg, b, a.S_max), k = seq_keep(a.rg, b, a.k_max, S);
  int r0, r1;
  share_of(k, a.nsplit, split, r0, r1);
  const int form_now = form_of_launch(a.rg, a.S_max, a.k_max);

  float qr[NH][EPC];  // this lane's slice of the query vectors, on its way during the selection
#pragma unroll
  for (int g = 0; g < NH; ++g)
#pragma unroll
    for (int e = 0; e < EPC; ++e) qr[g][e] = qhat[(head0 + g) * kD + c * EPC + e];
  float* score = REUSE_LO ? s_a : nullptr;
  __shared__ int32_t s_pages[GROWING ? kSaThreads * KPT / 256 : 1];
  SelectShare<KPT> share;
  int there = 0;
  if constexpr (GROWING) there = share.begin(a, sel, b, hkv, S, k, r0, r1, split == 0, s_sel, s_pages, s_idx, score);
  else select_share<KPT>(a, sel, b, hkv, S, k, r0, r1, split == 0, s_sel, s_idx, score);

  const size_t unit = a.pg.table != nullptr ? (size_t)0 : (size_t)cache_unit(a.rg, b * a.Hkv + hkv, a.Hkv);
  const RowAddr ra = make_row_addr<T, REUSE_LO>(klo, khi, v, unit, a.S_cap, a.d, c);
  AttendAcc<T, NH> acc;
  acc.init();
  if constexpr (GROWING) {
    attend_growing<T, NH, kSaWaves * RPW, REUSE_LO>(
        acc, qr, ra, s_idx, s_a, wave * RPW + rg, r0, r1, there, form_now, [&]() __attribute__((always_inline)) {
          share.complete(a, hkv, r0, r1, s_sel, s_pages, s_idx, score);
        });
  } else {
    with_form<kPastCaches>(form_now, [&](auto form) __attribute__((always_inline)) {
      attend_rows<T, NH, kSaWaves * RPW, true, REUSE_LO, false, false, decltype(form)::value != kThroughCaches>(
          acc, qr, ra, s_idx, s_a, wave * RPW + rg, r0, r1);
    });
  }
  attend_publish<T, NH, kSaWaves>(acc, s_merge);
  finish_share<T, NH>(a, s_merge, head0, sel, split, out);
}

// Matrix-core form for 4 or 8 query heads that share a selection (bf16 caches, attend_mfma_impl.h).
template <int NH, int KPT, bool GROWING>
__global__ __launch_bounds__(kSaThreads, 2) void select_attend_mfma_kernel(
    const void* __restrict__ klo, const void* __restrict__ khi, const void* __restrict__ v,
    const float* __restrict__ qhat, uint16_t* __restrict__ out, SelectAttendArgs a) {
  __shared__ ResidentSelectSmem<kSaThreads> s_sel;
  __shared__ __align__(16) int32_t s_idx[kMaxGatherChunk];
  __shared__ __align__(16) MergeSmem<kSaWaves, NH> s_merge;

  const int lane = threadIdx.x & 63;
  const int r16 = lane & 15;
  const int split = blockIdx.x, unit = blockIdx.y;
  const size_t head0 = (size_t)unit * NH;
  const bool head_ok = r16 < NH;
  const int b = unit / a.Hkv;
  const int S = seq_rows(a.rg, b, a.S_max), k = seq_keep(a.rg, b, a.k_max, S);
  int r0, r1;
  share_of(k, a.nsplit, split, r0, r1);
  const int form_now = form_of_launch(a.rg, a.S_max, a.k_max);

  __shared__ int32_t s_pages[GROWING ? kSaThreads * KPT / 256 : 1];
  SelectShare<KPT> share;
  int there = 0;
  if constexpr (GROWING) there = share.begin(a, unit, b, unit % a.Hkv, S, k, r0, r1, split == 0, s_sel, s_pages, s_idx, nullptr);
  else select_share<KPT>(a, unit, b, unit % a.Hkv, S, k, r0, r1, split == 0, s_sel, s_idx, nullptr);

  am_bf16x8_t bq[4][2];
  am_query_operands<4, 2>(qhat + (head0 + (head_ok ? r16 : 0)) * kD, head_ok, kD, bq);
  const size_t addr_unit = a.pg.table != nullptr ? (size_t)0 : (size_t)cache_unit(a.rg, unit, a.Hkv);
  const AmAddr<4> ad = am_make_addr<4, false>(klo, khi, v, addr_unit, a.S_cap, a.d);
  AmState st;
  st.init();
  with_form<kPastCaches>(form_now, [&](auto form) __attribute__((always_inline)) {
    am_attend_rows<true, 4, 2, decltype(form)::value != kThroughCaches>(
        ad, bq, s_idx, r0, AmRoundRobin<kSaWaves>(r0, r1, there), st, [&]() __attribute__((always_inline)) {
          if constexpr (GROWING) share.complete(a, unit % a.Hkv, r0, r1, s_sel, s_pages, s_idx, nullptr);
        });
  });
  am_publish<NH, kSaWaves>(st, s_merge);
  finish_share<BF16, NH>(a, s_merge, head0, unit, split, out);
}

// ---- launchers ------------------------------------------------------------------------------------
static inline int div_up(int a, int b) { return (a + b - 1) / b; }

// Row splits: a block per CU, no more (a second one repeats the selection on a CU that is busy with
// it already: 4 tokens of 2 sequences, 32/8 heads, k = 1329 45.6 -> 30.2 us), each with two trips of its row
// loop (vector: 256 rows in bf16, 128 in fp32; against half as many, one sequence of 2 KV groups at
// k = 1341: 26.1 -> 23.6 us), on the matrix cores half a trip (128 rows; against 256, Llama-3 shape at
// batch 1: 24.3 -> 22.4 us).  Never more than the workspace has partials for (gather_splits).
static int select_attend_splits(const Shape& s, int select_mode) {
  const int NH = select_mode == 1 ? s.G : 1;
  const int min_rows = attend_mfma_applies(s, NH) || s.dtype == 0 ? 128 : 256, nsplit = gather_splits(s, select_mode);
  int n = device_cus() / (s.B * s.Hq / NH);
  if (n > s.k / min_rows) n = s.k / min_rows;
  if (n < div_up(s.k, kMaxGatherChunk)) n = div_up(s.k, kMaxGatherChunk);
  if (n >= nsplit) return nsplit;
  return n > 1 ? n : 1;
}

// One launch, or selection and attention in two?  Every block here selects for itself, on 512
// threads, so what counts is how often a CU has to do that.  Both ways timed behind the same
// scoring on 1239 shapes, us per step, one launch / two:
//   matrix cores, and eight heads on the vector units (one block per CU fits): one round of blocks
//     and no more.  128 units of 4 heads, S = 12000, k = 3000 (2 splits: one round) 75.4 / 76.6,
//     256 units (two rounds) 154 / 141, 512 units 325 / 291; 256 units of 8 heads, fp32, S = 8192,
//     k = 1024 136 / 143, 512 units, S = 4096 203 / 199
//   vector units, S <= 8192: one split per head always (4096 heads, S = 8192, k = 2048 488 / 529;
//     512 heads, S = 600 19.7 / 22.8), several in one round, and two of them in any number of
//     rounds (k up to 4096; 1024 heads, k = 2500 353 / 373) but for several tokens per sequence,
//     whose heads share their rows (768 heads, k = 2139 91 / 84)
//   vector units, S > 8192, where a thread holds 20 to 32 keys and the selection alone has twice
//     the threads: one split per head in more than one round (512 heads, S = 16384, k = 2048 227 /
//     236; 2048 heads 494 / 517); in one round the two are level (256 heads, S = 9000 43.4 / 44.1;
//     48 heads, 5 splits 42.8 / 38.0) and with forced splits every block selects again (4096 heads,
//     S = 16384, k = 4096, 4 tokens 983 / 847; 320 heads, S = 14745, k = 7372 219 / 180).
bool select_attend_applies(const Shape& s, int select_mode) {
  if (s.S > kSaThreads * 32) return false;
  const int NH = select_mode == 1 ? s.G : 1, n = select_attend_splits(s, select_mode);
  const bool one_round = (long long)n * s.B * s.Hq / NH <= device_cus();
  if (attend_mfma_applies(s, NH) || NH == 8) return one_round;
  if (s.S > 8192) return n == 1 && !one_round;
  return n == 1 || one_round || (n == 2 && s.rg.queries <= 1);
}

// Attention that begins before the list is complete: where its blocks wait for memory and nothing
// else runs beside them (one round of blocks, bf16), the heads do not walk shared rows in step in
// one ascending list (xcd_group_blocks, on the vector units), and the rows are between 2049, below
// which the selection is short, and 8192, beyond which a thread holds 32 keys. us per step, apart /
// begun early: 32 heads, S = 4096, k = 1024 19.1 / 18.2; 32 heads, S = 8000, k = 2000 26.5 / 24.6;
// 16 heads, S = 7544, k = 471 21.9 / 21.3; on the matrix cores, always one round, 32/8 heads, S =
// 8192 21.4 / 20.8, S = 4685, k = 146 19.9 / 18.4 (147 such shapes: 2 % less on average, single
// ones up to 8 % more, S = 3057, k = 764 19.7 / 21.1, where one unit's search among the candidates
// takes long); but S = 1200, k = 150 19.6 / 20.3, S = 11000, k = 2750 35.1 / 36.7, fp32, 24 heads,
// S = 3473, k = 217 17.4 / 18.3, and on the vector units 2 tokens of 4 sequences, S = 1920 24.5 /
// 25.5.
// Several tokens per sequence on the matrix cores: with lists of up to 1536 rows (336 shapes of 2
// and 4 tokens: 1 % less on average; 2 tokens of 2 sequences of 32/8 heads, S = 4374, k = 546 27.4
// / 26.1, 4 of 8, S = 8192, k = 1024 45.5 / 44.0), beyond which the bin often holds more candidates
// than the list (4 of 2, S = 7426, k = 1856 33.0 / 34.5, 4 of 8 54.4 / 59.0), and again from three
// tenths of the rows on, where the threshold lies nearer to 0 and its bin is narrower (2 of 1, S =
// 5100, k = 1700 27.9 / 25.4, S = 7704, k = 3852 31.1 / 28.4).
static bool attention_begins_early(const SelectAttendArgs& a, dim3 grid) {
  if (a.rg.queries > 1 && a.k_max > 1536 && 10 * a.k_max < 3 * a.S_max) return false;
  return a.S_max > 2048 && a.S_max <= 8192 && a.xcd_group_blocks == 0 && (int)(grid.x * grid.y) <= device_cus();
}

template <typename T, int NH>
static hipError_t launch_sa(const SelectAttendArgs& a, dim3 grid, const void* klo, const void* khi, const void* v,
                            const float* qhat, void* out, hipStream_t st) {
  auto* o = static_cast<typename T::store_t*>(out);
  if constexpr (T::kBytes == 2 && NH == 1)
    if (attention_begins_early(a, grid)) {
      if (a.per_thread <= 8)
        hipLaunchKernelGGL((select_attend_kernel<T, NH, 8, true>), grid, dim3(kSaThreads), 0, st, klo, khi, v, qhat, o, a);
      else
        hipLaunchKernelGGL((select_attend_kernel<T, NH, 16, true>), grid, dim3(kSaThreads), 0, st, klo, khi, v, qhat, o, a);
      return hipGetLastError();
    }
  if (a.per_thread <= 8)
    hipLaunchKernelGGL((select_attend_kernel<T, NH, 8, false>), grid, dim3(kSaThreads), 0, st, klo, khi, v, qhat, o, a);
  else if (a.per_thread <= 16)
    hipLaunchKernelGGL((select_attend_kernel<T, NH, 16, false>), grid, dim3(kSaThreads), 0, st, klo, khi, v, qhat, o, a);
  else
    hipLaunchKernelGGL((select_attend_kernel<T, NH, 32, false>), grid, dim3(kSaThreads), 0, st, klo, khi, v, qhat, o, a);
  return hipGetLastError();
}

template <int NH>
static hipError_t launch_sa_mfma(const SelectAttendArgs& a, dim3 grid, const void* klo, const void* khi, const void* v,
                                 const float* qhat, void* out, hipStream_t st) {
  auto* o = static_cast<uint16_t*>(out);
  if (attention_begins_early(a, grid)) {
    if (a.per_thread <= 8)
      hipLaunchKernelGGL((select_attend_mfma_kernel<NH, 8, true>), grid, dim3(kSaThreads), 0, st, klo, khi, v, qhat, o, a);
    else
      hipLaunchKernelGGL((select_attend_mfma_kernel<NH, 16, true>), grid, dim3(kSaThreads), 0, st, klo, khi, v, qhat, o, a);
    return hipGetLastError();
  }
  if (a.per_thread <= 8)
    hipLaunchKernelGGL((select_attend_mfma_kernel<NH, 8, false>), grid, dim3(kSaThreads), 0, st, klo, khi, v, qhat, o, a);
  else if (a.per_thread <= 16)
    hipLaunchKernelGGL((select_attend_mfma_kernel<NH, 16, false>), grid, dim3(kSaThreads), 0, st, klo, khi, v, qhat, o, a);
  else
    hipLaunchKernelGGL((select_attend_mfma_kernel<NH, 32, false>), grid, dim3(kSaThreads), 0, st, klo, khi, v, qhat, o, a);
  return hipGetLastError();
}

hipError_t launch_select_attend(const Shape& s, int select_mode, const float* scores, int32_t* user_idx,
                                const float* qhat, const void* klo, const void* khi, const void* v, float* partial,
                                int32_t* tickets, void* out, hipStream_t st) {
  if (!select_attend_applies(s, select_mode)) return hipErrorInvalidValue;
  const int NH = select_mode == 1 ? s.G : 1, nsplit = select_attend_splits(s, select_mode);
  if (div_up(s.k, nsplit) > kMaxGatherChunk) return hipErrorInvalidValue;
  const bool mfma = attend_mfma_applies(s, NH);
  SelectAttendArgs a;
  a.scores = scores;
  a.user_idx = user_idx;
  a.partial = partial;
  a.tickets = tickets;
  a.Hkv = s.Hkv;
  a.G = s.G;
  a.S_max = s.S;
  a.S_cap = s.S_cap;
  a.d = s.d;
  a.k_max = s.k;
  a.nsplit = nsplit;
  a.per_thread = ((s.S + kSaThreads - 1) / kSaThreads + 3) & ~3;
  a.xcd_group_blocks = a.xcd_sets = 0;
  a.rg = with_loads(s, select_mode);
  a.pg = s.pg;
  int blocks_y = s.B * s.Hq / NH;
  if (mfma) {
    const dim3 grid(nsplit, blocks_y);
    return NH == 8 ? launch_sa_mfma<8>(a, grid, klo, khi, v, qhat, out, st)
                   : launch_sa_mfma<4>(a, grid, klo, khi, v, qhat, out, st);
  }
  const int tokens = s.rg.queries > 1 ? s.rg.queries : 1;
  const int sharers = tokens * s.G, sets = s.B / tokens * s.Hkv, rounds = (sets + 7) / 8;
  if (NH == 1 && sharers > 1 && (long long)rounds * 8 * sharers <= 65535) {
    a.xcd_group_blocks = sharers * nsplit;
    a.xcd_sets = sets;
    blocks_y = rounds * 8 * sharers;
  }
  const dim3 grid(nsplit, blocks_y);
#define LOKI_SA(T, NHV) return launch_sa<T, NHV>(a, grid, klo, khi, v, qhat, out, st)
  if (s.dtype == 0) {
    switch (NH) {
      case 1: LOKI_SA(F32, 1);
      case 2: LOKI_SA(F32, 2);
      case 4: LOKI_SA(F32, 4);
      case 8: LOKI_SA(F32, 8);
      default: return hipErrorInvalidValue;
    }
  }
  switch (NH) {  // (4 and 8 heads: the matrix-core form above)
    case 1: LOKI_SA(BF16, 1);
    case 2: LOKI_SA(BF16, 2);
    default: return hipErrorInvalidValue;
  }
#undef LOKI_SA
}

}  // namespace loki
