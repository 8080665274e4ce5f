// The whole decode step of Loki (Algorithm 1 lines 3 and 5-9 of arXiv 2406.02542) for one
// (batch, head) unit in ONE block, for shapes where a unit's scores fit in LDS and there are
// enough units to fill the chip: rotate q, score the low-rank slab into LDS, select the top-k
// in LDS, then attend over the selected rows — no score buffer, index list or partial result
// ever leaves the CU, and there is no launch boundary between the stages.
#pragma once

#include <type_traits>

#include "attend_impl.h"
#include "block_order.h"
#include "score_impl.h"
#include "select_impl.h"

namespace loki {

constexpr int kFusedThreads = 512;
constexpr int kFusedWaves = kFusedThreads / 64;
constexpr int kFusedKPT = kFusedMaxS / kFusedThreads;  // keys a thread may hold in the select stage

// positions per thread in the select stage: ceil(S / threads) rounded up to a multiple of 4
__host__ __device__ inline int fused_keys_per_thread(int S) {
  const int c = (S + kFusedThreads - 1) / kFusedThreads;
  return (c + 3) & ~3;
}

// Beyond 16 keys a thread (S > 8192) the selection runs on keys in LDS, whose leading 11 bits the
// scoring has counted (contiguous_select), else on scores read back into registers
// (block_select_topk_resident).  us per step, registers / LDS: groups of 4, every head for itself,
// 512 heads, S = 12345, k = 1543 88.4 / 85.9; 256 heads, S = 12000 54.6 / 51.3; 512 heads, S =
// 9000, d = 64, pages of unequal sequences 58.8 / 54.6; 64 heads, S = 14000 42.9 / 42.8; but 256
// heads, S = 7900 72.4 / 72.1, 512 groups' heads, S = 8000 58.3 / 58.4, and 8 fp32 heads, S = 1024
// 12.0 / 12.9, where one wave's search among the candidates is a longer chain than the whole
// block's.
constexpr int kFusedRegisterKeys = 16;
__host__ __device__ inline bool fused_keys_in_lds(int S) { return fused_keys_per_thread(S) > kFusedRegisterKeys; }

// bytes of the region that holds the rotation's partial sums (query, new key) and then the scores
// or their keys (padded)
__host__ __device__ inline size_t fused_region_bytes(int S) {
  const size_t words = fused_keys_in_lds(S) ? padded_words((size_t)S) : (size_t)S;
  const size_t scores = (words * 4 + 15) & ~(size_t)15, rot = 2 * kRotParts * kD * sizeof(float);
  return scores > rot ? scores : rot;
}

// Which (sequence, head) unit a block works on, with the sequence's rows and the rows it keeps.  Uniform
// batches: unit = block.  Ragged batches (up to 64 sequences): the sequences are ranked by length and
// handed out so that the two blocks that share a CU (block i and block i + half the grid, when the whole
// grid is resident) get a long and a short sequence: the first half of the grid takes the longest
// sequences in descending order, the second half the rest in ascending order.  Every wave computes the
// same answer from the length array (lane l holds and ranks sequence l), so no barrier is needed; all of
// the chain behind it waits for this, so each length is loaded once.  (us, the other
// lengths of the ranking and the block's own length and k from memory again / so: 4 sequences of 32
// heads, S = 700 13.3 / 12.9, 60 of 16, S = 1000 47.4 / 46.7, 16 of 8 on pages, S = 2000 17.5 / 17.3.)
struct FusedWork {
  int unit, S, k, form;  // form: see RowLoads
};
__device__ __forceinline__ FusedWork fused_work_of_block(const Ragged& rag, int B, int Hkv, int block, int S_max, int k_max) {
  if (rag.seq_lens != nullptr && B <= 64 && B >= 2) {
    const int lane = threadIdx.x & 63;
    const int mine = lane < B ? rag.seq_lens[lane] : 0;
    const int keep = lane < B && rag.ks != nullptr ? rag.ks[lane] : k_max;
    int rank = 0;
    for (int j = 0; j < B; ++j) {
      const int other = __builtin_amdgcn_readlane(mine, j);
      rank += (other > mine || (other == mine && j < lane)) ? 1 : 0;
    }
    const int want = paired_rank(block / Hkv, B);
    const unsigned long long hit = __ballot(lane < B && rank == want);
    if (hit != 0ull) {  // (always: the ranks are a permutation of 0..B-1, exactly one lane holds each)
      const int b = __ffsll((long long)hit) - 1;
      const int S = min(max(__builtin_amdgcn_readlane(mine, b), 1), S_max);  // as seq_rows and seq_keep
      int form = rag.loads.form;
      if (form == kByLengths) {
        // loads_form, of which one list a head and no slab read again leave the bytes: one sum, in front of the
        // first loads (16 sequences of 32 heads on pages, S = 4096: 0.4 us of 46, with rows and kept rows apart 0.55)
        const int S_l = min(max(mine, 1), S_max), k_l = max(1, min(keep, min(k_max, S_l)));
        const float bytes = wave_sum_f32(lane < B ? (float)S_l * rag.loads.row_bytes + (float)k_l * rag.loads.kept_bytes : 0.f);
        form = __builtin_amdgcn_readfirstlane(bytes < kPastBytes ? kThroughCaches : kPastCaches);
      }
      return {b * Hkv + block % Hkv, S, max(1, min(__builtin_amdgcn_readlane(keep, b), min(k_max, S))), form};
    }
  }
  const int S = seq_rows(rag, block / Hkv, S_max);
  return {block, S, seq_keep(rag, block / Hkv, k_max, S), form_of_launch(rag, S_max, k_max)};
}

// APPEND: the block also rotates the unit's new key with the P_h entries it already holds and
// writes it, with the new value, into row S-1 of the unit's cache before it scores.  The block's
// own later reads of that row go through the same L1 and see it after the barrier; no other
// block reads this unit's rows.
constexpr int kFusedMaxPages = kFusedMaxS / 256;  // pages are at least 256 rows

// PAGED: the three slabs are pools addressed through the sequence's page list (see Paging). Two
// blocks share a CU (4 waves per SIMD) as far as LDS allows: the register budget is 128 VGPRs and
// the compiler is told not to trade load-level parallelism for a higher occupancy that cannot
// happen.  LDS allows it (fused_two_per_cu) while the dynamic part, 4 (33/32 S + k) bytes (4 S + 8
// k up to 8192 rows, 33/8 S + 8 k on a paged cache), leaves room for the static arrays in half of
// 160 KB: S = 13800, k = 1725 fits, S = 16384 does not, and a block has its CU to itself at the
// same budget.
// KPT = keys a thread holds in the select stage (8 for S <= 4096, 16 for S <= 8192, else 32).
// GROUPED: G query heads to a KV head, every one selecting for itself.  STREAM: the rows are loaded past the
// caches, see row_loads (not with groups, whose heads read the same slab and largely the same rows: 90.5 us
// either way, with the slab's loads streamed too 96.7).
template <typename T, int LPR, bool REUSE_LO, int KPT, bool APPEND, bool PAGED, bool GROUPED, bool STREAM, int NEW, int PAGES>
__device__ __forceinline__ void fused_decode_body(
    const FusedWork& work, float (&s_q)[kD], float (&s_qhat)[1][kD], float (&s_kn)[NEW] /* the new key */,
    ResidentSelectSmem<kFusedThreads>& s_sel, int32_t (&s_pages)[PAGES],
    const typename T::store_t* klo, const typename T::store_t* khi, const typename T::store_t* v,
    const typename T::store_t* __restrict__ q, const float* __restrict__ P,
    typename T::store_t* __restrict__ out, int32_t* __restrict__ out_idx, int n_seq, int Hkv, int G, int S_max,
    int S_cap, int d, int k_max, bool long_trips, Ragged rag, Append ap, Paging pg) {
  using ST = typename T::store_t;
  constexpr int EPC = T::EPC;
  constexpr int LPRV = kD / EPC;
  constexpr int RPW = 64 / LPRV;

  // The rotation's partial sums and then the scores' keys, the index list, and the scores of its entries;
  // long sequences (KPT = 32) leave those out, so that two blocks share a CU's LDS for longer, and look a
  // row's score up by its position (a paged cache's entries are pool rows and need the copy).
  constexpr bool kKeysInLds = KPT > kFusedRegisterKeys, kScoreByRow = kKeysInLds && !PAGED;
  extern __shared__ __align__(16) unsigned char dyn_smem[];
  const int per_thread = kKeysInLds ? KPT : fused_keys_per_thread(S_max);  // multiple of 4, <= KPT
  float* s_score = reinterpret_cast<float*>(dyn_smem);           // [S_max]
  uint32_t* s_key = reinterpret_cast<uint32_t*>(dyn_smem);       // kKeysInLds: instead, padded
  float(*s_part)[kD] = reinterpret_cast<float(*)[kD]>(dyn_smem);   // [kRotParts][kD]: the query's; then the new key's
  int32_t* s_idx = reinterpret_cast<int32_t*>(dyn_smem + fused_region_bytes(S_max));  // [k_max]
  float* s_a = kScoreByRow ? reinterpret_cast<float*>(s_key) : reinterpret_cast<float*>(s_idx + k_max);

  static_assert(kFusedWaves == kRotParts, "one wave per part of the rotation");
  MergeSmem<kFusedWaves, 1>& s_merge = *reinterpret_cast<MergeSmem<kFusedWaves, 1>*>(&s_sel);  // behind the selection
  static_assert(sizeof(s_merge) <= sizeof(s_sel), "the merge fits the histograms");

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // head = b * Hq + query head; unit = b * Hkv + KV head, whose cache it reads
  const int unit = work.unit, S = work.S, k = work.k;
  const int head = GROUPED ? unit * G + grouped_head((int)blockIdx.x, G) : unit;
  const int h = unit % Hkv;

  LOKI_STAMP(0);
#ifdef LOKI_PHASE_TIMING
  if (threadIdx.x == 0 && blockIdx.x < 8192) {
    g_phase_ts[blockIdx.x * kPhaseSlots + 9] = __builtin_amdgcn_s_getreg((31 << 11) | 4);    // HW_ID
    g_phase_ts[blockIdx.x * kPhaseSlots + 10] = __builtin_amdgcn_s_getreg((31 << 11) | 20);  // XCC_ID
  }
#endif
  resident_select_clear<kFusedThreads>(s_sel);  // covered by the barriers of the next stages

  // this lane's place in the low-rank slab
  const int cs = lane % LPR;
  const bool cact = cs < d / EPC;
  const size_t slab_row_bytes = (size_t)d * T::kBytes;
  using Rows = std::conditional_t<PAGED, PagedRows, ContiguousRows>;
  Rows slab;
  if constexpr (PAGED) {
    // the pages of the sequence's rows, clamped into the pool; readable after the first barrier below
    if (tid <= (S_max - 1) >> pg.lg_rows && tid < kFusedMaxPages && tid < pg.pages_per_seq)
      s_pages[tid] = min(max(pg.table[(size_t)(unit / Hkv) * pg.pages_per_seq + tid], 0), pg.n_pages - 1);
    slab = PagedRows{reinterpret_cast<const char*>(klo) + (size_t)(cact ? cs : 0) * 16, slab_row_bytes,
                     s_pages, pg.lg_rows, Hkv, h};
  } else {
    slab = ContiguousRows{reinterpret_cast<const char*>(klo) + (size_t)unit * S_cap * slab_row_bytes +
                              (size_t)(cact ? cs : 0) * 16,
                          slab_row_bytes};
  }
  constexpr bool kPipelined = LPR <= 8;
  // Issue order = the order the results are needed in (loads return in order): q, then this
  // thread's 16 x 2 entries of P_h, then the first slab loads, which do not need qhat and stay
  // in flight during the rotation.
  const float q_mine = T::load1(q + (size_t)head * kD + (tid & (kD - 1)));  // no branch: no early wait
  float kn_mine = 0.f, vn_mine = 0.f;
  if constexpr (APPEND) {
    kn_mine = T::load1(static_cast<const ST*>(ap.k_new) + (size_t)unit * kD + (tid & (kD - 1)));
    vn_mine = T::load1(static_cast<const ST*>(ap.v_new) + (size_t)unit * kD + (tid & (kD - 1)));
  }
  // qhat = q P_h with the association every path uses (8 parts of 16 terms, parts added in
  // order): wave w owns part w, lane l columns 2l and 2l+1; a load instruction of the wave
  // covers one 512-byte row of P_h.
  float2 pv[kRotPartLen];
  {
    const float* Ph = P + (size_t)h * kD * kD + (size_t)(wave * kRotPartLen) * kD + 2 * lane;
#pragma unroll
    for (int ii = 0; ii < kRotPartLen; ++ii)
      pv[ii] = *reinterpret_cast<const float2*>(Ph + (size_t)ii * kD);
  }
  ScoreTrip<kPipelined ? LPR : 8> first_trip, second_trip;
  constexpr int kTripRows = kFusedWaves * 64 * ScoreTrip<kPipelined ? LPR : 8>::TPI;
  if constexpr (kPipelined && !PAGED) {  // (a paged cache needs its page list in LDS first)
    score_load_trip<LPR, kFusedWaves, STREAM>(slab, wave * 64, S, first_trip);
    if constexpr (!APPEND)  // the appending variant has no registers to spare during the rotation
      score_load_trip<LPR, kFusedWaves, STREAM>(slab, wave * 64 + kTripRows, S, second_trip);
  }

  s_q[tid & (kD - 1)] = q_mine;  // four threads store the same value: no branch to sink the load into
  if constexpr (APPEND) s_kn[tid & (kD - 1)] = kn_mine;
  __syncthreads();
  if constexpr (kPipelined && PAGED && !APPEND) {  // the page list is in LDS now
    score_load_trip<LPR, kFusedWaves, STREAM>(slab, wave * 64, S, first_trip);
    score_load_trip<LPR, kFusedWaves, STREAM>(slab, wave * 64 + kTripRows, S, second_trip);
  }
  auto rotate_part = [&](const float* vec, float* part_row) {
    float a0 = 0.f, a1 = 0.f;
#pragma unroll
    for (int i4 = 0; i4 < kRotPartLen; i4 += 4) {
      const float4 qq = *reinterpret_cast<const float4*>(&vec[wave * kRotPartLen + i4]);
      a0 = fmaf(qq.x, pv[i4 + 0].x, a0);
      a1 = fmaf(qq.x, pv[i4 + 0].y, a1);
      a0 = fmaf(qq.y, pv[i4 + 1].x, a0);
      a1 = fmaf(qq.y, pv[i4 + 1].y, a1);
      a0 = fmaf(qq.z, pv[i4 + 2].x, a0);
      a1 = fmaf(qq.z, pv[i4 + 2].y, a1);
      a0 = fmaf(qq.w, pv[i4 + 3].x, a0);
      a1 = fmaf(qq.w, pv[i4 + 3].y, a1);
    }
    *reinterpret_cast<float2*>(&part_row[2 * lane]) = make_float2(a0, a1);
  };
  rotate_part(s_q, s_part[wave]);
  if constexpr (APPEND) rotate_part(s_kn, s_part[kRotParts + wave]);
  __syncthreads();
  if (tid < kD) {
    float sum = 0.f;
#pragma unroll
    for (int pp = 0; pp < kRotParts; ++pp) sum += s_part[pp][tid];
    s_qhat[0][tid] = sum;
  }
  if constexpr (APPEND) {
    // row S-1 of the unit's cache: rotated key (columns < d to the low-rank slab, the rest to
    // the residual slab) by threads 128..255, value by threads 256..383
    size_t row;
    if constexpr (PAGED) row = (size_t)slab.pool_row(S - 1);
    else row = (size_t)unit * S_cap + (size_t)(S - 1);
    if (tid >= kD && tid < 2 * kD) {
      const int j = tid - kD;
      float sum = 0.f;
#pragma unroll
      for (int pp = 0; pp < kRotParts; ++pp) sum += s_part[kRotParts + pp][j];
      ST* dst = j < d ? const_cast<ST*>(klo) + row * d + j : const_cast<ST*>(khi) + row * (kD - d) + (j - d);
      T::store1(dst, sum);
    } else if (tid >= 2 * kD && tid < 3 * kD) {
      T::store1(const_cast<ST*>(v) + row * kD + (tid - 2 * kD), vn_mine);
    }
  }
  __syncthreads();
  if constexpr (APPEND && kPipelined) {
    // the loads put in flight before the rotation may have read row S-1 before it was written
    if (PAGED || S - 1 < kTripRows)
      score_load_trip<LPR, kFusedWaves, STREAM>(slab, wave * 64, S, first_trip);
    score_load_trip<LPR, kFusedWaves, STREAM>(slab, wave * 64 + kTripRows, S, second_trip);
  }

  LOKI_STAMP(1);
  // ---- approximate scores over the low-rank slab, into LDS ------------------------------
  {
    float qr[1][EPC];
#pragma unroll
    for (int e = 0; e < EPC; ++e) qr[0][e] = cact ? s_qhat[0][cs * EPC + e] : 0.f;
    auto to_lds = [&](int row, const float (&sc)[1]) {
      if constexpr (kKeysInLds) {
        const uint32_t key = float_to_key(sc[0]);
        s_key[padded_pos(row)] = key;
        atomicAdd(&s_sel.hist[0][key >> 21], 1u);
      } else {
        s_score[row] = sc[0];
      }
    };
    if constexpr (kPipelined)
      score_rows_pipelined<T, LPR, 1, kFusedWaves, STREAM>(slab, qr, 0, S, first_trip, second_trip, to_lds);
    else
      score_rows<T, LPR, 1, kFusedWaves, STREAM>(slab, cact, qr, 0, S, to_lds);
  }
  __syncthreads();
  LOKI_STAMP(2);

  // ---- top-k in LDS ------------------------------------------------------------------------
  int32_t* gidx = out_idx ? out_idx + (size_t)head * k_max : nullptr;
  if (gidx)
    for (int i = k + tid; i < k_max; i += kFusedThreads) gidx[i] = -1;  // a sequence keeping fewer rows
  auto put = [&](int rank, int pos, float score) {
    if constexpr (PAGED) s_idx[rank] = (int32_t)slab.pool_row(pos);  // the attention stage reads pool rows
    else s_idx[rank] = pos;
    if constexpr (!kScoreByRow) s_a[rank] = score;
    if (gidx) gidx[rank] = pos;
  };
  if constexpr (kKeysInLds)
    contiguous_select<kFusedThreads, KPT>(s_key, S, per_thread, k, s_sel,
                                          [&](int rank, int pos, uint32_t key) { put(rank, pos, key_to_float(key)); });
  else
    block_select_topk_resident<kFusedThreads, KPT>(s_score, S, k, per_thread, s_sel, put);
  __syncthreads();
  LOKI_STAMP(6);

  // ---- exact attention over the selected rows -----------------------------------------------
  const int c = lane % LPRV, rg = lane / LPRV;
  float qr[1][EPC];
#pragma unroll
  for (int e = 0; e < EPC; ++e) qr[0][e] = s_qhat[0][c * EPC + e];
  const RowAddr ra = make_row_addr<T, REUSE_LO>(klo, khi, v, PAGED ? (size_t)0 : (size_t)unit, S_cap, d, c);
  AttendAcc<T, 1> acc;
  acc.init();
  auto attend = [&](auto rows, int r0, int r1) {
    attend_rows<T, 1, kFusedWaves * RPW, true, REUSE_LO, kScoreByRow, kKeysInLds, STREAM, decltype(rows)::value>(
        acc, qr, ra, s_idx + r0, kScoreByRow ? s_a : s_a + r0, wave * RPW + rg, r0, r1);
  };
  // fp32, whose rows take twice the lanes: a trip of 8 rows a lane group is as many rows as a bf16 trip of
  // 4.  us, 4 / 8: 8 heads, S = 1024, k = 256 11.9 / 11.5, 128, S = 4096, k = 1024 43.6 / 40.8, on pages
  // S = 8000, k = 2000 79.0 / 75.1; but with two blocks on a CU and short lists 512 heads, k = 175 24.6 /
  // 25.6, k = 256 26.1 / 27.2, in groups of 4, k = 375 41.7 / 42.4; bf16, 512 heads, S = 4096 60.8 / 63.3.
  // So: where every block has a CU, or the list is long (launch_fused_k).
  // What a trip of 4 can hold at the list's end is left to one (us, all in trips of 8 / so: 16
  // heads, S = 700, k = 42 10.1 / 9.5, k = 129 11.4 / 11.0; 64, S = 1500, k = 129 13.3 / 12.9).
  if constexpr (T::kBytes == 4 && !kKeysInLds) {
    constexpr int kTrip = kFusedWaves * RPW * kRowsInFlight;  // rows of a trip of 4
    const int long_rows = long_trips ? (k + kTrip - 1) / (2 * kTrip) * (2 * kTrip) : 0;
    attend(std::integral_constant<int, 2 * kRowsInFlight>{}, 0, min(long_rows, k));
    attend(std::integral_constant<int, kRowsInFlight>{}, long_rows, k);
  } else {
    attend(std::integral_constant<int, kRowsInFlight>{}, 0, k);
  }
  LOKI_STAMP(7);
  attend_publish<T, 1, kFusedWaves>(acc, s_merge);
  if (tid < kD) {
    float mn, ls, os;
    attend_merged<kFusedWaves, 1>(s_merge, 0, tid, mn, ls, os);
    T::store1(out + (size_t)head * kD + tid, os / ls);
  }
  LOKI_STAMP(8);
}

template <typename T, int LPR, bool REUSE_LO, int KPT, bool APPEND, bool PAGED, bool GROUPED>
__global__ __launch_bounds__(kFusedThreads) __attribute__((amdgpu_waves_per_eu(4, 4))) void
fused_decode_kernel(
    const typename T::store_t* klo, const typename T::store_t* khi, const typename T::store_t* v,
    const typename T::store_t* __restrict__ q, const float* __restrict__ P,
    typename T::store_t* __restrict__ out, int32_t* __restrict__ out_idx, int n_seq, int Hkv, int G, int S_max,
    int S_cap, int d, int k_max, bool long_trips, Ragged rag, Append ap, Paging pg) {
  __shared__ __align__(16) float s_q[kD];
  __shared__ float s_qhat[1][kD];
  __shared__ __align__(16) float s_kn[APPEND ? kD : 4];
  __shared__ __align__(16) ResidentSelectSmem<kFusedThreads> s_sel;
  __shared__ int32_t s_pages[PAGED ? kFusedMaxPages : 1];
  FusedWork work;
  if constexpr (!GROUPED) {
    work = fused_work_of_block(rag, (int)gridDim.x / Hkv, Hkv, (int)blockIdx.x, S_max, k_max);
  } else {
    // The G heads of a unit read the same slab and largely the same rows: blocks go to the 8 XCDs in
    // turn, so a unit's heads are blocks 8 apart, on one XCD and next to each other in time.
    const int slot = grouped_slot((int)blockIdx.x, G, n_seq * Hkv);
    if (slot < 0) return;  // (padding of the launch; uniform for the block)
    work = fused_work_of_block(rag, n_seq, Hkv, slot, S_max, k_max);
  }
  with_form<GROUPED ? kThroughCaches : kPastCaches>(work.form, [&](auto form) __attribute__((always_inline)) {
    fused_decode_body<T, LPR, REUSE_LO, KPT, APPEND, PAGED, GROUPED, decltype(form)::value != kThroughCaches>(
        work, s_q, s_qhat, s_kn, s_sel, s_pages, klo, khi, v, q, P, out, out_idx, n_seq, Hkv, G, S_max, S_cap, d, k_max, long_trips,
        rag, ap, pg);
  });
}

inline size_t fused_dynamic_lds(const Shape& s) {
  const bool score_by_row = fused_keys_in_lds(s.S) && s.pg.table == nullptr;
  return fused_region_bytes(s.S) + (size_t)s.k * (score_by_row ? 4 : 8);
}

template <typename T, int LPR, bool REUSE_LO, int KPT, bool APPEND, bool PAGED, bool GROUPED>
static hipError_t launch_fused_k(const Shape& s, const void* q, const float* P, void* klo, void* khi,
                                 void* v, void* out, int32_t* out_idx, hipStream_t st) {
  using ST = typename T::store_t;
  auto kern = fused_decode_kernel<T, LPR, REUSE_LO, KPT, APPEND, PAGED, GROUPED>;
  const size_t lds = fused_dynamic_lds(s);
  static std::atomic<unsigned long long> lds_allowed{0};  // per instantiation: devices already set up
  const hipError_t ea = allow_dynamic_lds(reinterpret_cast<const void*>(kern),
                                          (int)(fused_region_bytes(kFusedMaxS) + kFusedMaxK * 8), lds_allowed);
  if (ea != hipSuccess) return ea;
  const int blocks = GROUPED ? (s.B * s.Hkv + 7) / 8 * 8 * s.G : s.B * s.Hkv;
  const bool long_trips = blocks <= device_cus() || (!GROUPED && s.k >= 320);  // fp32: see the attention's trips
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(kFusedThreads), lds, st,
                     static_cast<const ST*>(klo), static_cast<const ST*>(khi),
                     static_cast<const ST*>(v), static_cast<const ST*>(q), P, static_cast<ST*>(out),
                     out_idx, s.B, s.Hkv, s.G, s.S, s.S_cap, s.d, s.k, long_trips, GROUPED ? s.rg : with_loads(s, 0), s.ap, s.pg);
  return hipGetLastError();
}

template <typename T, int LPR, bool REUSE_LO, int KPT>
static hipError_t launch_fused_a(const Shape& s, const void* q, const float* P, void* klo, void* khi,
                                 void* v, void* out, int32_t* out_idx, hipStream_t st) {
  const bool paged = s.pg.table != nullptr, append = s.ap.k_new != nullptr;
  if (s.G > 1) {
    if (append) return hipErrorInvalidValue;  // (G blocks read the row: it is appended by a launch before)
    const auto launch = paged ? launch_fused_k<T, LPR, REUSE_LO, KPT, false, true, true>
                              : launch_fused_k<T, LPR, REUSE_LO, KPT, false, false, true>;
    return launch(s, q, P, klo, khi, v, out, out_idx, st);
  }
  const auto launch = append ? (paged ? launch_fused_k<T, LPR, REUSE_LO, KPT, true, true, false>
                                      : launch_fused_k<T, LPR, REUSE_LO, KPT, true, false, false>)
                             : (paged ? launch_fused_k<T, LPR, REUSE_LO, KPT, false, true, false>
                                      : launch_fused_k<T, LPR, REUSE_LO, KPT, false, false, false>);
  return launch(s, q, P, klo, khi, v, out, out_idx, st);
}

template <typename T, int LPR, bool REUSE_LO>
static hipError_t launch_fused_r(const Shape& s, const void* q, const float* P, void* klo, void* khi,
                                 void* v, void* out, int32_t* out_idx, hipStream_t st) {
  if (fused_keys_per_thread(s.S) <= 8)
    return launch_fused_a<T, LPR, REUSE_LO, 8>(s, q, P, klo, khi, v, out, out_idx, st);
  if (!fused_keys_in_lds(s.S))
    return launch_fused_a<T, LPR, REUSE_LO, 16>(s, q, P, klo, khi, v, out, out_idx, st);
  return launch_fused_a<T, LPR, REUSE_LO, kFusedKPT>(s, q, P, klo, khi, v, out, out_idx, st);
}

template <typename T, int LPR>
static hipError_t launch_fused_l(const Shape& s, const void* q, const float* P, void* klo, void* khi,
                                 void* v, void* out, int32_t* out_idx, hipStream_t st) {
  // the ranking score is reused as the low-rank part of the exact logit; with d = 128
  // (Exact-TopK of Section 5) it is the whole logit and the attention stage reads no key
  return launch_fused_r<T, LPR, true>(s, q, P, klo, khi, v, out, out_idx, st);
}

template <typename T>
static hipError_t launch_fused_t(const Shape& s, const void* q, const float* P, void* klo, void* khi,
                                 void* v, void* out, int32_t* out_idx, hipStream_t st) {
  const int nch = s.d / T::EPC;
  int lpr = 1;
  while (lpr < nch) lpr <<= 1;
  switch (lpr) {
    case 1: return launch_fused_l<T, 1>(s, q, P, klo, khi, v, out, out_idx, st);
    case 2: return launch_fused_l<T, 2>(s, q, P, klo, khi, v, out, out_idx, st);
    case 4: return launch_fused_l<T, 4>(s, q, P, klo, khi, v, out, out_idx, st);
    case 8: return launch_fused_l<T, 8>(s, q, P, klo, khi, v, out, out_idx, st);
    case 16: return launch_fused_l<T, 16>(s, q, P, klo, khi, v, out, out_idx, st);
    case 32:
      if constexpr (T::EPC == 4) return launch_fused_l<T, 32>(s, q, P, klo, khi, v, out, out_idx, st);
      return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
}

}  // namespace loki
