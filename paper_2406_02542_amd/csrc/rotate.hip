// Key rotation into the PCA basis and append into the split cache
// (Algorithm 1 lines 3-4 of arXiv 2406.02542): khat = k P_h, fp32 accumulation, one
// rounding to the storage type, columns [0,d) to the low-rank slab and [d,D) to the residual.
//
// All rows that share a KV head share P_h, whatever their batch index, so a block works on rows
// of (batch, row) items of ONE head with P_h resident in its waves' registers.
#include "common.h"
#include "launch.h"

namespace loki {

typedef __bf16 rot_bf16x8_t __attribute__((ext_vector_type(8)));
typedef float rot_f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int rot_u32x4_t __attribute__((ext_vector_type(4)));

// What bounds it: memory, while a head has rows for its blocks. The rows of a trip go through LDS,
// loaded whole rows at a time and left whole rows at a time, and every wave multiplies all of them
// by its own 32 columns of P_h, so that P_h costs registers once and no LDS traffic. Blocks of four
// waves, two to a CU, whose barriers fall apart, with four trips of rows on their way: 16 x 32 x
// 4096 rows 220 us (4.9 TB/s read + write; a copy of the same bytes 204 to 218), with one block of
// eight waves per CU 233, and 245 with P_h in LDS in operand layout (96 KB read per 32 rows and
// wave) and every block on 8192 rows of its own: the blocks' positions are then megabytes apart and
// alike in their low address bits, which alone costs a tenth (a copy of the bytes in that order
// 231 us, in this one 210). Small calls: 11 x 124 rows of 8 heads 23 -> 8.4 us, where a block had at
// least 1024 rows; fp32, then on the vector units, 2848 rows of 32 heads 277 -> 37 us.
constexpr int kRotThreads = 256;
constexpr int kRotPerCU = 2;                                      // blocks that share a CU
constexpr int kRotColGroups = 4;                                  // waves side by side: 32 columns each
constexpr int kRotRowGroups = kRotThreads / 64 / kRotColGroups;   // waves on rows of their own
constexpr int kRotAhead = 4;                                      // trips whose rows are on their way
constexpr int kRotTripBytes = 8192 * kRotRowGroups;               // key rows of a trip
constexpr int kRotLoads = kRotTripBytes / 16 / kRotThreads;       // 16-byte loads a thread makes per trip

// The 32 columns of P_h that a wave multiplies by, in registers as the A operand (the columns of P_h
// are the rows of the product, the key rows its columns).  multiply(kv, acc): adds the products of a
// 16-row tile, kv[t] = the lane's 16 bytes of key row lane % 16 for step t.
template <typename T>
struct RotOperand;

// P_h enters as three bf16 terms (24 significant bits): every product is exact, and only the order of
// the fp32 sums differs from a vector product.  Lane l supplies
// k = 32 step + 8 (l / 16) .. + 7 of column 8 (m / 4) + 4 nb + m % 4, m = l % 16, so that the
// accumulators of nb = 0 and 1 hold eight neighbouring columns of one row.
template <>
struct RotOperand<BF16> {
  static constexpr int kTiles = 2;  // 16-row tiles of a trip per wave
  static constexpr int kSteps = 4;
  static constexpr int kTerms = 3;
  rot_bf16x8_t p[kTerms][kSteps][2];
  __device__ __forceinline__ void load(const float* Ph, int cg, int r16, int kgrp) {
    float x[kSteps][2][8];
#pragma unroll
    for (int t = 0; t < kSteps; ++t)
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int e = 0; e < 8; ++e)
          x[t][nb][e] = Ph[(32 * t + 8 * kgrp + e) * kD + 32 * cg + 8 * (r16 / 4) + 4 * nb + r16 % 4];
#pragma unroll
    for (int t = 0; t < kSteps; ++t)
#pragma unroll
      for (int nb = 0; nb < 2; ++nb) {
        uint32_t w[kTerms][4];
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2) {
          float a = x[t][nb][2 * e2], b = x[t][nb][2 * e2 + 1];
#pragma unroll
          for (int n = 0; n < kTerms; ++n) {
            const uint32_t pk = BF16::round2(a, b);
            a -= __uint_as_float(pk << 16);  // exact in fp32
            b -= __uint_as_float(pk & 0xffff0000u);
            w[n][e2] = pk;
          }
        }
#pragma unroll
        for (int n = 0; n < kTerms; ++n) p[n][t][nb] = __builtin_bit_cast(rot_bf16x8_t, make_uint4(w[n][0], w[n][1], w[n][2], w[n][3]));
      }
  }
  // acc[nb]: 16 rows of keys times 16 columns
  __device__ __forceinline__ void multiply(const uint4 (&kv)[kSteps], rot_f32x4_t (&acc)[2]) const {
#pragma unroll
    for (int n = kTerms - 1; n >= 0; --n)  // smallest terms first
#pragma unroll
      for (int t = 0; t < kSteps; ++t)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
          acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(p[n][t][nb], __builtin_bit_cast(rot_bf16x8_t, kv[t]), acc[nb], 0, 0, 0);
  }
  // the row's 16-byte chunks that this lane holds: one, columns 32 cg + 8 kgrp .. + 7
  static constexpr int kChunks = 1;
  __device__ static __forceinline__ int chunk(int cg, int kgrp, int) { return 4 * cg + kgrp; }
  __device__ static __forceinline__ uint4 packed(const rot_f32x4_t (&acc)[2], int) {
    return make_uint4(BF16::round2(acc[0][0], acc[0][1]), BF16::round2(acc[0][2], acc[0][3]),
                      BF16::round2(acc[1][0], acc[1][1]), BF16::round2(acc[1][2], acc[1][3]));
  }
};

// fp32 products and sums.  Step t holds k = 16 t .. + 15: lane l supplies k = 16 t + 4 (l / 16) + j to
// the step's matrix instruction j, which is what the lane's 16 bytes of a key row hold.
template <>
struct RotOperand<F32> {
  static constexpr int kTiles = 1;
  static constexpr int kSteps = 8;
  float p[kSteps][4][2];
  __device__ __forceinline__ void load(const float* Ph, int cg, int r16, int kgrp) {
#pragma unroll
    for (int t = 0; t < kSteps; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) p[t][j][nb] = Ph[(16 * t + 4 * kgrp + j) * kD + 32 * cg + 16 * nb + r16];
  }
  __device__ __forceinline__ void multiply(const uint4 (&kv)[kSteps], rot_f32x4_t (&acc)[2]) const {
#pragma unroll
    for (int t = 0; t < kSteps; ++t) {
      float f[4];
      F32::unpack(kv[t], f);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(p[t][j][nb], f[j], acc[nb], 0, 0, 0);
    }
  }
  static constexpr int kChunks = 2;  // columns 32 cg + 16 nb + 4 kgrp .. + 3
  __device__ static __forceinline__ int chunk(int cg, int kgrp, int nb) { return 8 * cg + 4 * nb + kgrp; }
  __device__ static __forceinline__ uint4 packed(const rot_f32x4_t (&acc)[2], int nb) {
    return __builtin_bit_cast(uint4, acc[nb]);
  }
};

// Block (x, head): trips x, x + gridDim.x, ... of the head's items, kRows rows each.
// PAGED: the output rows go through the page table (a separate instantiation, so that the
// contiguous kernel's store addresses stay plain arithmetic).
template <typename T, bool PAGED, bool PASS_CACHES>
__global__ __launch_bounds__(kRotThreads, kRotPerCU) void rotate_kernel(
    const char* __restrict__ k_new, const float* __restrict__ P, char* __restrict__ klo, char* __restrict__ khi,
    int Hkv, int S_cap, int d, int pos, int n_new, int n_items, Paging pg) {
  using Op = RotOperand<T>;
  constexpr int kTiles = Op::kTiles, kRows = 16 * kTiles * kRotRowGroups;
  constexpr int kRowBytes = kD * T::kBytes, kChunks = kRowBytes / 16;  // 16-byte chunks of a row
  static_assert(kRows * kRowBytes == kRotTripBytes, "a trip fills a buffer");
  constexpr int kRowStep = kRotThreads / kChunks;  // rows from one of a thread's chunks to the next
  // Chunk c of row r sits at c ^ (r % 16): 16 rows' equal chunks, and a row's chunks, are in different banks.
  __shared__ uint4 s_in[2][kRotTripBytes / 16], s_out[2][kRotTripBytes / 16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cg = wave % kRotColGroups, rg = wave / kRotColGroups;
  const int kgrp = lane >> 4, r16 = lane & 15;
  const int h = blockIdx.y;
  const int my_row = tid / kChunks, my_chunk = tid % kChunks;
  auto my_slot = [&](int n) {
    const int row = my_row + n * kRowStep;
    return row * kChunks + (my_chunk ^ (row & 15));
  };

  // item -> (batch, row), a scalar division per trip and a carry per lane; rows past the end are the last row
  const float inv_n = 1.0f / (float)n_new;
  auto place = [&](int trip, int off, int& b, int& r) {
    const int base = min(trip * kRows, n_items - 1);  // (uniform)
    const int b0 = base / n_new;
    const int x = base - b0 * n_new + min(off, n_items - 1 - base);  // < n_new + kRows
    const int carry = n_new >= kRows ? (x >= n_new ? 1 : 0) : (int)(((float)x + 0.5f) * inv_n);
    b = b0 + carry;
    r = x - carry * n_new;
  };
  auto load_trip = [&](int trip, uint4 (&raw)[kRotLoads]) {
#pragma unroll
    for (int n = 0; n < kRotLoads; ++n) {
      int b, r;
      place(trip, my_row + n * kRowStep, b, r);
      const char* src = k_new + ((size_t)(b * Hkv + h) * n_new + r) * kRowBytes + my_chunk * 16;
      raw[n] = load16(src);
    }
  };
  auto store_trip = [&](int trip, int buf) {
#pragma unroll
    for (int n = 0; n < kRotLoads; ++n) {
      const int off = my_row + n * kRowStep;
      int b, r;
      place(trip, off, b, r);
      size_t row;
      if constexpr (PAGED) row = (size_t)cache_row(pg, b, h, Hkv, S_cap, pos + r);
      else row = (size_t)(b * Hkv + h) * S_cap + pos + r;
      const int col = my_chunk * T::EPC;
      char* dst = col < d ? klo + (row * d + col) * T::kBytes : khi + (row * (kD - d) + (col - d)) * T::kBytes;
      const rot_u32x4_t val = __builtin_bit_cast(rot_u32x4_t, s_out[buf][my_slot(n)]);
      if (trip * kRows + off < n_items) {
        if constexpr (PASS_CACHES) __builtin_nontemporal_store(val, reinterpret_cast<rot_u32x4_t*>(dst));
        else *reinterpret_cast<rot_u32x4_t*>(dst) = val;
      }
    }
  };

  const int n_trips = (n_items + kRows - 1) / kRows, stride = gridDim.x;
  uint4 raw[kRotAhead][kRotLoads];
  load_trip(blockIdx.x, raw[0]);
  Op op;
  op.load(P + (size_t)h * kD * kD, cg, r16, kgrp);
#pragma unroll
  for (int a = 1; a < kRotAhead; ++a) load_trip(blockIdx.x + a * stride, raw[a]);

  int trip = blockIdx.x, buf = 0;
  bool first = true;
  for (bool more = true; more;) {
#pragma unroll
    for (int a = 0; a < kRotAhead; ++a) {
      if (trip >= n_trips) {
        more = false;
        break;
      }
#pragma unroll
      for (int n = 0; n < kRotLoads; ++n) s_in[buf][my_slot(n)] = raw[a][n];
      load_trip(trip + kRotAhead * stride, raw[a]);
      __syncthreads();
      if (!first) store_trip(trip - stride, buf ^ 1);
      first = false;
#pragma unroll
      for (int u = 0; u < kTiles; ++u) {
        const int row = (rg * kTiles + u) * 16 + r16;
        uint4 kv[Op::kSteps];
#pragma unroll
        for (int t = 0; t < Op::kSteps; ++t) kv[t] = s_in[buf][row * kChunks + ((4 * t + kgrp) ^ r16)];
        rot_f32x4_t acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
        op.multiply(kv, acc);
#pragma unroll
        for (int c = 0; c < Op::kChunks; ++c)
          s_out[buf][row * kChunks + (Op::chunk(cg, kgrp, c) ^ r16)] = Op::packed(acc, c);
      }
      trip += stride;
      buf ^= 1;
    }
  }
  __syncthreads();
  store_trip(trip - stride, buf ^ 1);
}

template <typename T>
static hipError_t launch_rotate_t(const Shape& s, const void* k_new, const float* P, void* klo, void* khi, int pos,
                                  int n_new, int n_items, hipStream_t st) {
  constexpr int kRows = 16 * RotOperand<T>::kTiles * kRotRowGroups;
  const int cus = device_cus(), trips = (n_items + kRows - 1) / kRows;
  // One round of blocks, or as many more (up to four) as leave the last round less idle: a round costs
  // its longest block's trips and about two trips of set-up (P_h into registers, the first rows).
  int blocks = 1;
  long long best = -1;
  for (int rounds = 1; rounds <= 4; ++rounds) {
    int nb = (int)((long long)rounds * kRotPerCU * cus / s.Hkv);
    nb = nb < 1 ? 1 : nb > trips ? trips : nb;
    const long long cost = (long long)rounds * ((trips + nb - 1) / nb + 2);
    if (best < 0 || cost < best) {
      best = cost;
      blocks = nb;
    }
  }
  // Rows are written past the caches while input and output fit the last-level cache (256 MiB), into
  // which a cache that has just been cleared has been written.  us, past / through the caches, a
  // repeated call and one on new buffers: 55 MB 14.8 / 16.7 and 54 / 58, 98 MB 23.0 / 25.9 and 62 / 67,
  // 268 MB 57.5 / 59.3 and 107 / 105, 537 MB 108.5 / 111.7 and 200 / 174.
  const bool pass_caches = 2ll * n_items * s.Hkv * kD * T::kBytes <= 256ll << 20;
  const dim3 grid(blocks, s.Hkv);
  const auto kernel = s.pg.table != nullptr ? (pass_caches ? rotate_kernel<T, true, true> : rotate_kernel<T, true, false>)
                                            : (pass_caches ? rotate_kernel<T, false, true> : rotate_kernel<T, false, false>);
  hipLaunchKernelGGL(kernel, grid, dim3(kRotThreads), 0, st, static_cast<const char*>(k_new), P, static_cast<char*>(klo),
                     static_cast<char*>(khi), s.Hkv, s.S_cap, s.d, pos, n_new, n_items, s.pg);
  return hipGetLastError();
}

hipError_t launch_rotate(const Shape& s, const void* k_new, const float* P, void* klo, void* khi,
                         int pos, int n_new, hipStream_t st) {
  const long long n_items = (long long)s.B * n_new;
  if (n_items > 0x7fffffffLL) return hipErrorInvalidValue;
  return s.dtype == 1 ? launch_rotate_t<BF16>(s, k_new, P, klo, khi, pos, n_new, (int)n_items, st)
                      : launch_rotate_t<F32>(s, k_new, P, klo, khi, pos, n_new, (int)n_items, st);
}

}  // namespace loki
