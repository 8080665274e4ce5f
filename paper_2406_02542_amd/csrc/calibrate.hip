// Calibration and diagnostics around the decode path (arXiv 2406.02542, Section 3.1): the PCA
// of a set of calibration keys that produces the per-head basis P, Rank@v of its spectrum
// (Eq. 2), and the Jaccard agreement of two index lists (the quantity of Figure 6, left).
//
//   gram_kernel        (chunk, head)  the upper half of G = sum_s k_s^T k_s and column sums over a run of rows,
//                                     on the matrix cores, operands made in registers; bf16 keys are
//                                     exact, fp32 keys enter as two bf16 terms
//   cov_reduce_kernel  (tiles, head)  chunk partials added in a fixed order in fp64; sample
//                                     covariance C = (G - s s^T / N) / (N - 1)
//   eigensolver.hip                   eigenpairs of C, sorted by decreasing eigenvalue, every
//                                     component's largest entry made positive
//   rank_at_kernel, layer_width_kernel, jaccard_kernel    small reductions
#include <algorithm>

#include "eigensolver.h"

namespace loki {

typedef __bf16 cal_bf16x8_t __attribute__((ext_vector_type(8)));
typedef float cal_f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kGramThreads = 256;
constexpr int kGramWaves = kGramThreads / 64;
constexpr int kGramStep = 32;    // rows a wave multiplies at a time = the k dimension of one MFMA
constexpr int kGramSets = 8;     // column set c: columns c, c + 8, .., c + 120
constexpr int kGramTiles = kGramSets * (kGramSets + 1) / 2;  // 16 x 16 tiles of G: pairs of sets c1 <= c2
constexpr int kGramPartWords = kGramTiles * 64 * 4;          // a partial: [tile][lane][4] as the accumulators lie
__host__ __device__ constexpr int gram_tile(int c1, int c2) { return c1 * kGramSets - c1 * (c1 - 1) / 2 + c2 - c1; }

// Four waves, each on 32-row steps of its own.  Lane (m, g) of a step loads columns 8 m .. 8 m + 7
// of rows 8 g .. 8 g + 7 (bf16: one 16-byte load a row, four whole rows an instruction) and pairs
// the rows up (v_perm_b32; fp32: the conversion packs them): operand c then holds eight consecutive
// rows of column 8 m + c, which is what v_mfma_f32_16x16x32_bf16 takes on either side, so a step
// needs no LDS, no barrier and, G being symmetric, 36 of 64 tiles.  Column sums: bf16 by a column
// of ones on the other side, fp32 by adding the fp32 values themselves.  What bounds it is the read
// of the keys: one wave per SIMD with 512 registers holds the 36 tiles and two steps' loads (bf16
// with three 2 us more, with four 18).  32 heads x 65536 keys, us: bf16 (512 MiB) 95 (5.6 TB/s), 82
// with STREAM (bf16 only: fp32 asks for half a line at a time), fp32 190; through a tile transposed in LDS, with two barriers a tile and all 64 tiles, 131 (4.1
// TB/s) and 267.
// NT = bf16 terms per element: 1 for bf16 storage, 2 for fp32 storage (value, remainder).
template <int NT, bool STREAM>
__global__ __launch_bounds__(kGramThreads, 1) void gram_kernel(const void* __restrict__ keys,
                                                               float* __restrict__ gram_part,
                                                               float* __restrict__ sum_part,
                                                               long long N, int rows_per_chunk) {
  constexpr int kBufs = 2;               // steps whose loads are in flight
  constexpr int kWords = 8 * NT;           // 16-byte loads of a step
  constexpr size_t kRowBytes = (size_t)kD * (NT == 1 ? 2 : 4);
  __shared__ __align__(16) float4 s_red[kGramWaves / 2][kGramTiles * 64];
  __shared__ float s_sum[kGramWaves][kD];

  const int lane = threadIdx.x & 63, r16 = lane & 15, kgrp = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int chunk = blockIdx.x, head = blockIdx.y, nchunks = gridDim.x;
  const long long r0 = (long long)chunk * rows_per_chunk;
  const int rows = (int)max(min(N - r0, (long long)rows_per_chunk), 0LL);
  const char* base = static_cast<const char*>(keys) + ((size_t)head * N + r0 + 8 * kgrp) * kRowBytes + (size_t)r16 * 16 * NT;

  cal_f32x4_t acc[kGramTiles], total[NT == 1 ? kGramSets : 1];
  float csum[NT == 1 ? 1 : kGramSets];  // of this k-group's rows, column 8 r16 + c
#pragma unroll
  for (int i = 0; i < kGramTiles; ++i) acc[i] = cal_f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (auto& t : total) t = cal_f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (auto& t : csum) t = 0.f;

  uint4 raw[kBufs][kWords];
  auto load_step = [&](int t0, uint4 (&x)[kWords]) {  // rows t0 .. t0 + 31 of the chunk, zeros past its end
    const char* p = base + (size_t)t0 * kRowBytes;
    if (t0 + kGramStep <= rows) {  // (uniform)
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int t = 0; t < NT; ++t) x[NT * e + t] = load16_hint<STREAM>(p + e * kRowBytes + 16 * t);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int t = 0; t < NT; ++t)
          x[NT * e + t] = t0 + 8 * kgrp + e < rows ? load16_hint<STREAM>(p + e * kRowBytes + 16 * t) : make_uint4(0, 0, 0, 0);
    }
  };
  auto word = [](const uint4& x, int i) { return i == 0 ? x.x : i == 1 ? x.y : i == 2 ? x.z : x.w; };
  const cal_bf16x8_t ones = __builtin_bit_cast(cal_bf16x8_t, make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u));

#pragma unroll
  for (int b = 0; b < kBufs; ++b) load_step((wave + kGramWaves * b) * kGramStep, raw[b]);
  for (int t0 = wave * kGramStep; t0 < rows; t0 += kGramWaves * kGramStep * kBufs) {
#pragma unroll
    for (int b = 0; b < kBufs; ++b) {
      cal_bf16x8_t op[NT][kGramSets];
#pragma unroll
      for (int c = 0; c < kGramSets; ++c) {
        uint32_t w[NT][4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if constexpr (NT == 1) {
            w[0][j] = __builtin_amdgcn_perm(word(raw[b][2 * j + 1], c / 2), word(raw[b][2 * j], c / 2), c % 2 ? 0x07060302u : 0x05040100u);
          } else {
            const float x0 = __uint_as_float(word(raw[b][4 * j + c / 4], c % 4));
            const float x1 = __uint_as_float(word(raw[b][4 * j + 2 + c / 4], c % 4));
            w[0][j] = BF16::round2(x0, x1);
            w[NT - 1][j] = BF16::round2(x0 - __uint_as_float(w[0][j] << 16), x1 - __uint_as_float(w[0][j] & 0xffff0000u));
          }
        }
        if constexpr (NT == 2) {
          float x[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) x[e] = __uint_as_float(word(raw[b][2 * e + c / 4], c % 4));
          csum[c] += ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) op[t][c] = __builtin_bit_cast(cal_bf16x8_t, make_uint4(w[t][0], w[t][1], w[t][2], w[t][3]));
      }
      load_step(t0 + (b + kBufs) * kGramWaves * kGramStep, raw[b]);
      if constexpr (NT == 2) {  // smallest terms first; remainder x remainder, at most 2^-18 of a term, is left out
#pragma unroll
        for (int c1 = 0; c1 < kGramSets; ++c1)
#pragma unroll
          for (int c2 = c1; c2 < kGramSets; ++c2) {
            const int i = gram_tile(c1, c2);
            acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(op[1][c1], op[0][c2], acc[i], 0, 0, 0);
          }
#pragma unroll
        for (int c1 = 0; c1 < kGramSets; ++c1)
#pragma unroll
          for (int c2 = c1; c2 < kGramSets; ++c2) {
            const int i = gram_tile(c1, c2);
            acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(op[0][c1], op[1][c2], acc[i], 0, 0, 0);
          }
      }
#pragma unroll
      for (int c1 = 0; c1 < kGramSets; ++c1)
#pragma unroll
        for (int c2 = c1; c2 < kGramSets; ++c2) {
          const int i = gram_tile(c1, c2);
          acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(op[0][c1], op[0][c2], acc[i], 0, 0, 0);
        }
      if constexpr (NT == 1)
#pragma unroll
        for (int c = 0; c < kGramSets; ++c) total[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, op[0][c], total[c], 0, 0, 0);
    }
  }

  // the waves' sums, added pairwise in a fixed order
#pragma unroll
  for (int half = kGramWaves / 2; half > 0; half >>= 1) {
    if (wave >= half && wave < 2 * half)
#pragma unroll
      for (int i = 0; i < kGramTiles; ++i)
        s_red[wave - half][i * 64 + lane] = make_float4(acc[i][0], acc[i][1], acc[i][2], acc[i][3]);
    __syncthreads();
    if (wave < half)
#pragma unroll
      for (int i = 0; i < kGramTiles; ++i) {
        const float4 o = s_red[wave][i * 64 + lane];
        acc[i] = cal_f32x4_t{acc[i][0] + o.x, acc[i][1] + o.y, acc[i][2] + o.z, acc[i][3] + o.w};
      }
    __syncthreads();
  }
  // (every row of a tile of column sums is the same; fp32: the four k-groups' sums are added pairwise)
#pragma unroll
  for (int c = 0; c < kGramSets; ++c) {
    float sum;
    if constexpr (NT == 1) {
      sum = total[c][0];
    } else {
      sum = csum[c] + __shfl_xor(csum[c], 16);
      sum += __shfl_xor(sum, 32);
    }
    if (kgrp == 0) s_sum[wave][8 * r16 + c] = sum;
  }
  const size_t part = (size_t)head * nchunks + chunk;
  if (wave == 0) {
    float4* gp = reinterpret_cast<float4*>(gram_part + part * kGramPartWords);
#pragma unroll
    for (int i = 0; i < kGramTiles; ++i) gp[i * 64 + lane] = make_float4(acc[i][0], acc[i][1], acc[i][2], acc[i][3]);
  }
  __syncthreads();
  if (threadIdx.x < kD)
    sum_part[part * kD + threadIdx.x] = (s_sum[0][threadIdx.x] + s_sum[1][threadIdx.x]) + (s_sum[2][threadIdx.x] + s_sum[3][threadIdx.x]);
}

// C = (G - s s^T / N) / (N - 1), chunk partials added in order in fp64.  Block (set, head): rows
// set, set + 8, .. of C, thread (c2, lane) the four entries that this lane holds of tile (set, c2),
// or of its mirror image where only that exists; the rows are put together in LDS and leave whole.
// Both places of an entry are computed from the same numbers, so C is exactly symmetric (a skew
// part, however small, never leaves a Jacobi iteration, which then took all of its 30 sweeps: 9.9
// ms for 4 heads).
constexpr int kCovThreads = kGramSets * 64;
constexpr int kCovPitch = kD + 4;  // doubles per row in LDS
__global__ __launch_bounds__(kCovThreads) void cov_reduce_kernel(const float* __restrict__ gram_part,
                                                                 const float* __restrict__ sum_part,
                                                                 double* __restrict__ cov, long long N,
                                                                 int nchunks) {
  __shared__ double s_sum[kD];
  __shared__ __align__(16) double s_row[kD / kGramSets][kCovPitch];
  const int set = blockIdx.x, head = blockIdx.y, tid = threadIdx.x;
  const int c2 = tid >> 6, lane = tid & 63;
  const int tile = set <= c2 ? gram_tile(set, c2) : gram_tile(c2, set);
  const float4* gp = reinterpret_cast<const float4*>(gram_part + (size_t)head * nchunks * kGramPartWords) + tile * 64 + lane;
  const float* sp = sum_part + (size_t)head * nchunks * kD + tid;
  double g[4] = {0.0, 0.0, 0.0, 0.0}, s = 0.0;
#pragma unroll 4
  for (int cc = 0; cc < nchunks; ++cc) {
    const float4 x = gp[(size_t)cc * (kGramPartWords / 4)];
    g[0] += (double)x.x;
    g[1] += (double)x.y;
    g[2] += (double)x.z;
    g[3] += (double)x.w;
    if (tid < kD) s += (double)sp[(size_t)cc * kD];
  }
  if (tid < kD) s_sum[tid] = s;
  __syncthreads();
  const double n = (double)N;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    // row i of the tile, column j; on the diagonal the upper half serves both
    const int i = 4 * (lane >> 4) + e, j = lane & 15;
    const bool swap = set > c2;
    const int row = kGramSets * i + (swap ? c2 : set), col = kGramSets * j + (swap ? set : c2);
    const double x = (g[e] - s_sum[row] * s_sum[col] / n) / (n > 1.0 ? n - 1.0 : 1.0);
    if (swap) {
      s_row[j][row] = x;
    } else if (set < c2 || i <= j) {
      s_row[i][col] = x;
      if (set == c2) s_row[j][row] = x;
    }
  }
  __syncthreads();
  double* C = cov + (size_t)head * kD * kD;
#pragma unroll
  for (int u = tid; u < kD / kGramSets * kD / 2; u += kCovThreads) {
    const int i = u / (kD / 2), at = 2 * (u % (kD / 2));
    *reinterpret_cast<double2*>(C + (size_t)(kGramSets * i + set) * kD + at) = *reinterpret_cast<const double2*>(&s_row[i][at]);
  }
}

// Eq. 2: the smallest d whose leading normalised eigenvalues sum to at least v percent.
__device__ inline int rank_at_of(const float* __restrict__ lam, int Dn, float v_percent) {
  double total = 0.0;
  for (int i = 0; i < Dn; ++i) total += (double)lam[i];
  double run = 0.0;
  for (int i = 0; i < Dn; ++i) {
    run += (double)lam[i];
    if (run / total >= (double)v_percent / 100.0) return i + 1;
  }
  return Dn;
}

__global__ __launch_bounds__(64) void rank_at_kernel(const float* __restrict__ eigenvalues, int Dn,
                                                     float v_percent, int32_t* __restrict__ ranks) {
  if (threadIdx.x != 0) return;
  ranks[blockIdx.x] = rank_at_of(eigenvalues + (size_t)blockIdx.x * Dn, Dn, v_percent);
}

// Rank_l@v of a layer (the head average of Eq. 2, Section 3.1) and the slab width that the
// variable-width policy of Appendix B.2 derives from it: the average taken up to a whole
// number, then to a multiple of the layout's granularity, at most D.  One block; the ranks are
// integers, so their sum is exact whatever the order.
__global__ __launch_bounds__(256) void layer_width_kernel(const float* __restrict__ eigenvalues,
                                                          int n_heads, int Dn, float v_percent,
                                                          int multiple, float* __restrict__ mean_rank,
                                                          int32_t* __restrict__ d_out) {
  __shared__ int s_sum;
  if (threadIdx.x == 0) s_sum = 0;
  __syncthreads();
  int mine = 0;
  for (int h = threadIdx.x; h < n_heads; h += 256)
    mine += rank_at_of(eigenvalues + (size_t)h * Dn, Dn, v_percent);
  if (mine) atomicAdd(&s_sum, mine);
  __syncthreads();
  if (threadIdx.x == 0) {
    const int sum = s_sum;
    if (mean_rank) *mean_rank = (float)((double)sum / (double)n_heads);
    int d = (sum + n_heads - 1) / n_heads;             // ceil of the average
    d = (d + multiple - 1) / multiple * multiple;
    *d_out = d < Dn ? d : Dn;
  }
}

// |A n B| / |A u B| of two ascending index lists of length k each (entries < 0 are padding).
__global__ __launch_bounds__(256) void jaccard_kernel(const int32_t* __restrict__ a,
                                                      const int32_t* __restrict__ b, int k,
                                                      float* __restrict__ out) {
  __shared__ int s_cnt[3];
  const int32_t* la = a + (size_t)blockIdx.x * k;
  const int32_t* lb = b + (size_t)blockIdx.x * k;
  if (threadIdx.x < 3) s_cnt[threadIdx.x] = 0;
  __syncthreads();
  int inter = 0, na = 0, nb = 0;
  for (int i = threadIdx.x; i < k; i += 256) {
    const int x = la[i];
    nb += lb[i] >= 0 ? 1 : 0;
    if (x < 0) continue;
    ++na;
    int lo = 0, hi = k;  // lower bound of x among the non-negative prefix-ordered entries of b
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      const int y = lb[mid];
      if (y >= 0 && y < x) lo = mid + 1; else hi = mid;
    }
    inter += (lo < k && lb[lo] == x) ? 1 : 0;
  }
  atomicAdd(&s_cnt[0], inter);
  atomicAdd(&s_cnt[1], na);
  atomicAdd(&s_cnt[2], nb);
  __syncthreads();
  if (threadIdx.x == 0) {
    const int uni = s_cnt[1] + s_cnt[2] - s_cnt[0];
    out[blockIdx.x] = uni > 0 ? (float)s_cnt[0] / (float)uni : 1.0f;
  }
}

// ---- launchers ----------------------------------------------------------------------------------
// What the workspace is laid out for: a partial Gram matrix of 64 KiB for every 1024 rows, at most
// two for every CU over all heads (the eigensolver uses the space again).
static int pca_chunks(int Hkv, long long N) {
  const long long want = (2 * device_cus() + Hkv - 1) / Hkv;
  long long rows = (N + want - 1) / want;
  if (rows < 1024) rows = 1024;
  rows = (rows + 31) / 32 * 32;
  return (int)((N + rows - 1) / rows);
}

// Chunks of a head in the Gram pass, never more than pca_chunks: a CU holds one block, so as many
// as make whole rounds of blocks, one round if that leaves no CU idle (32 heads: 8 chunks), else
// the number of rounds at which rounds x (rows of a chunk + the 256 that a block's start and end
// cost) is least.
static int gram_chunks(int Hkv, long long N, int* rows_per_chunk) {
  constexpr long long kWhole = kGramWaves * kGramStep;
  const int most = pca_chunks(Hkv, N);
  long long best = -1;
  int chunks = 1;
  for (int rounds = 1; rounds <= 4 || best < 0; ++rounds) {
    const long long n = std::min<long long>(most, (long long)rounds * device_cus() / Hkv);
    if (n < 1) continue;
    const long long rows = (N + n - 1) / n, used = ((N + rows - 1) / rows * Hkv + device_cus() - 1) / device_cus();
    const long long cost = used * (rows + 256);
    if (best < 0 || cost < best) {
      best = cost;
      chunks = (int)n;
    }
  }
  const long long rows = ((N + chunks - 1) / chunks + kWhole - 1) / kWhole * kWhole;
  *rows_per_chunk = (int)rows;
  return (int)((N + rows - 1) / rows);
}

size_t pca_workspace_bytes(int Hkv, long long N) {
  const int nc = pca_chunks(Hkv, N);
  size_t b = 0;
  b += (size_t)Hkv * nc * kD * kD * sizeof(float);  // partial Gram matrices
  b += (size_t)Hkv * nc * kD * sizeof(float);       // partial column sums
  b = (b + 255) / 256 * 256;
  b += (size_t)Hkv * kD * kD * sizeof(double);      // covariance
  b += (size_t)Hkv * kD * kD * sizeof(double);      // eigensolver: the vectors, later the projected matrix
  b += (size_t)Hkv * kEigReflBytes;                 // eigensolver: reflectors, later half of the vectors
  b += (size_t)2 * Hkv * sizeof(int);               // eigensolver: a state word per head
  return b;
}

// stage 0: partial Gram matrices; 1: covariance; 2: eigensolver
hipError_t launch_pca_stage(int stage, int Hkv, int dtype, const void* keys, long long N, float* P,
                            float* eigenvalues, void* workspace, hipStream_t st) {
  static_assert(kGramPartWords <= kD * kD, "a partial Gram matrix fits the space laid out for it");
  int rpc;
  const int nc = pca_chunks(Hkv, N), chunks = gram_chunks(Hkv, N, &rpc);
  char* w = static_cast<char*>(workspace);
  float* gram_part = reinterpret_cast<float*>(w);
  float* sum_part = gram_part + (size_t)Hkv * nc * kD * kD;
  size_t off = ((size_t)Hkv * nc * kD * kD + (size_t)Hkv * nc * kD) * sizeof(float);
  off = (off + 255) / 256 * 256;
  double* cov = reinterpret_cast<double*>(w + off);
  double* mat = cov + (size_t)Hkv * kD * kD;
  if (stage == 0) {
    if (dtype == 0)
      hipLaunchKernelGGL((gram_kernel<2, false>), dim3(chunks, Hkv), dim3(kGramThreads), 0, st, keys, gram_part,
                         sum_part, N, rpc);
    else  // (keys that fit the last-level cache may be there: 11 MB 285.2 / 286.2 us a fit, 88 MB 302.5 / 296.1)
      hipLaunchKernelGGL((2ll * Hkv * N * kD >= 80000000 ? gram_kernel<1, true> : gram_kernel<1, false>), dim3(chunks, Hkv),
                         dim3(kGramThreads), 0, st, keys, gram_part, sum_part, N, rpc);
  } else if (stage == 1) {
    hipLaunchKernelGGL(cov_reduce_kernel, dim3(kGramSets, Hkv), dim3(kCovThreads), 0, st, gram_part, sum_part, cov, N,
                       chunks);
  } else {
    EigRegions r;
    r.cov = cov;
    r.mat = mat;
    r.refl = reinterpret_cast<char*>(mat + (size_t)Hkv * kD * kD);
    r.state = reinterpret_cast<int*>(r.refl + (size_t)Hkv * kEigReflBytes);
    r.spare = w;  // the partial Gram matrices (64 KiB each) have been added up
    r.spare_halves = nc;
    return launch_eigensolver(Hkv, r, P, eigenvalues, st);
  }
  return hipGetLastError();
}

hipError_t launch_rank_at(const float* eigenvalues, int n, int Dn, float v_percent, int32_t* ranks,
                          hipStream_t st) {
  hipLaunchKernelGGL(rank_at_kernel, dim3(n), dim3(64), 0, st, eigenvalues, Dn, v_percent, ranks);
  return hipGetLastError();
}

hipError_t launch_layer_width(const float* eigenvalues, int n, int Dn, float v_percent, int multiple,
                              float* mean_rank, int32_t* d_out, hipStream_t st) {
  hipLaunchKernelGGL(layer_width_kernel, dim3(1), dim3(256), 0, st, eigenvalues, n, Dn, v_percent,
                     multiple, mean_rank, d_out);
  return hipGetLastError();
}

hipError_t launch_jaccard(const int32_t* a, const int32_t* b, int n_lists, int k, float* out,
                          hipStream_t st) {
  hipLaunchKernelGGL(jaccard_kernel, dim3(n_lists), dim3(256), 0, st, a, b, k, out);
  return hipGetLastError();
}

}  // namespace loki
