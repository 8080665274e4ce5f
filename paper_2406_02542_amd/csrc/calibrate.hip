// Calibration and diagnostics around the decode path (arXiv 2406.02542, Section 3.1): the PCA
// of a set of calibration keys that produces the per-head basis P, Rank@v of its spectrum
// (Eq. 2), and the Jaccard agreement of two index lists (the quantity of Figure 6, left).
//
//   gram_kernel        (chunk, head)  G = sum_s k_s^T k_s and column sums over a run of rows, on
//                                     the matrix cores: a 32-row tile is written transposed into
//                                     LDS (swizzled, see gram_swizzle) so that both operands of
//                                     v_mfma_f32_16x16x32_bf16 (eight consecutive rows of one
//                                     column per lane) are one 16-byte LDS read; bf16 keys are exact, fp32 keys enter as two bf16 terms
//   cov_reduce_kernel  (tiles, head)  chunk partials added in a fixed order in fp64; sample
//                                     covariance C = (G - s s^T / N) / (N - 1)
//   eigensolver.hip                   eigenpairs of C, sorted by decreasing eigenvalue, every
//                                     component's largest entry made positive
//   rank_at_kernel, layer_width_kernel, jaccard_kernel    small reductions
#include "eigensolver.h"

namespace loki {

typedef __bf16 cal_bf16x8_t __attribute__((ext_vector_type(8)));
typedef float cal_f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kGramThreads = 256;
constexpr int kGramTile = 32;    // rows per tile = the k dimension of one MFMA
constexpr int kGramPitch = 144;  // bytes per column of the transposed tile: 8 slots of 16 bytes + 16
// A column's four 16-byte granules (rows 8 g .. 8 g + 7) sit in slots g ^ gram_swizzle(column).
// Columns one 16-byte chunk of a key row apart (8 columns) are written by neighbouring lanes in
// the same instruction and lie a multiple of 128 bytes apart whatever the pitch, i.e. in the same
// bank; the swizzle spreads the 16 chunks of a row over 8 bank groups (2-way instead of 16-way
// conflicts of the 2-byte transposing writes).
__device__ __forceinline__ int gram_swizzle(int col) { return (col >> 3) & 7; }

// NT = bf16 terms per element: 1 for bf16 storage, 2 for fp32 storage (value, remainder).
template <int NT>
__global__ __launch_bounds__(kGramThreads) void gram_kernel(const void* __restrict__ keys,
                                                            float* __restrict__ gram_part,
                                                            float* __restrict__ sum_part,
                                                            long long N, int rows_per_chunk) {
  constexpr int kColsPerChunk = NT == 1 ? 8 : 4;          // columns in a 16-byte chunk
  constexpr int kChunksPerRow = kD / kColsPerChunk;       // 16 or 32
  constexpr int kRowsPerPass = kGramThreads / kChunksPerRow;  // 16 or 8
  constexpr int kPasses = kGramTile / kRowsPerPass;       // 2 or 4
  __shared__ __align__(16) unsigned char s_t[NT][kD * kGramPitch];
  __shared__ float s_sum[kRowsPerPass][kD];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, kgrp = lane >> 4;
  const int chunk = blockIdx.x, head = blockIdx.y, nchunks = gridDim.x;
  const long long r0 = (long long)chunk * rows_per_chunk;
  const long long r1 = min(N, r0 + rows_per_chunk);
  const int c = tid % kChunksPerRow, rr = tid / kChunksPerRow;
  const size_t row_bytes = (size_t)kD * (NT == 1 ? 2 : 4);
  const char* base = static_cast<const char*>(keys) + (size_t)head * N * row_bytes + (size_t)c * 16;

  cal_f32x4_t acc[2][8];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = cal_f32x4_t{0.f, 0.f, 0.f, 0.f};
  float csum[kColsPerChunk];
#pragma unroll
  for (int e = 0; e < kColsPerChunk; ++e) csum[e] = 0.f;

  auto load_tile = [&](long long t0, uint4 (&raw)[kPasses]) {
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {
      const long long row = t0 + p * kRowsPerPass + rr;
      raw[p] = row < r1 ? load16(base + (size_t)row * row_bytes) : make_uint4(0, 0, 0, 0);
    }
  };

  uint4 raw[kPasses];
  load_tile(r0, raw);
  for (long long t0 = r0; t0 < r1; t0 += kGramTile) {
    __syncthreads();  // the previous tile's operand reads are done
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {
      const int row = p * kRowsPerPass + rr;  // row inside the tile
      if constexpr (NT == 1) {
        float f[8];
        BF16::unpack(raw[p], f);
        const uint32_t w[4] = {raw[p].x, raw[p].y, raw[p].z, raw[p].w};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          csum[e] += f[e];
          const uint16_t h = (uint16_t)((e & 1) ? (w[e >> 1] >> 16) : (w[e >> 1] & 0xffffu));
          *reinterpret_cast<uint16_t*>(&s_t[0][(8 * c + e) * kGramPitch + (((row >> 3) ^ gram_swizzle(8 * c + e)) << 4) + (row & 7) * 2]) = h;
        }
      } else {
        float f[4];
        F32::unpack(raw[p], f);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          csum[e] += f[e];
          const uint16_t hi = BF16::round(f[e]);
          const uint16_t lo = BF16::round(f[e] - __uint_as_float((uint32_t)hi << 16));
          *reinterpret_cast<uint16_t*>(&s_t[0][(4 * c + e) * kGramPitch + (((row >> 3) ^ gram_swizzle(4 * c + e)) << 4) + (row & 7) * 2]) = hi;
          *reinterpret_cast<uint16_t*>(&s_t[NT - 1][(4 * c + e) * kGramPitch + (((row >> 3) ^ gram_swizzle(4 * c + e)) << 4) + (row & 7) * 2]) = lo;
        }
      }
    }
    __syncthreads();
    load_tile(t0 + kGramTile, raw);  // next tile's loads fly during the products (zeros past the end)
    // wave w owns output rows 32 w .. 32 w + 31 (two 16-row tiles) of all 128 columns
    cal_bf16x8_t a[NT][2];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < 2; ++i)
        a[t][i] = *reinterpret_cast<const cal_bf16x8_t*>(
            &s_t[t][(32 * wave + 16 * i + r16) * kGramPitch + ((kgrp ^ gram_swizzle(32 * wave + 16 * i + r16)) << 4)]);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      cal_bf16x8_t b[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t)
        b[t] = *reinterpret_cast<const cal_bf16x8_t*>(
            &s_t[t][(16 * j + r16) * kGramPitch + ((kgrp ^ gram_swizzle(16 * j + r16)) << 4)]);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        if constexpr (NT == 2) {  // smallest terms first; remainder x remainder is below fp32's last place
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1][i], b[0], acc[i][j], 0, 0, 0);
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0][i], b[1], acc[i][j], 0, 0, 0);
        }
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0][i], b[0], acc[i][j], 0, 0, 0);
      }
    }
  }

  // partial Gram matrix: lane holds rows 4 kgrp + e, column r16 of each 16 x 16 tile
  float* gp = gram_part + ((size_t)head * nchunks + chunk) * kD * kD;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        gp[(size_t)(32 * wave + 16 * i + 4 * kgrp + e) * kD + 16 * j + r16] = acc[i][j][e];
  // column sums: the kRowsPerPass threads that share a chunk are added in a fixed order
#pragma unroll
  for (int e = 0; e < kColsPerChunk; ++e) s_sum[rr][kColsPerChunk * c + e] = csum[e];
  __syncthreads();
  if (tid < kD) {
    float s = 0.f;
#pragma unroll
    for (int r = 0; r < kRowsPerPass; ++r) s += s_sum[r][tid];
    sum_part[((size_t)head * nchunks + chunk) * kD + tid] = s;
  }
}

// C = (G - s s^T / N) / (N - 1), chunk partials added in order in fp64, and exactly symmetric: G's two
// halves are averaged (with fp32 keys they differ in the last place, value x remainder and
// remainder x value being added in the opposite order; a skew part, however small, never leaves a
// Jacobi iteration, which then took all of its 30 sweeps: 9.9 ms for 4 heads).  Block (tile pair,
// head): a 32 x 32 tile on or above the diagonal and its mirror image, exchanged through LDS.
constexpr int kCovTile = 32;
constexpr int kCovTiles = kD / kCovTile;
constexpr int kCovPairs = kCovTiles * (kCovTiles + 1) / 2;
__global__ __launch_bounds__(kCovTile * kCovTile) void cov_reduce_kernel(const float* __restrict__ gram_part,
                                                                         const float* __restrict__ sum_part,
                                                                         double* __restrict__ cov, long long N,
                                                                         int nchunks) {
  __shared__ double s_mirror[kCovTile][kCovTile + 1];
  const int head = blockIdx.y;
  int ti = 0, tj = blockIdx.x;
  while (tj >= kCovTiles - ti) {
    tj -= kCovTiles - ti;
    ++ti;
  }
  tj += ti;
  const int r = threadIdx.x / kCovTile, c = threadIdx.x % kCovTile;
  const int row = ti * kCovTile + r, col = tj * kCovTile + c;            // this thread's entry of the tile
  const int mrow = tj * kCovTile + r, mcol = ti * kCovTile + c;          // and of its mirror image
  const float* gp = gram_part + (size_t)head * nchunks * kD * kD;
  const float* sp = sum_part + (size_t)head * nchunks * kD;
  double g = 0.0, gm = 0.0, sr = 0.0, sc = 0.0;
  for (int cc = 0; cc < nchunks; ++cc) {
    g += (double)gp[(size_t)cc * kD * kD + (size_t)row * kD + col];
    gm += (double)gp[(size_t)cc * kD * kD + (size_t)mrow * kD + mcol];
    sr += (double)sp[cc * kD + row];
    sc += (double)sp[cc * kD + col];
  }
  s_mirror[r][c] = gm;
  __syncthreads();
  const double n = (double)N;
  const double x = (0.5 * (g + s_mirror[c][r]) - sr * sc / n) / (n > 1.0 ? n - 1.0 : 1.0);
  cov[(size_t)head * kD * kD + (size_t)row * kD + col] = x;
  __syncthreads();
  s_mirror[c][r] = x;
  __syncthreads();
  cov[(size_t)head * kD * kD + (size_t)mrow * kD + mcol] = s_mirror[r][c];
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
int pca_chunks(int Hkv, long long N, int* rows_per_chunk) {
  long long want = (2 * device_cus() + Hkv - 1) / Hkv;  // about two blocks per CU over all heads
  long long rows = (N + want - 1) / want;
  if (rows < 1024) rows = 1024;
  rows = (rows + kGramTile - 1) / kGramTile * kGramTile;
  *rows_per_chunk = (int)rows;
  return (int)((N + rows - 1) / rows);
}

size_t pca_workspace_bytes(int Hkv, long long N) {
  int rpc;
  const int nc = pca_chunks(Hkv, N, &rpc);
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
  int rpc;
  const int nc = pca_chunks(Hkv, N, &rpc);
  char* w = static_cast<char*>(workspace);
  float* gram_part = reinterpret_cast<float*>(w);
  float* sum_part = gram_part + (size_t)Hkv * nc * kD * kD;
  size_t off = ((size_t)Hkv * nc * kD * kD + (size_t)Hkv * nc * kD) * sizeof(float);
  off = (off + 255) / 256 * 256;
  double* cov = reinterpret_cast<double*>(w + off);
  double* mat = cov + (size_t)Hkv * kD * kD;
  if (stage == 0) {
    if (dtype == 0)
      hipLaunchKernelGGL(gram_kernel<2>, dim3(nc, Hkv), dim3(kGramThreads), 0, st, keys, gram_part,
                         sum_part, N, rpc);
    else
      hipLaunchKernelGGL(gram_kernel<1>, dim3(nc, Hkv), dim3(kGramThreads), 0, st, keys, gram_part,
                         sum_part, N, rpc);
  } else if (stage == 1) {
    hipLaunchKernelGGL(cov_reduce_kernel, dim3(kCovPairs, Hkv), dim3(kCovTile * kCovTile), 0, st, gram_part,
                       sum_part, cov, N, nc);
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
