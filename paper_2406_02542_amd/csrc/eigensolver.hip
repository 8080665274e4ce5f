// Symmetric eigensolver in fp64 for the 128 x 128 covariances of a calibration (Section 3.1 of
// arXiv 2406.02542), one matrix per KV head.
//
//   tridiag_kernel        (head)         Householder tridiagonalisation, the matrix in registers
//   eigvec_kernel         (slice, head)  16 eigenpairs of the tridiagonal matrix per block: the
//                                        eigenvalues by multisection on Sturm counts, the vectors by
//                                        the twisted factorisation, taken back through the reflectors
//   orthonormalise_kernel (slice, head)  one Newton-Schulz step on the vectors; a head whose vectors
//                                        are far from orthonormal (equal eigenvalues: rank-deficient
//                                        keys, dead columns) is marked
//   project_kernel        (slice, head)  B = V C V^T; a marked head gets B = C, V = I instead
//   jacobi_kernel         (role, head)   cyclic Jacobi on B until its off-diagonal mass is at rounding
//                                        level.  An unmarked head passes that test at once (measured
//                                        5e-31 against the test's 1e-28), a marked one is solved here
//   finish_kernel         (slice, head)  pairs by decreasing eigenvalue, largest entry positive, fp32
//
// What bounds it: chains of dependent fp64 steps, not throughput (4 M multiply-adds per head and
// product).  Jacobi alone, one block per head, needed 12 sweeps of 127 rounds at 2.1 us a round and
// 74 us a sweep more for the vectors: 4.1 of the 4.23 ms of a fit of 32 heads x 65536 keys, now
// 0.31 ms (tridiag 125 us, eigvec 64, orthonormalise 13, project 13, the two Jacobi launches 9,
// finish 6; the Gram pass 83, the covariance 8).  Tridiagonalisation is 126 steps of one barrier, and
// everything behind it is spread over 8 blocks per head.
#include "eigensolver.h"

#include <algorithm>
#include <type_traits>

namespace loki {

constexpr int kEigSliceRows = 16;               // eigenvectors a block of the sliced kernels owns
constexpr int kEigSlices = kD / kEigSliceRows;
constexpr int kEigThreads = 256;
constexpr int kJacThreads = 1024;
constexpr int kJacPitch = kD + 1;               // doubles per row of the LDS-resident matrix
constexpr int kJacMaxSweeps = 30;
constexpr int kJacRounds = kD - 1;
constexpr int kJacSliceCols = 32;               // columns of V an accumulating block owns
constexpr int kJacSlices = kD / kJacSliceCols;
constexpr int kJacMaxPolls = 1 << 22;           // of about a microsecond
constexpr size_t kMatBytes = (size_t)kD * kD * sizeof(double);
constexpr size_t kHalfBytes = kMatBytes / 2;
constexpr size_t kLogBytes = (size_t)kJacRounds * (kD / 2) * sizeof(double);  // one sweep's tangents
static_assert(kLogBytes <= kHalfBytes, "a sweep's log fits half a matrix");
constexpr double kOrthTolerance = 1e-7;  // a Newton-Schulz step leaves its square
constexpr double kOffTolerance = 1e-28;  // off-diagonal over diagonal mass (squares) of a solved matrix

// Where everything lives (see eigen_regions): the partial Gram matrices are dead by now and their
// space is used again.
struct EigBufs {
  double* cov;          // [heads][128][128]; dead after project_kernel: the first two sweep logs of a head
  double* mat;          // [heads][128][128]  Z, the vectors before orthonormalisation; then B
  char* vec_lo;         // [heads] 64 KiB: d, e of the tridiagonal matrix; then rows 0..63 of V
  char* refl;           // [heads][kEigReflBytes]: the reflectors; then rows 64..127 of V and the progress words
  char* more_logs;      // [heads][n_logs - 2] 64 KiB each
  int* state;           // [heads] kStateMarked, and kStateSolvedIn (1 + the Jacobi launch that solved the head)
  int n_heads;
  int n_logs;           // sweep logs a head has room for (2 or more)
  int defer;            // of a launch's sweeps, how many are replayed in the next (0 or 1)
};
constexpr int kStateMarked = 1, kStateSolvedIn = 2;

__device__ __forceinline__ double* eig_tri(const EigBufs& b, int head) {  // d[128], e[128], tau[128]
  return reinterpret_cast<double*>(b.vec_lo + (size_t)head * kHalfBytes);
}
__device__ __forceinline__ double* eig_refl(const EigBufs& b, int head) {
  return reinterpret_cast<double*>(b.refl + (size_t)head * kEigReflBytes);
}
__device__ __forceinline__ double* eig_vec_row(const EigBufs& b, int head, int row) {
  char* base = row < kD / 2 ? b.vec_lo + (size_t)head * kHalfBytes : b.refl + (size_t)head * kEigReflBytes;
  return reinterpret_cast<double*>(base) + (size_t)(row & (kD / 2 - 1)) * kD;
}
// [2], behind the rows of V: sweeps logged so far + kJacLaunchEnded for each launch whose sweeps have
// ended, and the blocks that have come to the head's launches
__device__ __forceinline__ int* eig_progress(const EigBufs& b, int head) {
  return reinterpret_cast<int*>(b.refl + (size_t)head * kEigReflBytes + kHalfBytes);
}
constexpr int kJacLaunchEnded = 1 << 16;
__device__ __forceinline__ double* eig_mass(const EigBufs& b, int head) {  // [slices][2]: off-diagonal, diagonal squares
  return reinterpret_cast<double*>(b.refl + (size_t)head * kEigReflBytes + kHalfBytes) + 2;
}
__device__ __forceinline__ double* eig_log(const EigBufs& b, int head, int i) {
  return reinterpret_cast<double*>(
      i < 2 ? reinterpret_cast<char*>(b.cov) + (size_t)head * kMatBytes + (size_t)i * kHalfBytes
            : b.more_logs + ((size_t)head * (b.n_logs - 2) + (i - 2)) * kHalfBytes);
}

template <int CTRL>
__device__ __forceinline__ double dpp_mov_f64(double x) {
  const long long v = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(v & 0xffffffffLL), CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double readlane_f64(double x, int lane) {
  const long long v = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readlane((int)(v & 0xffffffffLL), lane);
  const int hi = __builtin_amdgcn_readlane((int)(v >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
// sum over each aligned group of 16 lanes, to every lane of it
__device__ __forceinline__ double row_sum_f64(double x) {
  x += dpp_mov_f64<kDppQuadXor1>(x);
  x += dpp_mov_f64<kDppQuadXor2>(x);
  x += dpp_mov_f64<kDppRowHalfMirror>(x);
  x += dpp_mov_f64<kDppRowMirror>(x);
  return x;
}
__device__ __forceinline__ double wave_sum_f64(double x) {  // all 64 lanes active
  x = row_sum_f64(x);
  return (readlane_f64(x, 0) + readlane_f64(x, 16)) + (readlane_f64(x, 32) + readlane_f64(x, 48));
}

// ---- Householder tridiagonalisation ------------------------------------------------------------
__device__ __forceinline__ double fast_rcp_f64(double x) {  // two Newton steps: full precision but for the last place
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  r = fma(fma(-x, r, 1.0), r, r);
  return r;
}
__device__ __forceinline__ double fast_rsqrt_f64(double x) {  // likewise
  double y = __builtin_amdgcn_rsq(x);
  y = fma(y, 0.5 * fma(-x * y, y, 1.0), y);
  y = fma(y, 0.5 * fma(-x * y, y, 1.0), y);
  return y;
}

// Four waves: wave w holds rows 4 u + w, u = 0..31, lane l columns l and l + 64 (128 registers), so
// all waves keep live rows to the end, every wave sees whole rows (norms and dot products need no
// exchange) and a row's value read from LDS serves two columns.  Reflector j is u = x - beta e(j+1)
// with x the row's part beyond j (zeros up to j) and H = I - u u^T / h: u differs from x in one
// place, so the product with A starts on x while the norm is still being taken.  A step is one
// barrier, behind which the four partial sums of p = A u and row j + 1 as it was are in LDS: every
// wave then has all of p and brings that row up to date for itself, so the next step begins without
// an exchange.  What bounds it is the chain of a step (two sums over a wave, a square root, a
// reciprocal), about 2000 cycles.  Measured, 32 heads: 125 us; with a second barrier, for the next
// row from the wave that owns it, 131; with eight waves and that barrier 146; as two 64-row halves
// with four barriers a step, the library's square root and divisions and a branch around every
// group of rows 197.
// PER_CU = 2, for more heads than CUs: two blocks share a CU, a wave having at most 256 registers.
// The next row is then taken before the rows of the matrix are updated, so that it need not be kept
// beside them (240 registers for 292, 2 us more for a block alone).  257 heads: 177 us as before
// that kernel had one barrier, with one block per CU 254.
template <int PER_CU>
__global__ __launch_bounds__(kEigThreads, PER_CU) void tridiag_kernel(EigBufs bufs) {
  constexpr int kWaves = kEigThreads / 64, kRows = kD / kWaves, kPitch = kRows + 2;
  constexpr int kChunk = 4;  // rows of a wave that are skipped together once they are done
  static_assert(kWaves == 4, "four partial sums");
  // (a wave is at most one barrier ahead of another: two sets take turns)
  __shared__ __align__(16) double s_p[2][kWaves][kD], s_row[2][kD];
  __shared__ __align__(16) double s_pr[kWaves][kPitch], s_xr[kWaves][kPitch];  // a wave's own rows, for itself
  const int tid = threadIdx.x, lane = tid & 63, head = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const double* C = bufs.cov + (size_t)head * kD * kD;
  double* tri = eig_tri(bufs, head);
  double* refl = eig_refl(bufs, head);
  if (tid == 0) bufs.state[head] = 0;

  double a[kRows][2], x[2];
#pragma unroll
  for (int u = 0; u < kRows; ++u)
#pragma unroll
    for (int h = 0; h < 2; ++h) a[u][h] = C[(size_t)(kWaves * u + wave) * kD + lane + 64 * h];
  // `row` up to date: its entries beyond the diagonal become x, the diagonal is done
  auto take_row = [&](int row, const double (&v)[2]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int c = lane + 64 * h;
      x[h] = c > row ? v[h] : 0.0;
      if (wave == 0 && c == row) tri[row] = v[h];
      if (c % kWaves == wave) s_xr[wave][c / kWaves] = x[h];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  auto at_column = [&](const double (&v)[2], int c) { return readlane_f64(c < 64 ? v[0] : v[1], c & 63); };
  {
    const double first[2] = {C[lane], C[lane + 64]};
    take_row(0, first);
  }

  // the steps whose next row lies in rows 16 seg .. 16 seg + 15: straight-line code over the live rows
  auto steps = [&](auto seg) {
    constexpr int kLive = decltype(seg)::value * kChunk;  // first live row index of a wave
    for (int j = max(kWaves * kLive - 1, 0); j < min(kWaves * (kLive + kChunk) - 1, kD - 2); ++j) {
      const int next = j + 1, next_wave = next % kWaves, next_u = next / kWaves, set = j & 1;
      double u[2], xr[kRows], p[2] = {0.0, 0.0}, p2[2] = {0.0, 0.0};
      const double alpha = at_column(x, next);
#pragma unroll
      for (int i = kLive; i < kRows; i += 2) {
        const double2 v = *reinterpret_cast<const double2*>(&s_xr[wave][i]);
        xr[i] = v.x;
        xr[i + 1] = v.y;
      }
      double sel[2];  // row j + 1 in its wave, else 0
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        sel[h] = a[kLive][h];
#pragma unroll
        for (int i = kLive + 1; i < kLive + kChunk; ++i) sel[h] = i == next_u ? a[i][h] : sel[h];
        if (wave == next_wave) s_row[set][lane + 64 * h] = sel[h];
        sel[h] = wave == next_wave ? sel[h] : 0.0;
      }
      const double t0 = lane > next ? x[0] : 0.0, t1 = lane + 64 > next ? x[1] : 0.0;
      const double tail = wave_sum_f64(fma(t0, t0, t1 * t1));
#pragma unroll
      for (int i = kLive; i < kRows; i += 2)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          p[h] = fma(a[i][h], xr[i], p[h]);
          p2[h] = fma(a[i + 1][h], xr[i + 1], p2[h]);
        }
      double beta = alpha, inv_h = 0.0, top = 0.0;  // nothing to clear: no reflector
      if (tail != 0.0) {
        const double s2 = fma(alpha, alpha, tail), rs = fast_rsqrt_f64(s2);
        const double nrm = fma(0.5 * rs, fma(-(s2 * rs), s2 * rs, s2), s2 * rs);
        beta = -copysign(nrm, alpha);
        top = alpha - beta;                          // u[j + 1]
        inv_h = fast_rcp_f64(fma(fabs(alpha), nrm, s2));
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        u[h] = lane + 64 * h == next ? top : x[h];
        s_p[set][wave][lane + 64 * h] = fma(-beta, sel[h], p[h] + p2[h]);
      }
      if (wave == 0) {
#pragma unroll
        for (int h = 0; h < 2; ++h) refl[(size_t)j * kD + lane + 64 * h] = u[h];
        if (lane == 0) {
          tri[kD + j] = beta;
          tri[2 * kD + j] = inv_h;
        }
      }
      __syncthreads();
      double row[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int c = lane + 64 * h;
        row[h] = s_row[set][c];
        p[h] = (s_p[set][0][c] + s_p[set][1][c]) + (s_p[set][2][c] + s_p[set][3][c]);
        if (c % kWaves == wave) s_pr[wave][c / kWaves] = p[h];
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      // A -= u w^T + w u^T with w = p / h - k u: row r, column c lose u_r (p_c / h - 2 k u_c) + p_r u_c / h
      const double k2 = inv_h * inv_h * wave_sum_f64(fma(p[0], u[0], p[1] * u[1]));
      const double pn = at_column(p, next);
      double f[2], g[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        f[h] = fma(-k2, u[h], p[h] * inv_h);
        g[h] = inv_h * u[h];
        row[h] = fma(-top, f[h], fma(-pn, g[h], row[h]));
      }
      if constexpr (PER_CU == 2) take_row(next, row);  // (this step's own rows are in xr)
#pragma unroll
      for (int i = kLive; i < kRows; i += 2) {  // (row j + 1, where u is not x, is done)
        const double2 pr = *reinterpret_cast<const double2*>(&s_pr[wave][i]);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          a[i][h] = fma(-xr[i], f[h], fma(-pr.x, g[h], a[i][h]));
          a[i + 1][h] = fma(-xr[i + 1], f[h], fma(-pr.y, g[h], a[i + 1][h]));
        }
      }
      if constexpr (PER_CU == 1) take_row(next, row);
    }
  };
  steps(std::integral_constant<int, 0>{});
  steps(std::integral_constant<int, 1>{});
  steps(std::integral_constant<int, 2>{});
  steps(std::integral_constant<int, 3>{});
  steps(std::integral_constant<int, 4>{});
  steps(std::integral_constant<int, 5>{});
  steps(std::integral_constant<int, 6>{});
  steps(std::integral_constant<int, 7>{});
  static_assert(kRows == 8 * kChunk, "eight segments");
  // rows 126 (left in x) and 127
  if (tid == 63) tri[kD + kD - 2] = x[1];
  if (tid == kEigThreads - 1) tri[kD - 1] = a[kRows - 1][1];
}

// v_mfma_f64_16x16x4_f64: lane l gives row (column) l % 16 of A (B) at k = l / 16 and holds column
// l % 16, rows l / 16 + 4 i of the result.
typedef double f64x4_t __attribute__((ext_vector_type(4)));

// lane N of each aligned group of 16 lanes, to every lane of it
template <int N>
__device__ __forceinline__ double row_bcast_f64(double x) { return dpp_mov_f64<0x150 + N>(x); }

// ---- eigenpairs of the tridiagonal matrix ------------------------------------------------------
// Block (head, slice): eigenvalues 16 slice .. 16 slice + 15 in increasing order, 16 threads each.
// Multisection: a pass evaluates the Sturm count at 16 points of the bracket, 13 passes of 1/17 take
// the Gershgorin interval to 2e-16 of its length (a pass is a chain of 128 dependent steps
// whatever the number of points).  The counts use the determinants' recurrence, one dependent
// multiply-add a step, and not the quotients', whose reciprocal makes the chain six times as
// long (the kernel, 32 heads: 89 us against 169, with the reflectors still on the vector units);
// the determinants are scaled by a power of two every 8 steps, and the matrix to norm 1, so that
// nothing over- or underflows.  The twisted factorisation runs its two directions in two lane groups
// at once and needs no starting vector; the reflectors are applied sixteen at a time on the matrix
// cores, the vectors lying in the accumulators (64 us).
__global__ __launch_bounds__(kEigThreads) void eigvec_kernel(EigBufs bufs) {
  constexpr int kN = kEigSliceRows;
  constexpr int kPasses = 13;
  constexpr int kReflChunk = 16;  // reflectors applied at a time
  constexpr int kChunks = kD / kReflChunk, kGramPitch = kReflChunk + 1;
  constexpr double kTiny = 1e-30;
  __shared__ __align__(16) double2 s_de[kD];  // (d_i, e_(i-1)^2) of the scaled matrix
  __shared__ double s_e[kD], s_invh[kD], s_lam[kN], s_sq[2][kN];
  __shared__ int s_r[kN];
  // products of a chunk's reflectors with each other, row > column; the parts and the whole of their
  // products with the vectors
  __shared__ double s_gram[kChunks][kReflChunk][kGramPitch];
  __shared__ double s_w[kEigThreads / 64][kReflChunk][kN + 1], s_c[kReflChunk][kN + 1];
  __shared__ __align__(16) double s_buf[2 * kD * kN];  // the factors L, U
  __shared__ double s_dp[kD][kN], s_z[kD][kN + 1], s_dd[kD][kN + 1];
  double(*s_l)[kN] = reinterpret_cast<double(*)[kN]>(s_buf);
  double(*s_u)[kN] = reinterpret_cast<double(*)[kN]>(s_buf + kD * kN);
  static_assert(kN == 16 && kReflChunk == 16 && kEigThreads == 256, "a matrix instruction's tile, a thread for each of its entries");
  const int tid = threadIdx.x, lane = tid & 63, slice = blockIdx.y, head = blockIdx.x;
  if (head >= bufs.n_heads) return;
  const int n16 = tid >> 4, sub = tid & 15;
  const double* tri = eig_tri(bufs, head);
  // the Gershgorin interval (every wave for itself)
  double lo = 1e300, hi = -1e300;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int i = lane + 64 * h;
    const double r = (i < kD - 1 ? fabs(tri[kD + i]) : 0.0) + (i > 0 ? fabs(tri[kD + i - 1]) : 0.0);
    lo = fmin(lo, tri[i] - r);
    hi = fmax(hi, tri[i] + r);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, off));
    hi = fmax(hi, __shfl_xor(hi, off));
  }
  const double inv_norm = 1.0 / fmax(fmax(fabs(lo), fabs(hi)), 1e-290);
  lo = fma(lo, inv_norm, -1e-15);
  hi = fma(hi, inv_norm, 1e-15);
  if (tid < kD) {
    const double e = tid < kD - 1 ? tri[kD + tid] * inv_norm : 0.0;
    const double ep = tid > 0 ? tri[kD + tid - 1] * inv_norm : 0.0;
    s_e[tid] = e;
    // (a floor far below rounding: the determinants never vanish twice in a row)
    s_de[tid] = make_double2(tri[tid] * inv_norm, fmax(ep * ep, kTiny * kTiny));
    s_invh[tid] = tid < kD - 2 ? tri[2 * kD + tid] : 0.0;
  }
  __syncthreads();
  const int want = slice * kN + n16;
#pragma unroll 1
  for (int pass = 0; pass < kPasses; ++pass) {
    const double step = (hi - lo) * (1.0 / 17.0);
    const double x = fma((double)(sub + 1), step, lo);
    // eigenvalues below x = sign changes of the leading determinants of T - x
    double p0 = 0.0, p = 1.0;
    unsigned below = 0, last = 0;
    double2 da[8], db[8];  // 8 rows in use, 8 on their way
    auto fetch = [&](double2 (&de)[8], int i0) {
#pragma unroll
      for (int e = 0; e < 8; ++e) de[e] = s_de[i0 + e];
    };
    unsigned signs = 0;  // of the last 32 determinants, one bit each
    auto advance = [&](const double2 (&de)[8]) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const double pn = fma(de[e].x - x, p, -(de[e].y * p0));
        p0 = p;
        p = pn;
        signs = __builtin_amdgcn_alignbit(signs, (unsigned)__double2hiint(p), 31);
      }
      const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(p), fabs(p0)));
      p = __builtin_amdgcn_ldexp(p, ex);
      p0 = __builtin_amdgcn_ldexp(p0, ex);
    };
    fetch(da, 0);
#pragma unroll 1
    for (int i0 = 0; i0 < kD; i0 += 32) {
      fetch(db, i0 + 8);
      advance(da);
      fetch(da, i0 + 16);
      advance(db);
      fetch(db, i0 + 24);
      advance(da);
      fetch(da, min(i0 + 32, kD - 8));
      advance(db);
      below += __popc(signs ^ ((signs >> 1) | (last << 31)));
      last = signs & 1u;
    }
    // points with at most `want` eigenvalues below them lie left of eigenvalue `want`
    const unsigned long long left = __ballot((int)below <= want);
    const int m = __popc((unsigned)(left >> (lane & 48)) & 0xffffu);
    const double nlo = m > 0 ? fma((double)m, step, lo) : lo;
    hi = m < 16 ? fma((double)(m + 1), step, lo) : hi;
    lo = nlo;
  }
  if (sub == 0) s_lam[n16] = 0.5 * (lo + hi);
  __syncthreads();

  // T - lambda = L+ D+ L+^T from the top (lanes 0-15) and U- D- U-^T from the bottom (lanes 16-31):
  // the pivots are the quotients of neighbouring determinants, so the chain is the one above and
  // the divisions are done side by side afterwards
  if (tid < 2 * kN) {
    const int n = sub;
    const bool up = tid >= kN;
    const double lam = s_lam[n];
    double p0 = 0.0, p = 1.0;
    double(*num)[kN] = up ? s_u : s_l;
    double(*den)[kN + 1] = up ? s_dd : s_z;
    double da[8], ea[8], db[8], eb[8];  // 8 rows in use, 8 on their way
    auto fetch = [&](double (&d)[8], double (&e2)[8], int i0) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int i = up ? kD - 1 - (i0 + e) : i0 + e;
        d[e] = s_de[i].x;
        e2[e] = s_de[up ? min(i + 1, kD - 1) : i].y;  // (the first step's meets p0 = 0)
      }
    };
    auto advance = [&](const double (&d)[8], const double (&e2)[8], int i0) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int i = up ? kD - 1 - (i0 + e) : i0 + e;
        const double pn = fma(d[e] - lam, p, -(e2[e] * p0));
        num[i][n] = pn;
        den[i][n] = p;
        p0 = p;
        p = pn;
      }
      const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(p), fabs(p0)));
      p = __builtin_amdgcn_ldexp(p, ex);
      p0 = __builtin_amdgcn_ldexp(p0, ex);
    };
    fetch(da, ea, 0);
#pragma unroll 1
    for (int i0 = 0; i0 < kD; i0 += 16) {
      fetch(db, eb, i0 + 8);
      advance(da, ea, i0);
      fetch(da, ea, min(i0 + 16, kD - 8));
      advance(db, eb, i0 + 8);
    }
  } else if (tid >= 64) {
    // meanwhile the other waves: the products of a chunk's reflectors with each other (k permuted alike
    // for both operands, which are then the same registers; reflectors 126 and 127 do not exist)
    const int r16 = lane & 15, kg = lane >> 4;
    for (int c = (tid >> 6) - 1; c < kChunks; c += kEigThreads / 64 - 1) {
      const int row = kReflChunk * c + r16;
      const double* v = eig_refl(bufs, head) + (size_t)min(row, kD - 3) * kD + 2 * kg;
      double2 x[kD / 8];
#pragma unroll
      for (int t = 0; t < kD / 8; ++t) x[t] = *reinterpret_cast<const double2*>(v + 8 * t);
      f64x4_t g0{0.0, 0.0, 0.0, 0.0}, g1{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int t = 0; t < kD / 8; ++t) {
        if (row > kD - 3) x[t] = make_double2(0.0, 0.0);
        g0 = __builtin_amdgcn_mfma_f64_16x16x4f64(x[t].x, x[t].x, g0, 0, 0, 0);
        g1 = __builtin_amdgcn_mfma_f64_16x16x4f64(x[t].y, x[t].y, g1, 0, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) s_gram[c][kg + 4 * i][r16] = kg + 4 * i > r16 ? g0[i] + g1[i] : 0.0;
    }
  }
  __syncthreads();
  {
    // thread (n16, sub): rows sub + 16 u of vector n16
    auto pivot = [&](double num, double den, double& q, double& rq) {
      const bool small = fabs(num) < kTiny * fabs(den);
      q = small ? (num < 0.0 ? -kTiny : kTiny) : num * fast_rcp_f64(den);
      rq = small ? (num < 0.0 ? -1.0 / kTiny : 1.0 / kTiny) : den * fast_rcp_f64(num);
    };
    double l[kD / 16], u[kD / 16];
#pragma unroll
    for (int k = 0; k < kD / 16; ++k) {
      const int i = sub + 16 * k, j = min(i + 1, kD - 1);
      double q, rq, q2, rq2;
      pivot(s_l[i][n16], s_z[i][n16], q, rq);     // D+[i]
      pivot(s_u[j][n16], s_dd[j][n16], q2, rq2);  // D-[i + 1]
      s_dp[i][n16] = q;
      l[k] = s_e[i] * rq;
      u[k] = s_e[i] * rq2;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kD / 16; ++k) {
      s_l[sub + 16 * k][n16] = l[k];
      s_u[sub + 16 * k][n16] = u[k];
    }
  }
  __syncthreads();
  // the twist: the smallest |D+[r] - U-[r] e[r]| (the last row has no U)
  {
    double best = 1e300;
    int at = 0;
    for (int i = sub; i < kD; i += 16) {
      const double g = fabs(i < kD - 1 ? fma(-s_u[i][n16], s_e[i], s_dp[i][n16]) : s_dp[i][n16]);
      if (g < best) {
        best = g;
        at = i;
      }
    }
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) {
      const double b2 = __shfl_xor(best, off);
      const int a2 = __shfl_xor(at, off);
      if (b2 < best || (b2 == best && a2 < at)) {
        best = b2;
        at = a2;
      }
    }
    if (sub == 0) s_r[n16] = at;
  }
  __syncthreads();
  if (tid < kN) {  // the vector above its twist ...
    const int r = s_r[tid];
    double z = 1.0, sq = 1.0;
    s_z[r][tid] = 1.0;
#pragma unroll 4
    for (int i = r - 1; i >= 0; --i) {
      z *= -s_l[i][tid];
      s_z[i][tid] = z;
      sq = fma(z, z, sq);
    }
    s_sq[0][tid] = sq;
  } else if (tid < 2 * kN) {  // ... and below it
    const int n = tid - kN, r = s_r[n];
    double z = 1.0, sq = 0.0;
#pragma unroll 4
    for (int i = r; i < kD - 1; ++i) {
      z *= -s_u[i][n];
      s_z[i + 1][n] = z;
      sq = fma(z, z, sq);
    }
    s_sq[1][n] = sq;
  }
  __syncthreads();
  // Back through the reflectors, z <- (I - u u^T / h) z, last reflector first, 16 at a time: their
  // products with the 16 vectors on the matrix cores (every wave's 32 entries for themselves, added
  // up in LDS), corrected one reflector after the other by their products with each other, and the
  // vectors less the reflectors times the result, on the matrix cores again.  A wave holds entries
  // 32 wave + 16 t + 4 (lane / 16) + i of vector lane % 16 as the accumulators lie, which is also how
  // the first product takes them.
  {
    const int wave = tid >> 6, r16 = lane & 15, kg = lane >> 4;
    const double* refl = eig_refl(bufs, head);
    f64x4_t z[2];
    {
      const double inv = 1.0 / sqrt(s_sq[0][r16] + s_sq[1][r16]);
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) z[t][i] = s_z[32 * wave + 16 * t + 4 * kg + i][r16] * inv;
    }
    double2 aw[2][2];   // this wave's entries of reflector r16
    double au[2][4];    // entry 4 (r16 % 4) + r16 / 4 of its tiles, reflectors kg, kg + 4, ..
    auto fetch = [&](int c) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int e0 = 32 * wave + 16 * t;
        const double* v = refl + (size_t)min(kReflChunk * c + r16, kD - 3) * kD + e0 + 4 * kg;
        aw[t][0] = *reinterpret_cast<const double2*>(v);
        aw[t][1] = *reinterpret_cast<const double2*>(v + 2);
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4)
          au[t][s4] = refl[(size_t)min(kReflChunk * c + 4 * s4 + kg, kD - 3) * kD + e0 + 4 * (r16 & 3) + (r16 >> 2)];
      }
    };
    fetch(kChunks - 1);
#pragma unroll 1
    for (int c = kChunks - 1; c >= 0; --c) {
      f64x4_t w{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        w = __builtin_amdgcn_mfma_f64_16x16x4f64(aw[t][0].x, z[t][0], w, 0, 0, 0);
        w = __builtin_amdgcn_mfma_f64_16x16x4f64(aw[t][0].y, z[t][1], w, 0, 0, 0);
        w = __builtin_amdgcn_mfma_f64_16x16x4f64(aw[t][1].x, z[t][2], w, 0, 0, 0);
        w = __builtin_amdgcn_mfma_f64_16x16x4f64(aw[t][1].y, z[t][3], w, 0, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) s_w[wave][kg + 4 * i][r16] = w[i];
      double u[2][4];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) u[t][s4] = au[t][s4];
      fetch(max(c - 1, 0));
      // thread (n16, sub): reflector sub of the chunk, vector n16 (a reflector that does not exist: inv_h = 0)
      double g[kReflChunk];
#pragma unroll
      for (int n = 1; n < kReflChunk; ++n) g[n] = s_gram[c][n][sub];
      const bool exists = kReflChunk * c + sub < kD - 2;
      const double ih = -s_invh[kReflChunk * c + sub];
      __syncthreads();
      double x = (s_w[0][sub][n16] + s_w[1][sub][n16]) + (s_w[2][sub][n16] + s_w[3][sub][n16]);
      if (!exists) x = 0.0;
      x = fma(row_bcast_f64<15>(ih * x), g[15], x);
      x = fma(row_bcast_f64<14>(ih * x), g[14], x);
      x = fma(row_bcast_f64<13>(ih * x), g[13], x);
      x = fma(row_bcast_f64<12>(ih * x), g[12], x);
      x = fma(row_bcast_f64<11>(ih * x), g[11], x);
      x = fma(row_bcast_f64<10>(ih * x), g[10], x);
      x = fma(row_bcast_f64<9>(ih * x), g[9], x);
      x = fma(row_bcast_f64<8>(ih * x), g[8], x);
      x = fma(row_bcast_f64<7>(ih * x), g[7], x);
      x = fma(row_bcast_f64<6>(ih * x), g[6], x);
      x = fma(row_bcast_f64<5>(ih * x), g[5], x);
      x = fma(row_bcast_f64<4>(ih * x), g[4], x);
      x = fma(row_bcast_f64<3>(ih * x), g[3], x);
      x = fma(row_bcast_f64<2>(ih * x), g[2], x);
      x = fma(row_bcast_f64<1>(ih * x), g[1], x);
      s_c[sub][n16] = ih * x;
      __syncthreads();
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4) {
        const double cf = s_c[4 * s4 + kg][r16];
#pragma unroll
        for (int t = 0; t < 2; ++t) z[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(u[t][s4], cf, z[t], 0, 0, 0);
      }
    }
    double* Z = bufs.mat + (size_t)head * kD * kD + (size_t)(slice * kN + r16) * kD + 32 * wave + 4 * kg;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      *reinterpret_cast<double2*>(Z + 16 * t) = make_double2(z[t][0], z[t][1]);
      *reinterpret_cast<double2*>(Z + 16 * t + 2) = make_double2(z[t][2], z[t][3]);
    }
  }
}

// ---- products of whole matrices with a 16-row slice ----------------------------------------------
// Four waves, two 16-row tiles of the whole matrix each;
// operands come straight from the matrix in L2 (16 bytes a lane, k permuted alike for both: k =
// 8 t + 2 (l / 16) + {0, 1}), so all loads of a product can be in flight at once.  Through tiles
// staged in LDS and the vector units, with a barrier per tile, the two kernels took 28 and 33 us.
constexpr int kSlicePitch = kD + 2;     // doubles per row of a slice in LDS
constexpr int kTilesPerWave = kD / 16 / (kEigThreads / 64);

// acc[n] += X[16-row tile n of this wave] Y^T; x(row), y: this lane's rows
template <typename RowX>
__device__ __forceinline__ void slice_product(RowX x, const double* y, f64x4_t (&acc)[kTilesPerWave]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, at = 2 * (lane >> 4);
  const double* xr[kTilesPerWave];
#pragma unroll
  for (int n = 0; n < kTilesPerWave; ++n) {
    xr[n] = x(16 * (kTilesPerWave * wave + n) + (lane & 15)) + at;
    acc[n] = f64x4_t{0.0, 0.0, 0.0, 0.0};
  }
#pragma unroll
  for (int t = 0; t < kD / 8; ++t) {
    const double2 b = *reinterpret_cast<const double2*>(y + at + 8 * t);
#pragma unroll
    for (int n = 0; n < kTilesPerWave; ++n) {
      const double2 a = *reinterpret_cast<const double2*>(xr[n] + 8 * t);
      acc[n] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, acc[n], 0, 0, 0);
      acc[n] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.y, acc[n], 0, 0, 0);
    }
  }
}

// V <- V - (V V^T - I) V / 2 for rows 16 slice .. of V (components are rows): the Newton-Schulz step
// towards the nearest orthonormal set.  Marks the head when a product of two rows, or a norm, is off
// by more than kOrthTolerance (also when it is not a number).
__global__ __launch_bounds__(kEigThreads) void orthonormalise_kernel(EigBufs bufs) {
  __shared__ __align__(16) double s_m[kEigSliceRows * kSlicePitch];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r16 = lane & 15, kg = lane >> 4;
  const int slice = blockIdx.y, head = blockIdx.x, r0 = slice * kEigSliceRows;
  if (head >= bufs.n_heads) return;
  const double* Z = bufs.mat + (size_t)head * kD * kD;
  f64x4_t acc[kTilesPerWave];
  slice_product([&](int k) { return Z + (size_t)k * kD; }, Z + (size_t)(r0 + r16) * kD, acc);
  bool off = false;
#pragma unroll
  for (int n = 0; n < kTilesPerWave; ++n)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k = 16 * (kTilesPerWave * wave + n) + kg + 4 * i;
      const double m = acc[n][i] - (k == r0 + r16 ? 1.0 : 0.0);
      off |= !(fabs(m) <= kOrthTolerance);
      s_m[r16 * kSlicePitch + k] = m;
    }
  if (off) atomicOr(&bufs.state[head], kStateMarked);
  __syncthreads();
  // (M Z)[s][i]: A = M's rows from LDS, B = 16 columns of Z
#pragma unroll
  for (int n = 0; n < kTilesPerWave; ++n) {
    const int i0 = 16 * (kTilesPerWave * wave + n);
    f64x4_t o{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < kD; k += 4)
      o = __builtin_amdgcn_mfma_f64_16x16x4f64(s_m[r16 * kSlicePitch + k + kg], Z[(size_t)(k + kg) * kD + i0 + r16], o, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int s = kg + 4 * i;
      eig_vec_row(bufs, head, r0 + s)[i0 + r16] = fma(-0.5, o[i], Z[(size_t)(r0 + s) * kD + i0 + r16]);
    }
  }
}

// Columns 16 slice .. of B = V C V^T (symmetric) and their share of its diagonal and off-diagonal
// mass; B = C and V = I for a marked head.
__global__ __launch_bounds__(kEigThreads) void project_kernel(EigBufs bufs) {
  __shared__ __align__(16) double s_t[kEigSliceRows * kSlicePitch];
  __shared__ double s_mass[kEigThreads / 64][2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r16 = lane & 15, kg = lane >> 4;
  const int slice = blockIdx.y, head = blockIdx.x, r0 = slice * kEigSliceRows;
  if (head >= bufs.n_heads) return;
  const double* C = bufs.cov + (size_t)head * kD * kD;
  double* B = bufs.mat + (size_t)head * kD * kD;
  if (slice == 0 && tid < 2) eig_progress(bufs, head)[tid] = 0;
  if (bufs.state[head] & kStateMarked) {  // (uniform; set by the launch before)
    for (int e = tid; e < kEigSliceRows * kD; e += kEigThreads) {
      const int r = r0 + e / kD, i = e % kD;
      B[(size_t)r * kD + i] = C[(size_t)r * kD + i];
      eig_vec_row(bufs, head, r)[i] = r == i ? 1.0 : 0.0;
    }
    return;
  }
  f64x4_t acc[kTilesPerWave];
  slice_product([&](int k) { return C + (size_t)k * kD; }, eig_vec_row(bufs, head, r0 + r16), acc);  // C is symmetric
#pragma unroll
  for (int n = 0; n < kTilesPerWave; ++n)
#pragma unroll
    for (int i = 0; i < 4; ++i) s_t[r16 * kSlicePitch + 16 * (kTilesPerWave * wave + n) + kg + 4 * i] = acc[n][i];
  __syncthreads();
  slice_product([&](int k) { return eig_vec_row(bufs, head, k); }, s_t + r16 * kSlicePitch, acc);
  double off = 0.0, dg = 0.0;
#pragma unroll
  for (int n = 0; n < kTilesPerWave; ++n)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k = 16 * (kTilesPerWave * wave + n) + kg + 4 * i;
      const double x = acc[n][i];
      B[(size_t)k * kD + r0 + r16] = x;
      if (k == r0 + r16) dg += x * x; else off += x * x;
    }
  off = wave_sum_f64(off);
  dg = wave_sum_f64(dg);
  if (lane == 0) {
    s_mass[wave][0] = off;
    s_mass[wave][1] = dg;
  }
  __syncthreads();
  if (tid < 2) eig_mass(bufs, head)[2 * slice + tid] = (s_mass[0][tid] + s_mass[1][tid]) + (s_mass[2][tid] + s_mass[3][tid]);
}

// ---- cyclic Jacobi -------------------------------------------------------------------------------
// round-robin pairing of 128 indices: slot 0 pairs (round, 127), slot t pairs
// ((round + t) % 127, (round - t) % 127); returned with p < q
__device__ __forceinline__ void jacobi_pair(int round, int slot, int& p, int& q) {
  if (slot == 0) {
    p = round;
    q = kD - 1;
  } else {
    p = (round + slot) % (kD - 1);
    q = (round - slot + (kD - 1)) % (kD - 1);
  }
  if (p > q) {
    const int t = p;
    p = q;
    q = t;
  }
}

__device__ __forceinline__ void jacobi_rotation(double t, double& cs, double& sn) {
  cs = 1.0 / sqrt(t * t + 1.0);
  sn = t * cs;
}

// One launch takes a head through as many sweeps as it has logs.  Of its five blocks the first to come
// runs the sweeps on B, resident in LDS (129 KiB), and logs every rotation's tangent; the others replay the
// logs on V, whose columns never mix, 32 columns each in LDS, a sweep as soon as it is logged.  So they
// wait for a block that runs already and itself waits for nobody, however many of the launch's blocks the
// device holds.  The host, which cannot know how many sweeps a head will need, enqueues kJacMaxSweeps / n_logs
// launches whose blocks leave at once when the head is solved; with the sweeps of one launch replayed in the
// next, which takes two sets of logs, it was over twice as many, 2 to 4 us each: fit of 32 x 65536 keys
// 321 -> 315 us, 8 x 7000 (9 launches -> 4) 253 -> 242.  A sweep is 127 rounds of 64 disjoint rotations; rows and
// columns of a round are rotated in one pass over 2 x 2 blocks of the upper triangle.
__device__ void jacobi_sweeps(const EigBufs& bufs, int head, int launch, double* A) {
  __shared__ double s_c[kD / 2], s_s[kD / 2];
  __shared__ int s_p[kD / 2], s_q[kD / 2];
  __shared__ double s_red[kJacThreads / 64];
  const int tid = threadIdx.x, per_launch = bufs.n_logs - bufs.defer;
  int* progress = eig_progress(bufs, head);
  bool solved = false;
  double* Ag = bufs.mat + (size_t)head * kD * kD;
  for (int e = tid; e < kD * kD; e += kJacThreads) A[(e / kD) * kJacPitch + e % kD] = Ag[e];
  __syncthreads();
  if (launch == 0) {  // B's two halves were computed apart: equal but for rounding
    for (int e = tid; e < kD * kD; e += kJacThreads) {
      const int i = e / kD, j = e % kD;
      if (i < j) A[i * kJacPitch + j] = A[j * kJacPitch + i] = 0.5 * (A[i * kJacPitch + j] + A[j * kJacPitch + i]);
    }
    __syncthreads();
  }
  auto block_sum = [&](double x) -> double {
    x = wave_sum_f64(x);
    __syncthreads();
    if ((tid & 63) == 0) s_red[tid >> 6] = x;
    __syncthreads();
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kJacThreads / 64; ++w) t += s_red[w];
    return t;
  };
  int sweep = 0;
  for (; sweep < per_launch; ++sweep) {
    // solved when the off-diagonal mass is at rounding level of the diagonal's
    double off = 0.0, dg = 0.0;
    for (int e = tid; e < kD * kD; e += kJacThreads) {
      const double x = A[(e / kD) * kJacPitch + e % kD];
      if (e / kD == e % kD) dg += x * x; else if (e / kD < e % kD) off += 2.0 * x * x;
    }
    off = block_sum(off);
    dg = block_sum(dg);
    solved = off <= kOffTolerance * dg || dg == 0.0;  // uniform: every thread holds the same sums
    if (solved) break;
    double* log = eig_log(bufs, head, (launch * per_launch + sweep) % bufs.n_logs);
    for (int round = 0; round < kJacRounds; ++round) {
      if (tid < kD / 2) {
        int p, q;
        jacobi_pair(round, tid, p, q);
        const double app = A[p * kJacPitch + p], aqq = A[q * kJacPitch + q], apq = A[p * kJacPitch + q];
        double t = 0.0;
        if (fabs(apq) > 1e-300) {
          const double theta = (aqq - app) / (2.0 * apq);
          t = (theta >= 0.0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
        }
        double cs, sn;
        jacobi_rotation(t, cs, sn);
        s_p[tid] = p; s_q[tid] = q; s_c[tid] = cs; s_s[tid] = sn;
        log[round * (kD / 2) + tid] = t;
        // the pair's own 2 x 2 block
        A[p * kJacPitch + p] = fma(-t, apq, app);
        A[q * kJacPitch + q] = fma(t, apq, aqq);
        A[p * kJacPitch + q] = t != 0.0 ? 0.0 : apq;
      }
      __syncthreads();
      // the 2 x 2 blocks of two different pairs, each once (only the upper triangle is kept): slots
      // (i, i + 1 ..) of row i and (63 - i, ..) of row 63 - i make 63 blocks for every i < 32
      for (int it = tid; it < (kD / 4) * (kD / 2 - 1); it += kJacThreads) {
        const int i = it / (kD / 2 - 1), b = it % (kD / 2 - 1);
        const bool first = b < kD / 2 - 1 - i;
        const int pr = first ? i : kD / 2 - 1 - i, pc = first ? i + 1 + b : b + 1;
        const int p = s_p[pr], q = s_q[pr], p2 = s_p[pc], q2 = s_q[pc];
        const double cs = s_c[pr], sn = s_s[pr], cs2 = s_c[pc], sn2 = s_s[pc];
        double& app = A[min(p, p2) * kJacPitch + max(p, p2)];
        double& apq = A[min(p, q2) * kJacPitch + max(p, q2)];
        double& aqp = A[min(q, p2) * kJacPitch + max(q, p2)];
        double& aqq = A[min(q, q2) * kJacPitch + max(q, q2)];
        const double xpp = app, xpq = apq, xqp = aqp, xqq = aqq;
        const double tpp = cs * xpp - sn * xqp, tqp = sn * xpp + cs * xqp;  // rows p, q at column p2
        const double tpq = cs * xpq - sn * xqq, tqq = sn * xpq + cs * xqq;  // rows p, q at column q2
        app = cs2 * tpp - sn2 * tpq;
        apq = sn2 * tpp + cs2 * tpq;
        aqp = cs2 * tqp - sn2 * tqq;
        aqq = sn2 * tqp + cs2 * tqq;
      }
      __syncthreads();
    }
    if (tid == 0)  // (behind a barrier: the block's stores of the log have left its waves)
      __hip_atomic_fetch_add(progress, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (tid == 0) {
    if (solved) bufs.state[head] |= kStateSolvedIn * (launch + 1);
    __hip_atomic_fetch_add(progress, kJacLaunchEnded, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (sweep > 0)
    for (int e = tid; e < kD * kD; e += kJacThreads) Ag[e] = A[(e / kD) * kJacPitch + e % kD];
}

// A wave owns two columns and a lane one pair of a round, so rounds need no barrier.
__device__ void jacobi_accumulate(const EigBufs& bufs, int head, int slice, int launch, double* s_v) {
  constexpr int kPitch = kJacSliceCols + 1;
  __shared__ int s_seen;
  const int tid = threadIdx.x, lane = tid & 63, i0 = slice * kJacSliceCols;
  // every launch before went to its last log
  const int per_launch = bufs.n_logs - bufs.defer, end = (launch + 1) * per_launch;
  const int first = launch * per_launch - (launch > 0 ? bufs.defer : 0);
  const int last = end < kJacMaxSweeps ? end - bufs.defer : end;
  for (int e = tid; e < kD * kJacSliceCols; e += kJacThreads)
    s_v[(e / kJacSliceCols) * kPitch + e % kJacSliceCols] = eig_vec_row(bufs, head, e / kJacSliceCols)[i0 + e % kJacSliceCols];
  double* column = s_v + 2 * (tid >> 6);
  for (int sweep = first;; ++sweep) {
    __syncthreads();
    if (tid == 0) {
      int seen = 0;
      for (int polls = 0; polls < kJacMaxPolls; ++polls) {
        seen = __hip_atomic_load(eig_progress(bufs, head), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (seen % kJacLaunchEnded > sweep || seen / kJacLaunchEnded > launch || sweep >= last) break;
        __builtin_amdgcn_s_sleep(8);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      s_seen = seen;
    }
    __syncthreads();
    const bool logged = s_seen % kJacLaunchEnded > sweep, ended = s_seen / kJacLaunchEnded > launch;
    // (a launch that ended before its last sweep solved the head: nothing is left to the next)
    if (!logged && !ended && sweep < last) {
      // the wait was given up: no result rather than a wrong one (no sweep takes a thousandth of that time)
      for (int e = tid; e < kD * kJacSliceCols; e += kJacThreads)
        eig_vec_row(bufs, head, e / kJacSliceCols)[i0 + e % kJacSliceCols] = __builtin_nan("");
      return;
    }
    if (!logged || sweep >= last) break;
    const double* log = eig_log(bufs, head, sweep % bufs.n_logs) + lane;
    double t = log[0], t1 = log[kD / 2];
    for (int round = 0; round < kJacRounds; ++round) {
      const double t2 = log[(size_t)min(round + 2, kJacRounds - 1) * (kD / 2)];
      int p, q;
      jacobi_pair(round, lane, p, q);
      double cs, sn;
      jacobi_rotation(t, cs, sn);
      double* vp = column + p * kPitch;
      double* vq = column + q * kPitch;
      const double x0 = vp[0], x1 = vp[1], y0 = vq[0], y1 = vq[1];
      vp[0] = cs * x0 - sn * y0;
      vp[1] = cs * x1 - sn * y1;
      vq[0] = sn * x0 + cs * y0;
      vq[1] = sn * x1 + cs * y1;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // the lanes' pairs of the next round
      t = t1;
      t1 = t2;
    }
  }
  for (int e = tid; e < kD * kJacSliceCols; e += kJacThreads)
    eig_vec_row(bufs, head, e / kJacSliceCols)[i0 + e % kJacSliceCols] = s_v[(e / kJacSliceCols) * kPitch + e % kJacSliceCols];
}

__global__ __launch_bounds__(kJacThreads) void jacobi_kernel(EigBufs bufs, int launch) {
  extern __shared__ __align__(16) unsigned char jac_smem[];
  __shared__ int s_turn;
  double* mem = reinterpret_cast<double*>(jac_smem);
  const int head = blockIdx.x;
  // Solved before this launch?  (uniform, and the same for all blocks of the head: what the sweeping block
  // writes meanwhile names this launch)
  const int state = bufs.state[head], solved_in = state / kStateSolvedIn;
  if (solved_in != 0 && solved_in <= launch) return;
  if (launch == 0 && !(state & kStateMarked)) {
    double off = 0.0, dg = 0.0;
    for (int s = 0; s < kEigSlices; ++s) {
      off += eig_mass(bufs, head)[2 * s];
      dg += eig_mass(bufs, head)[2 * s + 1];
    }
    if (off <= kOffTolerance * dg || dg == 0.0) {
      if (blockIdx.y == 0 && threadIdx.x == 0) bufs.state[head] = state | kStateSolvedIn;
      return;
    }
  }
  if (threadIdx.x == 0) s_turn = atomicAdd(eig_progress(bufs, head) + 1, 1) - launch * (1 + kJacSlices);
  __syncthreads();
  if (s_turn == 0) jacobi_sweeps(bufs, head, launch, mem);
  else jacobi_accumulate(bufs, head, s_turn - 1, launch, mem);
}

// ---- results ---------------------------------------------------------------------------------------
// Block (slice, head): components of rank 16 slice .. in decreasing eigenvalue order (ties: the lower
// index first), each with its largest entry positive (ties: the first); P's columns leave 64 bytes a row.
__global__ __launch_bounds__(kEigThreads) void finish_kernel(EigBufs bufs, float* __restrict__ P,
                                                             float* __restrict__ eigenvalues) {
  __shared__ double s_diag[kD];
  __shared__ int s_comp[kEigSliceRows];
  __shared__ float s_out[kD][kEigSliceRows + 1];
  const int tid = threadIdx.x, slice = blockIdx.y, head = blockIdx.x;
  if (head >= bufs.n_heads) return;
  const int n16 = tid >> 4, sub = tid & 15;
  if (tid < kD) s_diag[tid] = bufs.mat[(size_t)head * kD * kD + (size_t)tid * kD + tid];
  if (tid < kEigSliceRows) s_comp[tid] = slice * kEigSliceRows + tid;  // (stands only where values are not numbers)
  __syncthreads();
  if (tid < kD) {
    const double mine = s_diag[tid];
    int rank = 0;
    for (int j = 0; j < kD; ++j) {
      const double other = s_diag[j];
      rank += (other > mine || (other == mine && j < tid)) ? 1 : 0;
    }
    if (rank / kEigSliceRows == slice) {
      s_comp[rank % kEigSliceRows] = tid;
      eigenvalues[(size_t)head * kD + rank] = (float)mine;
    }
  }
  __syncthreads();
  const double* v = eig_vec_row(bufs, head, s_comp[n16]);
  double x[kD / 16], best = 0.0;
  int at = 0;
#pragma unroll
  for (int u = 0; u < kD / 16; ++u) {
    x[u] = v[sub + 16 * u];
    if (fabs(x[u]) > fabs(best)) {
      best = x[u];
      at = sub + 16 * u;
    }
  }
#pragma unroll
  for (int off = 8; off > 0; off >>= 1) {
    const double b2 = __shfl_xor(best, off);
    const int a2 = __shfl_xor(at, off);
    if (fabs(b2) > fabs(best) || (fabs(b2) == fabs(best) && a2 < at)) {
      best = b2;
      at = a2;
    }
  }
  const double sgn = best < 0.0 ? -1.0 : 1.0;
#pragma unroll
  for (int u = 0; u < kD / 16; ++u) s_out[sub + 16 * u][n16] = (float)(sgn * x[u]);
  __syncthreads();
  float* Ph = P + (size_t)head * kD * kD + slice * kEigSliceRows;
  for (int e = tid; e < kD * kEigSliceRows; e += kEigThreads)
    Ph[(size_t)(e / kEigSliceRows) * kD + e % kEigSliceRows] = s_out[e / kEigSliceRows][e % kEigSliceRows];
}

hipError_t launch_eigensolver(int Hkv, const EigRegions& r, float* P, float* eigenvalues, hipStream_t st) {
  EigBufs b;
  b.cov = r.cov;
  b.mat = r.mat;
  b.vec_lo = r.spare;
  b.refl = r.refl;
  b.more_logs = r.spare + (size_t)Hkv * kHalfBytes;
  b.state = r.state;
  b.n_heads = Hkv;
  b.n_logs = std::min(2 + (r.spare_halves - 1), kJacMaxSweeps);
  static std::atomic<unsigned long long> lds_allowed{0};  // devices already set up
  const size_t lds = (size_t)kD * kJacPitch * sizeof(double);
  const hipError_t ea = allow_dynamic_lds(reinterpret_cast<const void*>(jacobi_kernel), (int)lds, lds_allowed);
  if (ea != hipSuccess) return ea;
  // Blocks go to the 8 dies in turn, so with heads counted first, up to a multiple of 8, the slices of a head
  // share a die and find the head's matrices in its L2.  us per fit, slices first / so: 32 x 65536
  // keys 315 / 308, 8 x 7000 242 / 237.
  const dim3 slices((Hkv + 7) / 8 * 8, kEigSlices);
  if (Hkv > device_cus())
    hipLaunchKernelGGL(tridiag_kernel<2>, dim3(Hkv), dim3(kEigThreads), 0, st, b);
  else
    hipLaunchKernelGGL(tridiag_kernel<1>, dim3(Hkv), dim3(kEigThreads), 0, st, b);
  hipLaunchKernelGGL(eigvec_kernel, slices, dim3(kEigThreads), 0, st, b);
  hipLaunchKernelGGL(orthonormalise_kernel, slices, dim3(kEigThreads), 0, st, b);
  hipLaunchKernelGGL(project_kernel, slices, dim3(kEigThreads), 0, st, b);
  // The replay of a launch's last sweep is all that runs when it has been logged.  With few logs, so few
  // rows that the keys may well be rank-deficient, it is left to the next launch, beside whose sweeps it runs
  // (us, left / not, and with a barrier in every round of the replay: 32 heads of 100 keys 3596 / 4118, 130 of 3000
  // with dead columns 4541 / 5034).
  b.defer = b.n_logs <= 4 ? 1 : 0;
  for (int l = 0; l * (b.n_logs - b.defer) < kJacMaxSweeps; ++l)
    hipLaunchKernelGGL(jacobi_kernel, dim3(Hkv, 1 + kJacSlices), dim3(kJacThreads), lds, st, b, l);
  hipLaunchKernelGGL(finish_kernel, slices, dim3(kEigThreads), 0, st, b, P, eigenvalues);
  return hipGetLastError();
}

}  // namespace loki
