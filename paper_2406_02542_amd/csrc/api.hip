// C ABI of the Loki decode-attention library: argument validation, workspace planning and
// kernel sequencing.  See include/loki.h for the contract of every entry point.
#include "../../include/loki.h"

#include <hip/hip_runtime.h>

#include <atomic>
#include <new>

#include "launch.h"

namespace loki {

static inline int div_up(int a, int b) { return (a + b - 1) / b; }
static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

int device_cus() {
  constexpr int kSlots = 64;
  static std::atomic<int> cached[kSlots];
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kSlots) {
    (void)hipGetLastError();  // a size query without a device is not an error of a later launch
    return kDefaultCUs;
  }
  int n = cached[dev].load(std::memory_order_relaxed);
  if (n > 0) return n;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) {
    (void)hipGetLastError();
    n = kDefaultCUs;
  }
  cached[dev].store(n, std::memory_order_relaxed);
  return n;
}

hipError_t allow_dynamic_lds(const void* kernel, int bytes, std::atomic<unsigned long long>& done) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return hipErrorInvalidDevice;
  const unsigned long long bit = 1ull << (dev & 63);
  if (dev < 64 && (done.load(std::memory_order_acquire) & bit)) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess && dev < 64) done.fetch_or(bit, std::memory_order_release);
  return e;
}

int score_rows_per_block(const Shape& s) {
  const int units = s.B * s.Hkv;
  int nchunks = div_up(kScoreBlocksPerCU * device_cus(), units);
  const int max_chunks = div_up(s.S, 2 * kScoreRowsPerStep);
  if (nchunks > max_chunks) nchunks = max_chunks;
  if (nchunks < 1) nchunks = 1;
  int rows = div_up(div_up(s.S, nchunks), kScoreRowsPerStep) * kScoreRowsPerStep;
  if (s.S > 16384) {
    // long sequences: a block stays inside one 16384-row chunk of the selection (it adds its
    // counts into that chunk's histogram): a power of two of at most 16384 rows
    int r = kScoreRowsPerStep;
    while (2 * r <= rows && 2 * r <= 16384) r *= 2;
    rows = r;
  }
  if (s.pg.table != nullptr) {
    // a block must lie inside one page: the largest power of two (>= 256) within rows and the page
    const int page_rows = 1 << s.pg.lg_rows;
    int r = kScoreRowsPerStep;
    while (2 * r <= rows && 2 * r <= page_rows) r *= 2;
    rows = r;
  }
  return rows;
}

// From 90 MB a call on, the bytes it reads of its caches.  The last-level cache holds 256 MiB, so a
// smaller call finds rows there that it read itself a call or two before, or that the step before it
// in a model left there, and loads past the caches are slower then; larger ones find none and read
// 8 to 12 % faster.  us, through / past the caches, each over three copies of its inputs in turn:
//   one block per head: 602 MB of cache, 80 heads, S = 5230 49.8 / 45.3; 16 x 32 heads, S = 4096,
//     384 MB read 68.8 / 61.0, on pages 55.4 / 49.5; 96 heads, S = 4853, 82 MB 32.4 / 33.2, 64
//     heads, S = 4122, 16 MB 16.3 / 18.1
//   groups, values only: 151 MB 43.6 / 40.5, 125 MB 35.1 / 33.7, 93 MB 39.2 / 36.4; 46 MB 36.7 /
//     37.9, 24 MB 33.1 / 33.7
//   dense: 241 MB 48.1 / 42.6, 123 MB 28.7 / 26.0; 83 MB 18.5 / 19.2, 73 MB 19.7 / 19.9, 46 MB 13.8
//     / 15.1
// Heads that select for themselves in a group, or tokens of a sequence, find rows that the others
// have just read: not beyond half of the rows (72 units of 8 heads, k = S / 8 42.1 / 44.4; 2 tokens,
// k = S / 4, one head 63.8 / 57.8; groups of 4, k = S / 16 91.1 / 86.8).  At the line, lists of one row more and
// of half together: 16 x 32/8 heads, S = 16384 142.9 / 131.9, 8 x 32/16, S = 16000 132.6 / 129.1, 32 x 64/8,
// S = 8192, d = 64 171.6 / 163.1; 2 tokens of 4 x 32 heads, S = 6000 58.4 / 54.4.
// And not in groups beyond 16384 rows, where it turns on how much the heads' lists have in common (4 x 32/8
// heads, S = 131072, k = 8192 207 / 203, 169 / 173 with attention peaked on the same rows).
// Lengths of their own are not known here, so the blocks add them up and decide.  us, through / past / as the
// blocks decide, batches laid out for S rows of which every sequence holds an eighth, a quarter, half and all:
//   16 x 32 heads, S = 4096      46 MB 19.8 / 21.6 / 19.9   92 26.6 / 27.8 / 27.9   185 39.5 / 35.0 / 35.2   369 71.0 / 63.0 / 63.0
//   8 x 32 fp32 heads, S = 3000  34 MB 15.3 / 16.5 / 15.5   67 18.3 / 19.3 / 18.4   135 32.5 / 29.3 / 29.4   270 54.4 / 48.9 / 48.9
//   dense, 10 x 32, S = 2000     41 MB 14.2 / 16.8 / 14.9   82 20.8 / 22.6 / 20.9   164 37.3 / 33.6 / 34.0   328 60.8 / 54.3 / 54.5
// (Adding up costs 0 to 0.5 us of a launch, in those of groups up to 1.4, whose first loads wait for it.)
//
// The attention of a group with one selection reads the slab again, for the selected rows, a line of 128 bytes
// for each; a slab that was loaded past the caches is not there then.  So it pays while the lines read again are
// few beside the slab, and from 80 MB of slab on.  Time through / past the caches by the slab's size and by
// `again`, the lines' bytes over the slab's (2, 4 and 8 heads, 64 to 512 units, d = 16 and 32, contiguous
// and paged, 150 shapes):
//   again   50-60 MB     90 MB        110-134 MB   160 MB       200 MB       260 MB
//   0.12    0.98-1.00    1.03-1.06    1.05-1.10    1.10-1.11    1.09-1.12    1.06-1.09
//   0.17                 1.04-1.05    1.05-1.08                 1.07-1.09    1.03
//   0.25    0.97-1.00    1.03-1.05    1.04-1.08    1.03-1.04    0.99-1.01    0.99
//   0.4     1.01         1.02         0.97-1.01    0.97-0.98    0.97         0.98-0.99
//   0.5     1.01-1.02    0.97-0.98    0.96-0.97
// Slab rows of more than 64 bytes take two loads of half a line: never (d = 64: 0.87 to 0.94).
RowLoads row_loads(const Shape& s, int select_mode) {
  const int tokens = s.rg.queries > 1 ? s.rg.queries : 1;
  const bool known = s.rg.seq_lens == nullptr && s.rg.ks == nullptr;
  const float head_bytes = (float)s.Hkv * (float)s.elem_bytes, rows = (float)s.B * (float)s.S, kept = (float)s.B * (float)s.k;
  RowLoads l;
  if (select_mode == 0 && s.G > 1 && s.S > 16384) return l;
  l.entries = s.B;
  l.max_share = 1e30f;
  if (select_mode == kEveryRow) {
    l.row_bytes = head_bytes * 2 * kD;
  } else if (select_mode == kLowRankRows) {
    l.row_bytes = head_bytes * (float)(kD + s.d);
  } else {
    const int lists = select_mode == 0 ? s.G : 1;  // of a KV head and batch entry
    l.row_bytes = head_bytes * (float)s.d / (float)tokens;
    l.kept_bytes = head_bytes * (float)(lists * (2 * kD - (select_mode == 0 ? s.d : 0)));
    if (tokens * lists > 1) l.max_share = 0.5f / (float)(tokens * lists);
    if (select_mode == kGroupLaunch && s.d <= 8 * kSlabChunksPast) l.again_bytes = 128.0f * (float)s.Hkv;
  }
  if (known)
    l.form = loads_form(l, rows, kept);
  else if (rows * l.row_bytes + kept * l.kept_bytes >= kPastBytes)  // (else no lengths up to S reach it)
    l.form = kByLengths;
  return l;
}

int gather_splits(const Shape& s, int select_mode) {
  const int heads = (select_mode == 1) ? s.B * s.Hkv : s.B * s.Hq;
  // about two blocks per CU: a block's set-up and merge cost as much as a few hundred rows, and
  // a launch that needs no split also needs no combine kernel
  int n = div_up(2 * device_cus(), heads);
  const int max_n = s.k / 128 > 0 ? s.k / 128 : 1;
  if (n > max_n) n = max_n;
  const int min_n = div_up(s.k, kMaxGatherChunk);
  if (n < min_n) n = min_n;
  return n;
}

// Eight blocks per CU of at least 256 rows: at least dense_splits at any length up to S, which a workspace is
// sized for (one sized at the longest length serves all shorter ones).
static int max_dense_splits(const Shape& s) {
  const int n = div_up(8 * device_cus(), s.B * s.Hkv);
  const int max_n = s.S / 256 > 0 ? s.S / 256 : 1;
  return n > max_n ? max_n : n;
}

// Row splits of dense attention and of Algorithm 2, of at least 256 rows.  As many as make two
// blocks per CU in bf16 and four in fp32, where that fills nine tenths of those places: a block's
// set-up and merge, and the parts the combine launch reads, cost more than a smoother last round
// gains, and a few blocks over a full round cost most.  Against eight per CU, us: 16 sequences of
// 32/8 heads at S = 16384 191 -> 181 (three per CU 183, four 186), 7 of them at S = 12000 73 -> 66
// (rounded up to 2.2 per CU: 80), 32/32 heads at S = 4096 188 -> 178, 64/8 heads at S = 8192 105 ->
// 97; Algorithm 2 121 -> 114, 129 -> 120, 136 -> 125; fp32, 9 sequences of 32/16 heads at S = 5790
// 154 -> 149.  Otherwise eight per CU (10 sequences of 32 heads, S = 4000: 116, unsplit 120), and
// also where that makes one full round of three small blocks per CU (48 units, S = 4186: 25.2, two
// larger per CU 26.0), and for long blocks of fp32 groups of 8, of which a CU holds three (132
// units, S = 16159: eight 439, four 467; short ones, 33 units, S = 10370: 92.5, 82.1). Sequences of
// unequal length: the same counts, and for bf16 first three per CU, as many as are resident (16 of
// 32/8 heads, S = 16384: two 133, three 130, four 131), where the blocks are dealt out by length
// (dense_balanced); never unsplit, which ends with the longest sequence (25 of 40 fp32 heads, S =
// 2076, most of them short: eight 46, unsplit 78), and in fp32 from eight sequences on only dealt
// out (14 of 24/12 heads, S = 1798, eight 16.0, four 17.3; 6 of 32/4, S = 15561, 79.0, 69.4).
int dense_splits(const Shape& s, bool ragged) {
  const int units = s.B * s.Hkv, cus = device_cus();
  const int max_n = s.S / 256 > 0 ? s.S / 256 : 1;
  const int many = max_dense_splits(s);
  auto full = [&](int n, int per_cu) { return n >= 1 && n <= max_n && 10LL * units * n >= 9LL * per_cu * cus; };
  if (ragged && s.dtype == 1) {
    const int n = 3 * cus / units;
    if (full(n, 3) && dense_balanced(s, n)) return n;
  }
  const int per_cu = s.dtype == 1 ? 2 : 4;
  const int n = per_cu * cus / units;
  if (!full(n, per_cu) || (ragged && (n == 1 || (s.dtype == 0 && s.B >= 8 && !dense_balanced(s, n))))) return many;
  if (!ragged && s.dtype == 0 && s.G == 8 && s.S >= 1024 * n) return many;
  if (s.S < 512 * n && full(many, 3) && many * units <= 3 * cus) return many;
  return n;
}

// Whether dense attention over sequences of unequal length deals its blocks out by length
// (dense_runs; a kernel variant of its own): up to 64 sequences, and only where a block has at
// least 512 rows of the longest: working it out takes about 1 us, which shorter blocks do not win
// back (16 units, S = 3000: 14.1 -> 15.0 us).  Every round of blocks pays it anew; with eight per
// CU, as cut / dealt out: 288 units of one head, S = 6338, lengths from S / 4 on 128 / 114, 320
// units, S = 18990 417 / 399; but 800 units, S = 2687, most of them an eighth as long 26.6 / 28.7.
bool dense_balanced(const Shape& s, int nsplit) {
  return s.rg.seq_lens != nullptr && nsplit > 1 && s.B <= kDenseMaxRagged && s.S >= 512 * nsplit;
}

Workspace plan_workspace(const Shape& s, int select_mode, int nsplit, void* base, bool with_cluster) {
  Workspace w{};
  char* p = static_cast<char*>(base);
  size_t off = 0;
  const size_t heads_q = (size_t)s.B * s.Hq;
  auto take = [&](size_t bytes) {
    char* r = p ? p + off : nullptr;
    off += align_up(bytes, 256);
    return r;
  };
  if (select_mode == -2) w.qhat = reinterpret_cast<float*>(take(heads_q * kD * sizeof(float)));
  if (select_mode >= 0) {
    const size_t heads_sel = (select_mode == 1) ? (size_t)s.B * s.Hkv : heads_q;
    w.cluster_ctl = reinterpret_cast<uint32_t*>(take(kClusterCtlBytes));  // at offset 0 for every shape
    w.qhat = reinterpret_cast<float*>(take(heads_q * kD * sizeof(float)));
    w.scores = reinterpret_cast<float*>(take(heads_sel * s.S * sizeof(float)));
    w.sel_idx = reinterpret_cast<int32_t*>(take(heads_sel * s.k * sizeof(int32_t)));
    w.sel_score = reinterpret_cast<float*>(take(heads_sel * s.k * sizeof(float)));
    w.ticket_words = align_up(heads_q * sizeof(int32_t), 256) / 4;
    w.tickets = reinterpret_cast<int32_t*>(take(w.ticket_words * 4));
    const size_t scratch_words = select_scratch_words(s.S, (int)heads_sel);
    w.sel_scratch = scratch_words ? reinterpret_cast<uint32_t*>(take(scratch_words * 4)) : nullptr;
    if (scratch_words && !p) w.sel_scratch = nullptr;
    const size_t cluster_bytes = with_cluster ? fused_gqa_cluster_bytes(s, select_mode) : 0;
    w.cluster = cluster_bytes ? take(cluster_bytes) : nullptr;
  }
  w.partial = reinterpret_cast<float*>(
      take(nsplit > 1 ? heads_q * nsplit * (size_t)(kD + 2) * sizeof(float) : 0));
  w.total_bytes = off;
  return w;
}

// ---- stage timing ---------------------------------------------------------------------
}  // namespace loki

struct loki_profile {
  hipEvent_t ev[2 * LOKI_PROFILE_MAX_KERNELS];
  const char* names[LOKI_PROFILE_MAX_KERNELS];
  int n;
};

namespace loki {

static thread_local loki_profile* t_profile = nullptr;

struct StageTimer {
  hipStream_t st;
  explicit StageTimer(hipStream_t s) : st(s) {
    if (t_profile) t_profile->n = 0;
  }
  void begin(const char* name) {
    loki_profile* p = t_profile;
    if (!p || p->n >= LOKI_PROFILE_MAX_KERNELS) return;
    p->names[p->n] = name;
    (void)hipEventRecord(p->ev[2 * p->n], st);
  }
  void end() {
    loki_profile* p = t_profile;
    if (!p || p->n >= LOKI_PROFILE_MAX_KERNELS) return;
    (void)hipEventRecord(p->ev[2 * p->n + 1], st);
    p->n++;
  }
};

static int check_layout(const loki_layout* L, Shape* s) {
  if (!L) return LOKI_ERR_INVALID_ARG;
  if (L->B < 1 || L->Hq < 1 || L->Hkv < 1 || L->S_cap < 1) return LOKI_ERR_INVALID_ARG;
  if (L->Hq % L->Hkv != 0) return LOKI_ERR_INVALID_ARG;
  if (L->dtype != LOKI_F32 && L->dtype != LOKI_BF16) return LOKI_ERR_UNSUPPORTED;
  if (L->D != 128) return LOKI_ERR_UNSUPPORTED;
  const int eb = L->dtype == LOKI_F32 ? 4 : 2;
  if (L->d_split < 1 || L->d_split > L->D) return LOKI_ERR_INVALID_ARG;
  if ((L->d_split * eb) % 16 != 0) return LOKI_ERR_UNSUPPORTED;
  const int G = L->Hq / L->Hkv;
  if (G != 1 && G != 2 && G != 4 && G != 8) return LOKI_ERR_UNSUPPORTED;
  // heads index the second grid dimension of several kernels (at most 65 535 blocks)
  if ((long long)L->B * L->Hq > 65535) return LOKI_ERR_UNSUPPORTED;
  s->B = L->B;
  s->Hq = L->Hq;
  s->Hkv = L->Hkv;
  s->G = G;
  s->S_cap = L->S_cap;
  s->S = 0;
  s->d = L->d_split;
  s->k = 0;
  s->dtype = L->dtype;
  s->elem_bytes = eb;
  return LOKI_OK;
}

static inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
static inline bool aligned256(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 255u) == 0; }

// ---- built-in scratch for callers that cannot allocate (loki_decode_attn_static) -----------
// Every GPU the library runs on holds its own copy of this array, at its own address, until the
// process ends.  In host code the array's name is only a handle for hipGetSymbolAddress: the
// device address is looked up once per device (with that device current) and kept, and only
// that address is ever handed to a kernel.
static __device__ __align__(256) unsigned char scratch[LOKI_STATIC_SCRATCH_BYTES];
constexpr int kMaxDevices = 64;
static std::atomic<void*> g_scratch_ptr[kMaxDevices];

static int static_scratch_address(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return LOKI_ERR_HIP;
  if (dev < 0 || dev >= kMaxDevices) return LOKI_ERR_UNSUPPORTED;
  void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (ptr == nullptr) {
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr)
      return LOKI_ERR_HIP;
    g_scratch_ptr[dev].store(ptr, std::memory_order_release);  // every thread finds the same address
  }
  *out = ptr;
  return LOKI_OK;
}

}  // namespace loki

using namespace loki;

// Measurement aid: streams `n16` 16-byte words through the load path and discards them.  The
// time of this kernel over as many bytes as a decode step moves is the practical ceiling of
// a read-bound kernel on the device it runs on.
namespace loki {
__device__ unsigned g_stream_read_sink;
__global__ __launch_bounds__(512) void stream_read_kernel(const uint4* __restrict__ p, size_t n16) {
  unsigned acc = 0;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (; i + 3 * stride < n16; i += 4 * stride) {
    uint4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = p[i + u * stride];
#pragma unroll
    for (int u = 0; u < 4; ++u) acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
  }
  for (; i < n16; i += stride) {
    const uint4 v = p[i];
    acc ^= v.x ^ v.y ^ v.z ^ v.w;
  }
  if (acc == 0x9e3779b9u) g_stream_read_sink = acc;  // keeps the loads alive
}
}  // namespace loki

extern "C" {

int loki_version(void) { return 110; }

const char* loki_status_string(int status) {
  switch (status) {
    case LOKI_OK: return "ok";
    case LOKI_ERR_INVALID_ARG: return "invalid argument";
    case LOKI_ERR_UNSUPPORTED: return "unsupported configuration";
    case LOKI_ERR_ALIGNMENT: return "pointer not sufficiently aligned";
    case LOKI_ERR_WORKSPACE: return "workspace too small";
    case LOKI_ERR_HIP: return "HIP runtime error";
    case LOKI_ERR_SCRATCH_LIMIT: return "shape needs more than the built-in scratch buffer";
    default: return "unknown status";
  }
}

int loki_cache_bytes(const loki_layout* layout, size_t* klo_bytes, size_t* khi_bytes,
                     size_t* v_bytes) {
  Shape s;
  const int rc = check_layout(layout, &s);
  if (rc != LOKI_OK) return rc;
  if (!klo_bytes || !khi_bytes || !v_bytes) return LOKI_ERR_INVALID_ARG;
  const size_t rows = (size_t)s.B * s.Hkv * s.S_cap;
  *klo_bytes = rows * s.d * s.elem_bytes;
  *khi_bytes = rows * (128 - s.d) * s.elem_bytes;
  *v_bytes = rows * 128 * s.elem_bytes;
  return LOKI_OK;
}

int loki_workspace_bytes(const loki_layout* layout, int S, int d, int k, int select_mode,
                         size_t* bytes) {
  Shape s;
  const int rc = check_layout(layout, &s);
  if (rc != LOKI_OK) return rc;
  if (!bytes) return LOKI_ERR_INVALID_ARG;
  if (S < 1 || S > s.S_cap) return LOKI_ERR_INVALID_ARG;
  s.S = S;
  if (select_mode == -1 || select_mode == -2) {  // dense baseline; PCAAttn (rotated queries too)
    *bytes = plan_workspace(s, select_mode, max_dense_splits(s), nullptr).total_bytes;
    return LOKI_OK;
  }
  if (select_mode < 0) return LOKI_ERR_INVALID_ARG;
  select_mode &= ~(LOKI_PATH_MASK | LOKI_WORKSPACE_ZEROED);
  if (select_mode != LOKI_SELECT_PER_QUERY_HEAD && select_mode != LOKI_SELECT_PER_KV_GROUP)
    return LOKI_ERR_INVALID_ARG;
  if (d != s.d) return LOKI_ERR_UNSUPPORTED;
  if (k < 1 || k > S) return LOKI_ERR_INVALID_ARG;
  s.k = k;
  *bytes = plan_workspace(s, select_mode, gather_splits(s, select_mode), nullptr).total_bytes;
  return LOKI_OK;
}

static int paging_from_args(const int32_t* page_table, int page_rows, int pages_per_seq, int n_pages,
                            int Hkv, long long rows_needed, Paging* pg) {
  int lg = 0;
  while (lg < 31 && (1 << lg) < page_rows) ++lg;
  if (page_rows < 1 || (1 << lg) != page_rows) return LOKI_ERR_INVALID_ARG;
  if (lg < 8 || lg > 24 || pages_per_seq < 1 || n_pages < 1) return LOKI_ERR_INVALID_ARG;
  if ((long long)pages_per_seq * page_rows < rows_needed) return LOKI_ERR_INVALID_ARG;
  if ((long long)n_pages * Hkv * page_rows > 0x7fffffffLL) return LOKI_ERR_UNSUPPORTED;
  if (reinterpret_cast<uintptr_t>(page_table) & 3u) return LOKI_ERR_ALIGNMENT;
  pg->table = page_table;
  pg->lg_rows = lg;
  pg->pages_per_seq = pages_per_seq;
  pg->n_pages = n_pages;
  return LOKI_OK;
}

static int rotate_impl(const loki_layout* layout, const void* k_new, const float* P, void* klo,
                       void* khi, int pos, int n_new, const Paging* pg, void* stream) {
  Shape s;
  const int rc = check_layout(layout, &s);
  if (rc != LOKI_OK) return rc;
  if (!k_new || !P || !klo) return LOKI_ERR_INVALID_ARG;
  if (s.d < 128 && !khi) return LOKI_ERR_INVALID_ARG;
  if (pos < 0 || n_new < 1 || (long long)pos + n_new > s.S_cap) return LOKI_ERR_INVALID_ARG;
  if (!aligned16(k_new) || !aligned16(P) || !aligned16(klo) || !aligned16(khi))
    return LOKI_ERR_ALIGNMENT;
  if (pg) s.pg = *pg;
  hipStream_t st = static_cast<hipStream_t>(stream);
  StageTimer tm(st);
  tm.begin("rotate_keys");
  const hipError_t e = launch_rotate(s, k_new, P, klo, khi, pos, n_new, st);
  tm.end();
  return e == hipSuccess ? LOKI_OK : LOKI_ERR_HIP;
}

int loki_rotate_keys(const loki_layout* layout, const void* k_new, const float* P, void* klo,
                     void* khi, int pos, int n_new, void* stream) {
  return rotate_impl(layout, k_new, P, klo, khi, pos, n_new, nullptr, stream);
}

int loki_rotate_keys_paged(const loki_layout* layout, const void* k_new, const float* P, void* klo,
                           void* khi, const int32_t* page_table, int page_rows, int pages_per_seq,
                           int n_pages, int pos, int n_new, void* stream) {
  if (!layout || !page_table) return LOKI_ERR_INVALID_ARG;
  if (pos < 0 || n_new < 1) return LOKI_ERR_INVALID_ARG;
  Paging pg;
  const int rc = paging_from_args(page_table, page_rows, pages_per_seq, n_pages, layout->Hkv,
                                  (long long)pos + n_new, &pg);
  if (rc != LOKI_OK) return rc;
  return rotate_impl(layout, k_new, P, klo, khi, pos, n_new, &pg, stream);
}

// The decode step behind loki_decode_attn (no per-sequence sizes, no append) and
// loki_decode_step.
static int decode_impl(const loki_layout* layout, const void* q, const float* P, void* klo, void* khi,
                       void* v, int S, int d, int k, int select_mode, const Ragged& rg,
                       const Append& ap, const Paging& pg, void* workspace, size_t workspace_bytes,
                       void* out, int32_t* out_idx, void* stream) {
  Shape s;
  const int rc = check_layout(layout, &s);
  if (rc != LOKI_OK) return rc;
  if (rg.queries < 1 || rg.queries > 64) return LOKI_ERR_INVALID_ARG;
  if (rg.queries > 1) {
    // every query of a sequence is a batch entry of its own from here on; the kernels map
    // entry b back to the cache of sequence b / queries
    if ((long long)s.B * rg.queries * s.Hq > 65535) return LOKI_ERR_UNSUPPORTED;
    if (rg.seq_lens == nullptr) return LOKI_ERR_INVALID_ARG;  // each query has its own causal length
    s.B *= rg.queries;
  }
  if (!q || !P || !klo || !v || !out || !workspace) return LOKI_ERR_INVALID_ARG;
  if (s.d < 128 && !khi) return LOKI_ERR_INVALID_ARG;
  const int path = select_mode & LOKI_PATH_MASK;
  const bool ws_zeroed = (select_mode & LOKI_WORKSPACE_ZEROED) != 0;
  select_mode &= ~(LOKI_PATH_MASK | LOKI_WORKSPACE_ZEROED);
  if (select_mode != LOKI_SELECT_PER_QUERY_HEAD && select_mode != LOKI_SELECT_PER_KV_GROUP)
    return LOKI_ERR_INVALID_ARG;
  if (path != 0 && path != LOKI_PATH_SPLIT && path != LOKI_PATH_FUSED && path != LOKI_PATH_CLUSTER)
    return LOKI_ERR_INVALID_ARG;
  if (S < 1 || S > s.S_cap) return LOKI_ERR_INVALID_ARG;
  if (k < 1 || k > S) return LOKI_ERR_INVALID_ARG;
  if (d != s.d) return LOKI_ERR_UNSUPPORTED;
  if ((ap.k_new == nullptr) != (ap.v_new == nullptr)) return LOKI_ERR_INVALID_ARG;
  if (!aligned16(q) || !aligned16(P) || !aligned16(klo) || !aligned16(khi) || !aligned16(v) ||
      !aligned16(out) || !aligned16(out_idx) || !aligned16(ap.k_new) || !aligned16(ap.v_new))
    return LOKI_ERR_ALIGNMENT;
  if ((reinterpret_cast<uintptr_t>(rg.seq_lens) & 3u) || (reinterpret_cast<uintptr_t>(rg.ks) & 3u))
    return LOKI_ERR_ALIGNMENT;
  if (!aligned256(workspace)) return LOKI_ERR_ALIGNMENT;
  s.S = S;
  s.k = k;
  s.rg = rg;
  s.ap = ap;
  s.pg = pg;
  if (s.G == 1) select_mode = LOKI_SELECT_PER_QUERY_HEAD;  // identical; one code path
  const int nsplit = gather_splits(s, select_mode);
  Workspace w = plan_workspace(s, select_mode, nsplit, workspace);
  if (w.total_bytes > workspace_bytes && w.cluster != nullptr && path != LOKI_PATH_CLUSTER)
    w = plan_workspace(s, select_mode, nsplit, workspace, false);  // no room for the exchange area: the other sequences
  if (w.total_bytes > workspace_bytes) return LOKI_ERR_WORKSPACE;

  hipStream_t st = static_cast<hipStream_t>(stream);
  const int heads_sel = (select_mode == 1) ? s.B * s.Hkv : s.B * s.Hq;
  int32_t* idx = out_idx ? out_idx : w.sel_idx;
  StageTimer tm(st);
  hipError_t e;
  // (pinned, the single launches of groups refuse page tables of more than 64 pages per sequence, that of one
  // query head per KV head of more than 32 (fused_pinnable): a promise to callers who pin a path, no limit of
  // the kernels, which hold the pages of the rows there are)
  const bool wide_table = pg.table != nullptr && pg.pages_per_seq > 64;
  if (path == LOKI_PATH_CLUSTER && (s.G == 1 || wide_table || !fused_gqa_cluster_eligible(s, select_mode)))
    return LOKI_ERR_UNSUPPORTED;
  if (s.G == 1 && path == LOKI_PATH_FUSED && !fused_pinnable(s)) return LOKI_ERR_UNSUPPORTED;
  if (select_mode == LOKI_SELECT_PER_QUERY_HEAD &&
      ((s.G == 1 && path == LOKI_PATH_FUSED) || (path == 0 && fused_preferred(s)))) {
    if (s.G > 1 && s.ap.k_new != nullptr) {
      tm.begin("append");
      e = launch_qrot(s, q, P, w.qhat, klo, khi, v, nullptr, 0, st);
      tm.end();
      if (e != hipSuccess) return LOKI_ERR_HIP;
      s.ap = Append{};
    }
    tm.begin("fused_decode");
    e = launch_fused(s, q, P, klo, khi, v, out, out_idx, st);
    tm.end();
    return e == hipSuccess ? LOKI_OK : LOKI_ERR_HIP;
  }
  if (s.G > 1) {
    if (path == LOKI_PATH_CLUSTER || (path == 0 && w.cluster != nullptr && fused_gqa_cluster_preferred(s, select_mode))) {
      tm.begin("fused_decode");
      e = launch_fused_gqa_cluster(s, q, P, klo, khi, v, out, out_idx, w.cluster_ctl, ws_zeroed, w.cluster, st);
      tm.end();
      return e == hipSuccess ? LOKI_OK : LOKI_ERR_HIP;
    }
    if (path == LOKI_PATH_FUSED && (wide_table || !fused_gqa_eligible(s, select_mode))) return LOKI_ERR_UNSUPPORTED;
    if (path == LOKI_PATH_FUSED || (path == 0 && fused_gqa_preferred(s, select_mode))) {
      tm.begin("fused_decode");
      e = launch_fused_gqa(s, q, P, klo, khi, v, out, out_idx, st);
      tm.end();
      return e == hipSuccess ? LOKI_OK : LOKI_ERR_HIP;
    }
  }
  // long sequences, one token each: the score kernel counts the leading key bits into the
  // chunk histograms at the head of the select scratch (cleared by the rotation kernel), and the
  // selection leaves its list as two ascending runs, merged only for the caller's copy
  const int hist_chunks = w.sel_scratch ? select_hist_chunks(s, select_mode) : 0;
  uint32_t* hist_part = hist_chunks ? w.sel_scratch : nullptr;
  if (hist_chunks) idx = w.sel_idx;
  if (rotate_score_applies(s, select_mode) && hist_chunks == 0) {  // (histograms have to be clear before the scoring begins)
    tm.begin("rotate_score");
    e = launch_rotate_score(s, select_mode, q, P, klo, khi, v, w.scores, w.qhat, reinterpret_cast<uint32_t*>(w.tickets),
                            w.ticket_words, st);
    tm.end();
    if (e != hipSuccess) return LOKI_ERR_HIP;
  } else {
    tm.begin("rotate_query");
    // (the tickets lie directly before the select scratch, whose first words the histograms are)
    e = launch_qrot(s, q, P, w.qhat, klo, khi, v, reinterpret_cast<uint32_t*>(w.tickets),
                    w.ticket_words + (size_t)heads_sel * hist_chunks * 2048, st);
    tm.end();
    if (e != hipSuccess) return LOKI_ERR_HIP;
    tm.begin("score");
    e = launch_score(s, select_mode, klo, w.scores, w.qhat, hist_part, hist_chunks, st);
    tm.end();
    if (e != hipSuccess) return LOKI_ERR_HIP;
  }
  if (select_attend_applies(s, select_mode)) {
    tm.begin("select_attend");
    e = launch_select_attend(s, select_mode, w.scores, out_idx, w.qhat, klo, khi, v, w.partial, w.tickets, out, st);
    tm.end();
    return e == hipSuccess ? LOKI_OK : LOKI_ERR_HIP;
  }
  tm.begin("select");
  e = launch_select(s, heads_sel, w.scores, idx, w.sel_score, w.sel_scratch, hist_chunks != 0,
                    hist_chunks ? out_idx : nullptr, st);
  tm.end();
  if (e != hipSuccess) return LOKI_ERR_HIP;
  tm.begin("gather_attend");
  // (with several row splits the block that finishes a head group last merges them)
  e = launch_gather(s, select_mode, nsplit, w.qhat, klo, khi, v, idx, w.sel_score, w.partial,
                    w.tickets, out, st);
  tm.end();
  return e == hipSuccess ? LOKI_OK : LOKI_ERR_HIP;
}

int loki_decode_attn(const loki_layout* layout, const void* q, const float* P, const void* klo,
                     const void* khi, const void* v, int S, int d, int k, int select_mode,
                     void* workspace, size_t workspace_bytes, void* out, int32_t* out_idx,
                     void* stream) {
  // nothing is appended, so the caches are only read
  return decode_impl(layout, q, P, const_cast<void*>(klo), const_cast<void*>(khi),
                     const_cast<void*>(v), S, d, k, select_mode, Ragged{}, Append{}, Paging{},
                     workspace, workspace_bytes, out, out_idx, stream);
}

int loki_decode_attn_static(const loki_layout* layout, const void* q, const float* P,
                            const void* klo, const void* khi, const void* v, int S, int d, int k,
                            int select_mode, void* out, int32_t* out_idx, void* stream) {
  size_t need = 0;
  const int rc = loki_workspace_bytes(layout, S, d, k, select_mode, &need);
  if (rc != LOKI_OK) return rc;
  if (need > (size_t)LOKI_STATIC_SCRATCH_BYTES) return LOKI_ERR_SCRATCH_LIMIT;
  void* ptr = nullptr;
  const int ra = static_scratch_address(&ptr);
  if (ra != LOKI_OK) return ra;
  // the array starts as zeros and only this library writes it: the condition of
  // LOKI_WORKSPACE_ZEROED (nothing else in the workspace has to start at zero)
  return decode_impl(layout, q, P, const_cast<void*>(klo), const_cast<void*>(khi),
                     const_cast<void*>(v), S, d, k, select_mode | LOKI_WORKSPACE_ZEROED, Ragged{}, Append{}, Paging{}, ptr,
                     (size_t)LOKI_STATIC_SCRATCH_BYTES, out, out_idx, stream);
}

int loki_decode_step(const loki_layout* layout, const void* q, const float* P, void* klo, void* khi,
                     void* v, int S_max, int d, int k_max, int select_mode,
                     const loki_step_args* args, void* workspace, size_t workspace_bytes, void* out,
                     int32_t* out_idx, void* stream) {
  Ragged rg;
  Append ap;
  Paging pg;
  if (args && args->page_table) {
    if (!layout) return LOKI_ERR_INVALID_ARG;
    const int rc = paging_from_args(args->page_table, args->page_rows, args->pages_per_seq,
                                    args->n_pages, layout->Hkv, S_max, &pg);
    if (rc != LOKI_OK) return rc;
  }
  if (args) {
    rg.seq_lens = args->seq_lens;
    rg.ks = args->ks;
    rg.queries = args->queries_per_seq > 0 ? args->queries_per_seq : 1;
    ap.k_new = args->k_new;
    ap.v_new = args->v_new;
  }
  return decode_impl(layout, q, P, klo, khi, v, S_max, d, k_max, select_mode, rg, ap, pg, workspace,
                     workspace_bytes, out, out_idx, stream);
}

static int dense_impl(const loki_layout* layout, const void* q, const void* k_full, const void* v,
                      int S, const int32_t* seq_lens, void* workspace, size_t workspace_bytes,
                      void* out, void* stream) {
  Shape s;
  loki_layout L;
  if (!layout) return LOKI_ERR_INVALID_ARG;
  L = *layout;
  L.d_split = 128;  // ignored by the dense path
  const int rc = check_layout(&L, &s);
  if (rc != LOKI_OK) return rc;
  if (!q || !k_full || !v || !out) return LOKI_ERR_INVALID_ARG;
  if (S < 1 || S > s.S_cap) return LOKI_ERR_INVALID_ARG;
  if (!aligned16(q) || !aligned16(k_full) || !aligned16(v) || !aligned16(out))
    return LOKI_ERR_ALIGNMENT;
  if (reinterpret_cast<uintptr_t>(seq_lens) & 3u) return LOKI_ERR_ALIGNMENT;
  s.S = S;
  s.rg.seq_lens = seq_lens;
  const int nsplit = dense_splits(s, seq_lens != nullptr);
  const Workspace w = plan_workspace(s, -1, nsplit, workspace);
  if (nsplit > 1) {
    if (!workspace) return LOKI_ERR_INVALID_ARG;
    if (!aligned256(workspace)) return LOKI_ERR_ALIGNMENT;
    if (w.total_bytes > workspace_bytes) return LOKI_ERR_WORKSPACE;
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  StageTimer tm(st);
  hipError_t e;
  tm.begin("dense_attend");
  e = launch_dense(s, nsplit, q, k_full, v, w.partial, out, st);
  tm.end();
  if (e != hipSuccess) return LOKI_ERR_HIP;
  if (nsplit > 1) {
    tm.begin("combine");
    e = launch_combine(s, nsplit, w.partial, out, st);
    tm.end();
    if (e != hipSuccess) return LOKI_ERR_HIP;
  }
  return LOKI_OK;
}

int dense_decode_attn(const loki_layout* layout, const void* q, const void* k_full, const void* v,
                      int S, void* workspace, size_t workspace_bytes, void* out, void* stream) {
  return dense_impl(layout, q, k_full, v, S, nullptr, workspace, workspace_bytes, out, stream);
}

int dense_decode_step(const loki_layout* layout, const void* q, const void* k_full, const void* v,
                      int S_max, const int32_t* seq_lens, void* workspace, size_t workspace_bytes,
                      void* out, void* stream) {
  return dense_impl(layout, q, k_full, v, S_max, seq_lens, workspace, workspace_bytes, out, stream);
}

int loki_pca_attn(const loki_layout* layout, const void* q, const float* P, const void* klo,
                  const void* v, int S, int d, void* workspace, size_t workspace_bytes, void* out,
                  void* stream) {
  Shape s;
  const int rc = check_layout(layout, &s);
  if (rc != LOKI_OK) return rc;
  if (!q || !P || !klo || !v || !out || !workspace) return LOKI_ERR_INVALID_ARG;
  if (S < 1 || S > s.S_cap) return LOKI_ERR_INVALID_ARG;
  if (d != s.d) return LOKI_ERR_UNSUPPORTED;
  if (!aligned16(q) || !aligned16(P) || !aligned16(klo) || !aligned16(v) || !aligned16(out))
    return LOKI_ERR_ALIGNMENT;
  if (!aligned256(workspace)) return LOKI_ERR_ALIGNMENT;
  s.S = S;
  const int nsplit = dense_splits(s, false);
  const Workspace w = plan_workspace(s, -2, nsplit, workspace);
  if (w.total_bytes > workspace_bytes) return LOKI_ERR_WORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  StageTimer tm(st);
  hipError_t e;
  tm.begin("rotate_query");
  e = launch_qrot(s, q, P, w.qhat, nullptr, nullptr, nullptr, nullptr, 0, st);
  tm.end();
  if (e != hipSuccess) return LOKI_ERR_HIP;
  tm.begin("pca_attend");
  e = launch_pca_attend(s, nsplit, w.qhat, klo, v, w.partial, out, st);
  tm.end();
  if (e != hipSuccess) return LOKI_ERR_HIP;
  if (nsplit > 1) {
    tm.begin("combine");
    e = launch_combine(s, nsplit, w.partial, out, st);
    tm.end();
    if (e != hipSuccess) return LOKI_ERR_HIP;
  }
  return LOKI_OK;
}

int loki_pca_workspace_bytes(const loki_layout* layout, long long n_rows, size_t* bytes) {
  Shape s;
  const int rc = check_layout(layout, &s);
  if (rc != LOKI_OK) return rc;
  if (!bytes || n_rows < 2 || n_rows > (1LL << 40)) return LOKI_ERR_INVALID_ARG;
  *bytes = pca_workspace_bytes(s.Hkv, n_rows);
  return LOKI_OK;
}

int loki_pca_fit(const loki_layout* layout, const void* keys, long long n_rows, float* P,
                 float* eigenvalues, void* workspace, size_t workspace_bytes, void* stream) {
  Shape s;
  const int rc = check_layout(layout, &s);
  if (rc != LOKI_OK) return rc;
  if (!keys || !P || !eigenvalues || !workspace) return LOKI_ERR_INVALID_ARG;
  if (n_rows < 2 || n_rows > (1LL << 40)) return LOKI_ERR_INVALID_ARG;
  if (!aligned16(keys) || !aligned16(P) || !aligned16(eigenvalues)) return LOKI_ERR_ALIGNMENT;
  if (!aligned256(workspace)) return LOKI_ERR_ALIGNMENT;
  if (pca_workspace_bytes(s.Hkv, n_rows) > workspace_bytes) return LOKI_ERR_WORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  StageTimer tm(st);
  static const char* const kStageNames[3] = {"pca_gram", "pca_covariance", "pca_eigensolve"};
  for (int stage = 0; stage < 3; ++stage) {
    tm.begin(kStageNames[stage]);
    const hipError_t e =
        launch_pca_stage(stage, s.Hkv, s.dtype, keys, n_rows, P, eigenvalues, workspace, st);
    tm.end();
    if (e != hipSuccess) return LOKI_ERR_HIP;
  }
  return LOKI_OK;
}

int loki_rank_at(const float* eigenvalues, int n_heads, int D, float v_percent, int32_t* ranks,
                 void* stream) {
  if (!eigenvalues || !ranks || n_heads < 1 || D < 1) return LOKI_ERR_INVALID_ARG;
  if (!(v_percent > 0.f) || v_percent > 100.f) return LOKI_ERR_INVALID_ARG;
  const hipError_t e = launch_rank_at(eigenvalues, n_heads, D, v_percent, ranks,
                                      static_cast<hipStream_t>(stream));
  return e == hipSuccess ? LOKI_OK : LOKI_ERR_HIP;
}

int loki_layer_width(const float* eigenvalues, int n_heads, int D, float v_percent, int multiple,
                     float* mean_rank, int32_t* d_out, void* stream) {
  if (!eigenvalues || !d_out || n_heads < 1 || D < 1) return LOKI_ERR_INVALID_ARG;
  if (!(v_percent > 0.f) || v_percent > 100.f) return LOKI_ERR_INVALID_ARG;
  if (multiple < 1 || multiple > D || D % multiple != 0) return LOKI_ERR_INVALID_ARG;
  if ((long long)n_heads * D > 0x7fffffffLL / 2) return LOKI_ERR_UNSUPPORTED;  // rank sum in int32
  const hipError_t e = launch_layer_width(eigenvalues, n_heads, D, v_percent, multiple, mean_rank,
                                          d_out, static_cast<hipStream_t>(stream));
  return e == hipSuccess ? LOKI_OK : LOKI_ERR_HIP;
}

int loki_index_jaccard(const int32_t* idx_a, const int32_t* idx_b, int n_lists, int k, float* out,
                       void* stream) {
  if (!idx_a || !idx_b || !out || n_lists < 1 || k < 1) return LOKI_ERR_INVALID_ARG;
  const hipError_t e = launch_jaccard(idx_a, idx_b, n_lists, k, out, static_cast<hipStream_t>(stream));
  return e == hipSuccess ? LOKI_OK : LOKI_ERR_HIP;
}

int loki_profile_create(loki_profile** out) {
  if (!out) return LOKI_ERR_INVALID_ARG;
  loki_profile* p = new (std::nothrow) loki_profile();
  if (!p) return LOKI_ERR_INVALID_ARG;
  p->n = 0;
  for (int i = 0; i < 2 * LOKI_PROFILE_MAX_KERNELS; ++i) {
    if (hipEventCreate(&p->ev[i]) != hipSuccess) {
      for (int j = 0; j < i; ++j) (void)hipEventDestroy(p->ev[j]);
      delete p;
      return LOKI_ERR_HIP;
    }
  }
  *out = p;
  return LOKI_OK;
}

int loki_profile_destroy(loki_profile* p) {
  if (!p) return LOKI_ERR_INVALID_ARG;
  if (t_profile == p) t_profile = nullptr;
  for (int i = 0; i < 2 * LOKI_PROFILE_MAX_KERNELS; ++i) (void)hipEventDestroy(p->ev[i]);
  delete p;
  return LOKI_OK;
}

int loki_profile_attach(loki_profile* p) {
  t_profile = p;
  return LOKI_OK;
}

int loki_profile_read(loki_profile* p, int* n_kernels, float* ms, const char** names) {
  if (!p || !n_kernels || !ms) return LOKI_ERR_INVALID_ARG;
  *n_kernels = p->n;
  if (p->n == 0) return LOKI_OK;
  if (hipEventSynchronize(p->ev[2 * p->n - 1]) != hipSuccess) return LOKI_ERR_HIP;
  for (int i = 0; i < p->n; ++i) {
    if (hipEventElapsedTime(&ms[i], p->ev[2 * i], p->ev[2 * i + 1]) != hipSuccess)
      return LOKI_ERR_HIP;
    if (names) names[i] = p->names[i];
  }
  return LOKI_OK;
}

int loki_debug_cluster_spin_limit(unsigned polls) {
  set_cluster_spin_limit(polls ? polls : kClusterSpinLimit);
  return LOKI_OK;
}

int loki_debug_cluster_give_up_at_list(int on) {
  set_cluster_give_up_at_list(on != 0);
  return LOKI_OK;
}

int loki_debug_row_loads(const loki_layout* layout, int S_max, int d, int k_max, int select_mode,
                         const loki_step_args* args, double rows, double kept, int* form) {
  Shape s;
  const int rc = check_layout(layout, &s);
  if (rc != LOKI_OK) return rc;
  select_mode = select_mode < 0 ? select_mode : select_mode & ~(LOKI_PATH_MASK | LOKI_WORKSPACE_ZEROED);
  if (!form || select_mode < kLowRankRows || select_mode > 1 || S_max < 1) return LOKI_ERR_INVALID_ARG;
  if (args) {
    s.rg.seq_lens = args->seq_lens;
    s.rg.ks = args->ks;
    s.rg.queries = args->queries_per_seq > 1 ? args->queries_per_seq : 1;
    s.ap.k_new = args->k_new;
    s.pg.table = args->page_table;
    s.pg.pages_per_seq = args->pages_per_seq;
    while (s.pg.lg_rows < 24 && (1 << s.pg.lg_rows) < args->page_rows) ++s.pg.lg_rows;
  }
  s.B *= s.rg.queries;
  s.S = S_max;
  s.k = k_max;
  if (select_mode >= 0) {
    if (d != s.d) return LOKI_ERR_UNSUPPORTED;
    if (k_max < 1 || k_max > S_max) return LOKI_ERR_INVALID_ARG;
  }
  if (s.G == 1 && select_mode == 1) select_mode = 0;
  int loads = select_mode;
  if (select_mode == 1 && (fused_gqa_cluster_preferred(s, 1) || fused_gqa_preferred(s, 1))) loads = kGroupLaunch;
  const RowLoads l = row_loads(s, loads);
  *form = l.form == kByLengths ? loads_form(l, (float)rows, (float)kept) : l.form;
  if (select_mode == 0 && s.G > 1 && fused_preferred(s)) *form = kThroughCaches;  // (the one block per head of a group: always)
  return LOKI_OK;
}

int loki_cluster_gave_up(const void* workspace, int* gave_up, void* stream) {
  if (!workspace || !gave_up) return LOKI_ERR_INVALID_ARG;
  if (!aligned256(workspace)) return LOKI_ERR_ALIGNMENT;
  // the error word sits behind the control words of the last unit, at the start of the workspace
  const uint32_t* word = static_cast<const uint32_t*>(workspace) + (size_t)kClusterMaxUnits * kClusterCounterStride;
  uint32_t v = 0;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (hipMemcpyAsync(&v, word, sizeof(v), hipMemcpyDeviceToHost, st) != hipSuccess) return LOKI_ERR_HIP;
  if (hipStreamSynchronize(st) != hipSuccess) return LOKI_ERR_HIP;
  *gave_up = v != 0u ? 1 : 0;
  return LOKI_OK;
}

int loki_stream_read(const void* buf, size_t bytes, void* stream) {
  if (!buf || bytes == 0 || (bytes & 15) || (reinterpret_cast<uintptr_t>(buf) & 15))
    return LOKI_ERR_INVALID_ARG;
  hipLaunchKernelGGL(loki::stream_read_kernel, dim3(loki::device_cus()), dim3(512), 0,
                     static_cast<hipStream_t>(stream), static_cast<const uint4*>(buf), bytes / 16);
  return hipGetLastError() == hipSuccess ? LOKI_OK : LOKI_ERR_HIP;
}

}  // extern "C"
