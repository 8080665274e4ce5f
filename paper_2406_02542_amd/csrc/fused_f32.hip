// The single-launch decode step of one block per query head (fused_impl.h), fp32 caches.
#include "fused_impl.h"

namespace loki {

#ifdef LOKI_PHASE_TIMING
extern "C" int loki_debug_read_phase_ts_f32(unsigned long long* host_dst, size_t count) {
  return (int)hipMemcpyFromSymbol(host_dst, HIP_SYMBOL(loki::g_phase_ts), count * sizeof(unsigned long long));
}
#endif

hipError_t launch_fused_f32(const Shape& s, const void* q, const float* P, void* klo, void* khi, void* v, void* out,
                            int32_t* out_idx, hipStream_t st) {
  return launch_fused_t<F32>(s, q, P, klo, khi, v, out, out_idx, st);
}

}  // namespace loki
