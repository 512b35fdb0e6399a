// The pair-by-pair prefill: float32 instances.
#include "prefill_direct_kernel.hpp"

namespace sata {

hipError_t launch_prefill_direct_f32(const void* q, const void* k, const void* v, void* y, int heads, int qg, int n,
                                     int dk, int dv, int P, hipStream_t s) {
  if (dk <= 16) return launch_nct<float, true, true, 1>(q, k, v, y, heads, qg, n, dk, dv, P, s);
  return dk <= 32 ? launch_nct<float, true, false, 1>(q, k, v, y, heads, qg, n, dk, dv, P, s)
                  : launch_nct<float, true, false, 2>(q, k, v, y, heads, qg, n, dk, dv, P, s);
}

}  // namespace sata
