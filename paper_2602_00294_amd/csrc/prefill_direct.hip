// The pair-by-pair prefill: bfloat16 instances and the entry (the float32 ones
// are a source of their own, so that the two compile side by side).
#include "prefill_direct_kernel.hpp"

namespace sata {

hipError_t launch_prefill_direct_f32(const void* q, const void* k, const void* v, void* y, int heads, int qg, int n,
                                     int dk, int dv, int P, hipStream_t s);

hipError_t launch_prefill_direct(const void* q, const void* k, const void* v, void* y, bool bf16, int heads, int qg,
                                 int n, int dk, int dv, int P, hipStream_t s) {
  if (!bf16) return launch_prefill_direct_f32(q, k, v, y, heads, qg, n, dk, dv, P, s);
  return dk <= 32 ? launch_nct<u16, false, false, 1>(q, k, v, y, heads, qg, n, dk, dv, P, s)
                  : launch_nct<u16, false, false, 2>(q, k, v, y, heads, qg, n, dk, dv, P, s);
}

}  // namespace sata
