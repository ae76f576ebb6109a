// What the kernels that multiply several messages' vectors on the matrix cores share.
#pragma once
#include "step_impl.h"

namespace mdi {
namespace MDI_STEP_CAT(step_w, MDI_STEP_WAVES) {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return (uint32_t)f32_to_bf16(lo) | ((uint32_t)f32_to_bf16(hi) << 16);
}
__device__ __forceinline__ float bf16_bits_to_f32(uint32_t b) { return __uint_as_float(b << 16); }
__device__ __forceinline__ void st_pair(tagged_t* p, uint32_t bits, unsigned tag) {
  __hip_atomic_store((MDI_GLOBAL tagged_t*)p, ((tagged_t)tag << 32) | (tagged_t)bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The low word of *p once its counter is `tag` (see settle in step_impl.h).
__device__ __forceinline__ uint32_t settle_bits(const tagged_t* p, tagged_t u, unsigned tag, int spin_limit, int* err) {
  int it = 0;
  while ((uint32_t)(u >> 32) != tag) {
    if (++it > spin_limit) { __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); break; }
    __builtin_amdgcn_s_sleep(1);
    u = ld_raw(p);
  }
  return (uint32_t)u;
}

}  // namespace step_w<waves>
}  // namespace mdi
