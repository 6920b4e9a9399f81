// hbm_vec.hpp -- access to VEC consecutive replicas of a vertex row in device
// memory ([n][R] layout), for the device-memory sweep forms.
#pragma once

#include <hip/hip_runtime.h>

#include "device_common.hpp"

namespace cosm {
namespace {

// VEC consecutive replicas of one vertex row in one access (8 or 16 bytes for
// FP32 and FIX32, 4 or 8 for the 16-bit formats); idx is a multiple of VEC.
typedef float hbm_f32x2 __attribute__((ext_vector_type(2)));
typedef float hbm_f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t hbm_u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t hbm_u32x4 __attribute__((ext_vector_type(4)));
template <typename T>
using gvec = T __attribute__((address_space(1))) *;

template <int ST, int VEC>
__device__ __forceinline__ void load_vec(const void *p, size_t idx, float (&x)[VEC]) {
  using F = Fmt<ST>;
  if constexpr (VEC == 1) {
    x[0] = F::load_elem(p, idx);
  } else if constexpr (ST == COSM_STORE_FP32) {
    const float *q = static_cast<const float *>(p) + idx;
    if constexpr (VEC == 4) {
      const hbm_f32x4 v = *(gvec<const hbm_f32x4>)(q);
      x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
    } else {
      const hbm_f32x2 v = *(gvec<const hbm_f32x2>)(q);
      x[0] = v.x; x[1] = v.y;
    }
  } else if constexpr (ST == COSM_STORE_FIX32) {
    const uint32_t *q = static_cast<const uint32_t *>(p) + idx;
    if constexpr (VEC == 4) {
      const hbm_u32x4 v = *(gvec<const hbm_u32x4>)(q);
      x[0] = F::dec(v.x); x[1] = F::dec(v.y); x[2] = F::dec(v.z); x[3] = F::dec(v.w);
    } else {
      const hbm_u32x2 v = *(gvec<const hbm_u32x2>)(q);
      x[0] = F::dec(v.x); x[1] = F::dec(v.y);
    }
  } else {
    const uint16_t *q = static_cast<const uint16_t *>(p) + idx;
    if constexpr (VEC == 4) {
      const hbm_u32x2 v = *(gvec<const hbm_u32x2>)(q);
      x[0] = F::dec(v.x & 0xffffu); x[1] = F::dec(v.x >> 16);
      x[2] = F::dec(v.y & 0xffffu); x[3] = F::dec(v.y >> 16);
    } else {
      const uint32_t v = *(gvec<const uint32_t>)(q);
      x[0] = F::dec(v & 0xffffu); x[1] = F::dec(v >> 16);
    }
  }
}
template <int ST, int VEC>
__device__ __forceinline__ void store_vec(void *p, size_t idx, const float (&x)[VEC]) {
  using F = Fmt<ST>;
  if constexpr (VEC == 1) {
    F::store_elem(p, idx, x[0]);
  } else if constexpr (ST == COSM_STORE_FP32) {
    float *q = static_cast<float *>(p) + idx;
    if constexpr (VEC == 4) {
      *(gvec<hbm_f32x4>)(q) = hbm_f32x4{x[0], x[1], x[2], x[3]};
    } else {
      *(gvec<hbm_f32x2>)(q) = hbm_f32x2{x[0], x[1]};
    }
  } else if constexpr (ST == COSM_STORE_FIX32) {
    uint32_t *q = static_cast<uint32_t *>(p) + idx;
    if constexpr (VEC == 4) {
      *(gvec<hbm_u32x4>)(q) = hbm_u32x4{F::enc(x[0]), F::enc(x[1]), F::enc(x[2]), F::enc(x[3])};
    } else {
      *(gvec<hbm_u32x2>)(q) = hbm_u32x2{F::enc(x[0]), F::enc(x[1])};
    }
  } else {
    uint16_t *q = static_cast<uint16_t *>(p) + idx;
    if constexpr (VEC == 4) {
      *(gvec<hbm_u32x2>)(q) = hbm_u32x2{F::enc(x[0]) | (F::enc(x[1]) << 16),
                                        F::enc(x[2]) | (F::enc(x[3]) << 16)};
    } else {
      *(gvec<uint32_t>)(q) = F::enc(x[0]) | (F::enc(x[1]) << 16);
    }
  }
}

}  // namespace
}  // namespace cosm
