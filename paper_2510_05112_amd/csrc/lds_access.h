// LDS accesses by 32-bit LDS address: the kernels that work out per-lane addresses keep them as integers, so that
// ring positions and table offsets can be OR-ed / multiplied into them.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fpsched {

#define FPSCHED_LDS __attribute__((address_space(3)))
template <class T>
__device__ __forceinline__ T lds_read(unsigned a) {
  typedef T access __attribute__((may_alias));   // (rings and states are written in dwords and read in halves or bytes)
  return *reinterpret_cast<const FPSCHED_LDS access*>(a);
}
typedef int lds_int4 __attribute__((ext_vector_type(4)));
typedef int lds_int3 __attribute__((ext_vector_type(3)));
typedef int lds_int2 __attribute__((ext_vector_type(2)));
template <>
__device__ __forceinline__ int4 lds_read<int4>(unsigned a) {
  const lds_int4 v = *reinterpret_cast<const FPSCHED_LDS lds_int4*>(a);
  return make_int4(v.x, v.y, v.z, v.w);
}
template <>
__device__ __forceinline__ int2 lds_read<int2>(unsigned a) {
  const lds_int2 v = *reinterpret_cast<const FPSCHED_LDS lds_int2*>(a);
  return make_int2(v.x, v.y);
}
template <class T>
__device__ __forceinline__ void lds_write(unsigned a, T v) {
  typedef T access __attribute__((may_alias));
  *reinterpret_cast<FPSCHED_LDS access*>(a) = v;
}
__device__ __forceinline__ unsigned lds_address(const void* p) {
  return (unsigned)(size_t)(const FPSCHED_LDS char*)p;
}

}  // namespace fpsched
