// Raw buffer loads for the gfx950 kernels.  A raw buffer load whose byte offset
// lies outside the buffer returns zero WITHOUT touching memory, so work that
// does not exist (a group past K, a token row past M, a weight tile past N) is
// expressed as an out-of-range offset instead of a branch around the load.
#pragma once
#include "common.hpp"

namespace qspec {

typedef __amdgpu_buffer_rsrc_t rsrc_t;
constexpr uint32_t kOutOfRange = 0x80000000u;     // beyond any buffer this library accepts (< 2 GiB)

__device__ inline rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}
__device__ inline uint4 buf_load16(rsrc_t r, uint32_t off) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
  return uint4{v.x, v.y, v.z, v.w};
}
// streaming variant (weights are read once: do not keep them in the caches)
__device__ inline uint4 buf_load16_stream(rsrc_t r, uint32_t off) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 2);
  return uint4{v.x, v.y, v.z, v.w};
}
// The same from a base pointer and a size (0: an empty buffer, so zeros and no traffic), with a
// wave-uniform part soff of the offset that is not range-checked: only voff is.  (Both uniform
// arguments are moved to scalar registers by hand: one the compiler happens to hold in a vector
// register would otherwise become a loop over its values around the load.)
__device__ inline uint32_t scalar_u32(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ inline uint4 buf_load16(const void* p, uint32_t bytes, uint32_t voff, uint32_t soff) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(make_rsrc(p, scalar_u32(bytes)), voff, scalar_u32(soff), 0);
  return uint4{v.x, v.y, v.z, v.w};
}
__device__ inline uint16_t buf_load_u16(const void* p, uint32_t bytes, uint32_t voff, uint32_t soff) {
  return (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(make_rsrc(p, scalar_u32(bytes)), voff, scalar_u32(soff), 0);
}
// two floats another workgroup of this launch has written through (past this XCD's caches)
__device__ inline float2 buf_load_f32x2_shared(const void* p, uint32_t bytes, uint32_t voff, uint32_t soff) {
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(make_rsrc(p, scalar_u32(bytes)), voff, scalar_u32(soff), 16);   // sc1
  const uint32_t a = v.x, b = v.y;       // (copies: bit_cast of a vector element lvalue reads element 0)
  return float2{__builtin_bit_cast(float, a), __builtin_bit_cast(float, b)};
}
// 16 bytes per lane straight into LDS: lane l to bytes 16 l .. 16 l + 15 from lds (wave-uniform)
typedef __attribute__((address_space(3))) void* lds_ptr_t;
__device__ inline void buf_load16_lds(const void* p, uint32_t bytes, uint8_t* lds, uint32_t voff, uint32_t soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(make_rsrc(p, scalar_u32(bytes)), (lds_ptr_t)lds, 16, voff, scalar_u32(soff), 0, 0);
}
__device__ inline uint2 buf_load8(rsrc_t r, uint32_t off) {
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
  return uint2{v.x, v.y};
}
// three consecutive floats (4-byte aligned; each component is range-checked on its own)
struct float3_t { float x, y, z; };
__device__ inline float3_t buf_load_f32x3(rsrc_t r, uint32_t off) {
  typedef unsigned int u32x3 __attribute__((ext_vector_type(3)));
  const u32x3 v = __builtin_amdgcn_raw_buffer_load_b96(r, off, 0, 0);
  const uint32_t a = v.x, b = v.y, c = v.z;      // (copies: bit_cast of a vector element lvalue reads element 0)
  return float3_t{__builtin_bit_cast(float, a), __builtin_bit_cast(float, b), __builtin_bit_cast(float, c)};
}
__device__ inline float buf_load_f32(rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}

}  // namespace qspec
