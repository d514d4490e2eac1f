// Device helpers shared by the tile kernels: wave-uniform values, scalar table
// loads and the block order over the XCDs.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace dd {

// Table entries of one (wave tile, input row).
typedef int32_t ent4_t __attribute__((ext_vector_type(4)));
typedef int32_t ent8_t __attribute__((ext_vector_type(8)));
typedef int32_t ent16_t __attribute__((ext_vector_type(16)));

#define LDS_AS __attribute__((address_space(3)))

// Blocks are dispatched round-robin over the 8 XCDs.  Give each XCD a
// contiguous range of work items (time-major, output rows fastest).
__device__ __forceinline__ int xcd_remap(int L, int N) {
  const int q = N >> 3, r = N & 7;
  const int x = L & 7, k = L >> 3;
  return (x < r) ? x * (q + 1) + k : r * (q + 1) + (x - r) * q + k;
}

__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// The lane index, recomputed where it is used: the asm keeps the compiler
// from hoisting lane-dependent offsets out of loops and holding them in
// registers the small register windows cannot spare.
__device__ __forceinline__ int lane_fresh() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}

// A pointer the compiler must keep in SGPRs (its value is wave-uniform).
template <typename T>
__device__ __forceinline__ T* uniform_ptr(T* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<T*>(((uint64_t)hi << 32) | lo);
}

// A table the kernel only reads, in the constant address space: wave-uniform
// elements become scalar loads that the compiler may issue early.
template <typename T>
using const_table = const T __attribute__((address_space(4))) *;
template <typename T>
__device__ __forceinline__ const_table<T> uniform_table(const T* p) {
  return (const_table<T>)reinterpret_cast<uint64_t>(uniform_ptr(p));
}

// Wave-uniform scalar loads (wait included) of a table entry and a weight.
typedef int32_t ent2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ ent2_t sload_entry2(const int32_t* p) {
  ent2_t r;
  asm volatile("s_load_dwordx2 %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=s"(r) : "s"(p));
  return r;
}
__device__ __forceinline__ ent4_t sload_entry4(const int32_t* p) {
  ent4_t r;
  asm volatile("s_load_dwordx4 %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=s"(r) : "s"(p));
  return r;
}
__device__ __forceinline__ ent8_t sload_entry8(const int32_t* p) {
  ent8_t r;
  asm volatile("s_load_dwordx8 %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=s"(r) : "s"(p));
  return r;
}
template <typename E>
__device__ __forceinline__ E sload_entry_t(const int32_t* p);
template <>
__device__ __forceinline__ ent4_t sload_entry_t<ent4_t>(const int32_t* p) {
  return sload_entry4(p);
}
template <>
__device__ __forceinline__ ent8_t sload_entry_t<ent8_t>(const int32_t* p) {
  return sload_entry8(p);
}
template <>
__device__ __forceinline__ ent16_t sload_entry_t<ent16_t>(const int32_t* p) {
  ent16_t r;
  asm volatile("s_load_dwordx16 %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=s"(r) : "s"(p));
  return r;
}
// Scalar buffer loads (reads past the resource's range return zero), wait included.
__device__ __forceinline__ ent8_t sbload8(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  ent8_t r;
  asm volatile("s_buffer_load_dwordx8 %0, %1, %2\n\ts_waitcnt lgkmcnt(0)" : "=s"(r) : "s"(rs), "s"(off));
  return r;
}
__device__ __forceinline__ ent16_t sbload16(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  ent16_t r;
  asm volatile("s_buffer_load_dwordx16 %0, %1, %2\n\ts_waitcnt lgkmcnt(0)" : "=s"(r) : "s"(rs), "s"(off));
  return r;
}
__device__ __forceinline__ ent4_t sbload4(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  ent4_t r;
  asm volatile("s_buffer_load_dwordx4 %0, %1, %2\n\ts_waitcnt lgkmcnt(0)" : "=s"(r) : "s"(rs), "s"(off));
  return r;
}
template <typename E>
__device__ __forceinline__ E sbload_t(__amdgpu_buffer_rsrc_t rs, uint32_t off);
template <>
__device__ __forceinline__ ent4_t sbload_t<ent4_t>(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  return sbload4(rs, off);
}
template <>
__device__ __forceinline__ ent8_t sbload_t<ent8_t>(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  return sbload8(rs, off);
}
template <>
__device__ __forceinline__ ent16_t sbload_t<ent16_t>(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  return sbload16(rs, off);
}
__device__ __forceinline__ float sload_f32(const float* p) {
  float r;
  asm volatile("s_load_dword %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=s"(r) : "s"(p));
  return r;
}

}  // namespace dd
