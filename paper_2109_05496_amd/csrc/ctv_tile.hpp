// Tile job description and wave-level helpers shared by the forward tile
// kernels (column-register tiles and the row-sweep tile).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ctv_types.hpp"

namespace ctv {

constexpr int kRW = 64;  // columns of a tile region: one per lane of a wave64

struct TileJob {
  const float2* b;       // image (m x n)
  const uint8_t* mask;   // image support or nullptr
  const float4* st_in;   // [2][m][n] (q plane, r plane) or nullptr = cold start
  bool foreign;          // st_in is a caller's state, or one iteration from it (column tiles)
  float4* st_out;        // [2][m][n] or nullptr
  float2* x;             // Eq. (18) output or nullptr
  int m, n;
  int tx, ty;
  int kind;              // read by the kernel that runs all kinds in one body only
  float lam, c;
  Radii R;
  int T;
  float4* r_hist;          // r after each fused iteration (plane 1 of consecutive states), or nullptr
  long long hist_stride;   // float4 elements from one iteration's state to the next
};

// Whole-wave lane shifts through DPP (row_shr / row_shl across the wave with
// bound control): the neighbouring column's value, 0 past the wave's edge.
__device__ __forceinline__ float lane_from_left(float v) {   // lane i <- lane i-1 (lane 0 <- 0)
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_from_right(float v) {  // lane i <- lane i+1 (lane 63 <- 0)
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, true));
}

// One row of an image, from its first column inside a tile's region on, as a
// buffer of `bytes` bytes (0 for a row outside the image): the hardware's bounds
// check returns 0 for loads past it and drops stores, so a tile at the image's
// border loads and stores without a branch per row, all rows in flight at once.
// A lane outside the image uses the offset kNoOffset.
constexpr int kNoOffset = (int)0x80000000;
template <class T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_buf(const T* row, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(row), (short)0, bytes, 0x00020000);
}
typedef int vint4 __attribute__((ext_vector_type(4)));
typedef int vint2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float4 buf_ld4(__amdgpu_buffer_rsrc_t r, int off) {
  const vint4 v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
  return make_float4(__int_as_float(v.x), __int_as_float(v.y), __int_as_float(v.z), __int_as_float(v.w));
}
__device__ __forceinline__ float2 buf_ld2(__amdgpu_buffer_rsrc_t r, int off) {
  const vint2 v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
  return make_float2(__int_as_float(v.x), __int_as_float(v.y));
}
__device__ __forceinline__ bool buf_ld_mask(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_amdgcn_raw_buffer_load_b8(r, off, 0, 0) != 0;
}
// AUX: cache policy bits (2 = non-temporal)
template <int AUX = 0>
__device__ __forceinline__ void buf_st4(__amdgpu_buffer_rsrc_t r, int off, float4 v) {
  const vint4 u = {__float_as_int(v.x), __float_as_int(v.y), __float_as_int(v.z), __float_as_int(v.w)};
  __builtin_amdgcn_raw_buffer_store_b128(u, r, off, 0, AUX);
}
template <int AUX = 0>
__device__ __forceinline__ void buf_st2(__amdgpu_buffer_rsrc_t r, int off, float2 v) {
  const vint2 u = {__float_as_int(v.x), __float_as_int(v.y)};
  __builtin_amdgcn_raw_buffer_store_b64(u, r, off, 0, AUX);
}

// A tile kernel runs its form for finite values first (FIN = true) and, where that
// returns false, the form for any value, behind a condition that the compiler cannot
// look through and with the job read again from the kernel's arguments: otherwise it
// places the second form before the loop of the first and keeps the first's registers
// through it (63 -> 102 of the forward 8 x 4 tile), or keeps the job in scalar registers
// that the first form spills (16 x 4: 2-3 % of a masked launch).
__device__ __forceinline__ bool opaque(int done) {
  done = __builtin_amdgcn_readfirstlane(done);
  asm volatile("" : "+s"(done) : : "memory");
  return __builtin_expect(done != 0, 1);
}
template <class A>
__device__ __forceinline__ const A& args_again() {  // of a kernel whose only argument is an A
  auto p = __builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const A*)p;
}

// Bits [max(a, 0), min(b, n)) set: the rows i of a wave with a <= i < b. a and b
// are the same in every lane; readfirstlane between the two bounds
// keeps them scalar (the compiler makes a vector median of them otherwise).
__device__ __forceinline__ unsigned row_bits(int a, int b, int n) {
  a = min(__builtin_amdgcn_readfirstlane(max(a, 0)), n);
  b = min(__builtin_amdgcn_readfirstlane(max(b, 0)), n);
  return ((1u << b) - 1u) & ~((1u << a) - 1u);
}

}  // namespace ctv
