// Device helpers shared by the library's kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cnnlib {

typedef uint16_t bf16_t;  // bfloat16 bit pattern (top half of an IEEE float32)

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16_t x) { return __uint_as_float((uint32_t)x << 16); }

template <typename T> __device__ __forceinline__ T from_f32(float x);
template <> __device__ __forceinline__ float from_f32<float>(float x) { return x; }
// float32 -> bfloat16, round to nearest, ties to even; NaN stays a quiet NaN.
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float x) {
  uint32_t u = __float_as_uint(x);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (bf16_t)0x7fc0;
  u += 0x7fffu + ((u >> 16) & 1u);
  return (bf16_t)(u >> 16);
}

// Two fp32 values as bf16 (round to nearest, ties to even), x in the low half.
__device__ __forceinline__ uint32_t pk_bf16(float x, float y) {
  typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
  typedef float f2 __attribute__((ext_vector_type(2)));
  const f2 v = {x, y};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf2));
}

// A buffer of `bytes` from base (just below 2 GiB of it at most).  The range ends
// with the last element's 4-byte word, in memory and not from the base, which may
// lie at any 2 bytes.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_words(const void* base, int64_t bytes) {
  bytes = (int64_t)((((uintptr_t)base + (uintptr_t)bytes + 3) & ~(uintptr_t)3) - (uintptr_t)base);
  const int32_t n = bytes > 0x7ffffffcLL ? 0x7ffffffc : (int32_t)bytes;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, n, 0x00020000);
}

// Division by a divisor d fixed for a launch (1 <= d < 2^31) of dividends
// n in [0, 2^31), as a multiply and a shift: with l = ceil(log2 d), s = 31 + l
// and m = ceil(2^s / d) (< 2^32), n / d = floor(n m / 2^s).  (m d - 2^s lies
// in [0, d), so n m / 2^s exceeds n / d by less than n / 2^s < 2^-l <= 1 / d,
// which never carries it past the next integer.)  The magic numbers are made
// on the host, once per launch; a runtime integer division costs some 25
// vector instructions, this one three.
struct FastDiv {
  uint32_t m, s;
};
__host__ __device__ inline FastDiv make_fastdiv(uint32_t d) {
  uint32_t l = 0;
  while (l < 31 && (1u << l) < d) ++l;
  FastDiv f;
  f.s = 31u + l;
  f.m = (uint32_t)(((1ull << f.s) + d - 1) / d);
  return f;
}
__host__ __device__ __forceinline__ int fdiv(int n, FastDiv f) {
  return (int)(((uint64_t)(uint32_t)n * f.m) >> f.s);
}

// Index of a tensor's last element from a tile's first row, for kernels that
// compare it with 32-bit offsets from there (below 2^30): the tensor may go on
// for 2^32 elements or more, so it is saturated where no offset reaches, not
// cut to 32 bits.
__host__ __device__ __forceinline__ uint32_t last_index(int64_t elems_from_row) {
  return elems_from_row > 0x7fffffffLL ? 0x7fffffffu : (uint32_t)(elems_from_row - 1);
}

// The hardware hands consecutive workgroup ids to the 8 XCDs round-robin
// (id % 8).  Renumber so that each XCD receives one contiguous run of
// logical tiles: tiles that share input data (the k-tiles of one pixel tile)
// then meet in the same XCD's L2.  A bijection on [0, grid).
__device__ __forceinline__ int xcd_remap(int bid, int grid) {
  const int q = grid >> 3, rem = grid & 7;
  const int x = bid & 7, i = bid >> 3;
  return x * q + (x < rem ? x : rem) + i;
}

}  // namespace cnnlib
