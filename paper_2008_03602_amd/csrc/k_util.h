// Device helpers shared by the kernel families.
#pragma once
#include <hip/hip_runtime.h>

#include "ct_internal.h"

namespace ct {

// Bounds-checked load without a branch: the address is clamped to element 0
// when `ok` is false and the value is replaced by zero. Keeping loads out of
// divergent branches lets the compiler issue a whole batch of them before the
// first wait, instead of waiting for each one in turn.
template <typename T>
__device__ __forceinline__ T load_or_zero(const T* __restrict__ p, int64_t idx, bool ok) {
  const T v = p[ok ? idx : 0];
  return ok ? v : T{};
}

// Raw buffer resource over `bytes` bytes at base: loads at byte offsets at or
// past `bytes` return 0 (the hardware range check), so an out-of-range
// element needs no branch and no clamped address.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}
// Byte offset beyond every buffer of the fp32 families, which hold fewer than 2^31 bytes in
// whole words: reads as 0. Offsets are unsigned, since the words after it, or a second part
// outside, pass the largest int.
constexpr unsigned kOob = 0x7FFFFFFCu;
// The same at a 16-byte offset, for copies of that width and where nothing is added.
constexpr unsigned kOobQuad = 0xFFFFFFF0u;

// One word at byte offset off of r (0 past the buffer's range).
__device__ __forceinline__ float bload1(__amdgpu_buffer_rsrc_t r, unsigned off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
}

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x3 __attribute__((ext_vector_type(3)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
// Three consecutive words at byte offset off (a multiple of 4) of r.
__device__ __forceinline__ void bload3(__amdgpu_buffer_rsrc_t r, unsigned off, float* v) {
  const u32x3 q = __builtin_amdgcn_raw_buffer_load_b96(r, (int)off, 0, 0);
  const unsigned a = q.x, b = q.y, c = q.z;
  v[0] = __builtin_bit_cast(float, a);
  v[1] = __builtin_bit_cast(float, b);
  v[2] = __builtin_bit_cast(float, c);
}
// N consecutive words at byte offset off (a multiple of 4) of r, in loads of up to four
// words; words past the buffer's range read 0.
template <int N>
__device__ __forceinline__ void bload_words(__amdgpu_buffer_rsrc_t r, unsigned off, float* v) {
  if constexpr (N >= 4) {
    const u32x4 q = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0);
    const unsigned a = q.x, b = q.y, c = q.z, d = q.w;
    v[0] = __builtin_bit_cast(float, a);
    v[1] = __builtin_bit_cast(float, b);
    v[2] = __builtin_bit_cast(float, c);
    v[3] = __builtin_bit_cast(float, d);
    bload_words<N - 4>(r, off + 16, v + 4);
  } else if constexpr (N == 3) {
    bload3(r, off, v);
  } else if constexpr (N == 2) {
    const u32x2 q = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0);
    const unsigned a = q.x, b = q.y;
    v[0] = __builtin_bit_cast(float, a);
    v[1] = __builtin_bit_cast(float, b);
  } else if constexpr (N == 1) {
    v[0] = bload1(r, off);
  }
}
__device__ __forceinline__ void bstore1(__amdgpu_buffer_rsrc_t r, unsigned off, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, (int)off, 0, 0);
}

typedef __attribute__((address_space(3))) void lds_void_t;
// One wave instruction: lane i copies the word at byte offset off of r to
// lds[i] (an inactive lane copies nothing), without a trip through registers.
__device__ __forceinline__ void copy_to_lds(__amdgpu_buffer_rsrc_t r, float* lds, unsigned off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t*)lds, 4, (int)off, 0, 0, 0);
}
// The same with 16 bytes per lane: lane i fills lds[4i .. 4i+3] (lds and the
// lane's source 16-byte aligned).
__device__ __forceinline__ void copy16_to_lds(__amdgpu_buffer_rsrc_t r, float* lds, unsigned off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t*)lds, 16, (int)off, 0, 0, 0);
}
// Waits for this wave's copies to land in LDS.
__device__ __forceinline__ void wait_copies() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// floor(n / d) for 0 <= n < 2^22 given inv = 1/d in fp32: (n + 1/2)/d lies at
// least 1/(2d) from an integer and the fp32 product errs by less than that.
__device__ __forceinline__ int qdiv(int n, float inv) { return (int)(((float)n + 0.5f) * inv); }

// floor(n / d) for 0 <= n < 2^31 with a host-computed multiplier: m = ceil(2^(31+s) / d)
// for the smallest 2^s >= d, so m * d exceeds 2^(31+s) by less than 2^s and n times that
// excess stays below 2^(31+s). On a uniform n this is two scalar multiplies.
struct FastDiv {
  uint32_t m;
  int32_t sh;  // 31 + s
  int32_t d;
};
inline FastDiv make_fastdiv(int64_t d) {
  int s = 0;
  while (((int64_t)1 << s) < d) ++s;
  const uint64_t p = (uint64_t)1 << (31 + s);
  return {(uint32_t)((p + (uint64_t)d - 1) / (uint64_t)d), 31 + s, (int32_t)d};
}
__host__ __device__ __forceinline__ int fdiv(int n, const FastDiv& f) {
  return (int)(((uint64_t)(uint32_t)n * f.m) >> f.sh);
}

// Block renumbering for XCD locality: the device deals consecutive blocks to
// its 8 XCDs in turn, so block b runs on XCD b mod 8. Tile of block b when
// each XCD takes one contiguous band of the T tiles (the first T mod 8 XCDs
// take one tile more), so neighbouring tiles share that XCD's L2.
__host__ __device__ inline int xcd_band_tile(int b, int T) {
  const int q = T / 8, r = T % 8, xcd = b % 8, idx = b / 8;
  return xcd < r ? xcd * (q + 1) + idx : r * (q + 1) + (xcd - r) * q + idx;
}

// The wave index as a scalar value, so loops bounded by per-wave values stay
// uniform (scalar branches, unrollable) instead of exec-masked.
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

}  // namespace ct
