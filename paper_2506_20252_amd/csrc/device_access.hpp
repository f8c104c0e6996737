// Device-side building blocks shared by the kernels: vector types, explicit
// global-memory accesses, rank arithmetic and the bf16 conversions.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace pat {
namespace {

// Native clang vectors (not HIP's wrapper structs), so that the nontemporal
// builtins apply directly to the 128-bit loads and stores.
typedef unsigned int v2u __attribute__((ext_vector_type(2)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

// Buffer addresses come from pointer tables, so the compiler cannot tell they
// are global memory and would emit flat accesses; every data access goes
// through an explicit global (address space 1) pointer instead.
#define PAT_GLOBAL __attribute__((address_space(1)))

// Access alignment A: 0 keeps the type's own; A > 0 lets a 16-byte vector
// sit at any A-byte-aligned address (the relaxed variants, for buffers that
// are only element-aligned).  Code objects for gfx950 run in unaligned-access
// mode, where such a vector is still one 128-bit load or store.
template <typename T, int A>
struct Access {
  typedef T type __attribute__((aligned(A)));
};
template <typename T>
struct Access<T, 0> {
  typedef T type;
};

template <typename T, bool NT, int A = 0>
__device__ __forceinline__ T ldg(const char* p) {
  using AT = typename Access<T, A>::type;
  const PAT_GLOBAL AT* q = (const PAT_GLOBAL AT*)(p);
  if constexpr (NT) return __builtin_nontemporal_load(q);
  return *q;
}

template <bool NT, int A = 0, typename T>
__device__ __forceinline__ void stg(char* p, const T& v) {
  using AT = typename Access<T, A>::type;
  PAT_GLOBAL AT* q = (PAT_GLOBAL AT*)(p);
  if constexpr (NT)
    __builtin_nontemporal_store(v, q);
  else
    *q = v;
}

// Word q of a vector, as raw bits.
__device__ __forceinline__ uint32_t word(v4u x, int q) { return x[q]; }
__device__ __forceinline__ uint32_t word(v2u x, int q) { return x[q]; }
__device__ __forceinline__ uint32_t word(v4f x, int q) { return __float_as_uint(x[q]); }

// Stores elements [from, n) of the vector x, taken as n elements of EB bytes
// each (EB = 2 or 4; 2-byte element 2j is the low half of word j).  Used for
// a chunk-piece's partial last vector, which is moved back to end at the
// piece's end: its first `from` elements belong to the vector before it.
template <bool NT, int EB, typename T>
__device__ __forceinline__ void stg_from(char* p, T x, int from) {
  static_assert(EB == 2 || EB == 4, "2- or 4-byte elements");
  constexpr int W = sizeof(T) / 4;
  if constexpr (EB == 4) {
#pragma unroll
    for (int q = 0; q < W; ++q)
      if (q >= from) stg<NT>(p + 4 * q, word(x, q));
  } else {
#pragma unroll
    for (int q = 0; q < 2 * W; ++q)
      if (q >= from) stg<NT>(p + 2 * q, (uint16_t)(word(x, q / 2) >> (16 * (q & 1))));
  }
}

__device__ __forceinline__ int wrap_add(int a, int b, int n) {
  const int s = a + b;
  return s >= n ? s - n : s;
}

__device__ __forceinline__ int wrap_sub(int a, int b, int n) {
  const int s = a - b;
  return s < 0 ? s + n : s;
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// float32 -> bf16, round to nearest, ties to even (NaN stays a quiet NaN).
__device__ __forceinline__ uint32_t bf16_rne(float f) {
  const uint32_t u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (u >> 16) | 0x40u;
  return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

}  // namespace
}  // namespace pat
