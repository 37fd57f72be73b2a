// Storage types of the kernel library as the contraction kernels read them:
// loads of VEC values.
#pragma once

#include <hip/hip_runtime.h>

namespace pat {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));

struct bf16_t { unsigned short bits; };
struct f16_t { unsigned short bits; };

// VEC values per load (16 bytes if not said otherwise)
template <typename HT, int V = 16 / (int)sizeof(HT)> struct Slab;

template <> struct Slab<float, 4> {
  static constexpr int VEC = 4;
  typedef v4f raw_t;
  __device__ static __forceinline__ float get(const raw_t& r, int v) { return r[v]; }
};

template <int V> struct Slab<bf16_t, V> {
  static constexpr int VEC = V;
  typedef unsigned int raw_t __attribute__((ext_vector_type(V / 2)));
  __device__ static __forceinline__ float get(const raw_t& r, int v) {
    const unsigned w = r[v >> 1];
    const unsigned b = (v & 1) ? (w & 0xFFFF0000u) : (w << 16);
    return __uint_as_float(b);
  }
};

template <int V> struct Slab<f16_t, V> {
  static constexpr int VEC = V;
  typedef unsigned int raw_t __attribute__((ext_vector_type(V / 2)));
  __device__ static __forceinline__ float get(const raw_t& r, int v) {
    const unsigned w = r[v >> 1];
    const unsigned short h = (v & 1) ? (unsigned short)(w >> 16) : (unsigned short)(w & 0xFFFFu);
    _Float16 x;
    __builtin_memcpy(&x, &h, 2);
    return (float)x;
  }
};

}  // namespace pat
