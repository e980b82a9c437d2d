// Carriers and loads shared by the row kernels (hp_rows.hip) and the segment kernels
// (hp_segs.hip): a reduction whose operator and element type are known at compile time.
#pragma once

#include "hp_nest.h"

namespace hp {

namespace {

template <class Raw>
struct Vec;
template <>
struct Vec<float> {
  typedef f32x4 A;                                                            // 16-byte aligned
  typedef float E __attribute__((ext_vector_type(4), aligned(4)));            // element aligned
  static constexpr int N = 4;
  __device__ static __forceinline__ float get(A x, int e) { return x[e]; }
};
template <>
struct Vec<int32_t> {
  typedef i32x4 A;
  typedef int E __attribute__((ext_vector_type(4), aligned(4)));
  static constexpr int N = 4;
  __device__ static __forceinline__ int get(A x, int e) { return x[e]; }
};
template <>
struct Vec<uint16_t> {
  typedef u32x4 A;
  typedef unsigned int E __attribute__((ext_vector_type(4), aligned(2)));
  static constexpr int N = 8;
  __device__ static __forceinline__ float get(A x, int e) { return e & 1 ? bf16_hi(x[e >> 1]) : bf16_lo(x[e >> 1]); }
};
__device__ __forceinline__ float value_of(float x) { return x; }
__device__ __forceinline__ int value_of(int32_t x) { return x; }
__device__ __forceinline__ float value_of(uint16_t x) { return bf16_lo(x); }

// The carrier of one reduction: vec() folds a whole vector whose first element has
// index t, one() an element,
// lanes() the groups of 2^lb neighbouring lanes, bits() / of_bits() the 64-bit form in
// LDS and in the partials.
template <class Raw, int OP>
struct Red;

template <class Raw>
struct Red<Raw, HP_OP_SUM> {
  typedef typename std::conditional<std::is_same<Raw, int32_t>::value, long long, double>::type Acc;
  static constexpr bool kSum = true;
  __device__ static __forceinline__ Acc identity() { return 0; }
  __device__ static __forceinline__ void vec(Acc& a, typename Vec<Raw>::A x, uint32_t) {
    Acc p[Vec<Raw>::N];
#pragma unroll
    for (int e = 0; e < Vec<Raw>::N; ++e) p[e] = (Acc)Vec<Raw>::get(x, e);
#pragma unroll
    for (int h = 1; h < Vec<Raw>::N; h *= 2)
#pragma unroll
      for (int e = 0; e + h < Vec<Raw>::N; e += 2 * h) p[e] = add(p[e], p[e + h]);
    a = add(a, p[0]);
  }
  __device__ static __forceinline__ Acc add(Acc a, Acc b) {
    if constexpr (std::is_same<Acc, long long>::value) return (long long)((unsigned long long)a + (unsigned long long)b);
    else return a + b;
  }
  __device__ static __forceinline__ void one(Acc& a, Raw x, uint32_t) { a = add(a, (Acc)value_of(x)); }
  __device__ static __forceinline__ Acc merge(Acc a, Acc b) { return add(a, b); }
  template <int B>
  __device__ static __forceinline__ Acc step(Acc a, int lane) {
    if constexpr (std::is_same<Acc, long long>::value) return key_sum_step<B>(a, true, lane);
    else return lane_step<B>(a, true, lane);
  }
  __device__ static __forceinline__ Acc lanes(Acc a, int lb, int lane) {
    if (lb > 0) a = step<0>(a, lane);
    if (lb > 1) a = step<1>(a, lane);
    if (lb > 2) a = step<2>(a, lane);
    if (lb > 3) a = step<3>(a, lane);
    if (lb > 4) a = step<4>(a, lane);
    if (lb > 5) a = step<5>(a, lane);
    return a;
  }
  __device__ static __forceinline__ unsigned long long bits(Acc a) {
    if constexpr (std::is_same<Acc, long long>::value) return (unsigned long long)a;
    else return (unsigned long long)__double_as_longlong(a);
  }
  __device__ static __forceinline__ Acc of_bits(unsigned long long b) {
    if constexpr (std::is_same<Acc, long long>::value) return (long long)b;
    else return __longlong_as_double((long long)b);
  }
  __device__ static __forceinline__ void store(void* out, long long o, Acc a, bool f32_out) {
    if constexpr (std::is_same<Acc, long long>::value) {
      reinterpret_cast<long long*>(out)[o] = a;
    } else {
      const double v = float_result(a);
      if (f32_out) reinterpret_cast<float*>(out)[o] = (float)v;
      else reinterpret_cast<double*>(out)[o] = v;
    }
  }
};

// MIN and MAX: the value itself
template <int OP>
struct RedMinMax {
  typedef int Acc;
  static constexpr bool kSum = false;
  static constexpr bool kMin = OP == HP_OP_MIN;
  __device__ static __forceinline__ Acc identity() { return kMin ? 0x7FFFFFFF : (int)0x80000000; }
  __device__ static __forceinline__ Acc merge(Acc a, Acc b) { return kMin ? min(a, b) : max(a, b); }
  __device__ static __forceinline__ void vec(Acc& a, i32x4 x, uint32_t) {
    a = merge(merge(a, merge(x.x, x.y)), merge(x.z, x.w));
  }
  __device__ static __forceinline__ void one(Acc& a, int x, uint32_t) { a = merge(a, x); }
  __device__ static __forceinline__ Acc lanes(Acc a, int lb, int lane) {
    const uint32_t m = (1u << lb) - 1u;
    return word_allreduce<kMin, int>(a, m, m, lane);
  }
  __device__ static __forceinline__ unsigned long long bits(Acc a) { return (unsigned long long)(long long)a; }
  __device__ static __forceinline__ Acc of_bits(unsigned long long b) { return (int)(uint32_t)b; }
  __device__ static __forceinline__ void store(void* out, long long o, Acc a, bool) { reinterpret_cast<int*>(out)[o] = a; }
};
template <>
struct Red<int32_t, HP_OP_MIN> : RedMinMax<HP_OP_MIN> {};
template <>
struct Red<int32_t, HP_OP_MAX> : RedMinMax<HP_OP_MAX> {};

// ARGMIN and ARGMAX: (value, index), the smaller index among equal values.  An empty
// carrier has the index 2^31 - 1 beside the value no element beats.
template <int OP>
struct RedArg {
  struct Acc {
    int v;
    uint32_t i;
  };
  static constexpr bool kSum = false;
  static constexpr bool kMin = OP == HP_OP_ARGMIN;
  __device__ static __forceinline__ Acc identity() { return Acc{kMin ? 0x7FFFFFFF : (int)0x80000000, 0x7FFFFFFFu}; }
  __device__ static __forceinline__ bool better(int x, int y) { return kMin ? x < y : x > y; }
  __device__ static __forceinline__ Acc merge(Acc a, Acc b) {
    return better(b.v, a.v) || (b.v == a.v && b.i < a.i) ? b : a;
  }
  __device__ static __forceinline__ void vec(Acc& a, i32x4 x, uint32_t t) {
    const int m = kMin ? min(min(x.x, x.y), min(x.z, x.w)) : max(max(x.x, x.y), max(x.z, x.w));
    const uint32_t p = x.x == m ? 0u : x.y == m ? 1u : x.z == m ? 2u : 3u;
    a = merge(a, Acc{m, t + p});
  }
  __device__ static __forceinline__ void one(Acc& a, int x, uint32_t t) { a = merge(a, Acc{x, t}); }
  // 64-bit keys whose signed order is that of (value, index), as IntK's
  __device__ static __forceinline__ unsigned long long bits(Acc a) {
    return (unsigned long long)(uint32_t)a.v << 32 | (kMin ? a.i : 0xFFFFFFFFu - a.i);
  }
  __device__ static __forceinline__ Acc of_bits(unsigned long long b) {
    const uint32_t lo = (uint32_t)b;
    return Acc{(int)(uint32_t)(b >> 32), kMin ? lo : 0xFFFFFFFFu - lo};
  }
  __device__ static __forceinline__ Acc lanes(Acc a, int lb, int lane) {
    const uint32_t m = (1u << lb) - 1u;
    return of_bits((unsigned long long)key_minmax<kMin>((long long)bits(a), m, m, lane));
  }
  __device__ static __forceinline__ void store(void* out, long long o, Acc a, bool) {
    reinterpret_cast<int*>(out)[o] = (int)a.i;
  }
};
template <>
struct Red<int32_t, HP_OP_ARGMIN> : RedArg<HP_OP_ARGMIN> {};
template <>
struct Red<int32_t, HP_OP_ARGMAX> : RedArg<HP_OP_ARGMAX> {};

// A vector's elements from number `drop` on, the others cleared: a mask per 32-bit word,
// made once per lane, so that dropping costs one `and` per word.
template <class Raw>
__device__ __forceinline__ u32x4 keep_from(int drop) {
  constexpr int per = Vec<Raw>::N / 4;  // elements per word
  u32x4 m;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const int lost = drop - w * per;  // elements of this word that go
    m[w] = lost <= 0 ? 0xFFFFFFFFu : (per == 2 && lost == 1) ? 0xFFFF0000u : 0u;
  }
  return m;
}
template <class Raw>
__device__ __forceinline__ typename Vec<Raw>::A kept(typename Vec<Raw>::A x, u32x4 m) {
  return __builtin_bit_cast(typename Vec<Raw>::A, __builtin_bit_cast(u32x4, x) & m);
}

// Workgroup b of n: the workgroups of one XCD (one residue b mod 8) take a contiguous
// run of the work, as logical_group does for grids that are a multiple of 8.
__device__ __forceinline__ uint32_t xcd_run(uint32_t b, uint32_t n) {
  const uint32_t x = b & 7u, q = n >> 3, r = n & 7u;
  return x * q + (x < r ? x : r) + (b >> 3);
}

}  // namespace

}  // namespace hp
