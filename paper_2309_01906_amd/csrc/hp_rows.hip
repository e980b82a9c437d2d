// Nests with one reduction per output over a contiguous block, planned automatically:
// float sums of sums, and int32 nests with one operator (or one ARG level).  The level
// map collapses to "outputs" and "elements of a block", so these kernels take a few
// plain arguments instead of a plan in memory (an empty nest through the plan kernels
// took 6.3 us, most of it their reads of the plan and the set-up of the odometer; the
// kernels here 3 us), and pick their shape by the block's length:
//   tiny   blocks shorter than one 16-byte vector: a lane per output;
//   short  up to four vectors per lane of a wave: 2^k lanes per output, 64 / 2^k
//          outputs per step of a wave, the loads of U steps in flight together;
//   long   a workgroup per output (or per part of one): the block's aligned vectors as
//          a stream, its up to two partial vectors as single elements.
// Short blocks start at any element, so their vectors are loaded at the element type's
// alignment (global memory takes any); the last vector of a block is moved back to end
// with it.  MIN, MAX and ARG may see an element twice; sums drop the repeated ones.
#include "hp_rows.h"

#include "hp_fold.h"

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
// index t (keep: the elements that count, a bit each; sums only), one() an element,
// lanes() the groups of 2^lb neighbouring lanes, bits() / of_bits() the 64-bit form in
// LDS and in the partials.
template <class Raw, int OP>
struct Red;

template <class Raw>
struct Red<Raw, HP_OP_SUM> {
  typedef typename std::conditional<std::is_same<Raw, int32_t>::value, long long, double>::type Acc;
  static constexpr bool kSum = true;
  __device__ static __forceinline__ Acc identity() { return 0; }
  __device__ static __forceinline__ void vec(Acc& a, typename Vec<Raw>::A x, uint32_t, uint32_t keep) {
    Acc p[Vec<Raw>::N];
#pragma unroll
    for (int e = 0; e < Vec<Raw>::N; ++e) p[e] = (Acc)((keep >> e) & 1u ? Vec<Raw>::get(x, e) : 0);
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
  __device__ static __forceinline__ void vec(Acc& a, i32x4 x, uint32_t, uint32_t) {
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
  __device__ static __forceinline__ void vec(Acc& a, i32x4 x, uint32_t t, uint32_t) {
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

// Workgroup b of n: the workgroups of one XCD (one residue b mod 8) take a contiguous
// run of the work, as logical_group does for grids that are a multiple of 8.
__device__ __forceinline__ uint32_t xcd_run(uint32_t b, uint32_t n) {
  const uint32_t x = b & 7u, q = n >> 3, r = n & 7u;
  return x * q + (x < r ? x : r) + (b >> 3);
}

constexpr int kRowWaves = 4;

// ---------------------------------------------------------------------------
// tiny blocks: a lane per output

template <class Raw, int OP>
__global__ void __launch_bounds__(256) k_rows_tiny(const Raw* __restrict__ in, void* __restrict__ out, long long n_out, int B,
                                                   int f32_out) {
  typedef Red<Raw, OP> R;
  for (long long o = (long long)xcd_run(blockIdx.x, gridDim.x) * 256 + threadIdx.x; o < n_out;
       o += (long long)gridDim.x * 256) {
    const Raw* p = in + o * B;
    Raw x[Vec<Raw>::N - 1];
#pragma unroll
    for (int e = 0; e < Vec<Raw>::N - 1; ++e) x[e] = p[e < B ? e : 0];
    typename R::Acc a = R::identity();
#pragma unroll
    for (int e = 0; e < Vec<Raw>::N - 1; ++e)
      if (e < B) R::one(a, x[e], (uint32_t)e);
    R::store(out, o, a, f32_out != 0);
  }
}

// ---------------------------------------------------------------------------
// short blocks: 2^lb lanes per output, K vectors per lane, U steps in flight

template <class Raw, int OP, int K, int U>
__global__ void __launch_bounds__(kRowWaves * kWave) k_rows_short(const Raw* __restrict__ in, void* __restrict__ out,
                                                                  long long n_out, int B, int lb, int f32_out) {
  typedef Red<Raw, OP> R;
  typedef typename Vec<Raw>::A V;
  typedef const __attribute__((address_space(1))) typename Vec<Raw>::E GV;
  constexpr int N = Vec<Raw>::N;
  const int lane = (int)(threadIdx.x & 63);
  const int g = lane >> lb, l = lane & ((1 << lb) - 1);
  const int rows = 64 >> lb;  // outputs per step
  // this lane's vectors in a block: where they are loaded, and which elements count
  // (an element the vector before already has does not; ARG indices follow `at`)
  int at[K];
  uint32_t keep[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int t = (k << (lb)) * N + l * N;
    at[k] = t < B - N ? t : B - N;
    const int drop = t - at[k];
    keep[k] = drop >= N ? 0u : (0xFFu << drop) & ((1u << N) - 1u);
  }
  const long long steps = (n_out + rows - 1) / rows;
  const long long w0 = ((long long)xcd_run(blockIdx.x, gridDim.x) * kRowWaves + (threadIdx.x >> 6)) * U;
  const long long stride = (long long)gridDim.x * kRowWaves * U;
  auto load = [&](long long s, V* x) {
    long long o = s * rows + g;
    if (o >= n_out) o = n_out - 1;
    const Raw* p = in + o * B;
#pragma unroll
    for (int k = 0; k < K; ++k) x[k] = *(GV*)(p + at[k]);
  };
  V x[U][K];
#pragma unroll
  for (int u = 0; u < U; ++u) load(w0 + u, x[u]);
  for (long long s0 = w0; s0 < steps; s0 += stride) {
    V y[U][K];
    const bool more = s0 + stride < steps;
    if (more) {
#pragma unroll
      for (int u = 0; u < U; ++u) load(s0 + stride + u, y[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      typename R::Acc a = R::identity();
#pragma unroll
      for (int k = 0; k < K; ++k) R::vec(a, x[u][k], (uint32_t)at[k], keep[k]);
      a = R::lanes(a, lb, lane);
      const long long o = (s0 + u) * rows + g;
      if (l == 0 && o < n_out) R::store(out, o, a, f32_out != 0);
    }
    if (more) {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < K; ++k) x[u][k] = y[u][k];
    }
  }
}

// ---------------------------------------------------------------------------
// long blocks: part q of `parts` of output o on one workgroup of NW waves

template <class Raw, int OP, int NW>
__global__ void __launch_bounds__(NW* kWave) k_rows_long(const Raw* __restrict__ in, void* __restrict__ out,
                                                         unsigned long long* __restrict__ ws, long long B, uint32_t parts,
                                                         long long part_len, int f32_out) {
  typedef Red<Raw, OP> R;
  typedef typename Vec<Raw>::A V;
  typedef const __attribute__((address_space(1))) V GV;
  constexpr int N = Vec<Raw>::N;
  constexpr int U = 4;
  constexpr long long T = NW * kWave;  // vectors per pass of the workgroup
  const uint32_t id = xcd_run(blockIdx.x, gridDim.x);
  const uint32_t o = id / parts, q = id - o * parts;
  const int tid = (int)threadIdx.x, lane = tid & 63;
  const long long row = (long long)o * B;                      // first element of the block
  const long long a0 = (long long)q * part_len;                // this part's elements of the block
  const long long a1 = a0 + part_len < B ? a0 + part_len : B;
  const long long s = row + a0, e = row + a1;
  const long long v0 = (s + N - 1) / N, v1 = e / N;            // its aligned vectors (blocks are longer than 2 N)
  const int head = (int)(v0 * N - s), tail = (int)(e - v1 * N);
  typename R::Acc a = R::identity();
  // partial vectors at both ends, an element per lane of the first wave
  Raw ends = 0;
  long long ei = 0;
  const bool has = tid < head + tail;
  if (has) {
    ei = tid < head ? s + tid : v1 * N + (tid - head);
    ends = in[ei];
  }
  const GV* base = (const GV*)(in + v0 * N);
  const long long n = v1 - v0;                                 // > 0
  const uint32_t t0 = (uint32_t)(v0 * N - row);                // block index of the first vector's first element
  auto fold = [&](V x, long long i) { R::vec(a, x, t0 + (uint32_t)i * N, ~0u); };
  const long long full = n / (U * T) * (U * T);
  if (full > 0) {
    V x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = __builtin_nontemporal_load(base + u * T + tid);
    for (long long i = U * T; i < full; i += U * T) {
      V y[U];
#pragma unroll
      for (int u = 0; u < U; ++u) y[u] = __builtin_nontemporal_load(base + i + u * T + tid);
#pragma unroll
      for (int u = 0; u < U; ++u) fold(x[u], i - U * T + u * T + tid);
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = y[u];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) fold(x[u], full - U * T + u * T + tid);
  }
  if (full < n) {  // the last, partial batch: vectors beyond it repeat the last one
    V x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long long i = full + u * T + tid;
      x[u] = __builtin_nontemporal_load(base + (i < n ? i : n - 1));
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long long i = full + u * T + tid;
      if (R::kSum && i >= n) x[u] = V{0, 0, 0, 0};
      fold(x[u], i < n ? i : n - 1);
    }
  }
  if (has) R::one(a, ends, (uint32_t)(ei - row));
  a = R::lanes(a, 6, lane);
  if constexpr (NW > 1) {
    __shared__ unsigned long long slot[NW];
    if (lane == 0) slot[tid >> 6] = R::bits(a);
    __syncthreads();
    if (tid != 0) return;
    a = R::of_bits(slot[0]);
#pragma unroll
    for (int w = 1; w < NW; ++w) a = R::merge(a, R::of_bits(slot[w]));
  }
  if (tid == 0) {
    if (parts > 1) ws[(long long)o * parts + q] = R::bits(a);
    else R::store(out, o, a, f32_out != 0);
  }
}

// The partials of output o, one workgroup: thread k takes partials k, k + 256, ...; the
// order is fixed by their number.  Float partials are added as (sum, error) pairs.
template <class Raw, int OP>
__global__ void __launch_bounds__(256) k_rows_fold(const unsigned long long* __restrict__ ws, void* __restrict__ out, uint32_t parts,
                                                   int f32_out) {
  typedef Red<Raw, OP> R;
  const unsigned long long* p = ws + (long long)blockIdx.x * parts;
  const int tid = (int)threadIdx.x, lane = tid & 63, w = tid >> 6;
  constexpr int U = 8;
  __shared__ unsigned long long slot[2 * kRowWaves];
  if constexpr (std::is_same<typename R::Acc, double>::value) {
    DPair a{0.0, 0.0};
    for (uint32_t k0 = tid; k0 < parts; k0 += U * 256) {
      double v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = k0 + u * 256 < parts ? R::of_bits(p[k0 + u * 256]) : 0.0;
#pragma unroll
      for (int u = 0; u < U; ++u) dpair_add(a, v[u]);
    }
#pragma unroll
    for (int b = 0; b < 6; ++b) a = dpair_merge(a, DPair{xor_move_d(a.s, 1 << b, lane), xor_move_d(a.c, 1 << b, lane)});
    if (lane == 0) {
      slot[2 * w] = (unsigned long long)__double_as_longlong(a.s);
      slot[2 * w + 1] = (unsigned long long)__double_as_longlong(a.c);
    }
    __syncthreads();
    if (tid != 0) return;
#pragma unroll
    for (int j = 1; j < kRowWaves; ++j)
      a = dpair_merge(a, DPair{__longlong_as_double((long long)slot[2 * j]), __longlong_as_double((long long)slot[2 * j + 1])});
    R::store(out, blockIdx.x, a.s + a.c, f32_out != 0);
  } else {
    typename R::Acc a = R::identity();
    for (uint32_t k0 = tid; k0 < parts; k0 += U * 256) {
      unsigned long long v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = k0 + u * 256 < parts ? p[k0 + u * 256] : R::bits(R::identity());
#pragma unroll
      for (int u = 0; u < U; ++u) a = R::merge(a, R::of_bits(v[u]));
    }
    a = R::lanes(a, 6, lane);
    if (lane == 0) slot[w] = R::bits(a);
    __syncthreads();
    if (tid != 0) return;
#pragma unroll
    for (int j = 1; j < kRowWaves; ++j) a = R::merge(a, R::of_bits(slot[j]));
    R::store(out, blockIdx.x, a, f32_out != 0);
  }
}

template <class Raw, int OP>
void rows_go(const RowRoute& r, const Raw* in, void* out, void* ws, hipStream_t st) {
  const int f = r.f32_out;
  const dim3 wg(kRowWaves * kWave);
  if (r.kind == ROWS_TINY) {
    hipLaunchKernelGGL((k_rows_tiny<Raw, OP>), dim3(r.grid), wg, 0, st, in, out, (long long)r.n_out, (int)r.block, f);
    return;
  }
  if (r.kind == ROWS_SHORT) {
    const dim3 g(r.grid);
    const long long n = r.n_out;
    const int B = (int)r.block, lb = r.lane_bits;
    if (r.vecs == 1 && r.ahead == 1) hipLaunchKernelGGL((k_rows_short<Raw, OP, 1, 1>), g, wg, 0, st, in, out, n, B, lb, f);
    else if (r.vecs == 1) hipLaunchKernelGGL((k_rows_short<Raw, OP, 1, 4>), g, wg, 0, st, in, out, n, B, lb, f);
    else if (r.vecs == 2 && r.ahead == 1) hipLaunchKernelGGL((k_rows_short<Raw, OP, 2, 1>), g, wg, 0, st, in, out, n, B, lb, f);
    else if (r.vecs == 2) hipLaunchKernelGGL((k_rows_short<Raw, OP, 2, 2>), g, wg, 0, st, in, out, n, B, lb, f);
    else if (r.vecs == 3) hipLaunchKernelGGL((k_rows_short<Raw, OP, 3, 1>), g, wg, 0, st, in, out, n, B, lb, f);
    else hipLaunchKernelGGL((k_rows_short<Raw, OP, 4, 1>), g, wg, 0, st, in, out, n, B, lb, f);
    return;
  }
  unsigned long long* w = reinterpret_cast<unsigned long long*>(ws);
  const long long B = r.block, pl = r.part_len;
  const uint32_t parts = r.parts;
  const dim3 g(r.grid);
  if (r.waves == 1) hipLaunchKernelGGL((k_rows_long<Raw, OP, 1>), g, dim3(64), 0, st, in, out, w, B, parts, pl, f);
  else if (r.waves == 2) hipLaunchKernelGGL((k_rows_long<Raw, OP, 2>), g, dim3(128), 0, st, in, out, w, B, parts, pl, f);
  else if (r.waves == 4) hipLaunchKernelGGL((k_rows_long<Raw, OP, 4>), g, dim3(256), 0, st, in, out, w, B, parts, pl, f);
  else hipLaunchKernelGGL((k_rows_long<Raw, OP, 8>), g, dim3(512), 0, st, in, out, w, B, parts, pl, f);
  if (parts > 1)
    hipLaunchKernelGGL((k_rows_fold<Raw, OP>), dim3((unsigned)r.n_out), dim3(256), 0, st, w, out, parts, f);
}

}  // namespace

hp_status launch_rows(const RowRoute& r, const void* in, void* out, void* ws, hipStream_t st) {
  if (r.dtype == HP_F32) {
    rows_go<float, HP_OP_SUM>(r, reinterpret_cast<const float*>(in), out, ws, st);
  } else if (r.dtype == HP_BF16) {
    rows_go<uint16_t, HP_OP_SUM>(r, reinterpret_cast<const uint16_t*>(in), out, ws, st);
  } else {
    const int32_t* x = reinterpret_cast<const int32_t*>(in);
    switch (r.op) {
      case HP_OP_MIN: rows_go<int32_t, HP_OP_MIN>(r, x, out, ws, st); break;
      case HP_OP_MAX: rows_go<int32_t, HP_OP_MAX>(r, x, out, ws, st); break;
      case HP_OP_ARGMIN: rows_go<int32_t, HP_OP_ARGMIN>(r, x, out, ws, st); break;
      case HP_OP_ARGMAX: rows_go<int32_t, HP_OP_ARGMAX>(r, x, out, ws, st); break;
      default: rows_go<int32_t, HP_OP_SUM>(r, x, out, ws, st); break;
    }
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(HP_EDEVICE, "kernel launch failed: %s", hipGetErrorString(e));
  return HP_OK;
}

}  // namespace hp
