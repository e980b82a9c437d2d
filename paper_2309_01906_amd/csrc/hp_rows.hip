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
//
// Measured, short blocks, from 8192 waves that walk the rows to a round of steps per wave
// and 16 or 32 lanes with up to three vectors each:
//   float 100000 x 600 (240 MB)    41.9 -> 34.2 us     bf16 100000 x 1000 (200 MB)  34.7 -> 29.6 us
//   float 300000 x 130             42.5 -> 26.2 us     bf16 500000 x 130            38.2 -> 30.4 us
//   int32 100003 x 129 ARGMIN      16.2 -> 10.4 us     float 2000000 x 16           26.9 -> 23.3 us
#include "hp_rows.h"

#include "hp_fold.h"
#include "hp_red.h"

namespace hp {

namespace {

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
  u32x4 keep[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int t = (k << (lb)) * N + l * N;
    at[k] = t < B - N ? t : B - N;
    keep[k] = keep_from<Raw>(t - at[k]);
  }
  const long long steps = (n_out + rows - 1) / rows;
  const long long w0 =
      ((long long)xcd_run(blockIdx.x, gridDim.x) * kRowWaves + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6))) * U;
  const long long stride = (long long)gridDim.x * kRowWaves * U;
  // a step's blocks lie within 64 KiB of its first: 32-bit offsets; outputs beyond the
  // last read it again, steps beyond the last too
  const uint32_t lane_off = (uint32_t)(g * B);
  auto load = [&](long long s, V* x) {
    const long long o = s * rows < n_out ? s * rows : n_out - 1;
    const long long left = n_out - 1 - o;
    const uint32_t most = (uint32_t)((left < rows ? (int)left : rows) * B);
    const Raw* p = in + o * B;
    const uint32_t off = min(lane_off, most);
#pragma unroll
    for (int k = 0; k < K; ++k) x[k] = __builtin_nontemporal_load((GV*)(p + (off + (uint32_t)at[k])));
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
      for (int k = 0; k < K; ++k) R::vec(a, R::kSum ? kept<Raw>(x[u][k], keep[k]) : x[u][k], (uint32_t)at[k]);
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
  auto fold = [&](V x, long long i) { R::vec(a, x, t0 + (uint32_t)i * N); };
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
