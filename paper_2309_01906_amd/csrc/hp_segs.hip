// Int32 nests of two or three reducing segments (runs of levels with one operator),
// planned automatically.  The view is out[o] = Q over q of M over m of L over the
// contiguous row (o, q, m) of eL elements, eQ = 1 for two segments.  No level has to be
// a multiple of anything: rows start at any element and are loaded as 16-byte vectors
// at 4-byte alignment.
//   rows of at most four vectors per lane: k_seg_rows reduces rows and M together.  A
//     wave takes 64 / 2^lb rows a step, 2^lb lanes each; a row's value goes into its
//     lane group's carrier of M, and the groups, the waves and (in the tail) the parts
//     of one (o, q) meet once at the end.
//   longer rows: the row kernels reduce every row to one value first.
//     With as many pairs as fill the chip a wave runs through several (k_seg_run), some
//     of them side by side when M is short.
// k_seg_tail then reduces what is left: the parts of M, or its values, and Q.
#include "hp_segs.h"

#include "hp_fold.h"
#include "hp_red.h"
#include "hp_rows.h"

namespace hp {

namespace {

template <int OP>
__device__ __forceinline__ long long child_of(typename Red<int32_t, OP>::Acc a) {
  if constexpr (OP == HP_OP_ARGMIN || OP == HP_OP_ARGMAX) return (long long)a.i;
  else return (long long)a;
}

// Fold child value x with index t into a, where t grows from call to call (so an equal
// value never replaces the one before it); one uniform branch per call.
__device__ __forceinline__ void outer_add(IAcc& a, long long x, int t, int op, bool ok) {
  if (op == HP_OP_SUM) {
    a.v = (long long)((unsigned long long)a.v + (unsigned long long)(ok ? x : 0));
  } else {
    const bool mn = op == HP_OP_MIN || op == HP_OP_ARGMIN;
    // the first child of an ARG level always enters: the identity's index is 2^31 - 1
    const bool first = (op == HP_OP_ARGMIN || op == HP_OP_ARGMAX) && a.i == 0x7FFFFFFF;
    const bool take = ok && ((mn ? x < a.v : x > a.v) || first);
    a.v = take ? x : a.v;
    a.i = take ? t : a.i;
  }
}

__device__ __forceinline__ IAcc iacc_shfl(IAcc a, int b, int lane) { return IntT::shfl(a, 1 << b, lane); }

// The carrier of M: one 64-bit key (IntK) while an ARG level's children fit 32 bits,
// else (an ARG of int64 sums) a (value, index) pair.  Children of one lane come with
// growing m.
struct KeyM {
  typedef long long Acc;
  __device__ static __forceinline__ Acc identity(int op) { return IntK::identity(op); }
  __device__ static __forceinline__ void add(Acc& a, long long x, int m, int op, bool ok) {
    const long long k = IntK::key(x, m, op);
    a = IntK::merge(a, ok ? k : IntK::identity(op), op);
  }
  // over the lane groups: bits lo .. hi - 1, the bits below lo hold one value
  __device__ static __forceinline__ Acc lanes(Acc a, int lo, int hi, int lane, int op) {
    const uint32_t vm = (1u << hi) - (1u << lo);
    if (!vm) return a;
    if (op == HP_OP_SUM) {
      if (vm & 1u) a = key_sum_step<0>(a, true, lane);
      if (vm & 2u) a = key_sum_step<1>(a, true, lane);
      if (vm & 4u) a = key_sum_step<2>(a, true, lane);
      if (vm & 8u) a = key_sum_step<3>(a, true, lane);
      if (vm & 16u) a = key_sum_step<4>(a, true, lane);
      if (vm & 32u) a = key_sum_step<5>(a, true, lane);
      return a;
    }
    if (IntK::minlike(op)) return key_minmax<true>(a, vm, vm, lane);
    return key_minmax<false>(a, vm, vm, lane);
  }
  __device__ static __forceinline__ IAcc pair(Acc a, int op) {
    if (!IntK::arg(op)) return IAcc{a, 0, 0};
    return IAcc{(long long)(int)(uint32_t)((unsigned long long)a >> 32), (int)IntK::emit(a, op), 0};
  }
};
struct PairM {
  typedef IAcc Acc;
  __device__ static __forceinline__ Acc identity(int op) { return IntT::identity(op); }
  __device__ static __forceinline__ void add(Acc& a, long long x, int m, int op, bool ok) { outer_add(a, x, m, op, ok); }
  __device__ static __forceinline__ Acc lanes(Acc a, int lo, int hi, int lane, int op) {
    for (int b = lo; b < hi; ++b) a = IntT::merge(a, iacc_shfl(a, b, lane), op);
    return a;
  }
  __device__ static __forceinline__ IAcc pair(Acc a, int) { return a; }
};

// One row on 2^lb lanes: where this lane's vectors lie, and which of their elements
// count (an element that the vector before already has does not; ARG indices follow).
template <int OP, int K>
struct SegRow {
  typedef Red<int32_t, OP> R;
  static constexpr int KK = K > 0 ? K : 1;
  int at[KK];
  u32x4 keep[KK];
  int eL, lb;
  __device__ __forceinline__ SegRow(const SegRoute& S, int lane) {
    eL = S.eL;
    lb = S.lane_bits;
    const int l = lane & ((1 << lb) - 1);
#pragma unroll
    for (int k = 0; k < KK; ++k) {
      const int t = (k << lb) * 4 + l * 4;
      at[k] = K < 0 ? 0 : (t < eL - 4 ? t : eL - 4);
      keep[k] = keep_from<int32_t>(t - at[k]);
    }
  }
  __device__ __forceinline__ void load(const int32_t* base, uint32_t off, i32x4* x) const {
    typedef const __attribute__((address_space(1))) Vec<int32_t>::E GV;
    if constexpr (K < 0) {
      typedef int E __attribute__((ext_vector_type(-K), aligned(4)));
      const E v = __builtin_nontemporal_load((const __attribute__((address_space(1))) E*)(base + off));
#pragma unroll
      for (int e = 0; e < -K; ++e) x[0][e] = v[e];
    } else {
#pragma unroll
      for (int k = 0; k < KK; ++k) x[k] = __builtin_nontemporal_load((GV*)(base + (off + (uint32_t)at[k])));
    }
  }
  // the row's value, on every lane of its group
  __device__ __forceinline__ long long reduce(const i32x4* x, int lane) const {
    typename R::Acc a = R::identity();
    if constexpr (K < 0) {
#pragma unroll
      for (int e = 0; e < -K; ++e) R::one(a, x[0][e], (uint32_t)e);
    } else {
#pragma unroll
      for (int k = 0; k < KK; ++k) R::vec(a, R::kSum ? kept<int32_t>(x[k], keep[k]) : x[k], (uint32_t)at[k]);
      a = R::lanes(a, lb, lane);
    }
    return child_of<OP>(a);
  }
};

// A complete carrier of M: to the tail, or the nest's output.
__device__ __forceinline__ void seg_out(const SegRoute& S, void* out, IAcc* ws, long long unit, IAcc acc) {
  if (S.tail) {
    ws[unit] = acc;
  } else {
    const long long v = IntT::emit(acc, S.opM);
    if (S.out64) reinterpret_cast<long long*>(out)[unit] = v;
    else reinterpret_cast<int*>(out)[unit] = (int)v;
  }
}

// One (o, q) pair and part per workgroup of NW waves.  K vectors per lane and row (-1
// to -3: rows of that many elements, a lane each), U steps in flight.
template <int OP, int K, class M, int NW, int U>
__global__ void __launch_bounds__(NW* kWave)
    k_seg_rows(const int32_t* __restrict__ in, void* __restrict__ out, IAcc* __restrict__ ws, SegRoute S) {
  typedef Red<int32_t, OP> R;
  const int lane = (int)(threadIdx.x & 63);
  const int w = (int)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t unit = xcd_run(blockIdx.x, gridDim.x);  // pair * parts + part
  const uint32_t pair = unit / S.parts, part = unit - pair * S.parts;
  const int lb = S.lane_bits, eM = S.eM;
  const int g = lane >> lb, rows = 64 >> lb;
  const SegRow<OP, K> row(S, lane);
  // rows lie within 2^31 bytes of their pair's first (the planner checked): 32-bit offsets
  const int32_t* base = in + (long long)pair * eM * S.eL;
  const uint32_t lane_off = (uint32_t)(g * S.eL), last_off = (uint32_t)((eM - 1) * S.eL);
  // this wave's steps: part * per + w, then every NW-th
  const int s1 = ((int)part + 1) * S.per < S.steps ? ((int)part + 1) * S.per : S.steps;
  const int s0 = (int)part * S.per + w;
  constexpr int KK = SegRow<OP, K>::KK;
  auto load = [&](int s, i32x4* x) {
    row.load(base, min((uint32_t)(s * rows * S.eL) + lane_off, last_off), x);
  };
  typename M::Acc acc = M::identity(S.opM);
  i32x4 x[U][KK];
#pragma unroll
  for (int u = 0; u < U; ++u) load(s0 + u * NW, x[u]);
  for (int s = s0; s < s1; s += U * NW) {
    i32x4 y[U][KK];
    const bool more = s + U * NW < s1;
    if (more) {
#pragma unroll
      for (int u = 0; u < U; ++u) load(s + (U + u) * NW, y[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int su = s + u * NW, m = su * rows + g;
      M::add(acc, row.reduce(x[u], lane), m, S.opM, m < eM && su < s1);
    }
    if (more) {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < KK; ++k) x[u][k] = y[u][k];
    }
  }
  // the wave's lane groups, then its workgroup's waves
  acc = M::lanes(acc, lb, 6, lane, S.opM);
  __shared__ IAcc slot[NW];
  if (lane == 0) slot[w] = M::pair(acc, S.opM);
  __syncthreads();
  if (w != 0 || lane != 0) return;
  IAcc r = slot[0];
#pragma unroll
  for (int j = 1; j < NW; ++j) r = IntT::merge(r, slot[j], S.opM);
  seg_out(S, out, ws, unit, r);
}

// A run of (o, q) pairs per wave.  A step is 64 / 2^lb rows: of 2^pb pairs at once when
// M has no more rows than that leaves each, else of one pair, whose carrier is complete
// after S.steps steps.  The loads of U steps are in flight across pairs.
template <int OP, int K, class M, int U>
__global__ void __launch_bounds__(256)
    k_seg_run(const int32_t* __restrict__ in, void* __restrict__ out, IAcc* __restrict__ ws, SegRoute S) {
  const int lane = (int)(threadIdx.x & 63);
  const int w = (int)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const long long wave = (long long)xcd_run(blockIdx.x, gridDim.x) * 4 + w;
  const int lb = S.lane_bits, top = 6 - S.pair_bits, eM = S.eM;
  const int pr = lane >> top, g = (lane & ((1 << top) - 1)) >> lb, rows = 1 << (top - lb);
  const bool lead = (lane & ((1 << top) - 1)) == 0;
  const long long pairs = S.n_out * S.eQ, groups = (pairs + (1 << S.pair_bits) - 1) >> S.pair_bits;
  const long long g0 = wave * S.run, g1 = g0 + S.run < groups ? g0 + S.run : groups;
  if (g0 >= g1) return;
  const SegRow<OP, K> row(S, lane);
  constexpr int KK = SegRow<OP, K>::KK;
  long long lg = g0;  // the step whose loads come next
  int ls = 0;
  // 32-bit offsets from the group's first element, as above; in the last group the lanes
  // of pairs that do not exist read its last pair
  const uint32_t block = (uint32_t)(eM * S.eL), step = (uint32_t)(rows * S.eL);
  const uint32_t lane_off = (uint32_t)(g * S.eL), last_off = (uint32_t)((eM - 1) * S.eL);
  const uint32_t here = (uint32_t)pr * block;
  const uint32_t over = min((uint32_t)pr, (uint32_t)(pairs - 1 - ((groups - 1) << S.pair_bits))) * block;
  const int32_t* base = in + (lg << S.pair_bits) * block;
  const long long hop = (long long)block << S.pair_bits;
  uint32_t off = 0;
  auto load = [&](i32x4* x) {
    row.load(base, (lg < groups - 1 ? here : over) + min(off + lane_off, last_off), x);
    off += step;
    if (++ls == S.steps) {
      ls = 0;
      off = 0;
      if (lg < groups - 1) {
        ++lg;
        base += hop;
      }
    }
  };
  i32x4 x[U][KK];
#pragma unroll
  for (int u = 0; u < U; ++u) load(x[u]);
  typename M::Acc acc = M::identity(S.opM);
  int cs = 0;
  long long cg = g0;
  for (long long left = (g1 - g0) * S.steps; left > 0; left -= U) {
    i32x4 y[U][KK];
    const bool more = left > U;
    if (more) {
#pragma unroll
      for (int u = 0; u < U; ++u) load(y[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int m = cs * rows + g;
      M::add(acc, row.reduce(x[u], lane), m, S.opM, m < eM);
      if (++cs == S.steps) {  // the pair is complete: its lane groups meet
        acc = M::lanes(acc, lb, top, lane, S.opM);
        const long long pair = (cg << S.pair_bits) + pr;
        if (lead && cg < g1 && pair < pairs) seg_out(S, out, ws, pair, M::pair(acc, S.opM));
        acc = M::identity(S.opM);
        cs = 0;
        ++cg;
      }
    }
    if (more) {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < KK; ++k) x[u][k] = y[u][k];
    }
  }
}

// Output o on one workgroup: for every q, the eM entries (o, q, m) -- carriers of M
// (PARTS: the parts of its rows) or its child values -- then Q over q.  A wave takes
// every NW-th q, or all waves share one when there is only one.
template <class In, bool PARTS>
__global__ void __launch_bounds__(1024) k_seg_tail(const In* __restrict__ ws, void* __restrict__ out, int eQ, int n, int opQ,
                                                   int opM, int out64) {
  const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6), nw = (int)(blockDim.x >> 6);
  const long long o = blockIdx.x;
  const In* p = ws + o * eQ * n;
  __shared__ IAcc slot[16];
  auto add = [&](IAcc& a, In x, int m) {
    if constexpr (PARTS) a = IntT::merge(a, x, opM);
    else outer_add(a, (long long)x, m, opM, true);
  };
  constexpr int U = 4;
  auto span = [&](const In* r, int first, int stride) {  // this lane's entries of one q
    IAcc a = IntT::identity(opM);
    for (int m0 = first; m0 < n; m0 += U * stride) {
      In x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = r[m0 + u * stride < n ? m0 + u * stride : m0];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (m0 + u * stride < n) add(a, x[u], m0 + u * stride);
    }
    return a;
  };
  IAcc r;
  int op;
  if (opQ == HP_OP_NONE) {  // M alone: the whole workgroup on its entries
    r = span(p, (int)threadIdx.x, (int)blockDim.x);
    op = opM;
  } else if (n <= 8) {  // few entries per q: a lane per q
    r = IntT::identity(opQ);
    op = opQ;
    for (int q = (int)threadIdx.x; q < eQ; q += (int)blockDim.x) {
      IAcc a = IntT::identity(opM);
      for (int m = 0; m < n; ++m) add(a, p[(long long)q * n + m], m);
      outer_add(r, IntT::emit(a, opM), q, opQ, true);
    }
  } else {  // a wave per q
    r = IntT::identity(opQ);
    op = opQ;
    for (int q = w; q < eQ; q += nw) {
      IAcc a = span(p + (long long)q * n, lane, 64);
#pragma unroll
      for (int b = 0; b < 6; ++b) a = IntT::merge(a, iacc_shfl(a, b, lane), opM);
      outer_add(r, IntT::emit(a, opM), q, opQ, true);
    }
    if (lane != 0) r = IntT::identity(opQ);  // every lane holds the wave's carrier
  }
#pragma unroll
  for (int b = 0; b < 6; ++b) r = IntT::merge(r, iacc_shfl(r, b, lane), op);
  if (nw > 1) {
    if (lane == 0) slot[w] = r;
    __syncthreads();
    if (w != 0) return;
    for (int j = 1; j < nw; ++j) r = IntT::merge(r, slot[j], op);
  }
  if (lane == 0) {
    const long long v = IntT::emit(r, op);
    if (out64) reinterpret_cast<long long*>(out)[o] = v;
    else reinterpret_cast<int*>(out)[o] = (int)v;
  }
}

template <int OP, int K, class M, int U>
void rows_nw(const SegRoute& S, const int32_t* in, void* out, IAcc* ws, hipStream_t st) {
  if (S.waves == 1)
    hipLaunchKernelGGL((k_seg_run<OP, K, M, U>), dim3(S.grid), dim3(256), 0, st, in, out, ws, S);
  else if (S.waves == 4)
    hipLaunchKernelGGL((k_seg_rows<OP, K, M, 4, U>), dim3(S.units), dim3(256), 0, st, in, out, ws, S);
  else
    hipLaunchKernelGGL((k_seg_rows<OP, K, M, 8, U>), dim3(S.units), dim3(512), 0, st, in, out, ws, S);
}

template <int OP, class M>
void rows_op(const SegRoute& S, const int32_t* in, void* out, IAcc* ws, hipStream_t st) {
  switch (S.vecs) {
    case -1: rows_nw<OP, -1, M, 8>(S, in, out, ws, st); break;
    case -2: rows_nw<OP, -2, M, 8>(S, in, out, ws, st); break;
    case -3: rows_nw<OP, -3, M, 8>(S, in, out, ws, st); break;
    case 1: rows_nw<OP, 1, M, 4>(S, in, out, ws, st); break;
    case 2: rows_nw<OP, 2, M, 2>(S, in, out, ws, st); break;
    case 3: rows_nw<OP, 3, M, 1>(S, in, out, ws, st); break;
    default: rows_nw<OP, 4, M, 1>(S, in, out, ws, st); break;
  }
}

// The same for many outputs of few entries: a lane per output.
template <class In, bool PARTS>
__global__ void __launch_bounds__(256) k_seg_tail_lane(const In* __restrict__ ws, void* __restrict__ out, long long n_out,
                                                       int eQ, int n, int opQ, int opM, int out64) {
  const long long o = (long long)blockIdx.x * 256 + threadIdx.x;
  if (o >= n_out) return;
  const In* p = ws + o * eQ * n;
  IAcc r = IntT::identity(opQ);
  for (int q = 0; q < eQ; ++q) {
    IAcc a = IntT::identity(opM);
    for (int m = 0; m < n; ++m) {
      if constexpr (PARTS) a = IntT::merge(a, p[(long long)q * n + m], opM);
      else outer_add(a, (long long)p[(long long)q * n + m], m, opM, true);
    }
    if (opQ == HP_OP_NONE) r = a;
    else outer_add(r, IntT::emit(a, opM), q, opQ, true);
  }
  const long long v = IntT::emit(r, opQ == HP_OP_NONE ? opM : opQ);
  if (out64) reinterpret_cast<long long*>(out)[o] = v;
  else reinterpret_cast<int*>(out)[o] = (int)v;
}

template <class In, bool PARTS>
void tail(const SegRoute& S, int n, const In* ws, void* out, hipStream_t st) {
  const long long per = (long long)S.eQ * n;
  if (per <= 64 && S.n_out >= 4096) {
    hipLaunchKernelGGL((k_seg_tail_lane<In, PARTS>), dim3((unsigned)((S.n_out + 255) / 256)), dim3(256), 0, st, ws, out,
                       (long long)S.n_out, S.eQ, n, S.opQ, S.opM, S.out64);
    return;
  }
  const unsigned threads = per <= 64 ? 64 : per <= 1024 ? 256 : 1024;
  hipLaunchKernelGGL((k_seg_tail<In, PARTS>), dim3((unsigned)S.n_out), dim3(threads), 0, st, ws, out, S.eQ, n, S.opQ, S.opM,
                     S.out64);
}

}  // namespace

hp_status launch_segs(const SegRoute& S, const void* in, void* out, void* ws, hipStream_t st) {
  const int32_t* x = reinterpret_cast<const int32_t*>(in);
  if (S.kind == SEGS_LONG) {
    const hp_status s = launch_rows(S.rows, in, ws, reinterpret_cast<unsigned char*>(ws) + S.parts_off, st);
    if (s != HP_OK) return s;
    if (S.rows.op == HP_OP_SUM) tail<long long, false>(S, S.eM, reinterpret_cast<const long long*>(ws), out, st);
    else tail<int, false>(S, S.eM, reinterpret_cast<const int*>(ws), out, st);
  } else {
    IAcc* w = reinterpret_cast<IAcc*>(ws);
    switch (S.opL) {
      case HP_OP_MIN: rows_op<HP_OP_MIN, KeyM>(S, x, out, w, st); break;
      case HP_OP_MAX: rows_op<HP_OP_MAX, KeyM>(S, x, out, w, st); break;
      case HP_OP_ARGMIN: rows_op<HP_OP_ARGMIN, KeyM>(S, x, out, w, st); break;
      case HP_OP_ARGMAX: rows_op<HP_OP_ARGMAX, KeyM>(S, x, out, w, st); break;
      default:
        if (S.opM == HP_OP_ARGMIN || S.opM == HP_OP_ARGMAX) rows_op<HP_OP_SUM, PairM>(S, x, out, w, st);
        else rows_op<HP_OP_SUM, KeyM>(S, x, out, w, st);
        break;
    }
    if (S.tail) tail<IAcc, true>(S, (int)S.parts, w, out, st);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(HP_EDEVICE, "kernel launch failed: %s", hipGetErrorString(e));
  return HP_OK;
}

}  // namespace hp
