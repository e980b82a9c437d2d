// Int32 nests of two or three reducing segments (runs of levels with one operator),
// planned automatically.  The view is out[o] = Q over q of M over m of L over the
// contiguous row (o, q, m) of eL elements, eQ = 1 for two segments.  No level has to be
// a multiple of anything: rows start at any element and are loaded as 16-byte vectors
// at 4-byte alignment.
//   rows of at most four vectors per lane: k_seg_rows reduces rows and M together.  A
//     wave takes 64 / 2^lb rows a step, 2^lb lanes each; a row's value goes into its
//     lane group's carrier of M, and the groups, the waves and (in the tail) the parts
//     of one (o, q) meet once at the end.
//     With as many pairs as fill the chip a wave runs through one or several (k_seg_run),
//     some of them side by side when M is short.
//   longer rows: the row kernels reduce every row to one value first.
// k_seg_tail then reduces what is left: the parts of M, or its values, and Q, in parts of
// its own where a few outputs have a long outermost level.
//
// Measured, from 4096 to 8192 waves that walk their pairs to waves of some 4 KiB:
//   64 x 128 x 64 x 64 SUM, MAX, ARGMIN (128 MiB)      32.0 -> 26.8 us
//   61 x 125 x 67 x 59 SUM, MAX, ARGMIN                31.4 -> 27.8 us
//   65536 x 33 x 17 SUM, MAX (147 MB)                  37.2 -> 27.7 us
//   20000 x 30 x 200 SUM, MAX (480 MB)                 85.8 -> 67.9 us
//   30000 x 7 x 30 ARGMIN, SUM (25 MB; keys instead of (value, index) pairs)  19.7 -> 11.9 us
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

// The carrier of M: a sum, or one 64-bit key of which the least or the greatest counts.
// An ARG level's key is value << shift | index (complemented for ARGMAX, so that the
// lower index wins), the shift 32 for 32-bit children and the bits of an index for int64
// sums, which leave it room: a row and M together have at most 2^28 elements.
struct KeyM {
  typedef long long Acc;
  int op, shift;
  long long mask;
  bool arg, minlike;
  __device__ __forceinline__ KeyM(const SegRoute& S, bool wide)
      : op(S.opM), shift(wide ? 32 - __builtin_clz((unsigned)S.eM) : 32), mask((1ll << shift) - 1), arg(IntK::arg(S.opM)),
        minlike(IntK::minlike(S.opM)) {}
  __device__ __forceinline__ Acc identity() const { return IntK::identity(op); }
  __device__ __forceinline__ void add(Acc& a, long long x, int m, bool ok) const {
    if (op == HP_OP_SUM) {
      a = (long long)((unsigned long long)a + (unsigned long long)(ok ? x : 0));
      return;
    }
    long long k = x;
    if (arg) k = (long long)((unsigned long long)x << shift) | (minlike ? (long long)m : mask ^ m);
    if (minlike) a = ok && k < a ? k : a;
    else a = ok && k > a ? k : a;
  }
  // over the lane groups: bits lo .. hi - 1, the bits below lo hold one value
  __device__ __forceinline__ Acc lanes(Acc a, int lo, int hi, int lane) const {
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
    if (minlike) return key_minmax<true>(a, vm, vm, lane);
    return key_minmax<false>(a, vm, vm, lane);
  }
  // of a carrier with at least one row: the identity's bits would unpack to a value and
  // index that win against rows of the extreme value
  __device__ __forceinline__ IAcc pair(Acc a) const {
    if (!arg) return IAcc{a, 0, 0};
    return IAcc{a >> shift, (int)((minlike ? a : ~a) & mask), 0};
  }
};

// Rows are read through a buffer descriptor, so that a step that does not exist -- past
// the end of a pair, where a wave has fewer steps than loads -- costs no memory traffic:
// its offset lies beyond the buffer, and the load returns zeros.  (Repeating the last row
// instead is no cheaper than reading another one: 16 steps on waves that load 4 at a time,
// 2 of them repeats, took 48.9 us, without repeats 26.4.)
constexpr uint32_t kNoRow = 0x80000000u;  // pairs and runs hold fewer bytes
constexpr int kNt = 2;                    // nontemporal
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const int32_t* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(base), 0, (int)bytes, 0x00027000);  // raw dwords
}

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
  // The row at byte `off` of a buffer; kNoRow loads nothing.
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t buf, uint32_t off, i32x4* x) const {
    if constexpr (K == -1) {
      x[0].x = (int)__builtin_amdgcn_raw_buffer_load_b32(buf, off, 0, kNt);
    } else if constexpr (K == -2) {
      const auto v = __builtin_amdgcn_raw_buffer_load_b64(buf, off, 0, kNt);
      x[0].x = (int)v[0], x[0].y = (int)v[1];
    } else if constexpr (K == -3) {
      const auto v = __builtin_amdgcn_raw_buffer_load_b96(buf, off, 0, kNt);
      x[0].x = (int)v[0], x[0].y = (int)v[1], x[0].z = (int)v[2];
    } else {
#pragma unroll
      for (int k = 0; k < KK; ++k) x[k] = (i32x4)__builtin_amdgcn_raw_buffer_load_b128(buf, off + 4u * (uint32_t)at[k], 0, kNt);
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

// Steps u = 0 .. U - 1 of a round, kTogether at a time (their chains overlap); `next`
// loads the step U later into the freed registers (kMore: there is another round).
constexpr int kTogether = 4;
template <int OP, int K, int U, bool kMore, class Row, class Next, class Done>
__device__ __forceinline__ void seg_round(const Row& row, i32x4 (&x)[U][SegRow<OP, K>::KK], int lane, int count, Next next,
                                          Done done) {
  constexpr int N = U < kTogether ? U : kTogether;
#pragma unroll
  for (int u = 0; u < U; u += N) {
    if (kMore || u == 0 || u < count) {
      long long v[N];
#pragma unroll
      for (int j = 0; j < N; ++j) {
        v[j] = row.reduce(x[u + j], lane);
        if constexpr (kMore) next(x[u + j]);
      }
#pragma unroll
      for (int j = 0; j < N; ++j) done(v[j], u + j);
    }
  }
}

// One (o, q) pair and part per workgroup of NW waves.  K vectors per lane and row (-1
// to -3: rows of that many elements, a lane each), U steps in flight.
template <int OP, int K, int NW, int U>
__global__ void __launch_bounds__(NW* kWave)
    k_seg_rows(const int32_t* __restrict__ in, void* __restrict__ out, IAcc* __restrict__ ws, SegRoute S) {
  const int lane = (int)(threadIdx.x & 63);
  const int w = (int)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t unit = xcd_run(blockIdx.x, gridDim.x);  // pair * parts + part
  const uint32_t pair = unit / S.parts, part = unit - pair * S.parts;
  const int lb = S.lane_bits, eM = S.eM;
  const int g = lane >> lb, rows = 64 >> lb;
  const SegRow<OP, K> row(S, lane);
  const KeyM M(S, OP == HP_OP_SUM);
  const uint32_t block = (uint32_t)(eM * S.eL);
  const __amdgpu_buffer_rsrc_t buf = buffer_of(in + (long long)pair * block, 4u * block);
  // this wave's steps: part * per + w, then every NW-th
  const int s1 = ((int)part + 1) * S.per < S.steps ? ((int)part + 1) * S.per : S.steps;
  const int s0 = (int)part * S.per + w;
  const uint32_t step = 4u * (uint32_t)(rows * S.eL), lane_off = 4u * (uint32_t)(g * S.eL);
  int ls = s0;  // the step that is loaded next
  auto next = [&](i32x4* x) {
    row.load(buf, ls < s1 && ls * rows + g < eM ? (uint32_t)ls * step + lane_off : kNoRow, x);
    ls += NW;
  };
  long long acc = M.identity();
  i32x4 x[U][SegRow<OP, K>::KK];
#pragma unroll
  for (int u = 0; u < U; ++u) next(x[u]);
  int s = s0;
  auto done = [&](long long v, int u) {
    const int su = s + u * NW, m = su * rows + g;
    M.add(acc, v, m, m < eM && su < s1);
  };
  if constexpr (U == 1) {  // 4 KiB a step: the next one is loaded while this one is reduced, no more
    for (; s < s1; s += NW) {
      i32x4 y[SegRow<OP, K>::KK];
      next(y);
      done(row.reduce(x[0], lane), 0);
#pragma unroll
      for (int k = 0; k < SegRow<OP, K>::KK; ++k) x[0][k] = y[k];
    }
  } else {
    for (; s + U * NW < s1; s += U * NW) seg_round<OP, K, U, true>(row, x, lane, U, next, done);
    seg_round<OP, K, U, false>(row, x, lane, (s1 - s + NW - 1) / NW, next, done);
  }
  // the wave's lane groups, then its workgroup's waves (the last part of a pair may have
  // fewer steps than waves)
  acc = M.lanes(acc, lb, 6, lane);
  __shared__ IAcc slot[NW];
  if (lane == 0) slot[w] = s0 < s1 ? M.pair(acc) : IntT::identity(S.opM);
  __syncthreads();
  if (w != 0 || lane != 0) return;
  IAcc a = slot[0];
#pragma unroll
  for (int j = 1; j < NW; ++j) a = IntT::merge(a, slot[j], S.opM);
  seg_out(S, out, ws, unit, a);
}

// A run of (o, q) pairs per wave.  A step is 64 / 2^lb rows: of 2^pb pairs at once when
// M has no more rows than that leaves each, else of one pair, whose carrier is complete
// after S.steps steps.  The loads of U steps are in flight across pairs.
template <int OP, int K, int U>
__global__ void __launch_bounds__(256)
    k_seg_run(const int32_t* __restrict__ in, void* __restrict__ out, IAcc* __restrict__ ws, SegRoute S) {
  const int lane = (int)(threadIdx.x & 63);
  const int w = (int)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const long long wave = (long long)xcd_run(blockIdx.x, gridDim.x) * 4 + w;
  const int lb = S.lane_bits, pb = S.pair_bits, top = 6 - pb, eM = S.eM;
  const int pr = lane >> top, g = (lane & ((1 << top) - 1)) >> lb, rows = 1 << (top - lb);
  const bool lead = (lane & ((1 << top) - 1)) == 0;
  const long long pairs = S.n_out * S.eQ, groups = (pairs + (1 << pb) - 1) >> pb;
  const long long g0 = wave * S.run, g1 = g0 + S.run < groups ? g0 + S.run : groups;
  if (g0 >= g1) return;
  const SegRow<OP, K> row(S, lane);
  const KeyM M(S, OP == HP_OP_SUM);
  // the run's pairs; what lies beyond them is beyond the buffer
  const uint32_t block = (uint32_t)(eM * S.eL);
  const long long p0 = g0 << pb, p1 = g1 << pb < pairs ? g1 << pb : pairs;
  const __amdgpu_buffer_rsrc_t buf = buffer_of(in + p0 * block, 4u * (uint32_t)(p1 - p0) * block);
  const uint32_t hop = (4u * block) << pb, step = 4u * (uint32_t)(rows * S.eL);
  uint32_t at = 4u * ((uint32_t)pr * block + (uint32_t)(g * S.eL));  // this lane's row of the step that is loaded next
  int ls = 0, n = (int)(g1 - g0) * S.steps, left = n;
  auto next = [&](i32x4* x) {
    row.load(buf, left > 0 && ls * rows + g < eM ? at : kNoRow, x);
    --left;
    at += step;
    if (++ls == S.steps) {
      ls = 0;
      at += hop - (uint32_t)S.steps * step;
    }
  };
  i32x4 x[U][SegRow<OP, K>::KK];
#pragma unroll
  for (int u = 0; u < U; ++u) next(x[u]);
  long long acc = M.identity(), pair = p0 + pr;
  int cs = 0;
  auto done = [&](long long v, int) {
    const int m = cs * rows + g;
    M.add(acc, v, m, m < eM);
    if (++cs == S.steps) {  // the pair is complete: its lane groups meet
      acc = M.lanes(acc, lb, top, lane);
      if (lead && pair < p1) seg_out(S, out, ws, pair, M.pair(acc));
      acc = M.identity();
      cs = 0;
      pair += 1ll << pb;
    }
  };
  for (; n > U; n -= U) seg_round<OP, K, U, true>(row, x, lane, U, next, done);
  seg_round<OP, K, U, false>(row, x, lane, n, next, done);
}

// Part `part` of output o on one workgroup: for every q, the n entries (o, q, m) --
// carriers of M (PARTS: the parts of its rows) or its child values -- then Q over q.  A
// wave takes every NW-th q, a lane one of few entries, or all waves share one where there
// is no Q.  One of several parts takes `per` iterations of Q (without Q, entries) and
// leaves its carrier for a second pass over the parts; without that, a few outputs of a
// long outermost level are a few workgroups' serial work: 1 x 1048576 x 4 x 8 SUM, MAX,
// SUM took 570 us, where the input is read in 25.
template <class In, bool PARTS, bool SPLIT>
__global__ void __launch_bounds__(1024) k_seg_tail(const In* __restrict__ ws, void* __restrict__ out, int eQ, int n, int opQ,
                                                   int opM, int out64, uint32_t parts, int per,
                                                   IAcc* __restrict__ carriers) {
  const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6), nw = (int)(blockDim.x >> 6);
  const uint32_t o = SPLIT ? blockIdx.x / parts : blockIdx.x;
  const int i0 = SPLIT ? (int)(blockIdx.x - o * parts) * per : 0;  // its first iteration of Q, or entry
  const In* p = ws + (long long)o * eQ * n;
  __shared__ IAcc slot[16];
  auto add = [&](IAcc& a, In x, int m) {
    if constexpr (PARTS) a = IntT::merge(a, x, opM);
    else outer_add(a, (long long)x, m, opM, true);
  };
  constexpr int U = 4;
  auto span = [&](const In* r, int first, int stride, int end) {  // this lane's entries of one q
    IAcc a = IntT::identity(opM);
    for (int m0 = first; m0 < end; m0 += U * stride) {
      In x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = r[m0 + u * stride < end ? m0 + u * stride : m0];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (m0 + u * stride < end) add(a, x[u], m0 + u * stride);
    }
    return a;
  };
  const int all = opQ == HP_OP_NONE ? n : eQ;
  const int i1 = SPLIT && i0 + per < all ? i0 + per : all;
  IAcc r;
  int op;
  if (opQ == HP_OP_NONE) {  // M alone: the whole workgroup on its entries
    r = span(p, i0 + (int)threadIdx.x, (int)blockDim.x, i1);
    op = opM;
  } else if (n <= kTailLane) {  // few entries per q: a lane per q
    r = IntT::identity(opQ);
    op = opQ;
    for (int q = i0 + (int)threadIdx.x; q < i1; q += (int)blockDim.x) {
      IAcc a = IntT::identity(opM);
      for (int m = 0; m < n; ++m) add(a, p[(long long)q * n + m], m);
      outer_add(r, IntT::emit(a, opM), q, opQ, true);
    }
  } else {  // a wave per q
    r = IntT::identity(opQ);
    op = opQ;
    for (int q = i0 + w; q < i1; q += nw) {
      IAcc a = span(p + (long long)q * n, lane, 64, n);
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
    if constexpr (SPLIT) {
      carriers[blockIdx.x] = r;
      return;
    }
    const long long v = IntT::emit(r, op);
    if (out64) reinterpret_cast<long long*>(out)[o] = v;
    else reinterpret_cast<int*>(out)[o] = (int)v;
  }
}

// Steps in flight: 8 KiB of a wave's input.
template <int OP, int K>
void rows_nw(const SegRoute& S, const int32_t* in, void* out, IAcc* ws, hipStream_t st) {
  constexpr int U = K < 0 ? 8 : K == 1 ? 4 : 2, UR = K <= 2 ? U : 1;
  if (S.waves == 1)
    hipLaunchKernelGGL((k_seg_run<OP, K, U>), dim3(S.grid), dim3(256), 0, st, in, out, ws, S);
  else if (S.waves == 4)
    hipLaunchKernelGGL((k_seg_rows<OP, K, 4, UR>), dim3(S.units), dim3(256), 0, st, in, out, ws, S);
  else
    hipLaunchKernelGGL((k_seg_rows<OP, K, 8, UR>), dim3(S.units), dim3(512), 0, st, in, out, ws, S);
}

template <int OP>
void rows_op(const SegRoute& S, const int32_t* in, void* out, IAcc* ws, hipStream_t st) {
  switch (S.vecs) {
    case -1: rows_nw<OP, -1>(S, in, out, ws, st); break;
    case -2: rows_nw<OP, -2>(S, in, out, ws, st); break;
    case -3: rows_nw<OP, -3>(S, in, out, ws, st); break;
    case 1: rows_nw<OP, 1>(S, in, out, ws, st); break;
    case 2: rows_nw<OP, 2>(S, in, out, ws, st); break;
    case 3: rows_nw<OP, 3>(S, in, out, ws, st); break;
    default: rows_nw<OP, 4>(S, in, out, ws, st); break;
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
void tail(const SegRoute& S, int n, const In* ws, void* out, unsigned char* base, hipStream_t st) {
  const long long per = (long long)S.eQ * n;
  // A lane walks its output's entries one after the other, so that takes as long for a few
  // outputs as for many: 4096 x 21 x 1 x 4 MAX, ARGMAX, ARGMIN 17.1 us, 11.0 by the plan's
  // kernels, 8.9 with a workgroup per output (18123 x 9 x 8 x 2: 14.2 us by lanes, 17.0 so).
  if (per <= 64 && S.n_out >= 4096 && (per <= 8 || per * 1400 <= S.n_out)) {
    hipLaunchKernelGGL((k_seg_tail_lane<In, PARTS>), dim3((unsigned)((S.n_out + 255) / 256)), dim3(256), 0, st, ws, out,
                       (long long)S.n_out, S.eQ, n, S.opQ, S.opM, S.out64);
    return;
  }
  unsigned threads = per <= 64 ? 64 : per <= 1024 ? 256 : kTailThreads;
  if (S.opQ != HP_OP_NONE && n > kTailLane) {  // a wave per iteration of Q
    const int q = S.tail_parts > 1 ? S.tail_per : S.eQ;
    threads = q < kTailThreads / kWave ? (unsigned)(q * kWave) : kTailThreads;
  }
  if (S.tail_parts == 1) {
    hipLaunchKernelGGL((k_seg_tail<In, PARTS, false>), dim3((unsigned)S.n_out), dim3(threads), 0, st, ws, out, S.eQ, n, S.opQ,
                       S.opM, S.out64, 1u, 0, (IAcc*)nullptr);
    return;
  }
  IAcc* carriers = reinterpret_cast<IAcc*>(base + S.tail_off);
  hipLaunchKernelGGL((k_seg_tail<In, PARTS, true>), dim3((unsigned)S.n_out * S.tail_parts), dim3(threads), 0, st, ws, out,
                     S.eQ, n, S.opQ, S.opM, S.out64, S.tail_parts, S.tail_per, carriers);
  const unsigned last = S.tail_parts <= 64 ? 64 : S.tail_parts <= 256 ? 256 : kTailThreads;
  hipLaunchKernelGGL((k_seg_tail<IAcc, true, false>), dim3((unsigned)S.n_out), dim3(last), 0, st, carriers, out, 1,
                     (int)S.tail_parts, (int)HP_OP_NONE, S.opQ == HP_OP_NONE ? S.opM : S.opQ, S.out64, 1u, 0, (IAcc*)nullptr);
}

}  // namespace

hp_status launch_segs(const SegRoute& S, const void* in, void* out, void* ws, hipStream_t st) {
  const int32_t* x = reinterpret_cast<const int32_t*>(in);
  unsigned char* base = reinterpret_cast<unsigned char*>(ws);
  if (S.kind == SEGS_LONG) {
    const hp_status s = launch_rows(S.rows, in, ws, base + S.parts_off, st);
    if (s != HP_OK) return s;
    if (S.rows.op == HP_OP_SUM) tail<long long, false>(S, S.eM, reinterpret_cast<const long long*>(ws), out, base, st);
    else tail<int, false>(S, S.eM, reinterpret_cast<const int*>(ws), out, base, st);
  } else {
    IAcc* w = reinterpret_cast<IAcc*>(ws);
    switch (S.opL) {
      case HP_OP_MIN: rows_op<HP_OP_MIN>(S, x, out, w, st); break;
      case HP_OP_MAX: rows_op<HP_OP_MAX>(S, x, out, w, st); break;
      case HP_OP_ARGMIN: rows_op<HP_OP_ARGMIN>(S, x, out, w, st); break;
      case HP_OP_ARGMAX: rows_op<HP_OP_ARGMAX>(S, x, out, w, st); break;
      default: rows_op<HP_OP_SUM>(S, x, out, w, st); break;
    }
    if (S.tail) tail<IAcc, true>(S, (int)S.parts, w, out, base, st);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(HP_EDEVICE, "kernel launch failed: %s", hipGetErrorString(e));
  return HP_OK;
}

}  // namespace hp
