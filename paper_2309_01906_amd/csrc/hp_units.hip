// Unit tasks: pieces of batched nests, one wavefront each (hp_units.h).
//
// A batch of uneven nests is bound by how long a wave takes from its task to its first
// data and by the longest task, not by arithmetic.  So a task is at most some tens of
// KiB of any nest's input, the kernels hold no general path (6 or 7 waves per SIMD where
// the plan kernels' persistent form has 4), every row is read as vectors at any
// alignment, and the workgroups are dealt by the dispatcher, largest tasks first (the
// persistent form's queue counters cost each wave an atomic per task).
//
// Measured, against the same batches as tasks of their plans on persistent workers:
//   10,000 uneven bf16 nests of one SUM, 415 MiB, from a graph   126 -> 79 us (5.5 TB/s)
//   1,000 of them                                         34.1 -> 14 us
//   1,500 mixed int32, float and bf16 nests of 1 to 3 segments  2026 -> 159 us
//     (the plan tasks of nested int32 reductions run the general kernel)
//   a batch of one small nest                              9.2 -> 3.4 us
//
// Rows of kLong vectors per lane and more are streamed one after the other, kLong of a
// row's vectors at a time; shorter rows kRows at a time (alone, the end of a row is a
// chain of some 800 cycles); rows below a vector a lane each.  The operators of int32 nests are
// run-time values: MAX and ARGMAX work on complemented values, so that a carrier is a sum
// or a minimum of 64-bit keys, and the kernel stays within the instruction cache (one
// body per operator took 235 KiB and was the slower the more operators a batch mixed).
#include "hp_units_dev.h"

#include "hp_fold.h"
#include "hp_red.h"

namespace hp {

namespace {

constexpr int kLong = 4;  // vectors of a long row in flight (with 8 the 10,000 bf16 nests take 82 us, not 79)
constexpr int kRows = 4;  // short rows taken together: their butterflies overlap

__device__ __forceinline__ bool op_max(int op) { return op == HP_OP_MAX || op == HP_OP_ARGMAX; }
__device__ __forceinline__ bool op_arg(int op) { return op == HP_OP_ARGMIN || op == HP_OP_ARGMAX; }

// The reduction of a row.  ints: SUM the int64 sum, MIN / MAX the (complemented) value,
// ARG (complemented) value << 32 | index; every merge but SUM's is a signed minimum.
template <class Raw>
struct Row {
  typedef double Acc;
  __device__ __forceinline__ Row(int) {}
  __device__ __forceinline__ Acc identity() const { return 0.0; }
  __device__ __forceinline__ void vec(Acc& a, typename Vec<Raw>::A x, uint32_t) const { Red<Raw, HP_OP_SUM>::vec(a, x, 0u); }
  __device__ __forceinline__ void last(Acc& a, typename Vec<Raw>::A x, uint32_t, u32x4 keep) const {
    Red<Raw, HP_OP_SUM>::vec(a, kept<Raw>(x, keep), 0u);
  }
  __device__ __forceinline__ void one(Acc& a, Raw x, uint32_t) const { Red<Raw, HP_OP_SUM>::one(a, x, 0u); }
  __device__ __forceinline__ Acc lanes(Acc a, int lb, int lane) const { return Red<Raw, HP_OP_SUM>::lanes(a, lb, lane); }
};
__device__ __forceinline__ long long key_min(long long a, long long b) { return b < a ? b : a; }
template <>
struct Row<int32_t> {
  typedef long long Acc;
  int op;
  bool sum, arg;
  int flip;  // -1 for MAX and ARGMAX
  __device__ __forceinline__ Row(int op_) : op(op_), sum(op_ == HP_OP_SUM), arg(op_arg(op_)), flip(op_max(op_) ? -1 : 0) {}
  __device__ __forceinline__ Acc identity() const { return sum ? 0 : 0x7FFFFFFFFFFFFFFFll; }
  __device__ __forceinline__ void vec(Acc& a, i32x4 x, uint32_t t) const {
    if (sum) {
      a = (long long)((unsigned long long)a + (unsigned long long)((long long)x.x + x.y) +
                      (unsigned long long)((long long)x.z + x.w));
    } else {
      const i32x4 y = x ^ flip;
      const int m = min(min(y.x, y.y), min(y.z, y.w));
      long long k = m;
      if (arg) {
        const uint32_t p = y.x == m ? 0u : y.y == m ? 1u : y.z == m ? 2u : 3u;
        k = (long long)((unsigned long long)(uint32_t)m << 32 | (t + p));
      }
      a = key_min(a, k);
    }
  }
  __device__ __forceinline__ void last(Acc& a, i32x4 x, uint32_t t, u32x4 keep) const {
    vec(a, sum ? kept<int32_t>(x, keep) : x, t);
  }
  __device__ __forceinline__ void one(Acc& a, int x, uint32_t t) const {
    if (sum) a = (long long)((unsigned long long)a + (unsigned long long)(long long)x);
    else if (arg) a = key_min(a, (long long)((unsigned long long)(uint32_t)(x ^ flip) << 32 | t));
    else a = key_min(a, x ^ flip);
  }
  __device__ __forceinline__ Acc lanes(Acc a, int lb, int lane) const {
    if (lb == 0) return a;
    if (sum) return Red<int32_t, HP_OP_SUM>::lanes(a, lb, lane);
    const uint32_t m = (1u << lb) - 1u;
    if (!arg) return word_allreduce<true, int>((int)min(a, 0x7FFFFFFFll), m, m, lane);
    return key_minmax<true>(a, m, m, lane);
  }
  __device__ __forceinline__ long long child(Acc a) const {  // what the enclosing level sees
    return sum ? a : arg ? (long long)(uint32_t)a : a ^ (long long)flip;
  }
  __device__ __forceinline__ IAcc carrier(Acc a) const {  // IntT's (value, index)
    if (!arg) return IAcc{child(a), 0, 0};
    return IAcc{(long long)((int)(uint32_t)((unsigned long long)a >> 32) ^ flip), (int)(uint32_t)a, 0};
  }
};

// The carrier of the middle segment M over rows: the same keys, or for an ARG over int64
// sums (kWide) a (value, index) pair.
template <bool kWide>
struct Mid {
  typedef long long Acc;
  int op;
  bool sum, arg;
  long long flip;
  __device__ __forceinline__ Mid(int op_) : op(op_), sum(op_ == HP_OP_SUM), arg(op_arg(op_)), flip(op_max(op_) ? -1 : 0) {}
  __device__ __forceinline__ Acc identity() const { return sum ? 0 : 0x7FFFFFFFFFFFFFFFll; }
  __device__ __forceinline__ void add(Acc& a, long long x, int m, bool ok) const {
    if (sum) {
      a = (long long)((unsigned long long)a + (unsigned long long)(ok ? x : 0));
    } else {
      long long k = x ^ flip;
      if (arg) k = (long long)((unsigned long long)(uint32_t)k << 32 | (uint32_t)m);
      a = key_min(a, ok ? k : 0x7FFFFFFFFFFFFFFFll);
    }
  }
  // over lane bits lo .. hi - 1 (the bits below lo hold one value)
  __device__ __forceinline__ Acc lanes(Acc a, int lo, int hi, int lane) const {
    const uint32_t vm = (1u << hi) - (1u << lo);
    if (!vm) return a;
    if (!sum) return key_minmax<true>(a, vm, vm, lane);
    if (vm & 1u) a = key_sum_step<0>(a, true, lane);
    if (vm & 2u) a = key_sum_step<1>(a, true, lane);
    if (vm & 4u) a = key_sum_step<2>(a, true, lane);
    if (vm & 8u) a = key_sum_step<3>(a, true, lane);
    if (vm & 16u) a = key_sum_step<4>(a, true, lane);
    if (vm & 32u) a = key_sum_step<5>(a, true, lane);
    return a;
  }
  __device__ __forceinline__ IAcc carrier(Acc a) const {
    if (!arg) return IAcc{a ^ flip, 0, 0};
    return IAcc{(long long)((int)(uint32_t)((unsigned long long)a >> 32) ^ (int)flip), (int)(uint32_t)a, 0};
  }
};
template <>
struct Mid<true> {
  typedef IAcc Acc;
  int op;
  __device__ __forceinline__ Mid(int op_) : op(op_) {}
  __device__ __forceinline__ Acc identity() const { return IntT::identity(op); }
  __device__ __forceinline__ void add(Acc& a, long long x, int m, bool ok) const {
    a = IntT::merge(a, ok ? IAcc{x, m, 0} : IntT::identity(op), op);
  }
  __device__ __forceinline__ Acc lanes(Acc a, int lo, int hi, int lane) const {
    for (int b = lo; b < hi; ++b) a = IntT::merge(a, IntT::shfl(a, 1 << b, lane), op);
    return a;
  }
  __device__ __forceinline__ IAcc carrier(Acc a) const { return a; }
};

// Row::lanes of kRows carriers at once, step by step
template <class Raw>
__device__ __forceinline__ void rows_lanes(const Row<Raw>& R, typename Row<Raw>::Acc (&a)[kRows], int lb, int lane) {
  auto steps = [&](auto step) {
    if (lb > 0) step(std::integral_constant<int, 0>{});
    if (lb > 1) step(std::integral_constant<int, 1>{});
    if (lb > 2) step(std::integral_constant<int, 2>{});
    if (lb > 3) step(std::integral_constant<int, 3>{});
    if (lb > 4) step(std::integral_constant<int, 4>{});
    if (lb > 5) step(std::integral_constant<int, 5>{});
  };
  if constexpr (!std::is_same<Raw, int32_t>::value) {
    steps([&](auto b) {
#pragma unroll
      for (int u = 0; u < kRows; ++u) a[u] = lane_step<decltype(b)::value>(a[u], true, lane);
    });
  } else if (R.sum) {
    steps([&](auto b) {
#pragma unroll
      for (int u = 0; u < kRows; ++u) a[u] = key_sum_step<decltype(b)::value>(a[u], true, lane);
    });
  } else if (!R.arg) {
    int v[kRows];
#pragma unroll
    for (int u = 0; u < kRows; ++u) v[u] = (int)min(a[u], 0x7FFFFFFFll);
    steps([&](auto b) {
#pragma unroll
      for (int u = 0; u < kRows; ++u) v[u] = word_step<decltype(b)::value, true, int>(v[u], true, lane);
    });
#pragma unroll
    for (int u = 0; u < kRows; ++u) a[u] = v[u];
  } else if (lb > 0) {  // the extreme high words, then the least low word among their lanes
    int h[kRows];
    uint32_t w[kRows];
#pragma unroll
    for (int u = 0; u < kRows; ++u) h[u] = (int)(uint32_t)((unsigned long long)a[u] >> 32);
    steps([&](auto b) {
#pragma unroll
      for (int u = 0; u < kRows; ++u) h[u] = word_step<decltype(b)::value, true, int>(h[u], true, lane);
    });
#pragma unroll
    for (int u = 0; u < kRows; ++u)
      w[u] = (int)(uint32_t)((unsigned long long)a[u] >> 32) == h[u] ? (uint32_t)a[u] : 0xFFFFFFFFu;
    steps([&](auto b) {
#pragma unroll
      for (int u = 0; u < kRows; ++u) w[u] = word_step<decltype(b)::value, true, uint32_t>(w[u], true, lane);
    });
#pragma unroll
    for (int u = 0; u < kRows; ++u) a[u] = (long long)((unsigned long long)(uint32_t)h[u] << 32 | w[u]);
  }
}

__device__ __forceinline__ void out_int(const UnitDesc& D, long long o, long long v) {
  if (D.out_kind == UNIT_I64) reinterpret_cast<long long*>(D.out)[o] = v;
  else reinterpret_cast<int*>(D.out)[o] = (int)v;
}

template <class Raw, bool kWide>
__device__ __forceinline__ void unit_task(const UnitDesc& D, uint32_t unit, int lane) {
  constexpr bool kFlt = !std::is_same<Raw, int32_t>::value;
  typedef typename Vec<Raw>::A V;
  typedef const __attribute__((address_space(1))) typename Vec<Raw>::E GV;
  typedef const __attribute__((address_space(1))) Raw G1;
  constexpr int N = Vec<Raw>::N;
  const Row<Raw> R(D.opL);
  const Mid<kWide> M(D.opM);
  typedef typename Row<Raw>::Acc Acc;
  const int eL = D.eL, eM = D.eM, lb = D.lane_bits, K = D.vecs, steps = D.steps;
  const Raw* in = reinterpret_cast<const Raw*>(D.in);
  // one vector of a row at element offset t, the last one moved back to end with the row
  auto vector = [&](const Raw* row, uint32_t t) -> V { return __builtin_nontemporal_load((GV*)(row + t)); };
  // groups [g0, g1) of pairs, steps [s0, s1) of each
  const long long pairs = D.pairs;
  const int pb = D.pair_bits;
  const bool cut = D.lparts > 1;  // a part of one row
  long long g0 = 0, g1 = 1;
  int s0 = 0, s1 = steps;
  if (D.mparts > 1) {
    g0 = unit / (uint32_t)D.mparts;
    s0 = (int)(unit - (uint32_t)g0 * (uint32_t)D.mparts) * D.per;
    s1 = min(s0 + D.per, steps);
    g1 = g0 + 1;
  } else if (!cut) {
    const long long groups = (pairs + (1 << pb) - 1) >> pb;
    g0 = (long long)unit * D.run;
    g1 = g0 + D.run < groups ? g0 + D.run : groups;
  }
  const int top = 6 - pb;
  const int pr = lane >> top, g = (lane & ((1 << top) - 1)) >> lb, rows = 1 << (top - lb);
  const bool lead = (lane & ((1 << top) - 1)) == 0;
  const long long block = (long long)eL * eM;  // elements of a pair, below 2^28
  // where a row's value goes
  long long cg = g0;
  int cs = s0;
  typename Mid<kWide>::Acc acc = M.identity();
  auto row_done = [&](Acc a) {  // every lane of the row holds its value
    const long long pair = (cg << pb) + pr;
    if constexpr (kFlt) {
      if (lead && pair < pairs) Red<Raw, HP_OP_SUM>::store(D.out, pair, a, D.out_kind == UNIT_F32);
      ++cg;
    } else {
      if (D.direct) {
        if (lead && pair < pairs) out_int(D, pair, R.child(a));
        ++cg;
        return;
      }
      const int m = cs * rows + g;
      M.add(acc, R.child(a), m, m < eM);
      if (++cs < s1) return;
      acc = M.lanes(acc, lb, top, lane);
      if (lead && pair < pairs) {
        const IAcc v = M.carrier(acc);
        if (D.partial) reinterpret_cast<IAcc*>(D.ws)[D.mparts > 1 ? (long long)unit : pair] = v;
        else out_int(D, pair, IntT::emit(v, D.opM));
      }
      acc = M.identity();
      cs = s0;
      ++cg;
    }
  };
  if ((K >= kLong && lb == 6) || cut) {  // one row, or part of a row, at a time on the 64 lanes
    const Raw* row = in + g0 * block + (long long)s0 * eL;
    int len = eL, t0 = 0;
    long long n = (g1 - g0) * (s1 - s0);
    if (cut) {
      const uint32_t r = unit / (uint32_t)D.lparts;
      t0 = (int)(unit - r * (uint32_t)D.lparts) * D.part_len;
      len = min(D.part_len, eL - t0);
      row = in + (long long)r * eL + t0;
      n = 1;
    }
    const int full = (len - 1) / (64 * N);  // whole passes before the last
    const uint32_t lt = (uint32_t)(full * 64 * N + lane * N), at = min(lt, (uint32_t)(len - N));
    const u32x4 keep = keep_from<Raw>((int)(lt - at));
#pragma unroll 1
    for (long long j = 0; j < n; ++j, row += eL) {
      const V xl = vector(row, at);
      Acc a = R.identity();
      if (full > 0) {
        // no load sits in a branch (the compiler would wait for all of them): the passes
        // of a batch past the row's end read its first vector, all lanes the same one
        // (repeating the last pass costs as much traffic as another one)
        auto pass_t = [&](int i) { return i < full ? (uint32_t)(i * 64 * N + lane * N) : 0u; };
        V x[kLong];
#pragma unroll
        for (int u = 0; u < kLong; ++u) x[u] = vector(row, pass_t(u));
        int i = kLong;
#pragma unroll 1
        for (; i < full; i += kLong) {
#pragma unroll
          for (int u = 0; u < kLong; ++u) {
            R.vec(a, x[u], (uint32_t)t0 + pass_t(i - kLong + u));
            x[u] = vector(row, pass_t(i + u));
          }
        }
#pragma unroll
        for (int u = 0; u < kLong; ++u)
          if (i - kLong + u < full) R.vec(a, x[u], (uint32_t)t0 + pass_t(i - kLong + u));
      }
      R.last(a, xl, (uint32_t)t0 + at, keep);
      a = R.lanes(a, 6, lane);
      if (!cut) row_done(a);
      else if (lane == 0) {
        if constexpr (kFlt) reinterpret_cast<double*>(D.ws)[2 * (long long)unit] = a;
        else reinterpret_cast<IAcc*>(D.ws)[unit] = R.carrier(a);
      }
    }
    return;
  }
  // Short rows, kRows steps together.  Element offsets from the unit's first element in
  // 32 bits (the partition keeps a unit below 2^28 elements); a group's pairs that do not
  // exist read its first pair, rows beyond M its last, and the steps beyond the unit its
  // first vector, all lanes the same one.
  const uint32_t lane_off = (uint32_t)(g * eL), last_off = (uint32_t)((eM - 1) * eL), row_step = (uint32_t)(rows * eL);
  const Raw* base = in + (g0 << pb) * block;
  const uint32_t hop = (uint32_t)block << pb;
  const int n_groups = (int)(g1 - g0);
  int lg = 0, ls = s0;  // the step whose offset comes next
  constexpr uint32_t kNone = 0xFFFFFFFFu;
  auto next_row = [&]() -> uint32_t {
    if (lg >= n_groups) return kNone;
    const uint32_t po = ((g0 + lg) << pb) + pr < pairs ? (uint32_t)pr * (uint32_t)block : 0u;
    const uint32_t ro = (uint32_t)lg * hop + po + min((uint32_t)ls * row_step + lane_off, last_off);
    if (++ls == s1) {
      ls = s0;
      ++lg;
    }
    return ro;
  };
  const int n_rows = n_groups * (s1 - s0);
  auto in_row = [&](uint32_t ro, uint32_t t) { return ro == kNone ? 0u : ro + t; };
  auto rows_done = [&](const Acc(&a)[kRows], int i) {
    if constexpr (kFlt) {
#pragma unroll
      for (int u = 0; u < kRows; ++u)
        if (i + u < n_rows) row_done(a[u]);
    } else {  // one copy of the code that ends a pair
      static_assert(kRows == 4, "picks one of four");
      const int k = min(kRows, n_rows - i);
#pragma unroll 1
      for (int u = 0; u < k; ++u) row_done(u == 0 ? a[0] : u == 1 ? a[1] : u == 2 ? a[2] : a[3]);
    }
  };
  if (K == 0) {  // rows below a vector: a lane each
    constexpr int E = N - 1;
    Raw x[E];
    auto load = [&]() {
      G1* q = (G1*)(base + in_row(next_row(), 0u));
#pragma unroll
      for (int e = 0; e < E; ++e) x[e] = q[e < eL ? e : 0];
    };
    load();
#pragma unroll 1
    for (int i = 0; i < n_rows; i += kRows) {
      Acc a[kRows];
#pragma unroll
      for (int u = 0; u < kRows; ++u) {
        a[u] = R.identity();
#pragma unroll
        for (int e = 0; e < E; ++e)
          if (e < eL) R.one(a[u], x[e], (uint32_t)e);
        if (i + u + 1 < n_rows) load();
      }
      rows_done(a, i);
    }
    return;
  }
  const int l = lane & ((1 << lb) - 1);
  const uint32_t first_t = (uint32_t)(l * N), pass = (uint32_t)(N << lb), end_t = (uint32_t)(eL - N);
  const uint32_t last_t = (uint32_t)(K - 1) * pass + first_t, last_at = min(last_t, end_t);
  const u32x4 keep = keep_from<Raw>((int)(last_t - last_at));
  uint32_t ro[kRows];
  V x[kRows];
  auto first = [&]() {
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
      ro[u] = next_row();
      x[u] = vector(base, in_row(ro[u], min(first_t, end_t)));
    }
  };
  first();
#pragma unroll 1
  for (int i = 0; i < n_rows; i += kRows) {
    Acc a[kRows];
#pragma unroll
    for (int u = 0; u < kRows; ++u) a[u] = R.identity();
    uint32_t t = first_t;
#pragma unroll 1
    for (int k = 1; k < K; ++k, t += pass) {
#pragma unroll
      for (int u = 0; u < kRows; ++u) {
        R.vec(a[u], x[u], t);
        x[u] = vector(base, in_row(ro[u], min(t + pass, end_t)));
      }
    }
#pragma unroll
    for (int u = 0; u < kRows; ++u) R.last(a[u], x[u], last_at, keep);
    if (i + kRows < n_rows) first();
    rows_lanes<Raw>(R, a, lb, lane);
    rows_done(a, i);
  }
}

template <class Raw>
__device__ __forceinline__ void unit_any(const UnitDesc& D, uint32_t unit, int lane) {
  if constexpr (std::is_same<Raw, int32_t>::value) {
    if (!D.direct && D.lparts == 1 && D.opL == HP_OP_SUM && op_arg(D.opM)) {
      unit_task<Raw, true>(D, unit, lane);
      return;
    }
  }
  unit_task<Raw, false>(D, unit, lane);
}

// Descriptors and tasks are read through the constant address space: scalar loads.
typedef const __attribute__((address_space(4))) UnitDesc CDesc;
typedef const __attribute__((address_space(4))) int CInt;

// Waves per SIMD the bodies fit without spills.
template <class Raw>
constexpr int kUnitWaves = std::is_same<Raw, float>::value ? 7 : 6;

template <class Raw>
__global__ void __launch_bounds__(256, kUnitWaves<Raw>) k_units(const UnitDesc* descs, const int2* tasks, int n) {
  const int t = (int)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
  if (t >= n) return;
  CInt* e = (CInt*)tasks;
  const int nest = e[2 * (long long)t], unit = e[2 * (long long)t + 1];
  unit_any<Raw>(*(const UnitDesc*)((CDesc*)descs + nest), (uint32_t)unit, (int)(threadIdx.x & 63));
}

template <class Raw>
__global__ void __launch_bounds__(256, kUnitWaves<Raw>) k_units_of(const UnitDesc* desc, int first, int n) {
  const int t = first + (int)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
  if (t >= n) return;
  unit_any<Raw>(*(const UnitDesc*)((CDesc*)desc), (uint32_t)t, (int)(threadIdx.x & 63));
}

// The carriers of one output: for each q, `rows` groups of `parts` carriers of `op` (rows:
// the iterations of M when rows were split, else 1), by wave w of nw; the waves' carriers
// meet in `slot`, and one lane ends the output.
template <int nw>
__device__ __forceinline__ void fold_ints(const UnitDesc& D, long long o, int lane, int w, IAcc* slot) {
  const bool cut = D.lparts > 1;
  const int rows = cut ? D.eM : 1, parts = cut ? D.lparts : D.mparts;
  const int op = cut ? D.opL : D.opM, opM = D.opM, eQ = D.eQ, inner = cut ? opM : op;
  // split rows: the child of M is the row's value; M of a single reduction passes it on
  const IAcc* p = reinterpret_cast<const IAcc*>(D.ws) + o * eQ * (long long)rows * parts;
  constexpr int U = 4;
  auto merged = [&](const IAcc* r, int first, int stride) {
    IAcc a = IntT::identity(op);
    for (int k = first; k < parts; k += U * stride) {
      IAcc x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = r[k + u * stride < parts ? k + u * stride : k];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (k + u * stride < parts) a = IntT::merge(a, x[u], op);
    }
    return a;
  };
  auto child = [&](IAcc& m, IAcc v, int t) {  // a row's value into M
    IAcc c{IntT::emit(v, op), t, 0};
    m = IntT::merge(m, c, opM);
  };
  auto lanes = [&](IAcc a, int o_) {
#pragma unroll
    for (int b = 0; b < 6; ++b) a = IntT::merge(a, IntT::shfl(a, 1 << b, lane), o_);
    return a;
  };
  auto waves = [&](IAcc a, int o_) {  // a is the wave's, on every lane
    if constexpr (nw > 1) {
      if (lane == 0) slot[w] = a;
      __syncthreads();
      a = slot[0];
      for (int j = 1; j < nw; ++j) a = IntT::merge(a, slot[j], o_);
    }
    return a;
  };
  auto value = [&](IAcc m) {  // of one q
    return cut ? (D.direct ? m.v : IntT::emit(m, opM)) : IntT::emit(m, op);
  };
  // M over rows first, first + stride, ... of one q, on the wave's lanes or a row at a time
  auto rows_of = [&](const IAcc* r, int first, int stride) {
    IAcc m = IntT::identity(opM);
    if (D.fold_form == FOLD_LANE_ROW) {
      for (int a = first * 64 + lane; a < rows; a += stride * 64) child(m, merged(r + (long long)a * parts, 0, 1), a);
      m = lanes(m, opM);
    } else {
      for (int a = first; a < rows; a += stride) child(m, lanes(merged(r + (long long)a * parts, lane, 64), op), a);
    }
    return m;
  };
  long long v;
  if (D.opQ == HP_OP_NONE) {
    IAcc m;
    if (!cut) m = waves(lanes(merged(p, w * 64 + lane, nw * 64), op), op);
    else if (rows > 1) m = waves(rows_of(p, w, nw), opM);
    else child(m = IntT::identity(opM), waves(lanes(merged(p, w * 64 + lane, nw * 64), op), op), 0);
    v = value(m);
  } else {
    IAcc Q = IntT::identity(D.opQ);
    if (D.fold_form == FOLD_LANE_Q) {
      for (int q = w * 64 + lane; q < eQ; q += nw * 64) {
        IAcc m = IntT::identity(inner);
        for (int a = 0; a < rows; ++a) {
          const IAcc x = merged(p + ((long long)q * rows + a) * parts, 0, 1);
          if (cut) child(m, x, a);
          else m = x;
        }
        Q = IntT::merge(Q, IAcc{value(m), q, 0}, D.opQ);
      }
      Q = lanes(Q, D.opQ);
    } else {
      for (int q = w; q < eQ; q += nw) {
        const IAcc* r = p + (long long)q * rows * parts;
        const IAcc m = cut ? rows_of(r, 0, 1) : lanes(merged(r, lane, 64), op);
        Q = IntT::merge(Q, IAcc{value(m), q, 0}, D.opQ);
      }
    }
    v = IntT::emit(waves(Q, D.opQ), D.opQ);
  }
  if (lane == 0 && w == 0) out_int(D, o, v);
}

// Float partials, in an order that their number fixes.
template <int nw>
__device__ __forceinline__ void fold_floats(const UnitDesc& D, long long o, int lane, int w, DPair* slot) {
  const double* p = reinterpret_cast<const double*>(D.ws) + 2 * o * D.lparts;
  DPair a{0.0, 0.0};
  constexpr int U = 4;
  const int stride = nw * 64;
  for (int k = w * 64 + lane; k < D.lparts; k += U * stride) {
    double x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = k + u * stride < D.lparts ? p[2 * (k + u * stride)] : 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u) dpair_add(a, x[u]);
  }
#pragma unroll
  for (int b = 0; b < 6; ++b) a = dpair_merge(a, DPair{xor_move_d(a.s, 1 << b, lane), xor_move_d(a.c, 1 << b, lane)});
  if constexpr (nw > 1) {
    if (lane == 0) slot[w] = a;
    __syncthreads();
    a = slot[0];
    for (int j = 1; j < nw; ++j) a = dpair_merge(a, slot[j]);
  }
  const double v = float_result(a.s + a.c);
  if (lane != 0 || w != 0) return;
  if (D.out_kind == UNIT_F32) reinterpret_cast<float*>(D.out)[o] = (float)v;
  else reinterpret_cast<double*>(D.out)[o] = v;
}

// A fold task per wave (kShared: per workgroup, whose waves share it).  Tasks of a wave go
// four to a workgroup, to spread a few hundred of them over the chip.
template <bool kShared>
__global__ void __launch_bounds__(kShared ? 64 * kFoldWaves : 256) k_unit_folds(const UnitDesc* descs, const int2* tasks, int n) {
  constexpr int nw = kShared ? kFoldWaves : 1;
  __shared__ IAcc slot[nw];
  static_assert(sizeof(IAcc) == sizeof(DPair), "one slot for either");
  const int w = (int)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int t = kShared ? (int)blockIdx.x : (int)blockIdx.x * 4 + w;
  if (t >= n) return;
  CInt* e = (CInt*)tasks;
  const int nest = e[2 * (long long)t], o = e[2 * (long long)t + 1];
  const UnitDesc& D = *(const UnitDesc*)((CDesc*)descs + nest);
  const int lane = (int)(threadIdx.x & 63);
  if (D.out_kind <= UNIT_F32) fold_floats<nw>(D, o, lane, kShared ? w : 0, reinterpret_cast<DPair*>(slot));
  else fold_ints<nw>(D, o, lane, kShared ? w : 0, slot);
}

hp_status launched() {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(HP_EDEVICE, "unit kernel launch failed: %s", hipGetErrorString(e));
  return HP_OK;
}


// `go` for every launch of n tasks: its first task, its tasks and its workgroups.
template <class Go>
hp_status in_launches(int64_t n, int64_t tasks_per_group, int64_t threads_per_task, Go go) {
  const int64_t most = launch_tasks(threads_per_task);
  hp_status s = HP_OK;
  for (int64_t t = 0; t < n && s == HP_OK; t += most) {
    const int64_t k = n - t < most ? n - t : most;
    go((int)t, (int)k, dim3((unsigned)((k + tasks_per_group - 1) / tasks_per_group)));
    s = launched();
  }
  return s;
}

}  // namespace

hp_status launch_units(int dtype, const UnitDesc* descs, const int2* tasks, int n, hipStream_t st) {
  return in_launches(n, 4, 64, [&](int t, int k, dim3 grid) {
    const dim3 wg(256);
    if (dtype == HP_F32) hipLaunchKernelGGL(k_units<float>, grid, wg, 0, st, descs, tasks + t, k);
    else if (dtype == HP_BF16) hipLaunchKernelGGL(k_units<uint16_t>, grid, wg, 0, st, descs, tasks + t, k);
    else hipLaunchKernelGGL(k_units<int32_t>, grid, wg, 0, st, descs, tasks + t, k);
  });
}

hp_status launch_units_of(int dtype, const UnitDesc* desc, int n, hipStream_t st) {
  return in_launches(n, 4, 64, [&](int t, int k, dim3 grid) {
    const dim3 wg(256);
    if (dtype == HP_F32) hipLaunchKernelGGL(k_units_of<float>, grid, wg, 0, st, desc, t, t + k);
    else if (dtype == HP_BF16) hipLaunchKernelGGL(k_units_of<uint16_t>, grid, wg, 0, st, desc, t, t + k);
    else hipLaunchKernelGGL(k_units_of<int32_t>, grid, wg, 0, st, desc, t, t + k);
  });
}

hp_status warm_unit_kernels(hipStream_t st) {
  const dim3 one(1), wg(256);
  hipLaunchKernelGGL(k_units<float>, one, wg, 0, st, nullptr, nullptr, 0);
  hipLaunchKernelGGL(k_units<uint16_t>, one, wg, 0, st, nullptr, nullptr, 0);
  hipLaunchKernelGGL(k_units<int32_t>, one, wg, 0, st, nullptr, nullptr, 0);
  hipLaunchKernelGGL(k_unit_folds<false>, one, wg, 0, st, nullptr, nullptr, 0);
  hipLaunchKernelGGL(k_unit_folds<true>, one, dim3(64 * kFoldWaves), 0, st, nullptr, nullptr, 0);
  return launched();
}

hp_status launch_unit_folds(const UnitDesc* descs, const int2* tasks, int n_shared, int n, hipStream_t st) {
  hp_status s = in_launches(n_shared, 1, 64 * kFoldWaves, [&](int t, int k, dim3 grid) {
    hipLaunchKernelGGL(k_unit_folds<true>, grid, dim3(64 * kFoldWaves), 0, st, descs, tasks + t, k);
  });
  if (s != HP_OK) return s;
  return in_launches(n - n_shared, 4, 64, [&](int t, int k, dim3 grid) {
    hipLaunchKernelGGL(k_unit_folds<false>, grid, dim3(256), 0, st, descs, tasks + n_shared + t, k);
  });
}

}  // namespace hp
