// Ordered products: associative, non-commutative reductions of affine maps and
// 2x2 matrices modulo 2^64 (HP_OP_PROD).  The paper points out that OpenMP
// reductions must be commutative (section 2); here siblings are combined strictly
// in iteration order at every level of the hierarchy.  The reduced block of one
// output is contiguous (row-major input), so every level of a nested product
// collapses into one ordered product over the block.
//
// A wave reads its range of the block as tiles of 8 adjacent KiB: whole lines at any
// alignment of the block.  (Lanes that each walk a part of their own, a line at a time,
// fetch every line twice where the block does not start on one: 300 x 20,011 affine maps
// took 28.6 us in that form, half of it the second fetch.)  Through LDS lane l gets the
// l-th 128 bytes of a tile and multiplies them alone, without a shuffle; the lanes of a
// tile are neighbours, so their products cannot be gathered tile by tile lane by lane.
// Instead 2^B tiles are turned as they are multiplied: on lane bit b two partial results
// of 2^b tiles become one of 2^(b+1), the lanes with the bit clear keep the first tiles
// and the others the second, and each lane multiplies its own value with its
// neighbour's in order.  That leaves a lane per tile, and 6 multiplies more end the
// group: 37 for 4 tiles of maps, where a butterfly per tile takes 52.
//
// Maps are bound by memory, matrices by the multiplies (a 64-bit product is three
// quarter-rate instructions, a matrix product eight of them: some 30 us for 256 MB).
// Measured, before (a part of its own per lane) and as here:
//   affine 300 x 20,011 (96 MB)      32.2 -> 18.6 us     2x2  300 x 20,011 (192 MB)  59.4 -> 34.7 us
//   affine 40 x 400,000 (256 MB)     42.1 -> 41.4 us     2x2  40 x 200,000 (256 MB)  45.5 -> 45.4 us
//   affine 1 x 16,777,216 (268 MB)   53.9 -> 48.9 us     2x2  1 x 8,388,608          60.9 -> 51.5 us
//   affine 4,096 x 8,192 (537 MB)    82.9 -> 80.5 us     2x2  4,096 x 4,096          83.7 -> 84.8 us
//   affine 4,000 x 700               13.6 -> 10.1 us     2x2  2,000 x 500             8.8 ->  7.9 us
//   affine 1 x 4,096                 11.0 ->  4.5 us     affine 100,000 x 32         82.8 -> 15.1 us
// Direct loads with a matrix or more per lane (32 bytes apart and up) read half of every
// line twice: 40 x 200,000 takes 51 us at 32 bytes and 92 at 64.
#include <hip/hip_runtime.h>

#include "hp_internal.h"
#include "hp_nest.h"

namespace hp {

typedef unsigned long long u64;

template <int W>
struct Elem {
  u64 v[W];
};

// x * y, x first.  Affine (a, b): x -> a x + b; matrices row-major.
template <int W>
__device__ __forceinline__ Elem<W> mul(const Elem<W>& x, const Elem<W>& y) {
  Elem<W> r;
  if constexpr (W == 2) {
    r.v[0] = x.v[0] * y.v[0];
    r.v[1] = y.v[0] * x.v[1] + y.v[1];
  } else {
    r.v[0] = x.v[0] * y.v[0] + x.v[1] * y.v[2];
    r.v[1] = x.v[0] * y.v[1] + x.v[1] * y.v[3];
    r.v[2] = x.v[2] * y.v[0] + x.v[3] * y.v[2];
    r.v[3] = x.v[2] * y.v[1] + x.v[3] * y.v[3];
  }
  return r;
}

template <int W>
__device__ __forceinline__ Elem<W> unit() {
  Elem<W> r;
#pragma unroll
  for (int k = 0; k < W; ++k) r.v[k] = 0;
  r.v[0] = 1;
  if constexpr (W == 4) r.v[3] = 1;
  return r;
}

// one element from global memory (16-byte nontemporal loads)
template <int W>
__device__ __forceinline__ Elem<W> load_elem(const u64* p) {
  typedef u64 u64x2 __attribute__((ext_vector_type(2)));
  typedef const __attribute__((address_space(1))) u64x2 G2;
  Elem<W> r;
#pragma unroll
  for (int h = 0; h < W / 2; ++h) {
    const u64x2 q = __builtin_nontemporal_load((G2*)(p + 2 * h));
    r.v[2 * h] = q.x;
    r.v[2 * h + 1] = q.y;
  }
  return r;
}

// One of the two halves of a step on lane bit B, for one 32-bit word: lanes with the
// bit clear keep a and receive their upper neighbour's a, the others keep b and
// receive their lower neighbour's b; l and r are the neighbours' values in lane order.
template <int B>
__device__ __forceinline__ void turn32(uint32_t a, uint32_t b, uint32_t& l, uint32_t& r, int lane) {
  if constexpr (B == 5) {
    const auto s = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    l = s[0], r = s[1];
  } else if constexpr (B == 4) {
    const auto s = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    l = s[0], r = s[1];
  } else if constexpr (B >= 2) {  // whole banks of four lanes are written, the others keep the old value
    constexpr int kDown = B == 3 ? kDppRowShr8 : kDppRowShr4, kUp = B == 3 ? kDppRowShl8 : kDppRowShl4;
    constexpr int kHigh = B == 3 ? 0xC : 0xA;
    l = (uint32_t)__builtin_amdgcn_update_dpp((int)a, (int)b, kDown, 0xF, kHigh, false);
    r = (uint32_t)__builtin_amdgcn_update_dpp((int)b, (int)a, kUp, 0xF, 0xF ^ kHigh, false);
  } else {
    constexpr int kSwap = B == 0 ? kDppQuad1032 : kDppQuad2301;
    const bool high = (lane >> B) & 1;
    const uint32_t ta = (uint32_t)dpp<kSwap>((int)a), tb = (uint32_t)dpp<kSwap>((int)b);
    l = high ? tb : a;
    r = high ? b : ta;
  }
}

template <int W, int B>
__device__ __forceinline__ Elem<W> turn(const Elem<W>& a, const Elem<W>& b, int lane) {
  Elem<W> l, r;
#pragma unroll
  for (int k = 0; k < W; ++k) {
    uint32_t l0, l1, r0, r1;
    turn32<B>((uint32_t)a.v[k], (uint32_t)b.v[k], l0, r0, lane);
    turn32<B>((uint32_t)(a.v[k] >> 32), (uint32_t)(b.v[k] >> 32), l1, r1, lane);
    l.v[k] = (u64)l1 << 32 | l0;
    r.v[k] = (u64)r1 << 32 | r0;
  }
  return mul<W>(l, r);
}

// Lane bits [LO, HI) of one value: every lane gets the product over them, in lane order.
template <int W, int LO, int HI>
__device__ __forceinline__ Elem<W> lanes_product(Elem<W> x, int lane) {
  if constexpr (LO < HI) x = lanes_product<W, LO + 1, HI>(turn<W, LO>(x, x, lane), lane);
  return x;
}

// What lanes beyond the end of a range read: the identity.
__device__ __align__(16) const u64 kIdentity2[2] = {1, 0};
__device__ __align__(16) const u64 kIdentity4[4] = {1, 0, 0, 1};
template <int W>
__device__ __forceinline__ const u64* identity() {
  if constexpr (W == 2) return kIdentity2;
  else return kIdentity4;
}

// A wave's tiles of a range: 512 adjacent 16-byte words (512 affine maps, 256 matrices),
// read as 8 loads of 1 KiB and staged in the wave's LDS slice, from which lane l takes
// the l-th run of 8 words, 128 bytes, as its elements.  A run's words are permuted so
// that the 16 lanes that are served together hit distinct banks, on both ways.
typedef u64 u64x2 __attribute__((ext_vector_type(2)));
constexpr int kRunWords = 8, kSliceBytes = 64 * kRunWords * 16;
__device__ __forceinline__ int word_slot(int run, int k) { return (run * kRunWords + (k ^ ((run >> 1) & 7))) * 16; }

template <int W>
struct Tiles {
  const u64* base;
  char* slice;
  uint32_t len, at;  // words of the range; this lane's first word of the next tile to load
  u64x2 g[kRunWords];
  __device__ __forceinline__ void load(int lane) {
    typedef const __attribute__((address_space(1))) u64x2 G2;
    const u64* none = identity<W>() + (W == 4 ? 2 * (lane & 1) : 0);
#pragma unroll
    for (int q = 0; q < kRunWords; ++q, at += 64)
      g[q] = __builtin_nontemporal_load((G2*)(at < len ? base + 2 * (size_t)at : none));
  }
  // The product of the lane's run of the loaded tile, as a balanced tree over adjacent
  // pairs; the next tile, if one follows, is loaded meanwhile.
  template <bool kMore>
  __device__ __forceinline__ Elem<W> product(int lane) {
    constexpr int K = 2 * kRunWords / W;
#pragma unroll
    for (int q = 0; q < kRunWords; ++q)
      *reinterpret_cast<u64x2*>(slice + word_slot(q * (64 / kRunWords) + lane / kRunWords, lane % kRunWords)) = g[q];
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
    Elem<W> x[K];
#pragma unroll
    for (int q = 0; q < kRunWords; ++q) {
      const u64x2 v = *reinterpret_cast<const u64x2*>(slice + word_slot(lane, q));
      x[2 * q / W].v[2 * q % W] = v.x;
      x[2 * q / W].v[2 * q % W + 1] = v.y;
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();
    if constexpr (kMore) load(lane);
#pragma unroll
    for (int h = 1; h < K; h *= 2) {
#pragma unroll
      for (int j = 0; j + h < K; j += 2 * h) x[j] = mul<W>(x[j], x[j + h]);
    }
    return x[0];
  }
};

// 2^B tiles, turned on lane bits 0 .. B - 1; kMore: tiles follow.
template <int W, int B, bool kMore>
__device__ __forceinline__ Elem<W> tiles_tree(Tiles<W>& T, int lane) {
  if constexpr (B == 0) {
    return T.template product<kMore>(lane);
  } else {
    const Elem<W> a = tiles_tree<W, B - 1, true>(T, lane);
    const Elem<W> b = tiles_tree<W, B - 1, kMore>(T, lane);
    return turn<W, B - 1>(a, b, lane);
  }
}

// The product of `len` adjacent elements (at least one), on every lane of a wave, in
// groups of G elements; kLoop: there may be more than one.
template <int W, int G, bool kLoop>
__device__ __forceinline__ Elem<W> range_product(const u64* base, uint32_t len, char* slice, int lane) {
  constexpr int kTiles = G * W / 2 / (64 * kRunWords);
  constexpr int B = kTiles == 1 ? 0 : kTiles == 2 ? 1 : kTiles == 4 ? 2 : 3;
  static_assert(1 << B == kTiles, "whole tiles");
  Tiles<W> T;
  T.base = base;
  T.slice = slice;
  T.len = len * (W / 2);
  T.at = (uint32_t)lane;
  T.load(lane);
  auto group = [&]() {
    Elem<W> g = tiles_tree<W, B, kLoop>(T, lane);  // a lane per tile, of the lanes that bits B .. 5 part
    g = lanes_product<W, B, 6>(g, lane);
    return lanes_product<W, 0, B>(g, lane);
  };
  if constexpr (!kLoop) return group();
  Elem<W> acc = unit<W>();
#pragma unroll 1
  for (uint32_t t = 0; t < len; t += G) acc = mul<W>(acc, group());
  return acc;
}

template <int W>
__device__ __forceinline__ void store_elem(u64* p, const Elem<W>& e) {
#pragma unroll
  for (int k = 0; k < W; ++k) p[k] = e.v[k];
}

__device__ __forceinline__ long long wave_id() {
  return (long long)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}

// Waves of their own: unit u is chunk u % C of output u / C.  (One tile of maps and no
// loop fits five waves per SIMD.)
template <int W, int G, bool kLoop>
__global__ void __launch_bounds__(256, W == 2 && !kLoop ? 5 : 4) k_ordered(const u64* __restrict__ in, u64* __restrict__ dst,
                                                                 long long units, long long C, long long block,
                                                                 long long span) {
  __shared__ __align__(16) char slices[4 * kSliceBytes];
  const int lane = (int)(threadIdx.x & 63);
  char* slice = slices + (threadIdx.x >> 6) * kSliceBytes;
  for (long long u = wave_id(); u < units; u += (long long)gridDim.x * 4) {
    const long long o = C == 1 ? u : ((u | C) >> 32) == 0 ? (long long)((uint32_t)u / (uint32_t)C) : u / C;
    const long long lo = (u - o * C) * span;
    const long long len = lo + span < block ? span : block - lo;
    const Elem<W> e = range_product<W, G, kLoop>(in + (size_t)(o * block + lo) * W, (uint32_t)len, slice, lane);
    if (lane == 0) store_elem<W>(dst + (size_t)u * W, e);
  }
}

// A workgroup per output, for short blocks and the products of chunks: `run` adjacent
// elements per lane, then the lanes, then the waves.  What counts here is the chain of
// multiplies, not the access: 98 products of 40 outputs take 5.2 us from tiles.
constexpr int kJoinWaves = 16, kJoinRun = 8;
template <int W>
__global__ void __launch_bounds__(64 * kJoinWaves) k_ordered_join(const u64* __restrict__ in, u64* __restrict__ out,
                                                                  long long n_out, int block, int run) {
  __shared__ u64 parts[kJoinWaves * W];
  const int lane = (int)(threadIdx.x & 63), w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  for (long long o = blockIdx.x; o < n_out; o += gridDim.x) {
    const u64* base = in + (size_t)(o * block) * W;
    const int e0 = (int)threadIdx.x * run;
    Elem<W> acc = unit<W>();
    if (w * 64 * run < block) {
      Elem<W> x[kJoinRun];
#pragma unroll
      for (int j = 0; j < kJoinRun; ++j)
        if (j < run) x[j] = load_elem<W>(e0 + j < block ? base + (size_t)(e0 + j) * W : identity<W>());
      acc = x[0];
#pragma unroll
      for (int j = 1; j < kJoinRun; ++j)
        if (j < run) acc = mul<W>(acc, x[j]);
      acc = lanes_product<W, 0, 6>(acc, lane);
    }
    if (lane == 0) store_elem<W>(parts + w * W, acc);
    __syncthreads();
    if (w == 0) {
      Elem<W> x;
#pragma unroll
      for (int k = 0; k < W; ++k) x.v[k] = parts[(lane & (kJoinWaves - 1)) * W + k];
      x = lanes_product<W, 0, 4>(x, lane);
      if (lane == 0) store_elem<W>(out + (size_t)o * W, x);
    }
    __syncthreads();
  }
}

// Blocks of at most 64 elements: 2^lb lanes per output, outputs side by side in a
// row, kRows rows together.
template <int W, int kRows>
__global__ void __launch_bounds__(256) k_ordered_short(const u64* __restrict__ in, u64* __restrict__ out,
                                                       long long n_out, int block, int lb) {
  const int lane = (int)(threadIdx.x & 63);
  const int e = lane & ((1 << lb) - 1), j = lane >> lb, per = 64 >> lb;
  for (long long o0 = wave_id() * kRows * per; o0 < n_out; o0 += (long long)gridDim.x * 4 * kRows * per) {
    Elem<W> x[kRows];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      const long long o = o0 + r * per + j;
      x[r] = load_elem<W>(o < n_out && e < block ? in + (size_t)(o * block + e) * W : identity<W>());
    }
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      if (lb > 0) x[r] = turn<W, 0>(x[r], x[r], lane);
      if (lb > 1) x[r] = turn<W, 1>(x[r], x[r], lane);
      if (lb > 2) x[r] = turn<W, 2>(x[r], x[r], lane);
      if (lb > 3) x[r] = turn<W, 3>(x[r], x[r], lane);
      if (lb > 4) x[r] = turn<W, 4>(x[r], x[r], lane);
      if (lb > 5) x[r] = turn<W, 5>(x[r], x[r], lane);
      const long long o = o0 + r * per + j;
      if (e == 0 && o < n_out) store_elem<W>(out + (size_t)o * W, x[r]);
    }
  }
}

// A nest without reducing levels: every element is its own output.
__global__ void __launch_bounds__(256) k_ordered_copy(const u64* __restrict__ in, u64* __restrict__ out, long long n) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    out[i] = in[i];
}

// A grid of g workgroups, held below 2^32 threads (the kernels walk what is left)
static dim3 grid_of(long long g) { return dim3((unsigned)(g < (1 << 21) ? g : 1 << 21)); }

// Four rows per wave where there are many (their chains overlap), else one.
template <int W>
static void launch_short(const u64* x, u64* y, long long n_out, long long block, hipStream_t st) {
  int lb = 0;
  while ((1 << lb) < block) ++lb;
  const long long outs = (long long)4 * (64 >> lb), g = (n_out + outs - 1) / outs;  // outputs of a workgroup's rows
  if (g > 1024)
    hipLaunchKernelGGL((k_ordered_short<W, 4>), grid_of((g + 3) / 4), dim3(256), 0, st, x, y, n_out, (int)block, lb);
  else
    hipLaunchKernelGGL((k_ordered_short<W, 1>), grid_of(g), dim3(256), 0, st, x, y, n_out, (int)block, lb);
}

template <int W>
static void launch_join(const u64* x, u64* y, long long n_out, long long block, hipStream_t st) {
  const int run = (int)((block + 64 * kJoinWaves - 1) / (64 * kJoinWaves));
  hipLaunchKernelGGL(k_ordered_join<W>, dim3((unsigned)(n_out < (1 << 16) ? n_out : 1 << 16)), dim3(64 * kJoinWaves), 0,
                     st, x, y, n_out, (int)block, run);
}

template <int W>
static void launch_w(const DevPlan& P, const u64* x, u64* y, u64* ws, hipStream_t st) {
  const long long n_out = P.n_out, block = P.ord_block, C = P.gsplit;
  if (block <= 64) return launch_short<W>(x, y, n_out, block, st);
  if (P.nw == kJoinWaves) return launch_join<W>(x, y, n_out, block, st);
  const long long units = n_out * C, span = P.ord_span;
  u64* dst = C > 1 ? ws : y;
  const dim3 grid = grid_of((units + 3) / 4);
  // One group of a tile (512 maps, 256 matrices), or a loop over groups: of 2048 maps, which
  // take 38 multiplies (37 and one for the running product), or of 512, which take 14,
  // whichever end a range with fewer; of 512 matrices only, since eight tiles' results spill
  // (4,096 x 4,000: 94 us, 82 in groups of 512).  Blocks of up to 256 matrices are a tile's
  // (17,657 x 89: 28.4 us in groups of 512, whose second tile is empty, 19.3 here), and
  // three tiles go one by one where there are more than a wave and a half per SIMD (3,687 x
  // 534: 16.3 and 15.2 us; 400 of them are 5 % faster in groups of two).
  const long long len = span < block ? span : block;
  if (W == 2 && len <= 512)
    hipLaunchKernelGGL((k_ordered<2, 512, false>), grid, dim3(256), 0, st, x, dst, units, C, block, span);
  else if (W == 4 && len <= 256)
    hipLaunchKernelGGL((k_ordered<4, 256, false>), grid, dim3(256), 0, st, x, dst, units, C, block, span);
  else if (W == 4 && len > 512 && len <= 768 && units > 1536)
    hipLaunchKernelGGL((k_ordered<4, 256, true>), grid, dim3(256), 0, st, x, dst, units, C, block, span);
  else if (W == 2 && (len + 2047) / 2048 * 38 <= (len + 511) / 512 * 14)
    hipLaunchKernelGGL((k_ordered<2, 2048, true>), grid, dim3(256), 0, st, x, dst, units, C, block, span);
  else
    hipLaunchKernelGGL((k_ordered<W, 512, true>), grid, dim3(256), 0, st, x, dst, units, C, block, span);
  if (C == 1) return;
  // the chunks' products are an ordered product themselves
  if (C <= 64) launch_short<W>(ws, y, n_out, C, st);
  else launch_join<W>(ws, y, n_out, C, st);
}

hp_status launch_ordered(const DevPlan& P, const void* in, void* out, void* ws, hipStream_t st) {
  const u64* x = reinterpret_cast<const u64*>(in);
  u64* y = reinterpret_cast<u64*>(out);
  u64* w = reinterpret_cast<u64*>(ws);
  if (P.p == P.depth) {
    const long long n = P.n_out * (P.dtype == HP_AFFINE64 ? 2 : 4), g = (n + 255) / 256;
    hipLaunchKernelGGL(k_ordered_copy, dim3((unsigned)(g < 4096 ? g : 4096)), dim3(256), 0, st, x, y, n);
  } else if (P.dtype == HP_AFFINE64) {
    launch_w<2>(P, x, y, w, st);
  } else {
    launch_w<4>(P, x, y, w, st);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(HP_EDEVICE, "kernel launch failed: %s", hipGetErrorString(e));
  return HP_OK;
}

}  // namespace hp
