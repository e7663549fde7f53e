// Model fitting shared by the encoder and the partitioner (section 3.1):
// the least-squares slope from exact integer sums, the residual width, and
// the choice between the fitted line and the constant model, with
// workgroup-wide reductions over 256 threads.  The reductions take any
// shared-memory struct with a `red[kEncWaves][4]` array and a `theta1` slot.
#pragma once

#include "leco_dev.hpp"

namespace leco {

constexpr int kEncBlock = 256;
constexpr int kEncWaves = kEncBlock / 64;

__device__ inline uint64_t load_value(const uint8_t* col, uint32_t dtype, uint64_t i) {
  return dtype == 8 ? reinterpret_cast<const uint64_t*>(col)[i]
                    : uint64_t(reinterpret_cast<const uint32_t*>(col)[i]);
}

__device__ inline uint64_t shfl_xor64(uint64_t x, int m) {
  return static_cast<uint64_t>(__shfl_xor(static_cast<unsigned long long>(x), m, 64));
}

// ---- wavefront reductions by lane permutations ----
//
// Data-parallel-primitive steps inside the vector unit (pairs, quads, half
// rows, rows of 16, then across rows) and reads of single lanes: no LDS
// pipe, no waits between steps, and the result is in scalar registers, so
// that the 128-bit arithmetic on it runs on the scalar unit.  Against
// ds_bpermute shuffles, encode of 1e8 u32 values at L = 1024 240 -> 226 us,
// at L = 128 1213 -> 1090 us, of 1e4 u64 values 14.1 -> 13.0 us.
// Every lane of the wavefront must be active.

// x permuted; lanes of the rows outside kRowMask keep x.  (A permutation of
// every row writes every lane, so it needs no copy of x to start from.)
template <int kCtrl, int kRowMask, class T>
__device__ inline T dpp(T x) {
  static_assert(sizeof(T) % 4 == 0, "whole registers");
  constexpr int kN = sizeof(T) / 4;
  struct Words { int w[kN]; };
  Words a = __builtin_bit_cast(Words, x);
#pragma unroll
  for (int i = 0; i < kN; ++i)
    a.w[i] = kRowMask == 0xf ? __builtin_amdgcn_mov_dpp(a.w[i], kCtrl, 0xf, 0xf, true)
                             : __builtin_amdgcn_update_dpp(a.w[i], a.w[i], kCtrl, kRowMask, 0xf, false);
  return __builtin_bit_cast(T, a);
}

template <int kLane, class T>
__device__ inline T lane_of(T x) {
  constexpr int kN = sizeof(T) / 4;
  struct Words { int w[kN]; };
  Words a = __builtin_bit_cast(Words, x);
#pragma unroll
  for (int i = 0; i < kN; ++i) a.w[i] = __builtin_amdgcn_readlane(a.w[i], kLane);
  return __builtin_bit_cast(T, a);
}
template <class T>
__device__ inline T lane63(T x) { return lane_of<63>(x); }

// op over the wavefront's x, in every lane.  kIdempotent: op(x, x) = x;
// else rows that a step does not add to must get op's neutral element.
template <bool kIdempotent, class T, class Op>
__device__ __attribute__((always_inline)) inline T wave_reduce(T x, const Op& op) {
  x = op(x, dpp<0xB1, 0xf>(x));   // quad_perm [1,0,3,2]
  x = op(x, dpp<0x4E, 0xf>(x));   // quad_perm [2,3,0,1]
  x = op(x, dpp<0x141, 0xf>(x));  // row_half_mirror
  x = op(x, dpp<0x140, 0xf>(x));  // row_mirror
  if constexpr (kIdempotent) {
    x = op(x, dpp<0x142, 0xa>(x));  // row_bcast15 into rows 1 and 3
    x = op(x, dpp<0x143, 0xc>(x));  // row_bcast31 into rows 2 and 3
    return lane63(x);
  } else {
    // rows 0 .. 3 hold their own totals
    const T a = lane_of<15>(x), b = lane_of<31>(x), c = lane_of<47>(x), d = lane_of<63>(x);
    return op(op(a, b), op(c, d));
  }
}

template <class T>
__device__ inline T wave_min(T x) {
  return wave_reduce<true>(x, [](T a, T b) { return b < a ? b : a; });
}
template <class T>
__device__ inline T wave_max(T x) {
  return wave_reduce<true>(x, [](T a, T b) { return b > a ? b : a; });
}
__device__ inline uint64_t wave_sum_u64(uint64_t x) {
  return wave_reduce<false>(x, [](uint64_t a, uint64_t b) { return a + b; });
}
__device__ inline U128 wave_sum_u128(U128 x) {
  return wave_reduce<false>(x, [](U128 a, U128 b) { return add128(a, b); });
}

__device__ inline void wave_minmax_u64(uint64_t& mn, uint64_t& mx) {
  mn = wave_min(mn);
  mx = wave_max(mx);
}

__device__ inline void wave_minmax_i64(int64_t& mn, int64_t& mx) {
  mn = wave_min(mn);
  mx = wave_max(mx);
}

__device__ inline void wave_sum_u128x2(U128& x, U128& y) {
  x = wave_sum_u128(x);
  y = wave_sum_u128(y);
}

__device__ inline void wave_sum_u64x2(uint64_t& x, uint64_t& y) {
  x = wave_sum_u64(x);
  y = wave_sum_u64(y);
}

// ---- workgroup reductions: one LDS slot per wavefront ----

// The workgroup's min and max of values the same in every lane of a
// wavefront, in every thread (two barriers).
template <class Sh>
__device__ inline void block_join_u64(Sh& sh, uint64_t& mn, uint64_t& mx) {
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
    sh.red[wave][0] = mn;
    sh.red[wave][1] = mx;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kEncWaves; ++w) {
    mn = sh.red[w][0] < mn ? sh.red[w][0] : mn;
    mx = sh.red[w][1] > mx ? sh.red[w][1] : mx;
  }
  __syncthreads();
}

template <class Sh>
__device__ inline void block_join_i64(Sh& sh, int64_t& mn, int64_t& mx) {
  // order-preserving map of int64 onto uint64
  uint64_t a = uint64_t(mn) ^ (1ull << 63), b = uint64_t(mx) ^ (1ull << 63);
  block_join_u64(sh, a, b);
  mn = int64_t(a ^ (1ull << 63));
  mx = int64_t(b ^ (1ull << 63));
}

// Every thread receives the workgroup's min and max (two barriers).
template <class Sh>
__device__ inline void block_minmax_u64(Sh& sh, uint64_t& mn, uint64_t& mx) {
  wave_minmax_u64(mn, mx);
  block_join_u64(sh, mn, mx);
}

template <class Sh>
__device__ inline void block_minmax_i64(Sh& sh, int64_t& mn, int64_t& mx) {
  wave_minmax_i64(mn, mx);
  block_join_i64(sh, mn, mx);
}

// Exact workgroup sums of two unsigned 128-bit values.
template <class Sh>
__device__ inline void block_sum_u128x2(Sh& sh, U128& x, U128& y) {
  wave_sum_u128x2(x, y);
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
    sh.red[wave][0] = x.lo;
    sh.red[wave][1] = x.hi;
    sh.red[wave][2] = y.lo;
    sh.red[wave][3] = y.hi;
  }
  __syncthreads();
  x = U128{0, 0};
  y = U128{0, 0};
#pragma unroll
  for (int w = 0; w < kEncWaves; ++w) {
    x = add128(x, U128{sh.red[w][0], sh.red[w][1]});
    y = add128(y, U128{sh.red[w][2], sh.red[w][3]});
  }
  __syncthreads();
}

// Exact workgroup sums of two 64-bit values that cannot overflow.
template <class Sh>
__device__ inline void block_sum_u64x2(Sh& sh, uint64_t& x, uint64_t& y) {
  wave_sum_u64x2(x, y);
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
    sh.red[wave][0] = x;
    sh.red[wave][1] = y;
  }
  __syncthreads();
  x = y = 0;
#pragma unroll
  for (int w = 0; w < kEncWaves; ++w) {
    x += sh.red[w][0];
    y += sh.red[w][1];
  }
  __syncthreads();
}

// Least-squares slope from exact sums S_y = sum y_t and S_ty = sum t y_t.
// Shifting every value by a constant c changes neither n S_ty - S_t S_y nor
// the slope, so the sums may be taken over v_t or over v_t - vmin; N is
// formed modulo 2^128 and its true magnitude is below 2^121, so it is exact.
__device__ inline double ls_slope(uint64_t len, U128 sv, U128 stv) {
  const uint64_t st = len * (len - 1) / 2;                         // < 2^39
  const uint64_t stt = ((len - 1) * len / 2) * (2 * len - 1) / 3;  // < 2^61, exact
  const U128 N = sub128(mul128x64(stv, len), mul128x64(sv, st));
  const U128 D = sub128(mul64x64(len, stt), mul64x64(st, st));
  double slope = i128_to_f64(N) / u128_to_f64(D);
  if (slope == 0.0) slope = 0.0;  // +0.0, never -0.0
  return slope;
}

// The same for at most 4096 values less than 2^30 above the smallest (sy < 2^42
// and sty < 2^54), in about a third of the operations: N in two parts whose
// binary64 products and differences are exact (below 2^47), joined by one
// rounding, and D = n^2 (n^2 - 1) / 12 < 2^45, exact (4 divides n^2 (n^2 - 1),
// and a multiple of 3 is divided by 3's inverse modulo 2^64).
__device__ inline double ls_slope_narrow(uint64_t len, uint64_t sy, uint64_t sty) {
  const uint32_t n = uint32_t(len), n2 = n * n, mask = (1u << 22) - 1;  // n^2 <= 2^24
  const double dn = double(n), st = double(n * (n - 1) / 2);
  const double hi = __builtin_fma(dn, double(uint32_t(sty >> 22)),
                                  -__dmul_rn(st, double(uint32_t(sy >> 22))));
  const double lo = __builtin_fma(dn, double(uint32_t(sty) & mask),
                                  -__dmul_rn(st, double(uint32_t(sy) & mask)));
  const uint64_t D = (uint64_t(n2) * (n2 - 1) / 4) * 0xaaaaaaaaaaaaaaabull;
  double slope = __builtin_fma(hi, 4194304.0, lo) / u64_to_f64(D);
  if (slope == 0.0) slope = 0.0;  // +0.0, never -0.0
  return slope;
}

// The slope computed once (by wave 0) and broadcast through LDS.
template <class Sh>
__device__ inline double block_slope(Sh& sh, uint64_t len, U128 sv, U128 stv) {
  if ((threadIdx.x >> 6) == 0) {
    const double th = ls_slope(len, sv, stv);
    if (threadIdx.x == 0) sh.theta1 = th;
  }
  __syncthreads();
  return sh.theta1;
}

template <class Sh>
__device__ inline double block_slope_narrow(Sh& sh, uint64_t len, uint64_t sy, uint64_t sty) {
  if ((threadIdx.x >> 6) == 0) {
    const double th = ls_slope_narrow(len, sy, sty);
    if (threadIdx.x == 0) sh.theta1 = th;
  }
  __syncthreads();
  return sh.theta1;
}

// The model of one partition, identical in every thread of the workgroup.
struct Model {
  uint64_t vmin, base;
  double theta1;
  uint32_t bits;
  bool linear;
  int64_t rmin;
  uint64_t range;  // vmax - vmin
};

// Chooses between the constant model and the fitted line (ties keep the
// constant model, whose width never exceeds bitlen(vmax - vmin)).
__device__ inline void choose_model(Model& md, double th, int64_t rmin, int64_t rmax) {
  const uint32_t b_ls = bitlen64(uint64_t(rmax) - uint64_t(rmin));
  if (b_ls < md.bits) {
    md.linear = true;
    md.theta1 = th;
    md.base = md.vmin + uint64_t(rmin);
    md.bits = b_ls;
    md.rmin = rmin;
  }
}

}  // namespace leco
