// Minimax line of a partition (section 3.1's fixed-width objective): the
// slope minimising the vertical width of the strip that holds every point
// (t, y_t).  The width W(theta) = max_t (y_t - theta t) - min_t (y_t - theta
// t) is convex and piecewise linear.  Its right derivative is t_lo - t_up,
// where t_up is the first of the points of largest y - theta t and t_lo the
// last of those of smallest: never zero for two or more points, so the
// minimiser is one slope, a bend of W, and a bend is the slope dy / dt of the
// line through two of the points.  The answer is that fraction.
//
// It is found by cutting planes.  A pair (upper point, lower point) bounds W
// from below by its own gap, a line in theta.  Two pairs are kept, the
// touching points just right of a slope left of the minimiser and of one
// right of it (at first of slopes -inf and +inf: the partition's ends).  The
// larger of the two upper points' lines minus the smaller of the two lower
// points' is a convex model of W with at most two bends; the model's
// minimum is one of them, the slope of two known points.  One pass over the
// partition finds the touching points there: if they are no further apart
// than the model, model and W share their minimum; otherwise they replace
// one of the pairs and the bracket shrinks.  2 passes on convex data, 3 to 5
// on noise and sorted keys, 16 on the worst of the point sets searched
// (arcs, exponentials and reciprocals against each other, 64 .. 4096 points).
//
// A pass orders the points by K_t = S (y_t dt - t dy) - t for S a power of
// two above every t: the largest K is the first point of largest y - theta
// t, the smallest K the last of smallest, and K gives back t and y.  All
// exact: in binary64 while 2 range S^2 < 2^53 (range below 2^32 for 1024
// values, 2^28 for 4096), where a value costs one fma, one add and two
// comparisons, else in int128 (range < 2^61, t < 2^20).
//
// This replaced convex hulls (per-thread chains of 16 points merged pairwise
// in LDS, every hull edge tested).  Encode of 1e8 values, before -> now: noisy
// line u32 L 1024 1.69 -> 0.30 ms, sorted keys u64 L 2000 3.66 -> 0.37, L 4096
// 2.14 -> 0.45 and L 10,000 (streamed) 3.76 -> 0.76; 2e7 u64 values in 4096s of
// range 2^29 to 2^40 (read again in every pass) 0.50 -> 0.15 to 0.17.  The
// register-held passes are bound by vector issue (64 binary64 instructions a
// pass and lane, about 40 more for the reduction): 1210 instructions a
// partition of 1024 values, 193 of the kernel's 215 us for 1e8.
#pragma once

#include "fit.hpp"

namespace leco {

// Slopes tried at most.  Every step ends the search or narrows the bracket;
// the bound only ends a search whose column changes under it.
constexpr int kStripSteps = 1024;

// A point of the partition: position and offset from its smallest value.
template <class C>
struct StripPoint {
  C t, y;
};

// The touching points of the strip at one slope, and their y dt - t dy.
template <class C, class P>
struct StripTouch {
  StripPoint<C> up, lo;
  P key_up, key_lo;
};

// The minimiser's fraction dy / dt, from the partition's first and last
// point (two or more in all); touch(dy, dt) is a pass over the points at
// slope dy / dt.  C holds coordinates, P products of two (both exact).
// Returns 0 once the width is known to be at least `beat` at every slope, 1
// with the answer, 2 when the steps ran out.
template <class C, class P, class Touch>
__device__ __attribute__((always_inline)) inline int strip_slope(StripPoint<C> first,
                                                                 StripPoint<C> last, P beat,
                                                                 const Touch& touch, C& dy, C& dt) {
  // touching points left (ul, ll) and right (ur, lr) of the minimiser
  StripPoint<C> ul = last, ll = first, ur = first, lr = last;
  for (int step = 0; step < kStripSteps; ++step) {
    const C du = ul.t - ur.t, dl = lr.t - ll.t;  // >= 0, not both 0
    const C yu = ul.y - ur.y, yl = lr.y - ll.y;
    // the model's bends yu / du and yl / dl: its minimum is at the first of
    // them when the gap already widens behind it, else at the other
    bool upper;
    if (du == 0)
      upper = false;
    else if (dl == 0)
      upper = true;
    else if (P(yu) * P(dl) <= P(yl) * P(du))
      upper = ll.t >= ur.t;
    else
      upper = lr.t < ul.t;
    dy = upper ? yu : yl;
    dt = upper ? du : dl;
    const auto key = [&](StripPoint<C> p) { return P(p.y) * P(dt) - P(p.t) * P(dy); };
    const P a = key(ul), b = key(ur), c = key(ll), d = key(lr);
    const P key_up = a > b ? a : b, key_lo = c < d ? c : d;
    if (key_up - key_lo >= beat * P(dt)) return 0;
    const StripTouch<C, P> x = touch(dy, dt);
    if (x.key_up == key_up && x.key_lo == key_lo) return 1;
    if (x.lo.t < x.up.t) {
      ul = x.up;
      ll = x.lo;
    } else {
      ur = x.up;
      lr = x.lo;
    }
  }
  return 2;
}

// The width from which a line cannot be stored instead of a model of `bits` >
// 0 bits, for offsets of range `range` < 2^61.  A stored prediction is floor(q),
// q the binary64 product, and q is within e of theta t: theta is rounded once
// or (from 2^53 on, where dy is no binary64 number) twice and the product
// once, so e <= 3 2^-53 |theta t|, and |theta t| <= 2 range at the minimiser,
// whose width is at most that of slope 0.  Residuals therefore span more than
// W - 1 - 2e, with 2e <= 3 2^-51 range, and 2^(bits-1) or more need `bits`
// bits again.  (A margin of 3 whatever the range lost lines from about 2^56
// on.)  Below 2^49 the range adds nothing.
__device__ inline int64_t strip_beat(uint32_t bits, uint64_t range) {
  return (int64_t(1) << (bits - 1)) + 3 + int64_t(range >> 49);
}

// Binary64 keys are exact for partitions of at most 2^log2s values (S =
// 2^log2s, log2s <= 20) whose range is below this; offsets fit 32 bits.
__device__ __host__ constexpr uint64_t strip_f64_range(uint32_t log2s) {
  return uint64_t(1) << (log2s <= 10 ? 32 : 52 - 2 * log2s);
}

// ---- group reductions of a (largest, smallest) pair -------------------------------

// Largest mx and smallest mn of a wavefront (maxNum / minNum: NaN passes).
__device__ inline void wave_maxmin(double& mx, double& mn) {
  mx = wave_reduce<true>(mx, [](double a, double b) { return fmax(a, b); });
  mn = wave_reduce<true>(mn, [](double a, double b) { return fmin(a, b); });
}

__device__ inline void wave_maxmin(__int128& mx, __int128& mn) {
  mx = wave_max(mx);
  mn = wave_min(mn);
}

// LDS of a workgroup's reductions, in two halves used in turn: one barrier
// per reduction (a half is rewritten two reductions later, behind the
// barrier of the one between).
struct StripShared {
  __int128 part[2][kEncWaves][2];
};

// A group of kT threads: one wavefront, or a workgroup of kEncBlock.
template <int kT>
struct StripGroup {
  StripShared* sh;
  uint32_t turn = 0;

  template <class P>
  __device__ void maxmin(P& mx, P& mn) {
    wave_maxmin(mx, mn);
    if constexpr (kT > 64) {
      P* part = reinterpret_cast<P*>(sh->part[turn]);
      turn ^= 1;
      const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
      if (lane == 0) {
        part[2 * wave] = mx;
        part[2 * wave + 1] = mn;
      }
      __syncthreads();
#pragma unroll
      for (int w = 0; w < kEncWaves; ++w) {
        mx = part[2 * w] > mx ? part[2 * w] : mx;
        mn = part[2 * w + 1] < mn ? part[2 * w + 1] : mn;
      }
    }
  }
};

// ---- passes -------------------------------------------------------------------------

// The touching points from the extreme keys of a binary64 pass.  y is the
// exact quotient (key + t dy) / dt, an integer below 2^52 / S^2: any
// reciprocal within 2^-34 rounds to it (one Newton step on v_rcp_f64).
__device__ inline StripTouch<double, double> touch_of(double kmx, double kmn, double dy, double dt,
                                                      double S, double inv_s) {
  const double r0 = __builtin_amdgcn_rcp(dt);
  const double r = __fma_rn(r0, __fma_rn(-dt, r0, 1.0), r0);
  StripTouch<double, double> x;
  x.key_up = ceil(kmx * inv_s);
  x.key_lo = ceil(kmn * inv_s);
  x.up.t = x.key_up * S - kmx;
  x.lo.t = x.key_lo * S - kmn;
  x.up.y = rint((x.key_up + x.up.t * dy) * r);
  x.lo.y = rint((x.key_lo + x.lo.t * dy) * r);
  return x;
}

// The minimax slope of a partition of len <= kT kR values held as binary64
// offsets, value k of thread tid at position tid + kT k (NaN from len on:
// maximum and minimum pass over NaN), range below strip_f64_range(kLog2S).
template <int kT, int kR, uint32_t kLog2S>
__device__ __attribute__((always_inline)) inline int strip_slope_regs(
    StripGroup<kT>& g, const double (&y)[kR], uint32_t tid, uint32_t len, double y_first,
    double y_last, uint32_t bits, double& dy, double& dt) {
  static_assert(kT * kR <= (1 << kLog2S), "positions below S");
  constexpr double S = double(1u << kLog2S);
  const auto touch = [&](double ey, double et) {
    const double m = et * S, s = ey * S + 1.0;
    const double step = s * double(kT);
    double c = -s * double(tid);
    double kmx = -__builtin_inf(), kmn = __builtin_inf();
#pragma unroll
    for (int k = 0; k < kR; ++k) {
      const double key = __fma_rn(y[k], m, c);
      kmx = fmax(kmx, key);
      kmn = fmin(kmn, key);
      c -= step;
    }
    g.maxmin(kmx, kmn);
    return touch_of(kmx, kmn, ey, et, S, 1.0 / S);
  };
  return strip_slope<double, double>({0.0, y_first}, {double(len - 1), y_last},
                                     double(strip_beat(bits, 0)), touch, dy, dt);
}

// The same for a partition of any length, its values read again in each
// pass, with S = 2^log2s >= len: in binary64 where the range allows it, else
// (range < 2^61) in int128.
template <int kT, class T>
__device__ __attribute__((always_inline)) inline int strip_slope_stream(
    StripGroup<kT>& g, const T* src, uint32_t tid, uint32_t len, uint64_t vmin, uint64_t range,
    uint32_t bits, double& theta) {
  const auto v = global_ptr(src);
  const auto offset = [&](uint32_t t) { return uint64_t(v[t]) - vmin; };
  const uint32_t log2s = 32 - uint32_t(__clz(int(len - 1)));
  if (range < strip_f64_range(log2s)) {
    const double S = double(1u << log2s), inv_s = 1.0 / S;
    const auto touch = [&](double ey, double et) {
      const double m = et * S, s = ey * S + 1.0;
      double kmx = -__builtin_inf(), kmn = __builtin_inf();
#pragma unroll 4
      for (uint32_t t = tid; t < len; t += kT) {
        const double key = __fma_rn(double(uint32_t(offset(t))), m, -s * double(t));
        kmx = fmax(kmx, key);
        kmn = fmin(kmn, key);
      }
      g.maxmin(kmx, kmn);
      return touch_of(kmx, kmn, ey, et, S, inv_s);
    };
    double dy, dt;
    const int r = strip_slope<double, double>({0.0, double(offset(0))},
                                              {double(len - 1), double(offset(len - 1))},
                                              double(strip_beat(bits, range)), touch, dy, dt);
    theta = dy / dt;
    return r;
  }
  // of equal y dt - t dy the first point is the larger key, or with `last`
  // the last one
  const auto pass = [&](int64_t ey, int64_t et, bool last) {
    __int128 kmx = -(__int128(1) << 126), kmn = __int128(1) << 126;
#pragma unroll 1
    for (uint32_t t = tid; t < len; t += kT) {
      const __int128 d = __int128(int64_t(offset(t))) * et - __int128(ey) * int64_t(t);
      const __int128 key = __int128(static_cast<unsigned __int128>(d) << log2s) +
                           (last ? int64_t(t) : -int64_t(t));
      kmx = key > kmx ? key : kmx;
      kmn = key < kmn ? key : kmn;
    }
    g.maxmin(kmx, kmn);
    StripTouch<int64_t, __int128> x;
    const __int128 mask = (__int128(1) << log2s) - 1;
    x.key_up = (kmx + (last ? 0 : mask)) >> log2s;
    x.key_lo = (kmn + (last ? 0 : mask)) >> log2s;
    x.up.t = int64_t((last ? kmx : -kmx) & mask);
    x.lo.t = int64_t((last ? kmn : -kmn) & mask);
    x.up.y = int64_t(offset(uint32_t(x.up.t)));
    x.lo.y = int64_t(offset(uint32_t(x.lo.t)));
    return x;
  };
  const auto touch = [&](int64_t ey, int64_t et) { return pass(ey, et, false); };
  int64_t dy, dt;
  const int r = strip_slope<int64_t, __int128>({0, int64_t(offset(0))},
                                               {int64_t(len - 1), int64_t(offset(len - 1))},
                                               __int128(strip_beat(bits, range)), touch, dy, dt);
  if (r == 1 && range >> 53) {
    // dy and its multiples may round differently: the fraction is that of
    // the upper touching points' whole edge, or when there is one point, of
    // the lower's
    const StripTouch<int64_t, __int128> x = pass(dy, dt, false), z = pass(dy, dt, true);
    const bool upper = z.up.t != x.up.t;
    dy = upper ? z.up.y - x.up.y : x.lo.y - z.lo.y;
    dt = upper ? z.up.t - x.up.t : x.lo.t - z.lo.t;
  }
  theta = static_cast<double>(dy) / static_cast<double>(dt);
  return r;
}

}  // namespace leco
