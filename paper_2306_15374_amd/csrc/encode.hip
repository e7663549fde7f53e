// LeCo encoder for gfx950 (section 3.1 regressor, section 3.3 encoder).  Every
// encode fits, lays out and packs:
//
//   fit    every partition's model: range, exact least-squares sums, slope,
//          residual range, the choice between the line and the constant
//          model (section 3.1), hence its width b and its word count; with
//          the minimax regressor also the minimax line (k_fit_minimax*,
//          minimax.hpp), with the polynomial regressor the degree-2 and
//          degree-3 polynomials (k_fit_poly*);
//   layout the exclusive prefix of the word counts gives every partition's
//          word offset; the records, starts, header and padding are written;
//   pack   every partition's residuals are bit-packed into its word span
//          (section 3.3 storage format).
//
// In two passes these are kernels of their own: no partition waits on another,
// and the packing reads the column a second time and recomputes the residuals
// from the stored models.  In one pass (k_encode_fused*, least squares) a
// partition's values stay in registers from the fit to the packing, and its
// word offset comes from a look-back over the counts that the partitions
// before it have published.  launch_encode_columns takes one pass for small
// launches, where launches and latency count, and for 8-byte columns whose
// partitions nearly fill a workgroup's registers.  Both work on a table of
// columns, so one sequence of launches encodes one column or thousands.
//
// The fits take one wavefront per partition when every partition holds at
// most kWaveEncodeMax values (2 to 16 per lane, by the partition's length) or
// twice that (32 per lane): values in registers, reductions by lane
// permutations, no workgroup barrier.  Longer partitions get a whole workgroup.
//
// Register-resident partitions whose range is below 2^30 (the usual case)
// fit on a narrow path: y = v - vmin fits 32 bits, the exact sums fit 64-bit
// lanes, and predictions and residuals fit int32.  The arithmetic and its
// results are the same as on the general path, only carried in fewer bits.
#include "fit.hpp"
#include "internal.hpp"
#include "leco_dev.hpp"
#include "minimax.hpp"

namespace leco {

constexpr int kEncRegs = 16;                           // values per thread in registers
constexpr uint32_t kEncRegLen = kEncBlock * kEncRegs;  // 4096
constexpr uint32_t kWaveEncMax = uint32_t(kWaveEncodeMax);
constexpr int kWaveRegs = int(kWaveEncMax / 64);      // values per lane, one wavefront
constexpr int kShortRegs = 2;                         // the fewest
constexpr uint64_t kNarrowRange = 1ull << 30;
constexpr uint32_t kScanItems = 1024;                  // word counts per scan workgroup

__device__ inline void raise(int* err, int bits) { atomicOr(err, bits); }

__device__ inline void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

struct FitShared {
  uint64_t red[kEncWaves][4];
  double theta1;
};

// ORs a residual u (< 2^b) into a stream of 32-bit words at bit q.
__device__ inline void or_bits(uint32_t* w, uint32_t q, uint32_t b, uint64_t u) {
  if (u == 0) return;
  const uint32_t i = q >> 5, s = q & 31;
  atomicOr(&w[i], uint32_t(u << s));
  if (s + b > 32) atomicOr(&w[i + 1], uint32_t(u >> (32 - s)));
  if (s + b > 64) atomicOr(&w[i + 2], uint32_t(u >> (64 - s)));
}

// p[i] read through the constant address space: a scalar load when i is
// uniform across the wavefront.  Only for data written before the launch.
template <class T>
__device__ inline T meta_load(const T* p, uint64_t i) {
  return ((const __attribute__((address_space(4))) T*)p)[i];
}

constexpr uint32_t kColWords = sizeof(EncColumn) / 8;
static_assert(sizeof(EncColumn) == 96 && offsetof(EncColumn, part_base) == 72 &&
                  offsetof(EncColumn, dtype) == 80 && offsetof(EncColumn, regressor) == 88,
              "column entry layout");

// The column holding partition P: the kernel argument of a one-column
// launch, else the last table entry with part_base <= P, read word by word
// with scalar loads when P is uniform.
__device__ inline EncColumn column_of(const EncColumn* cols, uint64_t ncols,
                                      const EncColumn& single, uint64_t P) {
  if (cols == nullptr) return single;
  const uint64_t* t = reinterpret_cast<const uint64_t*>(cols);
  uint64_t lo = 0, hi = ncols;
  while (hi - lo > 1) {
    const uint64_t mid = lo + ((hi - lo) >> 1);
    if (meta_load(t, mid * kColWords + 9) <= P) lo = mid; else hi = mid;
  }
  const uint64_t e = lo * kColWords;
  EncColumn c;
  c.col = reinterpret_cast<const uint8_t*>(meta_load(t, e + 0));
  c.blob = reinterpret_cast<uint8_t*>(meta_load(t, e + 1));
  c.starts = reinterpret_cast<const uint64_t*>(meta_load(t, e + 2));
  c.size_out = reinterpret_cast<uint64_t*>(meta_load(t, e + 3));
  c.n = meta_load(t, e + 4);
  c.m = meta_load(t, e + 5);
  c.fixed_len = meta_load(t, e + 6);
  c.cap = meta_load(t, e + 7);
  c.words_off = meta_load(t, e + 8);
  c.part_base = meta_load(t, e + 9);
  const uint64_t w = meta_load(t, e + 10);
  c.dtype = uint32_t(w);
  c.force_constant = uint32_t(w >> 32);
  c.regressor = uint32_t(meta_load(t, e + 11));
  c.pad = 0;
  return c;
}

// First value and length of partition j of column c.
__device__ inline void part_bounds(const EncColumn& c, uint64_t j, uint64_t& start,
                                   uint64_t& len) {
  if (c.fixed_len) {
    start = j * c.fixed_len;
    len = (start + c.fixed_len < c.n ? start + c.fixed_len : c.n) - start;
  } else {
    start = meta_load(c.starts, j);
    len = meta_load(c.starts, j + 1) - start;
  }
}

__device__ inline void write_header(const EncColumn& c, uint64_t total_words) {
  uint64_t* hd = reinterpret_cast<uint64_t*>(c.blob);
  const bool variable = c.fixed_len == 0;
  const uint64_t flags = (variable ? kFlagVariable : 0) | (c.regressor == 2 ? kFlagPoly : 0);
  hd[0] = uint64_t(kMagic) | (uint64_t(kVersion) << 32) | (uint64_t(c.dtype) << 48) |
          (flags << 56);
  hd[1] = c.n;
  hd[2] = c.m;
  hd[3] = c.fixed_len;
  hd[4] = kHeaderBytes;
  hd[5] = variable ? kHeaderBytes + kRecordBytes * c.m : 0;
  hd[6] = c.words_off;
  hd[7] = total_words;
}

// Header, the last start and the zero padding of a column whose total word
// count is known; size checked against the capacity.
__device__ inline void finish_column(const EncColumn& c, uint64_t total_words, int* err) {
  const uint64_t size = align16(c.words_off + 8 * total_words);
  if (c.size_out) *c.size_out = size;
  if (size > c.cap) {
    raise(err, kErrNoSpace);
    return;
  }
  write_header(c, total_words);
  const bool variable = c.fixed_len == 0;
  const uint64_t meta_end = kHeaderBytes + kRecordBytes * c.m + (variable ? 8 * (c.m + 1) : 0);
  if (variable) reinterpret_cast<uint64_t*>(c.blob + kHeaderBytes + kRecordBytes * c.m)[c.m] = c.n;
  // padding around the coefficient section, which k_layout fills
  const uint64_t coef = c.regressor == 2 ? align16(meta_end) : c.words_off;
  const uint64_t coef_end = c.regressor == 2 ? coef + 16 * c.m : c.words_off;
  for (uint64_t i = meta_end; i < coef; ++i) c.blob[i] = 0;
  for (uint64_t i = coef_end; i < c.words_off; ++i) c.blob[i] = 0;
  for (uint64_t i = c.words_off + 8 * total_words; i < size; ++i) c.blob[i] = 0;
}

// Record j of a column, its start (variable partitions) and its coefficients
// (polynomial columns; zero for a line or constant), as far as the capacity
// reaches.
__device__ inline void write_record(const EncColumn& c, uint64_t j, uint64_t base, uint64_t theta,
                                    uint64_t word_off, uint32_t bits, uint32_t kind, uint64_t c2,
                                    uint64_t c3) {
  const uint64_t rec = kHeaderBytes + kRecordBytes * j;
  if (rec + kRecordBytes <= c.cap) {
    uint4* r = reinterpret_cast<uint4*>(c.blob + rec);
    r[0] = make_uint4(uint32_t(base), uint32_t(base >> 32), uint32_t(theta), uint32_t(theta >> 32));
    r[1] = make_uint4(uint32_t(word_off), uint32_t(word_off >> 32), bits | kind << 8, 0);
  }
  const uint64_t starts = kHeaderBytes + kRecordBytes * c.m;
  if (c.fixed_len == 0 && starts + 8 * j + 8 <= c.cap)
    *reinterpret_cast<uint64_t*>(c.blob + starts + 8 * j) = c.starts[j];
  if (c.regressor == 2) {
    const uint64_t co = align16(starts + (c.fixed_len == 0 ? 8 * (c.m + 1) : 0)) + 16 * j;
    if (co + 16 <= c.cap) {
      uint64_t* q = reinterpret_cast<uint64_t*>(c.blob + co);
      q[0] = kind ? c2 : 0;
      q[1] = kind ? c3 : 0;
    }
  }
}

// Writes the fitted model of partition P.
__device__ inline void store_model(const EncScratch& s, uint64_t P, const Model& md,
                                   uint64_t len) {
  s.base[P] = md.base;
  s.theta[P] = uint64_t(__double_as_longlong(md.theta1));
  s.bits[P] = md.bits;
  s.nwords[P] = (len * md.bits + 63) >> 6;
}

// ---- fit: one thread per partition ------------------------------------------------

// Partitions of at most this many values are fitted by one thread each when
// a launch holds no longer ones (a wavefront per partition left 63 of its
// 64 lanes idle at one value per partition: 1.4 ms for the 2e6 sampled
// partitions of a size search's first length).
constexpr uint64_t kLaneFitMax = 32;

// The model fit_wave_regs computes, by one thread: the same exact sums (the
// slope is one function of them, whatever their order), the same residual
// range and the same choice.
__device__ inline Model fit_lane(const uint8_t* src, uint32_t dtype, uint64_t len,
                                 bool force_constant) {
  uint64_t vmin = ~uint64_t(0), vmax = 0;
  U128 sv{0, 0}, stv{0, 0};
  for (uint64_t t = 0; t < len; ++t) {
    const uint64_t x = load_value(src, dtype, t);
    vmin = x < vmin ? x : vmin;
    vmax = x > vmax ? x : vmax;
    sv = add128(sv, U128{x, 0});
    stv = add128(stv, mul64x64(t, x));
  }
  const uint64_t range = vmax - vmin;
  Model md{vmin, vmin, 0.0, bitlen64(range), false, 0, range};
  if (len > 1 && !force_constant && range < (uint64_t(1) << 61)) {
    const double th = ls_slope(len, sv, stv);
    int64_t rmin = INT64_MAX, rmax = INT64_MIN;
    for (uint64_t t = 0; t < len; ++t) {
      const int64_t rr = int64_t(load_value(src, dtype, t) - vmin) - predict(th, uint32_t(t));
      rmin = rr < rmin ? rr : rmin;
      rmax = rr > rmax ? rr : rmax;
    }
    choose_model(md, th, rmin, rmax);
  }
  return md;
}

// Least-squares partitions of at most kLaneFitMax values, one thread each
// (grid-stride over the launch's partitions).
__global__ __launch_bounds__(256) void k_fit_lane(const EncColumn* __restrict__ cols,
                                                  uint64_t ncols, EncColumn single,
                                                  uint64_t nparts, EncScratch scr) {
  const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
  for (uint64_t P = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; P < nparts; P += stride) {
    const EncColumn c = column_of(cols, ncols, single, P);
    uint64_t start, len;
    part_bounds(c, P - c.part_base, start, len);
    const Model md = fit_lane(c.col + start * c.dtype, c.dtype, len, c.force_constant != 0);
    store_model(scr, P, md, len);
  }
}

// ---- fit: one wavefront per partition ---------------------------------------------

// Exact sums of y = v - vmin (below 2^61) and of t y over kN register-held
// values (value k at position t0 + k * kStride, positions from len on
// ignored), each y split at bit 32: s = {sum y_lo, sum y_hi} and
// st = {sum t y_lo, sum t y_hi}.  With at most 4096 values (t < 2^12) every
// component stays below 2^56, so the wavefront and workgroup sums of U128
// pairs add them component-wise (no carry leaves a low half), and
// join_split makes the 128-bit sums.  The slope of the offsets is the
// slope of the values.
template <int kN, uint32_t kStride, class W>
__device__ __attribute__((always_inline)) inline void split_sums_regs(
    const W (&v)[kN], uint32_t t0, uint64_t len, uint64_t vmin, U128& s, U128& st) {
  uint64_t slo = 0, shi = 0, stlo = 0, sthi = 0;
#pragma unroll
  for (int k = 0; k < kN; ++k) {
    const uint32_t t = t0 + k * kStride;
    const uint64_t y = t < len ? uint64_t(v[k]) - vmin : 0;
    const uint64_t yl = y & 0xffffffffu, yh = y >> 32;
    slo += yl;
    shi += yh;
    stlo += uint64_t(t) * yl;
    sthi += uint64_t(t) * yh;
  }
  s = U128{slo, shi};
  st = U128{stlo, sthi};
}

__device__ inline U128 join_split(U128 p) {
  return add128(U128{p.lo, 0}, U128{p.hi << 32, p.hi >> 32});
}

// Range of the least-squares residuals of kN register-held values, value k
// at position t0 + k * kStride (positions from len on ignored), over the
// wavefront.  When small
// (values below vmin + 2^30, every |floor(theta1 t)| below 2^30, the same
// in every lane) each residual fits int32 and the range is taken in 32-bit
// operations; otherwise in 64-bit ones with the full prediction.
template <int kN, uint32_t kStride, class W>
__device__ __attribute__((always_inline)) inline void residual_range_regs(
    const W (&v)[kN], uint32_t t0, uint64_t len, uint64_t vmin, double th, bool small,
    int64_t& rmin, int64_t& rmax) {
  if (__builtin_amdgcn_readfirstlane(int(small))) {
    int32_t mn = INT32_MAX, mx = INT32_MIN;
#pragma unroll
    for (int k = 0; k < kN; ++k) {
      const uint32_t t = t0 + k * kStride;
      const int32_t rr = int32_t(uint32_t(v[k]) - uint32_t(vmin)) - predict32(th, t);
      if (t < len) {
        mn = rr < mn ? rr : mn;
        mx = rr > mx ? rr : mx;
      }
    }
    rmin = wave_min(mn);
    rmax = wave_max(mx);
  } else {
    rmin = INT64_MAX;
    rmax = INT64_MIN;
#pragma unroll
    for (int k = 0; k < kN; ++k) {
      const uint32_t t = t0 + k * kStride;
      const int64_t rr = int64_t(uint64_t(v[k]) - vmin) - predict(th, t);
      if (t < len) {
        rmin = rr < rmin ? rr : rmin;
        rmax = rr > rmax ? rr : rmax;
      }
    }
    wave_minmax_i64(rmin, rmax);
  }
}

// Loads of value t of a partition of len values: the index is clamped so
// every lane loads (no branch between loads), and callers mask t >= len.
template <class T>
__device__ inline uint64_t load_clamped(const T* src, uint32_t t, uint64_t len) {
  return uint64_t(global_ptr(src)[t < len ? t : uint32_t(len - 1)]);
}

// The model of a partition of len <= 64 kR values held by one wavefront,
// value lane + 64 k in v[k] (positions past len holding its last value;
// W: the column's value type, or uint64_t for either).
template <int kR, class W>
__device__ __attribute__((always_inline)) inline Model fit_wave_regs(const W (&v)[kR],
                                                                    uint64_t len,
                                                                    bool force_constant) {
  const uint32_t lane = threadIdx.x & 63;
  // clamped lanes hold the last value, which leaves min and max unchanged
  W lo = v[0], hi = v[0];
#pragma unroll
  for (int k = 1; k < kR; ++k) {
    lo = v[k] < lo ? v[k] : lo;
    hi = v[k] > hi ? v[k] : hi;
  }
  const uint64_t vmin = wave_min(lo), vmax = wave_max(hi);
  const uint64_t range = vmax - vmin;
  Model md{vmin, vmin, 0.0, bitlen64(range), false, 0, range};
  if (len > 1 && !force_constant && range < (uint64_t(1) << 61)) {
    const bool narrow = range < kNarrowRange;
    double th;
    if (narrow) {
      uint64_t sy = 0, sty = 0;  // < 2^40 and < 2^50
#pragma unroll
      for (int k = 0; k < kR; ++k) {
        const uint32_t t = lane + 64 * k;
        const uint64_t y = t < len ? uint32_t(v[k]) - uint32_t(vmin) : 0;
        sy += y;
        sty += uint64_t(t) * y;
      }
      wave_sum_u64x2(sy, sty);
      th = ls_slope_narrow(len, sy, sty);
    } else {
      U128 s, st;
      split_sums_regs<kR, 64>(v, lane, len, vmin, s, st);
      wave_sum_u128x2(s, st);
      th = ls_slope(len, join_split(s), join_split(st));
    }
    // |floor(theta1 t)| < 2^30 for every t < len: predictions fit int32
    const bool small = narrow && __dmul_rn(fabs(th), double(len)) < 1073741824.0;
    int64_t rmin, rmax;
    residual_range_regs<kR, 64>(v, lane, len, vmin, th, small, rmin, rmax);
    choose_model(md, th, rmin, rmax);
  }
  return md;
}

// The same, loading the partition (len <= 64 kR values) first.
template <int kR, class T>
__device__ __attribute__((always_inline)) inline Model fit_wave(const T* src, uint64_t len, bool force_constant) {
  const uint32_t lane = threadIdx.x & 63;
  T v[kR];
#pragma unroll
  for (int k = 0; k < kR; ++k) v[k] = T(load_clamped(src, lane + 64 * k, len));
  return fit_wave_regs<kR>(v, len, force_constant);
}

// Calls f with the smallest number of values per lane, kMin to kR halving,
// that holds a partition of len values: every loop of a fit runs over all of
// them, so at 16 a partition of 128 values paid for 1024 (encode of 5e7 u32
// values in such partitions: least squares 540 us, now 356, minimax 1020 and
// 660, polynomial 1153 and 744, with the packing's smaller last batch).
template <int kN>
struct Lanes {
  static constexpr int n = kN;
};

template <int kR, int kMin, class F>
__device__ __attribute__((always_inline)) inline auto by_length(uint64_t len, const F& f) {
  if constexpr (kR > kMin) {
    if (len <= 32 * kR) return by_length<kR / 2, kMin>(len, f);
  }
  return f(Lanes<kR>{});
}

// At 16 values per lane, held to five waves per SIMD (82 VGPRs instead of
// 104): 2% faster on u64 columns.
template <int kR>
__global__ __launch_bounds__(kEncBlock, kR == 16 ? 5 : 1) void k_fit_wave(const EncColumn* __restrict__ cols,
                                                       uint64_t ncols, EncColumn single,
                                                       uint64_t nparts, EncScratch scr,
                                                       int* err) {
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t P =
      uint64_t(blockIdx.x) * kEncWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (P >= nparts) return;
  // launches holding polynomial columns (k_fit_poly) never use this kernel
  const EncColumn c = column_of(cols, ncols, single, P);
  uint64_t start, len;
  part_bounds(c, P - c.part_base, start, len);
  if (len > 64 * kR) {  // the host sends such partitions to k_fit_block
    if (lane == 0) raise(err, kErrDevice);
    return;
  }
  const Model md = by_length<kR, kShortRegs>(len, [&](auto r) __attribute__((always_inline)) {
    return c.dtype == 8
               ? fit_wave<r.n>(reinterpret_cast<const uint64_t*>(c.col) + start, len, c.force_constant)
               : fit_wave<r.n>(reinterpret_cast<const uint32_t*>(c.col) + start, len, c.force_constant);
  });
  if (lane == 0) store_model(scr, P, md, len);
}

// Every thread receives the workgroup's min and max of int32 values.
__device__ inline void block_minmax_i32(FitShared& sh, int32_t& mn, int32_t& mx) {
  mn = wave_min(mn);
  mx = wave_max(mx);
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
    sh.red[wave][0] = uint64_t(uint32_t(mn));
    sh.red[wave][1] = uint64_t(uint32_t(mx));
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kEncWaves; ++w) {
    mn = min(mn, int32_t(uint32_t(sh.red[w][0])));
    mx = max(mx, int32_t(uint32_t(sh.red[w][1])));
  }
  __syncthreads();
}

// ---- fit: one workgroup per partition ----------------------------------------------

// The model of one partition, by the whole workgroup (identical in every
// thread).  Partitions of at most kEncRegLen values are held in registers;
// longer ones are streamed twice.  kKnown: at most kEncRegLen values, vmin and
// vmax are theirs.
template <bool kKnown, class T>
__device__ __attribute__((always_inline)) inline Model fit_block_range(FitShared& sh, const T* src, uint64_t len, bool force_constant,
                                                                      uint64_t vmin, uint64_t vmax) {
  const uint32_t tid = threadIdx.x;
  const bool in_regs = kKnown || len <= kEncRegLen;
  const auto gsrc = global_ptr(src);
  uint64_t v[kEncRegs];
  U128 sv{0, 0}, stv{0, 0};
  if (in_regs) {
#pragma unroll
    for (int k = 0; k < kEncRegs; ++k) v[k] = load_clamped(src, tid + k * kEncBlock, len);
    if (!kKnown) {
      vmin = vmax = v[0];
#pragma unroll
      for (int k = 1; k < kEncRegs; ++k) {
        vmin = v[k] < vmin ? v[k] : vmin;
        vmax = v[k] > vmax ? v[k] : vmax;
      }
    }
  } else {
    // streamed: range and raw sums in one pass
    for (uint64_t t = tid; t < len; t += kEncBlock) {
      const uint64_t x = uint64_t(gsrc[t]);
      vmin = x < vmin ? x : vmin;
      vmax = x > vmax ? x : vmax;
      sv = add128(sv, U128{x, 0});
      stv = add128(stv, mul64x64(t, x));
    }
  }
  if (!kKnown) block_minmax_u64(sh, vmin, vmax);
  const uint64_t range = vmax - vmin;
  Model md{vmin, vmin, 0.0, bitlen64(range), false, 0, range};
  if (len > 1 && !force_constant && range < (uint64_t(1) << 61)) {
    double th;
    bool small = false;
    if (in_regs && range < kNarrowRange) {
      uint64_t sy = 0, sty = 0;  // < 2^42 and < 2^54
#pragma unroll
      for (int k = 0; k < kEncRegs; ++k) {
        const uint32_t t = tid + k * kEncBlock;
        const uint64_t y = t < len ? uint32_t(v[k]) - uint32_t(vmin) : 0;
        sy += y;
        sty += uint64_t(t) * y;
      }
      block_sum_u64x2(sh, sy, sty);
      th = block_slope_narrow(sh, len, sy, sty);
      small = __dmul_rn(fabs(th), double(len)) < 1073741824.0;
    } else {
      if (in_regs) {
#pragma unroll
        for (int k = 0; k < kEncRegs; ++k) {
          const uint32_t t = tid + k * kEncBlock;
          const uint64_t x = t < len ? v[k] : 0;
          sv = add128(sv, U128{x, 0});
          stv = add128(stv, mul64x64(t, x));
        }
      }
      block_sum_u128x2(sh, sv, stv);
      th = block_slope(sh, len, sv, stv);
    }
    int64_t rmin = INT64_MAX, rmax = INT64_MIN;
    if (in_regs) {
      residual_range_regs<kEncRegs, kEncBlock>(v, tid, len, vmin, th, small, rmin, rmax);
    } else {
      for (uint64_t t = tid; t < len; t += kEncBlock) {
        const int64_t rr = int64_t(uint64_t(gsrc[t]) - vmin) - predict(th, uint32_t(t));
        rmin = rr < rmin ? rr : rmin;
        rmax = rr > rmax ? rr : rmax;
      }
      wave_minmax_i64(rmin, rmax);
    }
    block_join_i64(sh, rmin, rmax);
    choose_model(md, th, rmin, rmax);
  }
  return md;
}

template <class T>
__device__ __attribute__((always_inline)) inline Model fit_block(FitShared& sh, const T* src, uint64_t len, bool force_constant) {
  return fit_block_range<false>(sh, src, len, force_constant, ~uint64_t(0), 0);
}

// Six waves per SIMD (at most 80 VGPRs; 114 unconstrained): the extra
// waves of loads in flight outweigh the 26 registers the 128-bit-sum path
// spills.  (8-byte partitions of 3841..4096 values take one pass since.)
// Encode of 2e8 u64 values at L 4096: sorted keys 0.73-0.74 ->
// 0.70 ms (0.76 at four waves), a noisy line 0.66 -> 0.64 ms; partitions
// spanning 2^30 or more, which take that path, 1.07 -> 1.22 ms.
__global__ __launch_bounds__(kEncBlock) __attribute__((amdgpu_waves_per_eu(6))) void k_fit_block(
    const EncColumn* __restrict__ cols, uint64_t ncols, EncColumn single, uint64_t nparts,
    EncScratch scr) {
  __shared__ FitShared sh;
  const uint64_t P = blockIdx.x;
  if (P >= nparts) return;
  const EncColumn c = column_of(cols, ncols, single, P);
  if (c.regressor == 2) return;  // k_fit_poly
  uint64_t start, len;
  part_bounds(c, P - c.part_base, start, len);
  const Model md =
      c.dtype == 8
          ? fit_block(sh, reinterpret_cast<const uint64_t*>(c.col) + start, len, c.force_constant)
          : fit_block(sh, reinterpret_cast<const uint32_t*>(c.col) + start, len, c.force_constant);
  if (threadIdx.x == 0) store_model(scr, P, md, len);
}

// ---- fit with the minimax regressor ------------------------------------------------

// Takes the line of slope theta when its residuals, in [rmin, rmax], are
// strictly narrower than md's model.
__device__ inline void take_narrower(Model& md, double theta, int64_t rmin, int64_t rmax) {
  const uint32_t b = bitlen64(uint64_t(rmax) - uint64_t(rmin));
  if (b >= md.bits) return;
  md.linear = true;
  md.theta1 = theta;
  md.base = md.vmin + uint64_t(rmin);
  md.bits = b;
  md.rmin = rmin;
}

// Residual range of the slope theta over the offsets of strip_slope_regs
// (below 2^32; the predictions of a slope between two of them are below 2^33
// in magnitude, so every difference is exact), reduced over the group.
template <int kT, int kR>
__device__ __attribute__((always_inline)) inline void strip_residuals(StripGroup<kT>& g,
                                                                      const double (&y)[kR],
                                                                      uint32_t tid, double theta,
                                                                      int64_t& rmin,
                                                                      int64_t& rmax) {
  double mx = -__builtin_inf(), mn = __builtin_inf();
#pragma unroll
  for (int k = 0; k < kR; ++k) {
    const double r = y[k] - floor(__dmul_rn(theta, double(tid + kT * k)));
    mx = fmax(mx, r);
    mn = fmin(mn, r);
  }
  g.maxmin(mx, mn);
  rmax = int64_t(mx);
  rmin = int64_t(mn);
}

// The least-squares model of fit_wave_regs, then (minimax) the minimax line
// of section 3.1's fixed-width objective (minimax.hpp), stored instead when
// its residual width is strictly smaller: one wavefront, at most 64 kR
// values.
template <int kR, class T>
__device__ __attribute__((always_inline)) inline Model fit_minimax_wave(const T* src, uint64_t len,
                                                                        bool force_constant,
                                                                        bool minimax, int* err) {
  constexpr uint32_t kLog2S = kR <= 16 ? 10 : 11;
  const uint32_t lane = threadIdx.x & 63;
  T v[kR];
#pragma unroll
  for (int k = 0; k < kR; ++k) v[k] = T(load_clamped(src, lane + 64 * k, len));
  Model md = fit_wave_regs<kR>(v, len, force_constant);
  // the same partitions as the least-squares line: len > 1, range < 2^61
  if (!minimax || len < 2 || force_constant || md.bits == 0 || md.range >= (uint64_t(1) << 61))
    return md;
  StripGroup<64> g{nullptr};
  double theta;
  int64_t rmin, rmax;
  int found;
  if (md.range < strip_f64_range(kLog2S)) {
    double y[kR];
#pragma unroll
    for (int k = 0; k < kR; ++k)
      y[k] = lane + 64 * k < len ? double(uint32_t(uint64_t(v[k]) - md.vmin)) : __builtin_nan("");
    // lane 0 holds the first value, lane 63 (clamped or not) the last
    const double y_first = double(uint32_t(__builtin_amdgcn_readlane(int(uint32_t(v[0]) - uint32_t(md.vmin)), 0)));
    const double y_last = double(uint32_t(__builtin_amdgcn_readlane(int(uint32_t(v[kR - 1]) - uint32_t(md.vmin)), 63)));
    double dy, dt;
    found = strip_slope_regs<64, kR, kLog2S>(g, y, lane, uint32_t(len), y_first, y_last, md.bits,
                                             dy, dt);
    if (found != 1) {
      if (found == 2 && lane == 0) raise(err, kErrDevice);
      return md;
    }
    // one correctly rounded division of the exact fraction
    theta = dy / dt;
    if (theta == 0.0) theta = 0.0;  // +0.0, never -0.0
    strip_residuals<64, kR>(g, y, lane, theta, rmin, rmax);
  } else {
    found = strip_slope_stream<64>(g, src, lane, uint32_t(len), md.vmin, md.range, md.bits, theta);
    if (found != 1) {
      if (found == 2 && lane == 0) raise(err, kErrDevice);
      return md;
    }
    if (theta == 0.0) theta = 0.0;
    // the values read again: held across the search they cost an occupancy step
    rmin = INT64_MAX;
    rmax = INT64_MIN;
    const auto gsrc = global_ptr(src);
    for (uint32_t t = lane; t < len; t += 64) {
      const int64_t rr = int64_t(uint64_t(gsrc[t]) - md.vmin) - predict(theta, t);
      rmin = rr < rmin ? rr : rmin;
      rmax = rr > rmax ? rr : rmax;
    }
    wave_minmax_i64(rmin, rmax);
  }
  take_narrower(md, theta, rmin, rmax);
  return md;
}

// The same by one workgroup, any length: partitions of at most kEncRegLen
// values in registers where binary64 keys are exact, the others streamed.
template <class T>
__device__ __attribute__((always_inline)) inline Model fit_minimax(FitShared& fs, StripShared& ss,
                                                                   const T* src, uint64_t len,
                                                                   bool force_constant,
                                                                   bool minimax, int* err) {
  Model md = fit_block(fs, src, len, force_constant);
  if (!minimax || len < 2 || force_constant || md.bits == 0 || md.range >= (uint64_t(1) << 61))
    return md;
  constexpr uint32_t kLog2S = 12;
  static_assert(kEncRegLen == 1u << kLog2S, "register-held partitions");
  const uint32_t tid = threadIdx.x;
  StripGroup<kEncBlock> g{&ss};
  double theta;
  int64_t rmin = INT64_MAX, rmax = INT64_MIN;
  int found;
  if (len <= kEncRegLen && md.range < strip_f64_range(kLog2S)) {
    double y[kEncRegs];
    uint64_t v[kEncRegs];
#pragma unroll
    for (int k = 0; k < kEncRegs; ++k) v[k] = load_clamped(src, tid + k * kEncBlock, len);
    const double y_first = double(uint32_t(load_clamped(src, 0, len) - md.vmin));
    const double y_last = double(uint32_t(load_clamped(src, uint32_t(len), len) - md.vmin));
#pragma unroll
    for (int k = 0; k < kEncRegs; ++k)
      y[k] = tid + k * kEncBlock < len ? double(uint32_t(v[k] - md.vmin)) : __builtin_nan("");
    double dy, dt;
    found = strip_slope_regs<kEncBlock, kEncRegs, kLog2S>(g, y, tid, uint32_t(len), y_first, y_last,
                                                          md.bits, dy, dt);
    if (found == 1) {
      theta = dy / dt;
      if (theta == 0.0) theta = 0.0;  // +0.0, never -0.0
      strip_residuals<kEncBlock, kEncRegs>(g, y, tid, theta, rmin, rmax);
    }
  } else {
    found = strip_slope_stream<kEncBlock>(g, src, tid, uint32_t(len), md.vmin, md.range, md.bits,
                                          theta);
    if (found == 1) {
      if (theta == 0.0) theta = 0.0;
      const auto gsrc = global_ptr(src);
#pragma unroll 8
      for (uint32_t t = tid; t < len; t += kEncBlock) {
        const int64_t rr = int64_t(uint64_t(gsrc[t]) - md.vmin) - predict(theta, t);
        rmin = rr < rmin ? rr : rmin;
        rmax = rr > rmax ? rr : rmax;
      }
      block_minmax_i64(fs, rmin, rmax);
    }
  }
  if (found == 1) take_narrower(md, theta, rmin, rmax);
  else if (found == 2 && tid == 0) raise(err, kErrDevice);
  return md;
}

__global__ __launch_bounds__(kEncBlock) void k_fit_minimax(const EncColumn* __restrict__ cols,
                                                          uint64_t ncols, EncColumn single,
                                                          uint64_t nparts, EncScratch scr,
                                                          int* err) {
  __shared__ FitShared fs;
  __shared__ StripShared ss;
  const uint64_t P = blockIdx.x;
  if (P >= nparts) return;
  const EncColumn c = column_of(cols, ncols, single, P);
  if (c.regressor == 2) return;  // k_fit_poly
  uint64_t start, len;
  part_bounds(c, P - c.part_base, start, len);
  const bool minimax = c.regressor == 1;
  const Model md =
      c.dtype == 8
          ? fit_minimax(fs, ss, reinterpret_cast<const uint64_t*>(c.col) + start, len,
                        c.force_constant, minimax, err)
          : fit_minimax(fs, ss, reinterpret_cast<const uint32_t*>(c.col) + start, len,
                        c.force_constant, minimax, err);
  if (threadIdx.x == 0) store_model(scr, P, md, len);
}

// One wavefront per partition of at most 64 kR values (four per workgroup,
// no workgroup barrier).  Launches holding polynomial columns never use this
// kernel.
template <int kR>
__global__ __launch_bounds__(kEncBlock, kR == 16 ? 4 : 2) void k_fit_minimax_wave(const EncColumn* __restrict__ cols,
                                                               uint64_t ncols, EncColumn single,
                                                               uint64_t nparts, EncScratch scr,
                                                               int* err) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint64_t P = uint64_t(blockIdx.x) * kEncWaves + wave;
  if (P >= nparts) return;
  const EncColumn c = column_of(cols, ncols, single, P);
  uint64_t start, len;
  part_bounds(c, P - c.part_base, start, len);
  if (len > 64 * kR) {  // the host sends such partitions to k_fit_minimax
    if (lane == 0) raise(err, kErrDevice);
    return;
  }
  const bool minimax = c.regressor == 1;
  const Model md = by_length<kR, kShortRegs>(len, [&](auto r) __attribute__((always_inline)) {
    return c.dtype == 8
               ? fit_minimax_wave<r.n>(reinterpret_cast<const uint64_t*>(c.col) + start, len,
                                       c.force_constant, minimax, err)
               : fit_minimax_wave<r.n>(reinterpret_cast<const uint32_t*>(c.col) + start, len,
                                       c.force_constant, minimax, err);
  });
  if (lane == 0) store_model(scr, P, md, len);
}

// ---- fit with the polynomial regressor: one workgroup per partition ---------------

__device__ inline double i128_to_double(__int128 x) {
  return i128_to_f64(U128{uint64_t(x), uint64_t(static_cast<unsigned __int128>(x) >> 64)});
}

// The norms sum g_k(t)^2 over t < n have closed forms (the Gram
// polynomials' squared norms, exact integers): (n-1)n(n+1)/3,
// (n-2)...(n+2)/5 and (n-3)...(n+3)/7, below 2^84 for n <= 4096.  Each is
// a run of 3, 5 or 7 consecutive integers, one of which the divisor
// divides: that factor is divided first, so no 128-bit division is needed.
__device__ inline __int128 gram_norm(int64_t n, int64_t half, int64_t d) {
  __int128 q = 1;
  bool divided = false;
  for (int64_t f = n - half; f <= n + half; ++f) {
    int64_t x = f;
    if (!divided && x % d == 0) {
      x /= d;
      divided = true;
    }
    q *= x;
  }
  return q;
}

// The degree-2 and degree-3 least-squares polynomials of a partition of
// 3 <= n <= 4096 values of range below 2^50, in the Gram basis:
// c_k = fl(S_k) / fl(Q_k), S_k = sum y_t g_k(t) exact in int128 and
// Q_k = sum g_k(t)^2 from its closed form; md takes the narrower of them when
// strictly narrower than every simpler model.  Each of the group's kT
// threads holds kR <= 16 offsets y = v - vmin, at positions t = u + kT k
// (u = tid, k < kR); sum4 and minmax reduce over the group.
//
// S_k comes from the moments M_j = sum_t y_t t^j, j <= 3, by the
// coefficients of g_k:
//   S1 = 2 M1 - a M0,  S2 = 6 M2 - 6a M1 + e2 M0,
//   S3 = 20 M3 - 30a M2 + k3 M1 - e3 M0        (a = n - 1).
// A thread's positions come in chunks of up to 16 registers, t = u' + kT j
// (u' = u + 16 kT h for chunk h, j < 16); its share of M_j expands
// (u' + kT j)^j binomially over the chunk's sums T_i = sum_j y_j j^i, so
// the loop over values multiplies only by the constants j^i;
// T_3 <= 2^50 (0^3 + ... + 15^3) < 2^64, so every T_i fits 64 bits.  The
// group totals stay below 2^103 in magnitude.
template <int kT, int kR, class Sum4, class MinMax>
__device__ __attribute__((always_inline)) inline void poly_stage(
    Model& md, const uint64_t (&y)[kR], uint32_t tid, uint32_t n, const Sum4& sum4,
    const MinMax& minmax, uint32_t& kind, double& c2_out, double& c3_out) {
  constexpr int kC = kR < 16 ? kR : 16;  // registers per chunk
  static_assert(kR % kC == 0, "whole chunks");
  using u128 = unsigned __int128;
  u128 M0 = 0, M1 = 0, M2 = 0, M3 = 0;
#pragma unroll
  for (int h = 0; h < kR / kC; ++h) {
    uint64_t T0 = 0, T1 = 0, T2 = 0, T3 = 0;
#pragma unroll
    for (int j = 0; j < kC; ++j) {
      const int k = h * kC + j;
      const uint64_t yk = tid + uint32_t(k * kT) < n ? y[k] : 0;
      T0 += yk;
      T1 += yk * uint64_t(j);
      T2 += yk * uint64_t(j * j);
      T3 += yk * uint64_t(j * j * j);
    }
    const uint64_t u = tid + uint64_t(h) * kC * kT, S = kT;
    M0 += T0;
    M1 += u128(T0) * u + u128(T1) * S;
    M2 += u128(T0) * (u * u) + u128(T1) * (2 * u * S) + u128(T2) * (S * S);
    M3 += u128(T0) * (u * u * u) + u128(T1) * (3 * u * u * S) + u128(T2) * (3 * u * S * S) +
          u128(T3) * (S * S * S);
  }
  sum4(M0, M1, M2, M3);
  const int64_t N = n, a = N - 1;
  const int64_t k3 = 12 * N * N - 30 * N + 22, e2 = a * (N - 2), e3 = a * (N - 2) * (N - 3);
  const __int128 m0 = __int128(M0), m1 = __int128(M1), m2 = __int128(M2), m3 = __int128(M3);
  const __int128 S1 = 2 * m1 - a * m0;
  const __int128 S2 = 6 * m2 - 6 * a * m1 + e2 * m0;
  const __int128 S3 = 20 * m3 - 30 * a * m2 + k3 * m1 - e3 * m0;
  const __int128 Q1 = gram_norm(N, 1, 3), Q2 = gram_norm(N, 2, 5), Q3 = gram_norm(N, 3, 7);
  double c[3];
  const __int128 Sk[3] = {S1, S2, S3}, Q[3] = {Q1, Q2, Q3};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    c[k] = Q[k] != 0 ? i128_to_double(Sk[k]) / i128_to_double(Q[k]) : 0.0;
    if (c[k] == 0.0) c[k] = 0.0;  // +0.0, never -0.0
  }
  // the residuals of both degrees in one pass (the degree-2 prediction is
  // the degree-3 one with c3 = 0: the two share their Gram values, which
  // the thread steps by forward differences over its positions kT apart)
  int64_t mn2 = INT64_MAX, mx2 = INT64_MIN, mn3 = INT64_MAX, mx3 = INT64_MIN;
  GramWalk gw;
  gw.start(tid, n, kT);
#pragma unroll
  for (int k = 0; k < kR; ++k) {
    const uint32_t t = tid + k * kT;
    if (t < n) {
      const int64_t r2 = int64_t(y[k]) - poly_combine(c[0], c[1], 0.0, gw.g1, gw.g2, gw.g3);
      const int64_t r3 = int64_t(y[k]) - gw.predict(c[0], c[1], c[2]);
      mn2 = r2 < mn2 ? r2 : mn2;
      mx2 = r2 > mx2 ? r2 : mx2;
      mn3 = r3 < mn3 ? r3 : mn3;
      mx3 = r3 > mx3 ? r3 : mx3;
    }
    gw.next();
  }
  minmax(mn2, mx2);
  minmax(mn3, mx3);
  for (int deg = 2; deg <= 3; ++deg) {
    if (deg == 3 && n < 4) break;
    const int64_t rmin = deg == 2 ? mn2 : mn3, rmax = deg == 2 ? mx2 : mx3;
    const uint32_t b = bitlen64(uint64_t(rmax) - uint64_t(rmin));
    if (b < md.bits) {
      md.linear = true;
      md.theta1 = c[0];
      md.base = md.vmin + uint64_t(rmin);
      md.bits = b;
      md.rmin = rmin;
      kind = 1;
      c2_out = c[1];
      c3_out = deg == 3 ? c[2] : 0.0;
    }
  }
}

__device__ inline U128 to_u128(unsigned __int128 x) { return U128{uint64_t(x), uint64_t(x >> 64)}; }
__device__ inline unsigned __int128 from_u128(U128 x) {
  return (static_cast<unsigned __int128>(x.hi) << 64) | x.lo;
}

// Partitions whose range is below this take the narrow polynomial fit.
constexpr uint64_t kPolyNarrowRange = uint64_t(1) << 28;

// An integer below 2^52 held in binary64.
__device__ inline uint64_t f64_to_u64(double x) {
  return uint64_t(__double_as_longlong(x + 4503599627370496.0)) & ((uint64_t(1) << 52) - 1);
}

// The nearest int32 of an integer or infinity (v_cvt_i32_f64 saturates).
__device__ inline int32_t f64_to_i32(double x) {
  return static_cast<int32_t>(fmin(fmax(x, -2147483648.0), 2147483647.0));
}

__device__ inline uint64_t uniform64(uint64_t x) {
  const uint32_t lo = uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(x))));
  const uint32_t hi = uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(x >> 32))));
  return (uint64_t(hi) << 32) | lo;
}

// The line and both polynomials of a partition of 3 <= n <= kT kR values of
// range below kPolyNarrowRange, in one pass for the sums and one for the
// residuals, by a group of kT threads; value k of thread tid, at position tid
// + kT k, is the offset y[k] (0 from n on).  The same exact sums,
// slopes, predictions and choice as fit_wave / fit_block and poly_stage:
//   sums       the T_i of poly_stage reach 2^28 (0^3 + ... + 15^3) < 2^42,
//              exact in binary64; the line's sums are M_0 and M_1; M_0 .. M_2 fit 64 bits (2^28 2^36), M_3
//              takes 128;
//   residuals  y and every |floor| are below 2^52, so their differences and
//              extremes are exact in binary64, line, degree 2 and degree 3
//              side by side (25 instructions a value).
// Bound by vector issue: 1170 vector instructions a wavefront of 1000 values,
// 190 of the kernel's 235 us for 1e8.  Against integer sums and residuals in
// three passes, encode of 1e8 values: two sines u32 L 1000 586 -> 412 us,
// sorted keys u64 L 1000 620 -> 448, cubic blocks u64 L 2000 577 -> 415 and
// L 4096 (a workgroup each) 716 -> 474.
template <int kT, int kR, class Group>
__device__ __attribute__((always_inline)) inline Model fit_poly_narrow(
    const uint32_t (&y0)[kR], uint32_t tid, uint32_t n, uint64_t vmin, uint64_t range, Group& group,
    uint32_t& kind, double& c2_out, double& c3_out) {
  constexpr int kC = kR < 16 ? kR : 16;  // registers per chunk, as in poly_stage
  static_assert(kR % kC == 0, "whole chunks");
  using u128 = unsigned __int128;
  uint64_t M0 = 0, M1 = 0, M2 = 0;
  u128 M3 = 0;
#pragma unroll
  for (int h = 0; h < kR / kC; ++h) {
    // A_i = sum_j y_j C(j + i, i), by running sums from the last value down:
    // four additions a value and no constants
    double A0 = 0.0, A1 = 0.0, A2 = 0.0, A3 = 0.0;
#pragma unroll
    for (int j = kC - 1; j >= 0; --j) {
      A0 += double(y0[h * kC + j]);
      A1 += A0;
      A2 += A1;
      A3 += A2;
    }
    const uint64_t T0 = f64_to_u64(A0), T1 = f64_to_u64(A1 - A0),
                   T2 = f64_to_u64(2.0 * A2 - 3.0 * A1 + A0),
                   T3 = f64_to_u64(6.0 * A3 - 12.0 * A2 + 7.0 * A1 - A0);
    const uint64_t u = tid + uint64_t(h) * kC * kT, S = kT;
    M0 += T0;
    M1 += T0 * u + T1 * S;
    M2 += T0 * (u * u) + T1 * (2 * u * S) + T2 * (S * S);
    M3 += u128(T0) * (u * u * u) + u128(T1) * (3 * u * u * S) + u128(T2 * (3 * u * S * S)) +
          u128(T3) * (S * S * S);
  }
  group.sum(M0, M1, M2, M3);
  const int64_t N = n, a = N - 1;
  const int64_t k3 = 12 * N * N - 30 * N + 22, e2 = a * (N - 2), e3 = a * (N - 2) * (N - 3);
  // S1 < 2^54 and |S2| < 2^28 n^3 / 4 < 2^62 (the Gram polynomial of degree 2
  // is n^2 times a Legendre-like one) in 64-bit arithmetic modulo 2^64
  const int64_t S1 = int64_t(2 * M1 - uint64_t(a) * M0);
  const int64_t S2 = int64_t(6 * M2 - uint64_t(6 * a) * M1 + uint64_t(e2) * M0);
  const __int128 S3 = 20 * __int128(M3) - 30 * a * __int128(M2) + k3 * __int128(M1) - e3 * __int128(M0);
  // the norms of gram_norm: n (n^2 - 1) / 3, n (n^2 - 1)(n^2 - 4) / 5 < 2^60
  // and that product times (n^2 - 9) / 7, of which 7 divides one factor
  const uint64_t n2 = uint64_t(N) * uint64_t(N), w1 = uint64_t(N) * (n2 - 1), w2 = w1 * (n2 - 4);
  const bool in_w2 = w2 % 7 == 0;
  const __int128 Q3 = n < 4 ? 0
                            : __int128(u128(in_w2 ? w2 / 7 : w2) * (in_w2 ? n2 - 9 : (n2 - 9) / 7));
  double c[3];
  c[0] = i128_to_double(S1) / u64_to_f64(w1 / 3);
  c[1] = i128_to_double(S2) / u64_to_f64(w2 / 5);
  c[2] = Q3 != 0 ? i128_to_double(S3) / i128_to_double(Q3) : 0.0;
#pragma unroll
  for (int k = 0; k < 3; ++k)
    if (c[k] == 0.0) c[k] = 0.0;  // +0.0, never -0.0
  const double th = ls_slope_narrow(n, M0, M1);
  // an infinity stays only in threads without values: far outside int32
  double mx[3], mn[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    mx[k] = -__builtin_inf();
    mn[k] = __builtin_inf();
  }
  GramWalk gw;
  gw.start(tid, n, kT);
  double td = double(tid);
#pragma unroll
  for (int k = 0; k < kR; ++k) {
    // converted again, not kept in twice the registers since the sums
    uint32_t yk = y0[k];
    asm volatile("" : "+v"(yk));
    // past the end (of the partition's last rounds): NaN, which maximum and
    // minimum pass over
    double y = double(yk);
    if (uint32_t(kT * (k + 1)) > n) y = tid + kT * k < n ? y : __builtin_nan("");
    const double s2 = __dadd_rn(__dmul_rn(c[0], gw.g1), __dmul_rn(c[1], gw.g2));
    const double s3 = __dadd_rn(s2, __dmul_rn(c[2], gw.g3));
    const double r[3] = {y - floor(__dmul_rn(th, td)), y - floor(s2), y - floor(s3)};
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      mx[q] = fmax(mx[q], r[q]);
      mn[q] = fmin(mn[q], r[q]);
    }
    gw.next();
    td += double(kT);
  }
  // Residuals are below 2^31 in magnitude (y < 2^28; a least-squares
  // prediction, without its constant term, is below five times that), so
  // they are reduced as int32; the conversion saturates infinities.
  int32_t hi[3], lo[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    hi[q] = f64_to_i32(mx[q]);
    lo[q] = f64_to_i32(mn[q]);
    group.maxmin(hi[q], lo[q]);
  }
  Model md{vmin, vmin, 0.0, bitlen64(range), false, 0, range};
  choose_model(md, th, lo[0], hi[0]);
  kind = 0;
  c2_out = c3_out = 0.0;
#pragma unroll
  for (int deg = 2; deg <= 3; ++deg) {
    if (deg == 3 && n < 4) break;
    const int64_t rmin = lo[deg - 1], rmax = hi[deg - 1];
    const uint32_t b = bitlen64(uint64_t(rmax) - uint64_t(rmin));
    if (b < md.bits) {
      md.linear = true;
      md.theta1 = c[0];
      md.base = md.vmin + uint64_t(rmin);
      md.bits = b;
      md.rmin = rmin;
      kind = 1;
      c2_out = c[1];
      c3_out = deg == 3 ? c[2] : 0.0;
    }
  }
  return md;
}

// The group's reductions for fit_poly_narrow.
struct PolyWave {
  // m3 < 2^76 in two halves of 40 bits, which 64 lanes cannot overflow
  __device__ void sum(uint64_t& m0, uint64_t& m1, uint64_t& m2, unsigned __int128& m3) {
    m0 = wave_sum_u64(m0);
    m1 = wave_sum_u64(m1);
    m2 = wave_sum_u64(m2);
    const uint64_t lo = wave_sum_u64(uint64_t(m3) & ((uint64_t(1) << 40) - 1));
    m3 = (static_cast<unsigned __int128>(wave_sum_u64(uint64_t(m3 >> 40))) << 40) + lo;
  }
  __device__ void maxmin(int32_t& mx, int32_t& mn) {
    mx = wave_max(mx);
    mn = wave_min(mn);
  }
};

struct PolyBlock {
  FitShared& fs;
  __device__ void sum(uint64_t& m0, uint64_t& m1, uint64_t& m2, unsigned __int128& m3) {
    block_sum_u64x2(fs, m0, m1);
    U128 x = to_u128(m3), z{m2, 0};
    block_sum_u128x2(fs, x, z);
    m0 = uniform64(m0);  // every wavefront's, for the scalar unit
    m1 = uniform64(m1);
    m2 = uniform64(z.lo);
    m3 = (static_cast<unsigned __int128>(uniform64(x.hi)) << 64) | uniform64(x.lo);
  }
  __device__ void maxmin(int32_t& mx, int32_t& mn) { block_minmax_i32(fs, mn, mx); }
};

// The least-squares line and the polynomials, by the whole workgroup: in
// binary64 for narrow partitions, else the model of fit_block and then
// poly_stage.
template <class T>
__device__ __attribute__((always_inline)) inline Model fit_poly(FitShared& fs, const T* src, uint64_t len, bool force_constant,
                                 uint32_t& kind, double& c2_out, double& c3_out) {
  const uint32_t tid = threadIdx.x;
  kind = 0;
  c2_out = c3_out = 0.0;
  const bool in_regs = !force_constant && len >= 3 && len <= kEncRegLen;
  uint64_t vmin = 0, vmax = 0;
  if (in_regs) {
    T v[kEncRegs];
#pragma unroll
    for (int k = 0; k < kEncRegs; ++k) v[k] = T(load_clamped(src, tid + k * kEncBlock, len));
    T lo = v[0], hi = v[0];
#pragma unroll
    for (int k = 1; k < kEncRegs; ++k) {
      lo = v[k] < lo ? v[k] : lo;
      hi = v[k] > hi ? v[k] : hi;
    }
    vmin = lo;
    vmax = hi;
    block_minmax_u64(fs, vmin, vmax);
    if (vmax - vmin < kPolyNarrowRange) {
      uint32_t y[kEncRegs];
#pragma unroll
      for (int k = 0; k < kEncRegs; ++k)
        y[k] = tid + k * kEncBlock < len ? uint32_t(v[k]) - uint32_t(vmin) : 0u;
      PolyBlock g{fs};
      return fit_poly_narrow<kEncBlock, kEncRegs>(y, tid, uint32_t(len), vmin, vmax - vmin, g, kind,
                                                  c2_out, c3_out);
    }
  }
  // Wider: the values read again here and by the polynomials.  Kept in
  // registers (the same loads, as far as the compiler sees: it is told that
  // src may have changed) they cost the narrow fit an occupancy step, 6-9%.
  asm volatile("" : "+s"(src));
  Model md = in_regs ? fit_block_range<true>(fs, src, len, false, vmin, vmax)
                     : fit_block(fs, src, len, force_constant);
  asm volatile("" : "+s"(src));
  if (force_constant || len < 3 || len > kPolyMaxLen || md.range >= kPolyMaxRange) return md;
  uint64_t y[kEncRegs];
#pragma unroll
  for (int k = 0; k < kEncRegs; ++k) y[k] = load_clamped(src, tid + k * kEncBlock, len) - md.vmin;
  const auto sum4 = [&](unsigned __int128& m0, unsigned __int128& m1, unsigned __int128& m2,
                        unsigned __int128& m3) {
    U128 x = to_u128(m0), w = to_u128(m1);
    block_sum_u128x2(fs, x, w);
    m0 = from_u128(x);
    m1 = from_u128(w);
    x = to_u128(m2);
    w = to_u128(m3);
    block_sum_u128x2(fs, x, w);
    m2 = from_u128(x);
    m3 = from_u128(w);
  };
  const auto minmax = [&](int64_t& mn, int64_t& mx) { block_minmax_i64(fs, mn, mx); };
  poly_stage<kEncBlock, kEncRegs>(md, y, tid, uint32_t(len), sum4, minmax, kind, c2_out, c3_out);
  return md;
}

// The same by one wavefront, for partitions of at most 64 kR values (no
// barrier).
template <int kR, class T>
__device__ __attribute__((always_inline)) inline Model fit_poly_wave(const T* src, uint64_t len, bool force_constant,
                                      uint32_t& kind, double& c2_out, double& c3_out) {
  const uint32_t lane = threadIdx.x & 63;
  kind = 0;
  c2_out = c3_out = 0.0;
  T v[kR];
#pragma unroll
  for (int k = 0; k < kR; ++k) v[k] = T(load_clamped(src, lane + 64 * k, len));
  if (!force_constant && len >= 3) {
    T lo = v[0], hi = v[0];
#pragma unroll
    for (int k = 1; k < kR; ++k) {
      lo = v[k] < lo ? v[k] : lo;
      hi = v[k] > hi ? v[k] : hi;
    }
    const uint64_t vmin = wave_min(lo), vmax = wave_max(hi);
    if (vmax - vmin < kPolyNarrowRange) {
      uint32_t y[kR];
#pragma unroll
      for (int k = 0; k < kR; ++k)
        y[k] = lane + 64 * k < len ? uint32_t(v[k]) - uint32_t(vmin) : 0u;
      PolyWave g;
      return fit_poly_narrow<64, kR>(y, lane, uint32_t(len), vmin, vmax - vmin, g, kind, c2_out,
                                     c3_out);
    }
  }
  Model md = fit_wave<kR>(src, len, force_constant);
  if (force_constant || len < 3 || md.range >= kPolyMaxRange) return md;
  uint64_t y[kR];
#pragma unroll
  for (int k = 0; k < kR; ++k) y[k] = load_clamped(src, lane + 64 * k, len) - md.vmin;
  const auto sum4 = [](unsigned __int128& m0, unsigned __int128& m1, unsigned __int128& m2,
                       unsigned __int128& m3) {
    U128 x = to_u128(m0), w = to_u128(m1), z = to_u128(m2), q = to_u128(m3);
    wave_sum_u128x2(x, w);
    wave_sum_u128x2(z, q);
    m0 = from_u128(x);
    m1 = from_u128(w);
    m2 = from_u128(z);
    m3 = from_u128(q);
  };
  const auto minmax = [](int64_t& mn, int64_t& mx) { wave_minmax_i64(mn, mx); };
  poly_stage<64, kR>(md, y, lane, uint32_t(len), sum4, minmax, kind, c2_out, c3_out);
  return md;
}

__device__ inline void store_poly(const EncScratch& s, uint64_t P, uint32_t kind, double c2,
                                  double c3) {
  s.kind[P] = kind;
  s.c2[P] = uint64_t(__double_as_longlong(c2));
  s.c3[P] = uint64_t(__double_as_longlong(c3));
}

__global__ __launch_bounds__(kEncBlock, 4) void k_fit_poly(const EncColumn* __restrict__ cols,
                                                       uint64_t ncols, EncColumn single,
                                                       uint64_t nparts, EncScratch scr) {
  __shared__ FitShared fs;
  const uint64_t P = blockIdx.x;
  if (P >= nparts) return;
  const EncColumn c = column_of(cols, ncols, single, P);
  if (c.regressor != 2) return;  // the other fit kernels
  uint64_t start, len;
  part_bounds(c, P - c.part_base, start, len);
  uint32_t kind;
  double c2, c3;
  const Model md =
      c.dtype == 8
          ? fit_poly(fs, reinterpret_cast<const uint64_t*>(c.col) + start, len, c.force_constant,
                     kind, c2, c3)
          : fit_poly(fs, reinterpret_cast<const uint32_t*>(c.col) + start, len, c.force_constant,
                     kind, c2, c3);
  if (threadIdx.x == 0) {
    store_model(scr, P, md, len);
    store_poly(scr, P, kind, c2, c3);
  }
}

// Held to four waves per SIMD at 16 values per lane and three at 32: the
// narrow fit takes 84 and 134 VGPRs by itself, the wide one beside it 127 and
// 168 (some spilled).  Held to five and four, encode of 1e8 two-sine values
// 455 -> 515 us, of cubic blocks 470 -> 575.
template <int kR>
__global__ __launch_bounds__(kEncBlock, kR == 16 ? 4 : 3) void k_fit_poly_wave(const EncColumn* __restrict__ cols,
                                                            uint64_t ncols, EncColumn single,
                                                            uint64_t nparts, EncScratch scr,
                                                            int* err) {
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t P =
      uint64_t(blockIdx.x) * kEncWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (P >= nparts) return;
  const EncColumn c = column_of(cols, ncols, single, P);
  if (c.regressor != 2) return;  // the other fit kernels
  uint64_t start, len;
  part_bounds(c, P - c.part_base, start, len);
  if (len > 64 * kR) {  // the host sends such partitions to k_fit_poly
    if (lane == 0) raise(err, kErrDevice);
    return;
  }
  uint32_t kind;
  double c2, c3;
  const Model md = by_length<kR, kShortRegs>(len, [&](auto r) __attribute__((always_inline)) {
    return c.dtype == 8
               ? fit_poly_wave<r.n>(reinterpret_cast<const uint64_t*>(c.col) + start, len,
                                    c.force_constant, kind, c2, c3)
               : fit_poly_wave<r.n>(reinterpret_cast<const uint32_t*>(c.col) + start, len,
                                    c.force_constant, kind, c2, c3);
  });
  if (lane == 0) {
    store_model(scr, P, md, len);
    store_poly(scr, P, kind, c2, c3);
  }
}

// ---- layout: word offsets and records -----------------------------------------------

// Exclusive prefix sum of x over a workgroup of 64 W threads, with the
// workgroup's sum in *total.  wsum[W] is shared; a barrier has to lie between
// two calls.
template <int W>
__device__ inline uint64_t block_exclusive_scan_u64(uint64_t* wsum, uint64_t x, uint64_t* total) {
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint64_t inc = x;
#pragma unroll
  for (int delta = 1; delta < 64; delta <<= 1) {
    const uint64_t y = uint64_t(__shfl_up(static_cast<unsigned long long>(inc), delta, 64));
    if (int(lane) >= delta) inc += y;
  }
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  uint64_t before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    if (w < int(wave)) before += wsum[w];
    all += wsum[w];
  }
  *total = all;
  return before + inc - x;
}

// bsum[g] = word count of partitions [g * 1024, (g + 1) * 1024).
__global__ __launch_bounds__(kEncBlock) void k_scan_sums(EncScratch scr, uint64_t nparts) {
  __shared__ uint64_t wsum[kEncWaves];
  const uint64_t p0 = uint64_t(blockIdx.x) * kScanItems + threadIdx.x;
  uint64_t x = 0;
#pragma unroll
  for (uint32_t q = 0; q < kScanItems; q += kEncBlock)
    if (p0 + q < nparts) x += scr.nwords[p0 + q];
  uint64_t total;
  block_exclusive_scan_u64<kEncWaves>(wsum, x, &total);
  if (threadIdx.x == 0) scr.bsum[blockIdx.x] = total;
}

// Exclusive prefix of bsum[0, ng) in place, by one workgroup.
__global__ __launch_bounds__(kScanItems) void k_scan_top(EncScratch scr, uint64_t ng) {
  __shared__ uint64_t wsum[kScanItems / 64];
  uint64_t carry = 0;
  for (uint64_t g0 = 0; g0 < ng; g0 += kScanItems) {
    const uint64_t g = g0 + threadIdx.x;
    const uint64_t x = g < ng ? scr.bsum[g] : 0;
    uint64_t total;
    const uint64_t ex = block_exclusive_scan_u64<kScanItems / 64>(wsum, x, &total);
    __syncthreads();
    if (g < ng) scr.bsum[g] = carry + ex;
    carry += total;
  }
}

// What k_layout knows of the word counts before its workgroup's partitions.
constexpr uint32_t kLayoutCounts = 0;  // nothing: it sums the counts themselves
constexpr uint32_t kLayoutSums = 1;    // bsum holds the sums of k_scan_sums
constexpr uint32_t kLayoutPrefix = 2;  // bsum holds their prefixes (k_scan_top)
constexpr uint64_t kLayoutDirect = 32;
constexpr uint64_t kLayoutGroups = 4096;

// Word offsets within each column, records, starts and headers, one
// workgroup per kScanItems partitions; the workgroups together also write the
// blobs of empty columns, which have no partition.  Below 1e6 partitions
// latency is all there is here (about 5 us for each launch of such kernels),
// so the launches count: the prefixes, their application, the records and the
// empty columns were five kernels and are this one, after at most two that
// sum the counts.  1e6 values: polynomial 29.7 us, now 19.5, 1e7 in
// least-squares partitions of 1024 42 and 35.5.  The words that the column
// of the workgroup's first partition has before it come from the sums of
// whole groups, less what the column's first group holds of columns before
// it; columns that start further on start at 0.  A thread per partition
// while the workgroups fit the chip; more workgroups of 256 threads, which
// take fewer registers: for 1e7 partitions 154 us, 226 with 1024 threads.
template <uint32_t kThreads>
__global__ __launch_bounds__(kThreads) void k_layout(const EncColumn* __restrict__ cols,
                                                    uint64_t ncols, EncColumn single,
                                                    uint64_t nparts, EncScratch scr,
                                                    uint32_t mode, int* err) {
  constexpr uint32_t kPer = kScanItems / kThreads;
  __shared__ uint64_t prefix[kScanItems];
  __shared__ uint64_t wsum[2][kThreads / 64];
  const uint64_t stride = uint64_t(gridDim.x) * kThreads;
  for (uint64_t i = uint64_t(blockIdx.x) * kThreads + threadIdx.x; i < ncols; i += stride) {
    const EncColumn& e = cols ? cols[i] : single;
    if (e.m == 0) finish_column(e, 0, err);  // also writes starts[0] = 0 of a variable column
  }
  const uint64_t g = blockIdx.x, p0 = g * kScanItems;
  if (p0 >= nparts) return;
  uint64_t nw[kPer], sum = 0;
#pragma unroll
  for (uint32_t q = 0; q < kPer; ++q) {
    const uint64_t P = p0 + kPer * threadIdx.x + q;
    nw[q] = P < nparts ? scr.nwords[P] : 0;
    sum += nw[q];
  }
  // words of the first column's partitions before p0
  uint64_t before = 0;
  const uint64_t first = column_of(cols, ncols, single, p0).part_base;
  const uint64_t gf = first / kScanItems;
  if (first < p0) {
    if (mode == kLayoutCounts) {
      for (uint64_t q = first + threadIdx.x; q < p0; q += kThreads) before += scr.nwords[q];
    } else {
      if (mode == kLayoutSums)
        for (uint64_t q = gf + threadIdx.x; q < g; q += kThreads) before += scr.bsum[q];
      else if (threadIdx.x == 0)
        before = scr.bsum[g] - scr.bsum[gf];
      for (uint64_t q = gf * kScanItems + threadIdx.x; q < first; q += kThreads)
        before -= scr.nwords[q];
    }
  }
  uint64_t carry, total;
  block_exclusive_scan_u64<kThreads / 64>(wsum[0], before, &carry);
  uint64_t run = block_exclusive_scan_u64<kThreads / 64>(wsum[1], sum, &total);
#pragma unroll
  for (uint32_t q = 0; q < kPer; ++q) {
    prefix[kPer * threadIdx.x + q] = run;
    run += nw[q];
  }
  __syncthreads();
  for (uint32_t q = 0; q < kPer; ++q) {
    const uint32_t at = q * kThreads + threadIdx.x;
    const uint64_t P = p0 + at;
    if (P >= nparts) break;
    const EncColumn c = column_of(cols, ncols, single, P);
    const uint64_t j = P - c.part_base;
    const uint64_t word_off =
        c.part_base < p0 ? carry + prefix[at] : prefix[at] - prefix[c.part_base - p0];
    scr.woff[P] = word_off;
    const bool poly = c.regressor == 2;
    write_record(c, j, scr.base[P], scr.theta[P], word_off, scr.bits[P], poly ? scr.kind[P] : 0,
                 poly ? scr.c2[P] : 0, poly ? scr.c3[P] : 0);
    if (j + 1 == c.m) finish_column(c, word_off + scr.nwords[P], err);
  }
}

// ---- pack ----------------------------------------------------------------------------

constexpr uint32_t kPackBatch = 8;  // rounds of 64 residuals per batch

// Packs rounds [k_begin, k_end) of partition v[0, len) into its words, from
// the stored model: u = (v - base) - floor(theta1 t), the encoder's
// residual for both models (the constant model has theta1 = +0).  Round k
// holds residuals 64k .. 64k + 63, which fill exactly 2b 32-bit words, so a
// batch of consecutive rounds fills 2b words per round with no word shared
// with another batch.  A batch's values are loaded together, its words
// assembled in the wavefront's LDS buffer (kPackBatch * 128 words) and
// stored as one contiguous run; words at or beyond `limit` (the span's end,
// or the blob's capacity) are not stored.  Called by one wavefront.  A
// polynomial partition (kind 1) predicts with poly_predict(theta1, c2, c3).
template <uint32_t kBatch, class T>
__device__ __attribute__((always_inline)) inline void pack_batch(
    const T* src, uint64_t len, uint64_t base, double theta1, bool fits32, uint32_t kind, double c2,
    double c3, uint32_t b, __attribute__((address_space(1))) uint32_t* gdst, uint64_t limit,
    uint64_t k0, uint32_t nr, uint32_t* w32) {
  const uint32_t lane = threadIdx.x & 63;
  uint64_t u[kBatch];
#pragma unroll
  for (uint32_t r = 0; r < kBatch; ++r) u[r] = load_clamped(src, uint32_t(64 * (k0 + r) + lane), len);
#pragma unroll
  for (uint32_t r = 0; r < kBatch; ++r) {
    const uint32_t t = uint32_t(64 * (k0 + r) + lane);
    const uint64_t p = kind ? uint64_t(poly_predict(theta1, c2, c3, t, uint32_t(len)))
                            : fits32 ? uint64_t(int64_t(predict32(theta1, t)))
                                     : uint64_t(predict(theta1, t));
    u[r] = t < len ? (u[r] - base) - p : 0;
  }
  const uint32_t nw = 2 * b * nr;  // <= 1024
  for (uint32_t q = lane; q < nw; q += 64) w32[q] = 0;
  wave_fence();
#pragma unroll
  for (uint32_t r = 0; r < kBatch; ++r)
    if (r < nr) or_bits(w32, (64 * r + lane) * b, b, u[r]);
  wave_fence();
  const uint64_t first = 2 * b * k0;
  const uint64_t count = first >= limit ? 0 : (limit - first < nw ? limit - first : nw);
  for (uint32_t q = lane; q < count; q += 64) gdst[first + q] = w32[q];
  wave_fence();
}

// kTails: the last rounds in the smallest batch that holds them.
template <bool kTails, class T>
__device__ __attribute__((always_inline)) inline void pack_rounds(const T* src, uint64_t len, uint64_t base, double theta1,
                                   uint32_t kind, double c2, double c3, uint32_t b,
                                   uint32_t* gw32, uint64_t limit, uint64_t k_begin,
                                   uint64_t k_end, uint32_t* w32) {
  const bool fits32 = prediction_fits_i32(theta1, len);
  const auto gdst = global_ptr(gw32);
  uint64_t k0 = k_begin;
  for (; k0 + (kTails ? kPackBatch / 2 : 0) < k_end; k0 += kPackBatch)
    pack_batch<kPackBatch>(src, len, base, theta1, fits32, kind, c2, c3, b, gdst, limit, k0,
                           uint32_t(k_end - k0 < kPackBatch ? k_end - k0 : kPackBatch), w32);
  if (!kTails || k0 >= k_end) return;
  const uint32_t nr = uint32_t(k_end - k0);
  if (nr > 2)
    pack_batch<4>(src, len, base, theta1, fits32, kind, c2, c3, b, gdst, limit, k0, nr, w32);
  else if (nr == 2)
    pack_batch<2>(src, len, base, theta1, fits32, kind, c2, c3, b, gdst, limit, k0, nr, w32);
  else
    pack_batch<1>(src, len, base, theta1, fits32, kind, c2, c3, b, gdst, limit, k0, nr, w32);
}

// One wavefront per partition (kWave, four per workgroup), or one workgroup
// per partition whose four wavefronts take consecutive quarters of its
// rounds (each a whole number of batches).  Five waves per SIMD, as
// the fit had (95 VGPRs instead of 105).  kTails: a smaller last batch, whose
// code beside the full batches' spills 4 registers instead of 2 (2e8 u64
// values at L 1024 335 us with, 324 without).
template <bool kWave, bool kTails>
__global__ __launch_bounds__(kEncBlock) __attribute__((amdgpu_waves_per_eu(5))) void k_pack(
    const EncColumn* __restrict__ cols, uint64_t ncols, EncColumn single, uint64_t nparts,
    EncScratch scr) {
  __shared__ uint32_t lds[kEncWaves][kPackBatch * 128];
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint64_t P = kWave ? uint64_t(blockIdx.x) * kEncWaves + wave : uint64_t(blockIdx.x);
  if (P >= nparts) return;
  const uint32_t b = meta_load(scr.bits, P);
  if (b == 0) return;
  const EncColumn c = column_of(cols, ncols, single, P);
  uint64_t start, len;
  part_bounds(c, P - c.part_base, start, len);
  const uint64_t w0 = 2 * meta_load(scr.woff, P);
  uint32_t* gw32 = reinterpret_cast<uint32_t*>(c.blob + c.words_off) + w0;
  const uint64_t cap_w32 = c.cap > c.words_off ? (c.cap - c.words_off) / 4 : 0;
  const uint64_t nwords32 = 2 * ((len * b + 63) >> 6);
  const uint64_t avail = cap_w32 > w0 ? cap_w32 - w0 : 0;
  const uint64_t limit = nwords32 < avail ? nwords32 : avail;
  const uint64_t rounds = (len + 63) / 64;
  uint64_t k_begin = 0, k_end = rounds;
  if (!kWave) {
    const uint64_t quarter = ((rounds + kEncWaves - 1) / kEncWaves + kPackBatch - 1) / kPackBatch * kPackBatch;
    k_begin = wave * quarter < rounds ? wave * quarter : rounds;
    k_end = k_begin + quarter < rounds ? k_begin + quarter : rounds;
  }
  const double theta1 = __longlong_as_double(static_cast<long long>(meta_load(scr.theta, P)));
  const uint64_t base = meta_load(scr.base, P);
  uint32_t kind = 0;
  double c2 = 0.0, c3 = 0.0;
  if (c.regressor == 2) {
    kind = meta_load(scr.kind, P);
    c2 = __longlong_as_double(static_cast<long long>(meta_load(scr.c2, P)));
    c3 = __longlong_as_double(static_cast<long long>(meta_load(scr.c3, P)));
  }
  if (c.dtype == 8)
    pack_rounds<kTails>(reinterpret_cast<const uint64_t*>(c.col) + start, len, base, theta1, kind, c2, c3,
                b, gw32, limit, k_begin, k_end, lds[wave]);
  else
    pack_rounds<kTails>(reinterpret_cast<const uint32_t*>(c.col) + start, len, base, theta1, kind, c2, c3,
                b, gw32, limit, k_begin, k_end, lds[wave]);
}

// Packs partitions of kPackShortMin to kPackShortMax values of one column,
// as many per wavefront as make up to 512 values: 64 consecutive values of the
// column per round, each with its own partition's model from LDS, into words
// that are consecutive in the blob.  With a wavefront per partition a short
// one pays the latency of its metadata, and a round of its last few values, for
// itself.  magic = 2^20 / fixed_len + 1: position * magic >> 20 is the partition (exact
// below 512 positions and lengths to 256).
constexpr uint64_t kPackShortMin = 32, kPackShortMax = 256;
constexpr uint32_t kPackShortValues = 64 * kPackBatch;
constexpr uint32_t kPackShortParts = kPackShortValues / uint32_t(kPackShortMin);

struct ShortPart {
  uint64_t base;
  double theta1;
  uint32_t bit0, bits;  // first bit among the wavefront's words, residual width
};

template <class T>
__device__ __attribute__((always_inline)) inline void pack_short(
    const EncColumn& c, uint64_t P0, uint32_t count, uint32_t magic, const EncScratch& scr,
    ShortPart* part, uint32_t* w32) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t L = uint32_t(c.fixed_len);
  const uint64_t start = P0 * L;
  const uint32_t n = uint32_t(c.n - start < uint64_t(count) * L ? c.n - start : uint64_t(count) * L);
  const uint64_t woff = meta_load(scr.woff, P0);
  const uint64_t words = meta_load(scr.woff, P0 + count - 1) + meta_load(scr.nwords, P0 + count - 1) - woff;
  if (words == 0) return;
  const T* src = reinterpret_cast<const T*>(c.col) + start;
  uint64_t u[kPackBatch];
#pragma unroll
  for (uint32_t r = 0; r < kPackBatch; ++r) u[r] = load_clamped(src, 64 * r + lane, n);
  bool fits = true;
  if (lane < count) {
    const uint64_t P = P0 + lane;
    const double theta1 = __longlong_as_double(static_cast<long long>(scr.theta[P]));
    part[lane] = ShortPart{scr.base[P], theta1, uint32_t(64 * (scr.woff[P] - woff)), scr.bits[P]};
    fits = prediction_fits_i32(theta1, L);
  }
  const bool fits32 = __ballot(!fits) == 0;
  const uint32_t nw = 2 * uint32_t(words);  // <= 2 kPackShortValues
  for (uint32_t q = lane; q < nw; q += 64) w32[q] = 0;
  wave_fence();
#pragma unroll
  for (uint32_t r = 0; r < kPackBatch; ++r) {
    const uint32_t f = 64 * r + lane;
    if (f < n) {
      const uint32_t i = f * magic >> 20, t = f - i * L;
      const ShortPart m = part[i];
      uint64_t p;
      if (c.regressor == 2 && scr.kind[P0 + i]) {
        const uint32_t len = n - i * L < L ? n - i * L : L;
        p = uint64_t(poly_predict(m.theta1, __longlong_as_double(static_cast<long long>(scr.c2[P0 + i])),
                                  __longlong_as_double(static_cast<long long>(scr.c3[P0 + i])), t, len));
      } else {
        p = fits32 ? uint64_t(int64_t(predict32(m.theta1, t))) : uint64_t(predict(m.theta1, t));
      }
      or_bits(w32, m.bit0 + t * m.bits, m.bits, (u[r] - m.base) - p);
    }
  }
  wave_fence();
  const uint64_t cap_w32 = c.cap > c.words_off ? (c.cap - c.words_off) / 4 : 0;
  const uint64_t avail = cap_w32 > 2 * woff ? cap_w32 - 2 * woff : 0;
  const uint32_t limit = nw < avail ? nw : uint32_t(avail);
  const auto gdst = global_ptr(reinterpret_cast<uint32_t*>(c.blob + c.words_off) + 2 * woff);
  for (uint32_t q = lane; q < limit; q += 64) gdst[q] = w32[q];
}

__global__ __launch_bounds__(kEncBlock) void k_pack_short(EncColumn c, uint64_t nparts,
                                                         uint32_t per, uint32_t magic,
                                                         EncScratch scr) {
  __shared__ uint32_t lds[kEncWaves][2 * kPackShortValues];
  __shared__ ShortPart part[kEncWaves][kPackShortParts];
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint64_t P0 = (uint64_t(blockIdx.x) * kEncWaves + wave) * per;
  if (P0 >= nparts) return;
  const uint32_t count = uint32_t(nparts - P0 < per ? nparts - P0 : per);
  if (c.dtype == 8)
    pack_short<uint64_t>(c, P0, count, magic, scr, part[wave], lds[wave]);
  else
    pack_short<uint32_t>(c, P0, count, magic, scr, part[wave], lds[wave]);
}

// ---- one pass: fit, word offset by look-back, record and pack ----------------------
//
// For least-squares columns whose partitions hold at most kEncRegLen
// values: one workgroup per partition reads the values once into registers
// (wavefront w holds values 1024 w .. 1024 w + 1023, 16 per lane, so its
// rounds of 64 residuals are consecutive), fits the model as fit_block
// does, and takes the partition's word offset from the word counts of the
// partitions before it in its column (decoupled look-back: each partition
// publishes its count as soon as it is fitted, and its inclusive prefix as
// soon as it knows it).  The waits are bounded (lb_exclusive): a partition
// that is late is counted by the one that waits for it.  It then writes its record (and start) and packs its residuals from
// the registers; the last partition of a column writes the header.

// A look-back state: flag in the top two bits, a word count below them.
// Each state is one 64-bit word read and written with relaxed atomics at
// device scope: the word is the whole message, so nothing needs ordering
// around it (acquire / release at device scope would write back or
// invalidate the L2 of an XCD at every access).
constexpr uint64_t kLbCount = uint64_t(1) << 62;      // the partition's own count
constexpr uint64_t kLbInclusive = uint64_t(2) << 62;  // counts of its column up to it
constexpr uint64_t kLbValue = kLbCount - 1;

__device__ inline void lb_publish(uint64_t* st, uint64_t P, uint64_t v) {
  __hip_atomic_store(st + P, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline U128 wave_sum_carry(U128 x) {
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) x = add128(x, U128{shfl_xor64(x.lo, m), shfl_xor64(x.hi, m)});
  return x;
}

// The word count of a partition, by one wavefront that keeps none of its
// values: the model of fit_wave_regs from three reads.  Only for a partition
// whose own workgroup is late (lb_exclusive).
__device__ inline uint64_t count_words(const EncColumn& c, uint64_t j) {
  const uint32_t lane = threadIdx.x & 63;
  uint64_t start, len;
  part_bounds(c, j, start, len);
  const uint8_t* src = c.col + c.dtype * start;
  uint64_t lo = ~uint64_t(0), hi = 0;
  for (uint64_t t = lane; t < len; t += 64) {
    const uint64_t x = load_value(src, c.dtype, t);
    lo = x < lo ? x : lo;
    hi = x > hi ? x : hi;
  }
  const uint64_t vmin = wave_min(lo), range = wave_max(hi) - vmin;
  Model md{vmin, vmin, 0.0, bitlen64(range), false, 0, range};
  if (len > 1 && !c.force_constant && range < (uint64_t(1) << 61)) {
    U128 s{0, 0}, st{0, 0};
    for (uint64_t t = lane; t < len; t += 64) {
      const uint64_t y = load_value(src, c.dtype, t) - vmin;
      s = add128(s, U128{y, 0});
      st = add128(st, mul64x64(t, y));
    }
    s = wave_sum_carry(s);
    st = wave_sum_carry(st);
    const double th = ls_slope(len, s, st);
    int64_t rmin = INT64_MAX, rmax = INT64_MIN;
    for (uint64_t t = lane; t < len; t += 64) {
      const int64_t r =
          int64_t(load_value(src, c.dtype, t) - vmin) - predict(th, uint32_t(t));
      rmin = r < rmin ? r : rmin;
      rmax = r > rmax ? r : rmax;
    }
    choose_model(md, th, wave_min(rmin), wave_max(rmax));
  }
  return (len * md.bits + 63) >> 6;
}

// Words of the column's partitions before P, by one wavefront: kLbWindow
// predecessors per round (lane l reads the state of partition hi - 1 - l),
// down to the nearest one with an inclusive prefix; rounds wait (sleeping
// between reads) while a partition closer than that has published nothing
// yet.  What these reads fetch past the L2s is what bounds a large launch, so
// the window is no wider than the number in flight asks for: with 1024
// workgroups 16 (2e8 u64 values in partitions of 4096 564 us; 64: 584, 256:
// 751, 4: 739), with 4096 wavefronts 64 (1e8 u32 values in partitions of 1024
// 287 us; 16: 367, 256: 560).
//
// Workgroups start in the order of their index here, so that a predecessor
// is running or done; but nothing guarantees it, so the wait is bounded:
// after `polls` reads the wavefront counts the nearest missing partition
// itself and goes on.  (An index from an atomic counter is such a guarantee,
// at 13 ns for each of its workgroups: 680 us for 48,800 of them.)
template <uint32_t kLbWindow>
__device__ inline uint64_t lb_exclusive(uint64_t* st, const EncColumn& c, uint64_t P,
                                        uint32_t polls) {
  const uint32_t lane = threadIdx.x & 63;
  const uint64_t first = c.part_base;
  uint64_t acc = 0, hi = P;
  uint32_t left = polls;
  while (hi > first) {
    const uint64_t span = hi - first < kLbWindow ? hi - first : kLbWindow;
    const bool in = lane < span;
    const uint64_t s =
        in ? __hip_atomic_load(st + (hi - 1 - lane), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    const uint64_t inc = __ballot(in && (s >> 62) == 2);
    const int stop = inc ? __ffsll(static_cast<long long>(inc)) - 1 : int(span) - 1;
    const uint64_t need = stop >= 63 ? ~0ull : (2ull << stop) - 1;  // lanes 0..stop
    const uint64_t missing = __ballot(in && (s >> 62) == 0) & need;
    if (missing == 0) {
      acc += wave_sum_u64(in && int(lane) <= stop ? (s & kLbValue) : 0);
      if (inc != 0) break;  // always, where the column's first partition is in the span
      hi -= span;
      left = polls;
      continue;
    }
    if (left != 0) {
      --left;
      __builtin_amdgcn_s_sleep(8);
      continue;
    }
    const uint64_t late = hi - uint64_t(__ffsll(static_cast<long long>(missing)));
    const uint64_t nw = count_words(c, late - first);
    unsigned long long none = 0;  // what its workgroup published meanwhile stays
    if (lane == 0)
      __hip_atomic_compare_exchange_strong(
          reinterpret_cast<unsigned long long*>(st + late), &none,
          (unsigned long long)((late == first ? kLbInclusive : kLbCount) | nw),
          __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  return acc;
}

constexpr uint64_t kFusedFullLen = 3840;  // see launch_encode_columns

struct FusedShared {
  FitShared fit;
  uint64_t woff;
  uint64_t join[3][kEncWaves][2];  // one for each join of the fit: a barrier less than one reused
  // each wavefront's 16 rounds of residuals, packed: 2 b words per round, for
  // every b (4 workgroups to a CU, as many as its registers allow; wider than
  // 61 bits from a second read of the values, 5e7 full-width values took 254
  // us in partitions of 4096, more than two passes' 243, and take 202)
  uint32_t words[kEncWaves][2 * 64 * kEncRegs];
};

// The narrow fit of fit_regs, in binary64: offsets below 2^30 are exact
// there, and so are a lane's sums of 16 (below 2^34, and 2^38 times k); a
// conversion, an addition and a fused multiply-add per value where 64-bit
// integers took eight issue slots.  kFull: no position is masked.
template <bool kFull>
__device__ __attribute__((always_inline)) inline void fit_regs_narrow(
    FusedShared& sh, const uint64_t (&v)[kEncRegs], uint32_t t0, uint64_t len, Model& md,
    int32_t (&r32)[kEncRegs], bool& small) {
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t low = uint32_t(md.vmin);
  double sy = 0.0, sk = 0.0;  // sums of y and of k y, position t0 + 64 k
#pragma unroll
  for (int k = 0; k < kEncRegs; ++k) {
    const uint32_t y = kFull || t0 + 64 * k < len ? uint32_t(v[k]) - low : 0;
    const double d = double(y);
    sy += d;
    sk = __builtin_fma(d, double(k), sk);
  }
  uint64_t s = f64_to_u64(sy), st = uint64_t(t0) * s + 64 * f64_to_u64(sk);  // < 2^42 and < 2^54
  wave_sum_u64x2(s, st);
  if (lane == 0) {
    sh.join[1][wave][0] = s;
    sh.join[1][wave][1] = st;
  }
  __syncthreads();
  s = st = 0;
#pragma unroll
  for (int w = 0; w < kEncWaves; ++w) {
    s += sh.join[1][w][0];
    st += sh.join[1][w][1];
  }
  const double th = block_slope_narrow(sh.fit, len, s, st);
  small = __dmul_rn(fabs(th), double(len)) < 1073741824.0;
  if (!small) {
    md.theta1 = th;
    return;
  }
  int32_t mn = INT32_MAX, mx = INT32_MIN;
  double t = double(t0);
#pragma unroll
  for (int k = 0; k < kEncRegs; ++k) {
    r32[k] = int32_t(uint32_t(v[k]) - low) - int32_t(floor(__dmul_rn(th, t)));
    t += 64.0;
    if (kFull || t0 + 64 * k < len) {
      mn = min(mn, r32[k]);
      mx = max(mx, r32[k]);
    }
  }
  mn = wave_min(mn);
  mx = wave_max(mx);
  if (lane == 0) {
    sh.join[2][wave][0] = uint64_t(uint32_t(mn));
    sh.join[2][wave][1] = uint64_t(uint32_t(mx));
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kEncWaves; ++w) {
    mn = min(mn, int32_t(uint32_t(sh.join[2][w][0])));
    mx = max(mx, int32_t(uint32_t(sh.join[2][w][1])));
  }
  choose_model(md, th, mn, mx);
}

// The model of a partition held in registers as described above.  When
// the residuals v - vmin - floor(theta1 t) fit int32 (`small`), r32 keeps
// them for the packing.
__device__ __attribute__((always_inline)) inline Model fit_regs(FusedShared& sh, const uint64_t (&v)[kEncRegs],
                                                               uint32_t t0, uint64_t len,
                                                               bool force_constant,
                                                               int32_t (&r32)[kEncRegs],
                                                               bool& small_out) {
  small_out = false;
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // clamped loads hold the partition's last value: min and max unchanged.
  // While a wavefront's values agree in their high halves the low ones do.
  const uint32_t high = uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(v[0] >> 32))));
  uint32_t apart = 0, mn = uint32_t(v[0]), mx = mn;
#pragma unroll
  for (int k = 0; k < kEncRegs; ++k) {
    const uint32_t x = uint32_t(v[k]);
    apart |= uint32_t(v[k] >> 32) ^ high;
    mn = x < mn ? x : mn;
    mx = x > mx ? x : mx;
  }
  uint64_t vmin, vmax;
  if (__ballot(apart != 0) == 0) {
    vmin = uint64_t(high) << 32 | wave_min(mn);
    vmax = uint64_t(high) << 32 | wave_max(mx);
  } else {
    vmin = vmax = v[0];
#pragma unroll
    for (int k = 1; k < kEncRegs; ++k) {
      vmin = v[k] < vmin ? v[k] : vmin;
      vmax = v[k] > vmax ? v[k] : vmax;
    }
    vmin = wave_min(vmin);
    vmax = wave_max(vmax);
  }
  if (lane == 0) {
    sh.join[0][wave][0] = vmin;
    sh.join[0][wave][1] = vmax;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kEncWaves; ++w) {
    vmin = sh.join[0][w][0] < vmin ? sh.join[0][w][0] : vmin;
    vmax = sh.join[0][w][1] > vmax ? sh.join[0][w][1] : vmax;
  }
  const uint64_t range = vmax - vmin;
  Model md{vmin, vmin, 0.0, bitlen64(range), false, 0, range};
  if (len <= 1 || force_constant || range >= (uint64_t(1) << 61)) return md;
  double th;
  if (range < kNarrowRange) {
    if (len == kEncRegLen)
      fit_regs_narrow<true>(sh, v, t0, len, md, r32, small_out);
    else
      fit_regs_narrow<false>(sh, v, t0, len, md, r32, small_out);
    if (small_out) return md;
    th = md.theta1;
    md.theta1 = 0.0;
  } else {
    U128 sv{0, 0}, stv{0, 0};
#pragma unroll
    for (int k = 0; k < kEncRegs; ++k) {
      const uint32_t t = t0 + 64 * k;
      const uint64_t x = t < len ? v[k] : 0;
      sv = add128(sv, U128{x, 0});
      stv = add128(stv, mul64x64(t, x));
    }
    block_sum_u128x2(sh.fit, sv, stv);
    th = block_slope(sh.fit, len, sv, stv);
  }
  int64_t rmin = INT64_MAX, rmax = INT64_MIN;
#pragma unroll
  for (int k = 0; k < kEncRegs; ++k) {
    const uint32_t t = t0 + 64 * k;
    const int64_t rr = int64_t(v[k] - vmin) - predict(th, t);
    if (t < len) {
      rmin = rr < rmin ? rr : rmin;
      rmax = rr > rmax ? rr : rmax;
    }
  }
  block_minmax_i64(sh.fit, rmin, rmax);
  choose_model(md, th, rmin, rmax);
  return md;
}

// One workgroup per partition: values loaded
// once, model fitted, word count published; the residuals packed into LDS
// (which needs no offset) while the partitions before it publish theirs;
// then the look-back, the record, and the packed words copied out.
__device__ __attribute__((always_inline)) inline void encode_fused_part(
    FusedShared& sh, const EncColumn& c, uint64_t P, const EncScratch& scr, uint32_t polls,
    int* err) {
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint64_t start, len;
  const uint64_t j = P - c.part_base;
  part_bounds(c, j, start, len);
  const uint32_t t0 = wave * 64 * kEncRegs + lane;  // value t0 + 64 k is v[k]
  uint64_t v[kEncRegs];
  const bool full = len == kEncRegLen;  // no load clamped, no position masked
  if (c.dtype == 8) {
    const uint64_t* src = reinterpret_cast<const uint64_t*>(c.col) + start;
    if (full) {
#pragma unroll
      for (int k = 0; k < kEncRegs; ++k) v[k] = global_ptr(src)[t0 + 64 * k];
    } else {
#pragma unroll
      for (int k = 0; k < kEncRegs; ++k) v[k] = load_clamped(src, t0 + 64 * k, len);
    }
  } else {
    const uint32_t* src = reinterpret_cast<const uint32_t*>(c.col) + start;
    if (full) {
#pragma unroll
      for (int k = 0; k < kEncRegs; ++k) v[k] = global_ptr(src)[t0 + 64 * k];
    } else {
#pragma unroll
      for (int k = 0; k < kEncRegs; ++k) v[k] = load_clamped(src, t0 + 64 * k, len);
    }
  }
  int32_t r32[kEncRegs];
  bool small;
  const Model md = fit_regs(sh, v, t0, len, c.force_constant != 0, r32, small);
  const uint64_t nw = (len * md.bits + 63) >> 6;
  uint64_t* st = scr.woff;
  if (threadIdx.x == 0) lb_publish(st, P, (j == 0 ? kLbInclusive : kLbCount) | nw);
  // pack this wavefront's rounds 16 w .. 16 w + 15 into its LDS words
  const uint32_t b = md.bits;
  const uint64_t rounds = (len + 63) / 64;
  const uint64_t r0 = uint64_t(wave) * kEncRegs;
  const uint32_t nr = r0 >= rounds ? 0 : uint32_t(rounds - r0 < kEncRegs ? rounds - r0 : kEncRegs);
  const uint32_t nwb = 2 * b * nr;
  uint32_t* w32 = sh.words[wave];
  if (nwb) {
    for (uint32_t q = lane; q < nwb; q += 64) w32[q] = 0;
    wave_fence();
    // the encoder's residual: (v - vmin) - floor(theta1 t) - rmin for the
    // line (from the fit's registers when they hold it), v - vmin for the
    // constant model
    const bool fits32 = prediction_fits_i32(md.theta1, len);
    const bool reuse = md.linear && small;
    if (reuse && full) {
      // every round whole, widths below 32: each residual ORs into two words
      // (the second gets zero bits when it fits in one)
      const int32_t rmin = int32_t(md.rmin);
#pragma unroll
      for (int k = 0; k < kEncRegs; ++k) {
        const uint32_t q = (64 * k + lane) * b;
        const uint64_t x = uint64_t(uint32_t(r32[k] - rmin)) << (q & 31);
        atomicOr(&w32[q >> 5], uint32_t(x));
        atomicOr(&w32[(q >> 5) + 1], uint32_t(x >> 32));
      }
    } else {
#pragma unroll
      for (int k = 0; k < kEncRegs; ++k) {
        const uint32_t t = t0 + 64 * k;
        uint64_t u;
        if (reuse) {
          u = uint64_t(uint32_t(r32[k] - int32_t(md.rmin)));
        } else {
          const uint64_t p = !md.linear ? 0
                             : fits32   ? uint64_t(int64_t(predict32(md.theta1, t)))
                                        : uint64_t(predict(md.theta1, t));
          u = (v[k] - md.base) - p;
        }
        if (t >= len) u = 0;
        if (uint32_t(k) < nr) or_bits(w32, (64 * k + lane) * b, b, u);
      }
    }
    wave_fence();
  }
  if (j != 0 && wave == 0) {
    const uint64_t before = lb_exclusive<16>(st, c, P, polls);
    if (lane == 0) {
      lb_publish(st, P, kLbInclusive | (before + nw));
      sh.woff = before;
    }
  }
  __syncthreads();
  const uint64_t woff = j == 0 ? 0 : sh.woff;
  if (threadIdx.x == 0) {
    const uint64_t rec = kHeaderBytes + kRecordBytes * j;
    if (rec + kRecordBytes <= c.cap) {
      uint64_t* r = reinterpret_cast<uint64_t*>(c.blob + rec);
      r[0] = md.base;
      r[1] = uint64_t(__double_as_longlong(md.theta1));
      r[2] = woff;
      r[3] = uint64_t(md.bits);
    }
    if (c.fixed_len == 0) {
      const uint64_t so = kHeaderBytes + kRecordBytes * c.m + 8 * j;
      if (so + 8 <= c.cap) *reinterpret_cast<uint64_t*>(c.blob + so) = start;
    }
    if (j + 1 == c.m) finish_column(c, woff + nw, err);
  }
  if (nwb) {
    const auto gdst = global_ptr(reinterpret_cast<uint32_t*>(c.blob + c.words_off) + 2 * woff);
    const uint64_t cap_w32 = c.cap > c.words_off ? (c.cap - c.words_off) / 4 : 0;
    const uint64_t avail = cap_w32 > 2 * woff ? cap_w32 - 2 * woff : 0;
    const uint64_t limit = 2 * nw < avail ? 2 * nw : avail;
    const uint64_t first = 2 * b * r0;
    const uint64_t count = first >= limit ? 0 : (limit - first < nwb ? limit - first : nwb);
    for (uint32_t q = lane; q < count; q += 64) gdst[first + q] = w32[q];
  }
}

// Before a one-pass encode: the look-back states (scr.woff) start at 0, and every empty column's blob is written whole
// (one launch instead of two).
__global__ void k_fused_prepare(const EncColumn* __restrict__ cols, uint64_t ncols,
                                EncColumn single, EncScratch scr, uint64_t nparts, int* err) {
  const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
  const uint64_t first = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  for (uint64_t i = first; i < nparts; i += stride) scr.woff[i] = 0;
  for (uint64_t i = first; i < ncols; i += stride) {
    const EncColumn& c = cols ? cols[i] : single;
    if (c.m == 0) finish_column(c, 0, err);
  }
}

__global__ __launch_bounds__(kEncBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_encode_fused(
    const EncColumn* __restrict__ cols, uint64_t ncols, EncColumn single, uint64_t nparts,
    EncScratch scr, uint32_t polls, int* err) {
  __shared__ FusedShared sh;
  const uint64_t P = blockIdx.x;
  if (P >= nparts) return;
  const EncColumn c = column_of(cols, ncols, single, P);
  encode_fused_part(sh, c, P, scr, polls, err);
}

// Partition P of k_encode_fused_wave, of at most 64 kN values.
template <int kN>
__device__ __attribute__((always_inline)) inline void encode_fused_wave(
    const EncColumn& c, uint64_t P, uint64_t j, uint64_t start, uint64_t len,
    const EncScratch& scr, uint32_t polls, uint32_t* w32, int* err) {
  const uint32_t lane = threadIdx.x & 63;
  uint64_t v[kN];
  if (c.dtype == 8) {
    const uint64_t* src = reinterpret_cast<const uint64_t*>(c.col) + start;
#pragma unroll
    for (int k = 0; k < kN; ++k) v[k] = load_clamped(src, lane + 64 * k, len);
  } else {
    const uint32_t* src = reinterpret_cast<const uint32_t*>(c.col) + start;
#pragma unroll
    for (int k = 0; k < kN; ++k) v[k] = load_clamped(src, lane + 64 * k, len);
  }
  const Model md = fit_wave_regs<kN>(v, len, c.force_constant != 0);
  const uint64_t nw = (len * md.bits + 63) >> 6;
  uint64_t* st = scr.woff;
  if (lane == 0) lb_publish(st, P, (j == 0 ? kLbInclusive : kLbCount) | nw);
  const uint32_t b = md.bits;
  const uint32_t nr = uint32_t((len + 63) / 64);
  const uint32_t nwb = 2 * b * nr;
  if (nwb) {
    for (uint32_t q = lane; q < nwb; q += 64) w32[q] = 0;
    wave_fence();
    const bool fits32 = prediction_fits_i32(md.theta1, len);
#pragma unroll
    for (int k = 0; k < kN; ++k) {
      const uint32_t t = lane + 64 * k;
      const uint64_t p = !md.linear ? 0
                         : fits32   ? uint64_t(int64_t(predict32(md.theta1, t)))
                                    : uint64_t(predict(md.theta1, t));
      const uint64_t u = t < len ? (v[k] - md.base) - p : 0;
      if (uint32_t(k) < nr) or_bits(w32, t * b, b, u);
    }
    wave_fence();
  }
  uint64_t woff = 0;
  if (j != 0) {
    woff = lb_exclusive<64>(st, c, P, polls);
    if (lane == 0) lb_publish(st, P, kLbInclusive | (woff + nw));
  }
  if (lane == 0) {
    const uint64_t rec = kHeaderBytes + kRecordBytes * j;
    if (rec + kRecordBytes <= c.cap) {
      uint64_t* r = reinterpret_cast<uint64_t*>(c.blob + rec);
      r[0] = md.base;
      r[1] = uint64_t(__double_as_longlong(md.theta1));
      r[2] = woff;
      r[3] = uint64_t(md.bits);
    }
    if (c.fixed_len == 0) {
      const uint64_t so = kHeaderBytes + kRecordBytes * c.m + 8 * j;
      if (so + 8 <= c.cap) *reinterpret_cast<uint64_t*>(c.blob + so) = start;
    }
    if (j + 1 == c.m) finish_column(c, woff + nw, err);
  }
  if (nwb) {
    const auto gdst = global_ptr(reinterpret_cast<uint32_t*>(c.blob + c.words_off) + 2 * woff);
    const uint64_t cap_w32 = c.cap > c.words_off ? (c.cap - c.words_off) / 4 : 0;
    const uint64_t avail = cap_w32 > 2 * woff ? cap_w32 - 2 * woff : 0;
    const uint64_t limit = 2 * nw < avail ? 2 * nw : avail;
    const uint64_t count = limit < nwb ? limit : nwb;
    for (uint32_t q = lane; q < count; q += 64) gdst[q] = w32[q];
  }
}

// The one-pass encoder for partitions of at most 64 kR values: one
// wavefront per partition, no workgroup barrier.  Values in
// registers, model by wavefront shuffles, word count published, residuals
// packed in the wavefront's LDS slice, look-back, record and words written.
template <int kR>
__global__ __launch_bounds__(kEncBlock) void k_encode_fused_wave(
    const EncColumn* __restrict__ cols, uint64_t ncols, EncColumn single, uint64_t nparts,
    EncScratch scr, uint32_t polls, int* err) {
  __shared__ uint32_t words[kEncWaves][2 * 64 * kR];
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint64_t P = uint64_t(blockIdx.x) * kEncWaves + wave;
  if (P >= nparts) return;
  const EncColumn c = column_of(cols, ncols, single, P);
  uint64_t start, len;
  const uint64_t j = P - c.part_base;
  part_bounds(c, j, start, len);
  if (len > 64 * kR) {  // the host sends such launches to the two passes
    if (lane == 0) raise(err, kErrDevice);
    return;
  }
  by_length<kR, kShortRegs>(len, [&](auto r) __attribute__((always_inline)) {
    encode_fused_wave<r.n>(c, P, j, start, len, scr, polls, words[wave], err);
  });
}

uint64_t encode_scratch_bytes(uint64_t nparts) {
  const uint64_t k = nparts ? nparts : 1;
  const uint64_t ng = (k + kScanItems - 1) / kScanItems;
  return 8 * (6 * k + ng + 1) + 8 * k + 64;
}

EncScratch carve_encode_scratch(void* p, uint64_t nparts) {
  const uint64_t k = nparts ? nparts : 1;
  const uint64_t ng = (k + kScanItems - 1) / kScanItems;
  uint64_t* q = static_cast<uint64_t*>(p);
  EncScratch s;
  s.nwords = q;
  s.woff = q + k;
  s.base = q + 2 * k;
  s.theta = q + 3 * k;
  s.bsum = q + 4 * k;
  s.c2 = q + 4 * k + ng + 1;
  s.c3 = q + 5 * k + ng + 1;
  s.bits = reinterpret_cast<uint32_t*>(q + 6 * k + ng + 1);
  s.kind = s.bits + k;
  return s;
}

hipError_t launch_fit_columns(leco_ctx* ctx, const EncColumn* cols_dev, uint64_t ncols,
                              const EncColumn& single, uint64_t nparts, uint64_t max_len,
                              uint32_t regs, const EncScratch& scr, hipStream_t stream) {
  if (nparts == 0) return hipSuccess;
  // each fit kernel fits the columns of its regressors and skips the others
  const uint64_t pw = (nparts + kEncWaves - 1) / kEncWaves;
  // one wavefront per partition: 16 values per lane up to 1024 values, 32
  // up to 2048
  const bool wave16 = max_len <= kWaveEncMax && ctx->tune.encode_wave;
  const bool wave32 =
      max_len <= 2 * kWaveEncMax && ctx->tune.encode_wave && ctx->tune.encode_wave32;
  if ((regs & kRegPoly) && wave16)
    hipLaunchKernelGGL(k_fit_poly_wave<kWaveRegs>, dim3(uint32_t(pw)), dim3(kEncBlock), 0, stream,
                       cols_dev, ncols, single, nparts, scr, ctx->err_dev);
  else if ((regs & kRegPoly) && wave32)
    hipLaunchKernelGGL(k_fit_poly_wave<2 * kWaveRegs>, dim3(uint32_t(pw)), dim3(kEncBlock), 0,
                       stream, cols_dev, ncols, single, nparts, scr, ctx->err_dev);
  else if (regs & kRegPoly)
    hipLaunchKernelGGL(k_fit_poly, dim3(uint32_t(nparts)), dim3(kEncBlock), 0, stream, cols_dev,
                       ncols, single, nparts, scr);
  if (!(regs & (kRegLS | kRegMinimax))) return hipGetLastError();
  if (regs == kRegLS && max_len <= kLaneFitMax && ctx->tune.encode_wave) {
    const uint64_t g = (nparts + 255) / 256, cap = uint64_t(ctx->num_cus) * 16;
    hipLaunchKernelGGL(k_fit_lane, dim3(uint32_t(g < cap ? g : cap)), dim3(256), 0, stream,
                       cols_dev, ncols, single, nparts, scr);
    return hipGetLastError();
  }
  // k_fit_wave fits every column it is given: not with polynomial columns
  const bool poly = regs & kRegPoly;
  if ((regs & kRegMinimax) && wave16 && !poly)
    hipLaunchKernelGGL(k_fit_minimax_wave<kWaveRegs>, dim3(uint32_t(pw)), dim3(kEncBlock), 0,
                       stream, cols_dev, ncols, single, nparts, scr, ctx->err_dev);
  else if ((regs & kRegMinimax) && wave32 && !poly)
    hipLaunchKernelGGL(k_fit_minimax_wave<2 * kWaveRegs>, dim3(uint32_t(pw)), dim3(kEncBlock), 0,
                       stream, cols_dev, ncols, single, nparts, scr, ctx->err_dev);
  else if (regs & kRegMinimax)
    hipLaunchKernelGGL(k_fit_minimax, dim3(uint32_t(nparts)), dim3(kEncBlock), 0, stream, cols_dev,
                       ncols, single, nparts, scr, ctx->err_dev);
  else if (wave16 && !poly)
    hipLaunchKernelGGL(k_fit_wave<kWaveRegs>, dim3(uint32_t(pw)), dim3(kEncBlock), 0, stream,
                       cols_dev, ncols, single, nparts, scr, ctx->err_dev);
  else if (wave32 && !poly)
    hipLaunchKernelGGL(k_fit_wave<2 * kWaveRegs>, dim3(uint32_t(pw)), dim3(kEncBlock), 0, stream,
                       cols_dev, ncols, single, nparts, scr, ctx->err_dev);
  else
    hipLaunchKernelGGL(k_fit_block, dim3(uint32_t(nparts)), dim3(kEncBlock), 0, stream, cols_dev,
                       ncols, single, nparts, scr);
  return hipGetLastError();
}

hipError_t launch_encode_columns(leco_ctx* ctx, const EncColumn* cols_dev, uint64_t ncols,
                                 const EncColumn& single, uint64_t nparts, uint64_t max_len,
                                 uint32_t regs, const EncScratch& scr, hipStream_t stream) {
  const bool wave_fit = max_len <= kWaveEncMax ||
                        (max_len <= 2 * kWaveEncMax && ctx->tune.encode_wave32);
  const uint64_t pw = (nparts + kEncWaves - 1) / kEncWaves;
  const auto fused = [&](uint32_t mode, uint64_t workgroups, uint64_t per_cu) {
    return mode == 1 || (mode == 2 && workgroups <= per_cu * ctx->num_cus);
  };
  const bool one_pass_wave = nparts != 0 && regs == kRegLS && ctx->tune.encode_wave &&
                             max_len <= kWaveEncMax && fused(ctx->tune.encode_fused_wave, pw, kFusedWavePerCu);
  // One read of the column instead of two pays where the workgroups' registers
  // are full: 1e8 u64 values in partitions of 4096 288 us for 333, of 4000 305
  // for 332, of 3500 340 for 323; u32 values 250 for 229.  Whatever they span:
  // 5e7 values in 4096s of range 2^40 231 us for 338, full-width ones 202 for
  // 243.  Of tables and variable starts the host knows only the longest
  // partition, not how many are as full: two passes (1e8 values in 512 columns
  // of 4096s 389 us, 294 in one pass, and in variable ones 350 and 312).
  const bool full = cols_dev == nullptr && single.dtype == 8 && single.fixed_len > kFusedFullLen;
  const bool one_pass = nparts != 0 && regs == kRegLS && !one_pass_wave &&
                        max_len <= kEncRegLen && !(wave_fit && ctx->tune.encode_wave) &&
                        (fused(ctx->tune.encode_fused, nparts, kFusedPerCu) ||
                         (full && ctx->tune.encode_fused == 2));
  if (one_pass_wave || one_pass) {
    const uint64_t items = nparts > ncols ? nparts : ncols;
    const uint64_t g = (items + 255) / 256;
    hipLaunchKernelGGL(k_fused_prepare, dim3(uint32_t(g < 4096 ? g : 4096)), dim3(256), 0, stream,
                       cols_dev, ncols, single, scr, nparts, ctx->err_dev);
    if (one_pass_wave)
      hipLaunchKernelGGL(k_encode_fused_wave<kWaveRegs>, dim3(uint32_t(pw)), dim3(kEncBlock), 0,
                         stream, cols_dev, ncols, single, nparts, scr, ctx->tune.lookback_polls,
                         ctx->err_dev);
    else
      hipLaunchKernelGGL(k_encode_fused, dim3(uint32_t(nparts)), dim3(kEncBlock), 0, stream,
                         cols_dev, ncols, single, nparts, scr, ctx->tune.lookback_polls,
                         ctx->err_dev);
    return hipGetLastError();
  }
  if (nparts != 0) {
    const hipError_t e = launch_fit_columns(ctx, cols_dev, ncols, single, nparts, max_len, regs,
                                            scr, stream);
    if (e != hipSuccess) return e;
  }
  const bool wave = max_len <= kWaveEncMax && ctx->tune.encode_wave;  // pack only
  const uint64_t ng = (nparts + kScanItems - 1) / kScanItems;
  // Every workgroup of k_layout sums what lies before it: the counts of up to
  // kLayoutDirect groups (256 KB at most, about 2 us) in less time than the
  // launch that sums them first (5 us), the sums of up to kLayoutGroups
  // groups (32 KB at most) in less than the launch that scans those.
  const uint32_t mode = ng <= kLayoutDirect   ? kLayoutCounts
                        : ng <= kLayoutGroups ? kLayoutSums
                                              : kLayoutPrefix;
  if (mode != kLayoutCounts)
    hipLaunchKernelGGL(k_scan_sums, dim3(uint32_t(ng)), dim3(kEncBlock), 0, stream, scr, nparts);
  if (mode == kLayoutPrefix)
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(kScanItems), 0, stream, scr, ng);
  uint64_t lg = (ncols + kEncBlock - 1) / kEncBlock;
  lg = lg < 1 ? 1 : (lg > 1024 ? 1024 : lg);
  lg = ng > lg ? ng : lg;
  if (lg <= 2 * uint64_t(ctx->num_cus))
    hipLaunchKernelGGL(k_layout<kScanItems>, dim3(uint32_t(lg)), dim3(kScanItems), 0, stream,
                       cols_dev, ncols, single, nparts, scr, mode, ctx->err_dev);
  else
    hipLaunchKernelGGL(k_layout<kEncBlock>, dim3(uint32_t(lg)), dim3(kEncBlock), 0, stream,
                       cols_dev, ncols, single, nparts, scr, mode, ctx->err_dev);
  if (nparts == 0) return hipGetLastError();
  // Several short partitions to a wavefront once that leaves a wavefront for
  // every SIMD, or four where few share one: 1e6 u32 values in partitions of
  // 64 25.7 us, so 22.3, of 128 18.5 and 17.6, but of 256 15.3 and 15.5 (5e7
  // values: 605 and 374, 317 and 225, 188 and 153).
  const uint64_t per = single.fixed_len ? kPackShortValues / single.fixed_len : 0;
  const uint64_t waves = uint64_t(ctx->num_cus) * (single.fixed_len <= 128 ? 4 : 16);
  // Two whole batches of rounds to a partition of 8-byte values: without the
  // code of smaller ones (2e8 values 635-640 -> 613 us, 1e8 within noise).
  // u32 values (426 -> 437), one batch (u64 L 512 359 -> 368) and partly filled
  // ones (L 800 336 -> 344) are better with it.
  const uint64_t rounds = (single.fixed_len + 63) / 64;
  const bool tails = cols_dev != nullptr || single.dtype != 8 || rounds <= kPackBatch || rounds % kPackBatch != 0;
  if (wave && cols_dev == nullptr && single.fixed_len >= kPackShortMin &&
      single.fixed_len <= kPackShortMax && nparts >= per * waves)
    hipLaunchKernelGGL(k_pack_short, dim3(uint32_t((nparts + per * kEncWaves - 1) / (per * kEncWaves))),
                       dim3(kEncBlock), 0, stream, single, nparts, uint32_t(per),
                       uint32_t((1u << 20) / single.fixed_len + 1), scr);
  else if (wave && tails)
    hipLaunchKernelGGL((k_pack<true, true>), dim3(uint32_t(pw)), dim3(kEncBlock), 0, stream, cols_dev,
                       ncols, single, nparts, scr);
  else if (wave)
    hipLaunchKernelGGL((k_pack<true, false>), dim3(uint32_t(pw)), dim3(kEncBlock), 0, stream, cols_dev,
                       ncols, single, nparts, scr);
  else
    hipLaunchKernelGGL((k_pack<false, true>), dim3(uint32_t(nparts)), dim3(kEncBlock), 0, stream, cols_dev,
                       ncols, single, nparts, scr);
  return hipGetLastError();
}

// ---- sampled cost of a partitioning -------------------------------------------------

// *out += sum over P < nparts of 32 + 8 * nwords[P]: the record and word
// bytes the fitted partitions add to a blob.
__global__ __launch_bounds__(kEncBlock) void k_cost_sum(EncScratch scr, uint64_t nparts,
                                                       uint64_t extra, unsigned long long* out) {
  __shared__ uint64_t part[kEncWaves];
  uint64_t x = 0;
  const uint64_t stride = uint64_t(gridDim.x) * kEncBlock;
  for (uint64_t P = uint64_t(blockIdx.x) * kEncBlock + threadIdx.x; P < nparts; P += stride)
    x += kRecordBytes + extra + 8 * scr.nwords[P];
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) x += shfl_xor64(x, m);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t t = 0;
    for (int w = 0; w < kEncWaves; ++w) t += part[w];
    atomicAdd(out, static_cast<unsigned long long>(t));
  }
}

hipError_t launch_cost_sum(const EncScratch& scr, uint64_t nparts, uint64_t extra_per_part,
                           uint64_t* out, hipStream_t stream) {
  uint64_t blocks = (nparts + kEncBlock - 1) / kEncBlock;
  blocks = blocks < 1 ? 1 : (blocks > 2048 ? 2048 : blocks);
  hipLaunchKernelGGL(k_cost_sum, dim3(uint32_t(blocks)), dim3(kEncBlock), 0, stream, scr, nparts,
                     extra_per_part, reinterpret_cast<unsigned long long*>(out));
  return hipGetLastError();
}

// ---- diagnostics --------------------------------------------------------------

__global__ void k_diag_slope(const uint64_t* __restrict__ in, uint64_t k, double* __restrict__ out) {
  const uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= k) return;
  const U128 N{in[4 * i], in[4 * i + 1]};
  const U128 D{in[4 * i + 2], in[4 * i + 3]};
  double s = i128_to_f64(N) / u128_to_f64(D);
  if (s == 0.0) s = 0.0;
  out[i] = s;
}

hipError_t launch_diag_slope(const uint64_t* in, uint64_t k, double* out, hipStream_t stream) {
  if (k == 0) return hipSuccess;
  hipLaunchKernelGGL(k_diag_slope, dim3(uint32_t((k + 255) / 256)), dim3(256), 0, stream, in, k, out);
  return hipGetLastError();
}

}  // namespace leco
