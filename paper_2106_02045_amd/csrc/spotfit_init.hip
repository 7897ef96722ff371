// spotfit_init.hip -- start values on the device.  The paper takes start
// values as given and leaves them out of its timings (Results section); these
// passes let raw frames go in and fits come out without a host round trip.
//
// The centroid / second-moment estimate (its recipe with the device function
// in spotfit_start.h), and the recipe the paper gives for its accuracy runs
// (Results section): centre = brightest pixel of the 3 x 3 moving average,
// sigma = sqrt(M / pi) with M the pixels above alpha0 exp(-1/2) + beta0.
//
// 16-bit pixels: a lane per row, integer arithmetic (below).  Float pixels: a
// group of L lanes per spot, lane l owning the columns l + L*j, the groups
// stepping over the spots with a grid stride.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "lanegroup.h"
#include "spotfit.h"
#include "spotfit_internal.h"
#include "spotfit_start.h"

namespace sf {
namespace ini {

using namespace lg;

template <int L, int CPL>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void moment_init_kernel(const float* data,
                                                         const spotfit_shape_t* sizes,
                                                         const int64_t* offsets, int64_t n,
                                                         int max_side, int max_pixels,
                                                         float* out) {
  const int lane = __lane_id();
  const int li = lane % L;
  const int64_t stride = (int64_t)gridDim.x * (64 / L);
  // s is the same on every lane of a group, so groups stay whole in the loop
  for (int64_t s = (int64_t)blockIdx.x * (64 / L) + lane / L; s < n; s += stride) {
    const spotfit_shape_t sh = sizes[s];
    if (!usable<L * CPL>(sh, max_side, max_pixels)) {
      if (li == 0) write_nan(out, s);
      continue;
    }
    float o[4];
    moment_init_spot<L, CPL>(data, SPOTFIT_F32, sh, offsets[s], li, o);
    if (li == 0)
      for (int q = 0; q < 4; ++q) out[4 * s + q] = o[q];
  }
}

constexpr double kExpMinusHalf = 0x1.368b2fc6f960ap-1;  // e^(-1/2), correctly rounded
constexpr double kPi = 0x1.921fb54442d18p+1;

// ---------------------------------------------------------------------------
// 16-bit pixels: a group of L lanes per spot, lane r holding row r (w, h <= L),
// two pixels to a register.  Everything up to the last few operations is exact
// integer arithmetic, so the order of the sums does not matter and the values
// are those of the streamed kernels above and below.  A wavefront takes up to 64
// spots: their totals go to LDS, and then one lane per spot forms its start
// values, so that the divisions and square roots are shared by 64 spots.
// ---------------------------------------------------------------------------

// A row as read: windows of 4 pixels, each two registers; zeros past column w.
template <int W>
struct Row {
  uint32_t v[2 * W];
};

// Row r of a spot (zeros for r >= h).  A window that would read past the spot's
// end starts earlier; its pixels and the end of the row are shifted into place.
template <int W>
__device__ __forceinline__ void load_row(const uint16_t* px, int w, int h, int r, Row<W>& row) {
  typedef uint32_t vec __attribute__((ext_vector_type(2), aligned(2)));
  const int n = w * h, cols = r < h ? w : 0, first = r < h ? r * w : 0;
  uint64_t t[W];
#pragma unroll
  for (int q = 0; q < W; ++q) {
    const int p = first + 4 * q < n - 4 ? first + 4 * q : n - 4;
    const vec u = *reinterpret_cast<const vec*>(px + p);
    t[q] = (uint64_t)u[1] << 32 | u[0];
  }
#pragma unroll
  for (int q = 0; q < W; ++q) {
    int keep = cols - 4 * q;  // pixels of the row in this window
    keep = keep > 4 ? 4 : keep;
    const int p = first + 4 * q < n - 4 ? first + 4 * q : n - 4;
    const int late = first + 4 * q - p;  // they begin `late` pixels in: keep + late <= 4
    uint64_t x = t[q] << ((64 - 16 * (keep + late)) & 63);
    x = x >> ((64 - 16 * keep) & 63);
    row.v[2 * q] = keep > 0 ? (uint32_t)x : 0u;
    row.v[2 * q + 1] = keep > 0 ? (uint32_t)(x >> 32) : 0u;
  }
}

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
// Per half: max(a - b, 0).
__device__ __forceinline__ uint32_t sub_sat(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2, a),
                                                                    __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ uint32_t min2(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, a),
                                                                __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ uint32_t max2(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a),
                                                                __builtin_bit_cast(u16x2, b)));
}
// acc + a.lo b.lo + a.hi b.hi
__device__ __forceinline__ uint32_t dot2(uint32_t a, uint32_t b, uint32_t acc) {
  return __builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b), acc, false);
}

template <int L>
__device__ __forceinline__ uint32_t gmax_u(uint32_t v) {
  return ~gmin_u<L>(~v);
}

// The two middle values of the border ring (2 (w + h - 2) pixels, every lane of
// the group returns them): a select bit by bit, from the highest bit in which the
// ring's values differ anywhere in the wavefront.
template <int L>
__device__ __forceinline__ void ring_middle(const uint16_t* px, int w, int h, int r, uint32_t first,
                                            uint32_t& v1, uint32_t& v2) {
  const uint32_t none = 0xffffffffu;
  const bool col = r < w, side = r >= 1 && r < h - 1;
  // lane r: top and bottom pixel of column r, left and right pixel of row r
  uint32_t key[4];
  const int rc = col ? r : 0, rr = side ? r : 0;
  key[0] = px[rc];
  key[1] = px[(h - 1) * w + rc];
  key[2] = first;
  key[3] = px[rr * w + w - 1];
  key[0] = col ? key[0] : none;
  key[1] = col ? key[1] : none;
  key[2] = side ? key[2] : none;
  key[3] = side ? key[3] : none;
  const int k1 = w + h - 3;  // the middle order statistics: k1 and k1 + 1
  uint32_t lo = none, hi = 0;
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    lo = key[m] < lo ? key[m] : lo;
    const uint32_t t = key[m] == none ? 0u : key[m];
    hi = t > hi ? t : hi;
  }
  lo = gmin_u<L>(lo);
  hi = gmax_u<L>(hi);
  const uint32_t span = hi - lo;
  uint32_t v = lo;
#pragma unroll
  for (int bit = 15; bit >= 0; --bit) {
    if (__builtin_amdgcn_ballot_w64((span >> bit) != 0) == 0) continue;
    const uint32_t c = v + (1u << bit);
    int cnt = 0;
#pragma unroll
    for (int m = 0; m < 4; ++m) cnt += key[m] < c ? 1 : 0;
    cnt = gsum_i<L>(cnt);
    v = cnt <= k1 ? c : v;
  }
  int le = 0;
  uint32_t above = none;
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    le += key[m] <= v ? 1 : 0;
    above = key[m] > v && key[m] < above ? key[m] : above;
  }
  le = gsum_i<L>(le);
  above = gmin_u<L>(above);
  v1 = v;
  v2 = le >= k1 + 2 ? v : above;
}

// The spots of a wavefront, up to 64 from `base` on, their descriptions one per
// lane, and the usable ones in the order in which they are gone through: by the
// lanes that their rows (and, for the moments, whose ring has a lane per column too,
// their columns) take: 8, 16 or 32, whatever sides the launch is for.  100,000 spots of 9x9 with the default options (sides up to 32): moments 45.8
// us with groups of 16 lanes and two columns each, 57.6 with 32 lanes for every
// spot, 23.2 so; brightest-pixel values 24.3, 74.6 and 20.6 (of 7..16 px 20.8 instead
// of 75; of 17..32 px as before).
struct Batch {
  spotfit_shape_t sh;  // of spot `base + lane`
  int64_t off;
  bool ok;
  int cls;       // its class
  int first[4];  // class c (8 << c lanes) is order[first[c]] .. order[first[c + 1] - 1]
};

// Fills the batch for a kernel of up to LMAX lanes per spot; order: 64 words of LDS.
// ROWS: by the rows alone.
template <int LMAX, bool ROWS>
__device__ __forceinline__ Batch take_batch(const spotfit_shape_t* sizes, const int64_t* offsets, int64_t base,
                                            int count, int max_side, int max_pixels, int* order) {
  const int lane = __lane_id();
  Batch b{};
  if (lane < count) {
    b.sh = sizes[base + lane];
    b.off = offsets[base + lane];
  }
  b.ok = lane < count && usable<LMAX>(b.sh, max_side, max_pixels);
  const int side = !ROWS && b.sh.w > b.sh.h ? b.sh.w : b.sh.h;
  uint64_t m[3];  // the lanes of each class
  m[0] = __builtin_amdgcn_ballot_w64(b.ok && side <= 8);
  m[1] = __builtin_amdgcn_ballot_w64(b.ok && side > 8 && side <= 16);
  m[2] = __builtin_amdgcn_ballot_w64(b.ok && side > 16);
  // a few small spots among larger ones go along with those where that takes no
  // more rounds
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    if ((16 << c) > LMAX) continue;
    const int some = __builtin_popcountll(m[c]), more = __builtin_popcountll(m[c + 1]), G = 4 >> c;
    if ((some + more + G - 1) / G <= (some + 2 * G - 1) / (2 * G) + (more + G - 1) / G) {
      m[c + 1] |= m[c];
      m[c] = 0;
    }
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    if (m[c] >> lane & 1) b.cls = c;
    if (m[c] >> lane & 1)
      order[b.first[c] + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m[c] >> 32),
                                                        __builtin_amdgcn_mbcnt_lo((uint32_t)m[c], 0u))] = lane;
    b.first[c + 1] = b.first[c] + (int)__builtin_popcountll(m[c]);
  }
  __syncthreads();
  return b;
}

__device__ __forceinline__ int pick(int v, int lane) { return __builtin_amdgcn_ds_bpermute(lane << 2, v); }

// f(windows, from, valid, w, h, pixels) for the spots of the batch that take L
// lanes, 64 / L at a time: `from` the lane that describes the spot of this lane's
// group (the last one again where there are no more: not valid).  Rows are gone
// through in L / 4 windows of 4 columns, or LMAX / 4 where a spot has more columns
// than L; with 32 lanes in 6 where no spot has more than 24 columns, 58 us instead
// of 75 for the brightest-pixel values of 100,000 spots of 17x17.  Of 30x12 (w x h),
// by their larger side 73 us, by their rows 36 (54 before the row kernels).
template <int L, int LMAX, typename F>
__device__ __forceinline__ void for_spots(const Batch& b, const uint16_t* data, const int* order, F&& f) {
  constexpr int C = L == 8 ? 0 : L == 16 ? 1 : 2, G = 64 / L;
  const int begin = b.first[C], end = b.first[C + 1];
  if (begin == end) return;
  const int g = __lane_id() / L;
  const int2 o2 = __builtin_bit_cast(int2, b.off);
  const int whs = b.sh.w | b.sh.h << 8;
  auto go = [&](auto windows) {
#pragma unroll 1
    for (int i = begin; i < end; i += G) {
      const int from = order[i + g < end ? i + g : end - 1];
      const int wh = pick(whs, from);
      const int64_t o = __builtin_bit_cast(int64_t, make_int2(pick(o2.x, from), pick(o2.y, from)));
      f(windows, from, i + g < end, wh & 0xff, wh >> 8, data + o);
    }
  };
  auto wider = [&](int w) { return __builtin_amdgcn_ballot_w64(b.ok && b.cls == C && b.sh.w > w) != 0; };
  if constexpr (L == 32) {
    if (!wider(24)) return go(std::integral_constant<int, 6>{});
  } else if constexpr (LMAX > L) {
    if (wider(L)) return go(std::integral_constant<int, LMAX / 4>{});
  }
  go(std::integral_constant<int, L / 4>{});
}

// Start values from the moments of max(g - b0, 0), b0 the mean of the ring's
// middle values v1, v2: 2 max(g - b0, 0) = max(g - floor b0, 0) + max(g - ceil
// b0, 0), so all sums are integers.  Per spot ~85 vector instructions at 16
// rows (~35 of them the ring's select), against ~250 with every pixel read as a
// value of its own and four lanes repeating the spot's last steps: 1M spots of
// 15x15 in 0.196 ms instead of 0.50, of 32x32 in 0.60 instead of 1.19.
template <int L>
__device__ __forceinline__ void moment_rows(const Batch& b, const uint16_t* data, const int* order, double* sxx,
                                            double* syy, uint32_t* s0, uint32_t* sx, uint32_t* sy) {
  const int r = __lane_id() % L;
  for_spots<L, L>(b, data, order, [&](auto windows, int from, bool valid, int w, int h, const uint16_t* px) {
    constexpr int W = decltype(windows)::value;
    Row<W> row;
    load_row<W>(px, w, h, r, row);
    uint32_t v1, v2;
    ring_middle<L>(px, w, h, r, row.v[0] & 0xffffu, v1, v2);
    const uint32_t k0 = (v1 + v2) >> 1, k1 = (v1 + v2 + 1) >> 1;
    const uint32_t b0 = k0 | k0 << 16, b1 = k1 | k1 << 16;
    uint32_t a0 = 0, a1 = 0, a2 = 0;  // the row's sums of 2 wt, 2 wt c, 2 wt c^2 (below 2^31)
#pragma unroll
    for (int p = 0; p < 2 * W; ++p) {
      const uint32_t c = 2 * p, one = 0x10001u, lin = c | (c + 1) << 16, sq = c * c | (c + 1) * (c + 1) << 16;
      const uint32_t d = sub_sat(row.v[p], b0), e = sub_sat(row.v[p], b1);
      a0 = dot2(e, one, dot2(d, one, a0));
      a1 = dot2(e, lin, dot2(d, lin, a1));
      a2 = dot2(e, sq, dot2(d, sq, a2));
    }
    const double yy = gsum<L>(double(a0) * double(r * r)), xx = gsum<L>(double(a2));
    const uint32_t t0 = (uint32_t)gsum_i<L>((int)a0), t1 = (uint32_t)gsum_i<L>((int)a1);
    const uint32_t ty = (uint32_t)gsum_i<L>((int)(a0 * (uint32_t)r));
    if (r == 0 && valid) {
      sxx[from] = xx;
      syy[from] = yy;
      s0[from] = t0;
      sx[from] = t1;
      sy[from] = ty;
    }
  });
}

template <int LMAX>
__global__ __launch_bounds__(64) void moment_rows_kernel(const uint16_t* data, const spotfit_shape_t* sizes,
                                                         const int64_t* offsets, int64_t n, int per_block,
                                                         int max_side, int max_pixels, float* out) {
  __shared__ double sxx[64], syy[64];
  __shared__ uint32_t s0[64], sx[64], sy[64];
  __shared__ int order[64];
  const int lane = __lane_id();
  const int64_t base = (int64_t)blockIdx.x * per_block;
  const int count = n - base < per_block ? (int)(n - base) : per_block;
  const Batch b = take_batch<LMAX, false>(sizes, offsets, base, count, max_side, max_pixels, order);
  const spotfit_shape_t sh = b.sh;
  const bool ok = b.ok;
  moment_rows<8>(b, data, order, sxx, syy, s0, sx, sy);
  if constexpr (LMAX >= 16) moment_rows<16>(b, data, order, sxx, syy, s0, sx, sy);
  if constexpr (LMAX >= 32) moment_rows<32>(b, data, order, sxx, syy, s0, sx, sy);
  __syncthreads();
  if (lane < count) {
    float o[4];
    const float nanf = __builtin_nanf("");
    o[0] = o[1] = o[2] = o[3] = nanf;
    if (ok) {
      // about the ROI centre (w1 / 2, h1 / 2), exactly: the sums are of 2 wt
      const double t = s0[lane], w1 = sh.w - 1, h1 = sh.h - 1;
      const double x = sx[lane], y = sy[lane];
      const double swx = 0.25 * (2.0 * x - w1 * t), swy = 0.25 * (2.0 * y - h1 * t);
      const double swxx = 0.125 * (4.0 * sxx[lane] - 4.0 * w1 * x + w1 * w1 * t);
      const double swyy = 0.125 * (4.0 * syy[lane] - 4.0 * h1 * y + h1 * h1 * t);
      moment_values<1>(0.5 * t, swx, swy, swxx, swyy, sh, o);
    }
    float4* dst = reinterpret_cast<float4*>(out) + (base + lane);
    if ((reinterpret_cast<uintptr_t>(out) & 15) == 0) {
      *dst = make_float4(o[0], o[1], o[2], o[3]);
    } else {
      for (int q = 0; q < 4; ++q) out[4 * (base + lane) + q] = o[q];
    }
  }
}

// The paper's start values of 16-bit pixels, rows as above.  A window's sum is
// an integer and its pixel count 4, 6 or 9, so its mean times 36 is an integer
// (below 2^23) and orders the windows exactly, ties included, as the correctly
// rounded quotients do; with 31 - column below it, a row's largest such number is
// its first brightest window.  Measured: 1M spots of 15x15 in 0.188 ms instead
// of 0.79, of 32x32 in 0.67 instead of 1.50.
template <int L, int LMAX>
__device__ __forceinline__ void peak_rows(const Batch& b, const uint16_t* data, const int* order,
                                          uint32_t* where, uint32_t* area) {
  const int r = __lane_id() % L;
  for_spots<L, LMAX>(b, data, order, [&](auto windows, int from, bool valid, int w, int h, const uint16_t* px) {
    constexpr int W = decltype(windows)::value;
    Row<W> row;
    load_row<W>(px, w, h, r, row);
    // 36 / (rows x columns of the window), for inner and for edge columns
    const bool row_edge = r == 0 || r == h - 1;
    const uint32_t inner = r < h ? (row_edge ? 6u * 32 : 4u * 32) : 0u;
    const uint32_t edge = r < h ? (row_edge ? 9u * 32 : 6u * 32) : 0u;
    uint32_t best = 0, left = 0, mid = row.v[0] & 0xffffu;
    uint32_t hi2 = 0, lo2 = 0xffffffffu;
#pragma unroll
    for (int c = 0; c < 4 * W; ++c) {
      const uint32_t right = c + 1 < 4 * W ? (c & 1 ? row.v[(c + 1) / 2 < 2 * W ? (c + 1) / 2 : 0] & 0xffffu
                                                    : row.v[c / 2] >> 16)
                                           : 0u;
      const uint32_t across = left + mid + right;
      uint32_t up, down;
      if constexpr (L == 16) {  // a group is a DPP row: zeros come in at its ends
        up = (uint32_t)dpp_i<0x111>((int)across);    // row_shr:1
        down = (uint32_t)dpp_i<0x101>((int)across);  // row_shl:1
      } else {
        up = (uint32_t)dpp_i<0x138>((int)across);    // wave_shr:1
        down = (uint32_t)dpp_i<0x130>((int)across);  // wave_shl:1
        up = r == 0 ? 0u : up;
        down = r == L - 1 ? 0u : down;
      }
      const uint32_t mult = c == 0 ? edge : c < w - 1 ? inner : c == w - 1 ? edge : 0u;
      const uint32_t key = (across + up + down) * mult + uint32_t(31 - c);
      best = key > best ? key : best;
      left = mid;
      mid = right;
    }
    // smallest and largest pixel of the row
#pragma unroll
    for (int p = 0; p < 2 * W; ++p) {
      hi2 = max2(hi2, row.v[p]);
      const uint32_t past = 2 * p >= w ? 0xffffffffu : 2 * p + 1 >= w ? 0xffff0000u : 0u;
      lo2 = min2(lo2, row.v[p] | past);
    }
    uint32_t hi = (hi2 & 0xffffu) > hi2 >> 16 ? hi2 & 0xffffu : hi2 >> 16;
    uint32_t lo = (lo2 & 0xffffu) < lo2 >> 16 ? lo2 & 0xffffu : lo2 >> 16;
    lo = r < h ? lo : 0xffffu;
    hi = gmax_u<L>(hi);
    lo = gmin_u<L>(lo);
    // the group's brightest window: the first row among the largest means
    const uint32_t mean = best >> 5, top = gmax_u<L>(mean);
    const uint32_t at = gmin_u<L>(mean == top && r < h ? uint32_t(r) << 5 | (31u - (best & 31u)) : 0xffffffffu);
    const double thr = __builtin_fma(double(hi) - double(lo), kExpMinusHalf, double(lo));
    // g > thr is g > floor(thr): count max(g - floor(thr), 0) != 0
    const uint32_t f = (uint32_t)thr, f2 = f | f << 16;
    uint32_t m = 0;
#pragma unroll
    for (int p = 0; p < 2 * W; ++p) m = dot2(min2(sub_sat(row.v[p], f2), 0x10001u), 0x10001u, m);
    m = (uint32_t)gsum_i<L>((int)m);
    if (r == 0 && valid) {
      where[from] = at;
      area[from] = m;
    }
  });
}

template <int LMAX>
__global__ __launch_bounds__(64) void peak_rows_kernel(const uint16_t* data, const spotfit_shape_t* sizes,
                                                       const int64_t* offsets, int64_t n, int per_block,
                                                       int max_side, int max_pixels, float* out) {
  __shared__ uint32_t where[64], area[64];
  __shared__ int order[64];
  const int lane = __lane_id();
  const int64_t base = (int64_t)blockIdx.x * per_block;
  const int count = n - base < per_block ? (int)(n - base) : per_block;
  const Batch b = take_batch<LMAX, true>(sizes, offsets, base, count, max_side, max_pixels, order);
  const bool ok = b.ok;
  peak_rows<8, LMAX>(b, data, order, where, area);
  if constexpr (LMAX >= 16) peak_rows<16, LMAX>(b, data, order, where, area);
  if constexpr (LMAX >= 32) peak_rows<32, LMAX>(b, data, order, where, area);
  __syncthreads();
  if (lane < count) {
    const float nanf = __builtin_nanf("");
    float4 v = make_float4(nanf, nanf, nanf, nanf);
    if (ok) {
      double sig = sqrt(double(area[lane]) / kPi);
      sig = sig < 0.5 ? 0.5 : sig;
      v = make_float4(float(where[lane] & 31u), float(where[lane] >> 5), float(sig), float(sig));
    }
    float* dst = out + 4 * (base + lane);
    dst[0] = v.x;
    dst[1] = v.y;
    dst[2] = v.z;
    dst[3] = v.w;
  }
}

// ---------------------------------------------------------------------------
// The paper's start values of float pixels.  Per own pixel the 3 x 3 window sum is formed in
// double from the pixel's column and its two neighbours (clamped loads, masked
// outside the ROI) and divided by the number of in-ROI window pixels; the sums
// are exact for pixels within 2^26 of each other, so their order does not matter
// there.  The group keeps the largest mean
// and, among equal means, the smallest row-major index.
// ---------------------------------------------------------------------------
template <int L>
__device__ __forceinline__ double gmax_d(double v) {
  if constexpr (L >= 2) v = fmax(v, dpp_mov<0xB1>(v));
  if constexpr (L >= 4) v = fmax(v, dpp_mov<0x4E>(v));
  if constexpr (L >= 8) v = fmax(v, dpp_mov<0x141>(v));
  if constexpr (L >= 16) v = fmax(v, dpp_mov<0x140>(v));
  return v;
}

template <int L>
__device__ __forceinline__ float gmin_f(float v) {
  if constexpr (L >= 2) v = fminf(v, dpp_mov<0xB1>(v));
  if constexpr (L >= 4) v = fminf(v, dpp_mov<0x4E>(v));
  if constexpr (L >= 8) v = fminf(v, dpp_mov<0x141>(v));
  if constexpr (L >= 16) v = fminf(v, dpp_mov<0x140>(v));
  return v;
}

template <int L>
__device__ __forceinline__ float gmax_f(float v) {
  if constexpr (L >= 2) v = fmaxf(v, dpp_mov<0xB1>(v));
  if constexpr (L >= 4) v = fmaxf(v, dpp_mov<0x4E>(v));
  if constexpr (L >= 8) v = fmaxf(v, dpp_mov<0x141>(v));
  if constexpr (L >= 16) v = fmaxf(v, dpp_mov<0x140>(v));
  return v;
}

template <int L, int CPL>
__global__ __launch_bounds__(64) void peak_init_kernel(const float* data,
                                                       const spotfit_shape_t* sizes,
                                                       const int64_t* offsets, int64_t n,
                                                       int max_side, int max_pixels, float* out) {
  constexpr int HM = L * CPL;
  const int lane = __lane_id();
  const int li = lane % L;
  const int64_t stride = (int64_t)gridDim.x * (64 / L);
  for (int64_t s = (int64_t)blockIdx.x * (64 / L) + lane / L; s < n; s += stride) {
    const spotfit_shape_t sh = sizes[s];
    if (!usable<HM>(sh, max_side, max_pixels)) {
      if (li == 0) write_nan(out, s);
      continue;
    }
    const int w = sh.w, h = sh.h;
    const int64_t off = offsets[s];
    double best = -__builtin_inf();
    int bk = 0x7fffffff;
    float lo = __builtin_inff(), hi = -__builtin_inff();
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      const int c = li + L * j;
      const bool cin = c < w;
      const int cm = c - 1 < 0 ? 0 : (c - 1 < w ? c - 1 : w - 1);
      const int cc = c < w ? c : w - 1;
      const int cp = c + 1 < w ? c + 1 : w - 1;
      float g0[HM], g1[HM], g2[HM];  // columns c - 1, c, c + 1 (clamped)
#pragma unroll
      for (int r = 0; r < HM; ++r) {
        const int64_t row = off + (int64_t)(r < h ? r : h - 1) * w;
        g0[r] = data[row + cm];
        g1[r] = data[row + cc];
        g2[r] = data[row + cp];
      }
      const bool left = c >= 1, right = c + 1 < w;
      const int ncol = 1 + (left ? 1 : 0) + (right ? 1 : 0);
#pragma unroll
      for (int r = 0; r < HM; ++r) {
        if (!(cin && r < h)) continue;
        double acc = 0.0;
        int nrow = 0;
#pragma unroll
        for (int d = -1; d <= 1; ++d) {
          const int rr = r + d;
          if (rr < 0 || rr >= h) continue;
          ++nrow;
          acc += double(g1[rr]);
          if (left) acc += double(g0[rr]);
          if (right) acc += double(g2[rr]);
        }
        const double mean = acc / double(nrow * ncol);
        const int k = r * w + c;
        if (mean > best || (mean == best && k < bk)) {
          best = mean;
          bk = k;
        }
        lo = fminf(lo, g1[r]);
        hi = fmaxf(hi, g1[r]);
      }
    }
    const double top = gmax_d<L>(best);
    bk = (int)gmin_u<L>(best == top ? (uint32_t)bk : 0xFFFFFFFFu);
    lo = gmin_f<L>(lo);
    hi = gmax_f<L>(hi);
    const double beta0 = double(lo), alpha0 = double(hi) - double(lo);
    const double thr = __builtin_fma(alpha0, kExpMinusHalf, beta0);
    int m = 0;
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      const int c = li + L * j;
      if (c >= w) continue;
#pragma unroll
      for (int r = 0; r < HM; ++r)
        if (r < h) m += double(data[off + (int64_t)r * w + c]) > thr ? 1 : 0;
    }
    m = gsum_i<L>(m);
    double sig = sqrt(double(m) / kPi);
    sig = sig < 0.5 ? 0.5 : sig;
    if (li == 0) {
      out[4 * s + 0] = float(bk % w);
      out[4 * s + 1] = float(bk / w);
      out[4 * s + 2] = float(sig);
      out[4 * s + 3] = float(sig);
    }
  }
}

}  // namespace ini

namespace {

template <int L>
hipError_t launch_rows(int method, const uint16_t* data, const spotfit_shape_t* sizes, const int64_t* offsets,
                       int64_t n, int max_side, int max_pixels, float* out, hipStream_t st) {
  // up to 64 spots per wavefront, fewer where that leaves the chip idle (16
  // wavefronts per CU on 256 CUs); a launch takes fewer than 2^32 threads
  int per = 64;
  while (per > 64 / L && n < (int64_t)per * 4096) per /= 2;
  constexpr int64_t kSpots = (int64_t)1 << 30;
  if (n > kSpots) {
    const hipError_t e = launch_rows<L>(method, data, sizes, offsets, kSpots, max_side, max_pixels, out, st);
    return e != hipSuccess ? e
                           : launch_rows<L>(method, data, sizes + kSpots, offsets + kSpots, n - kSpots, max_side,
                                            max_pixels, out + 4 * kSpots, st);
  }
  const int64_t blocks = (n + per - 1) / per;
  if (method == kInitMoments)
    hipLaunchKernelGGL((ini::moment_rows_kernel<L>), dim3((unsigned)blocks), dim3(64), 0, st, data, sizes,
                       offsets, n, per, max_side, max_pixels, out);
  else
    hipLaunchKernelGGL((ini::peak_rows_kernel<L>), dim3((unsigned)blocks), dim3(64), 0, st, data, sizes,
                       offsets, n, per, max_side, max_pixels, out);
  return hipGetLastError();
}

template <int L, int CPL>
hipError_t launch_streamed(int method, const float* data, const spotfit_shape_t* sizes, const int64_t* offsets,
                           int64_t n, int max_side, int max_pixels, float* out, hipStream_t st) {
  int64_t blocks = (n + 64 / L - 1) / (64 / L);
  blocks = blocks < (1 << 20) ? blocks : (1 << 20);  // the kernels stride over the rest
  if (method == kInitMoments)
    hipLaunchKernelGGL((ini::moment_init_kernel<L, CPL>), dim3((unsigned)blocks), dim3(64), 0, st, data,
                       sizes, offsets, n, max_side, max_pixels, out);
  else
    hipLaunchKernelGGL((ini::peak_init_kernel<L, CPL>), dim3((unsigned)blocks), dim3(64), 0, st, data,
                       sizes, offsets, n, max_side, max_pixels, out);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_start_values(int method, const void* data, int dtype, const spotfit_shape_t* sizes,
                               const int64_t* offsets, int64_t n, int max_side, int max_pixels,
                               float* out, hipStream_t st, bool lane_per_column) {
  if (dtype == SPOTFIT_U16) {  // a lane per row
    const uint16_t* px = static_cast<const uint16_t*>(data);
    if (max_side <= 8) return launch_rows<8>(method, px, sizes, offsets, n, max_side, max_pixels, out, st);
    if (max_side <= 16) return launch_rows<16>(method, px, sizes, offsets, n, max_side, max_pixels, out, st);
    return launch_rows<32>(method, px, sizes, offsets, n, max_side, max_pixels, out, st);
  }
  const float* px = static_cast<const float*>(data);
  // a lane per column for the latency hint (raw floats with the fit, us with groups of 4
  // or 16 lanes / so: 32 of 15x15 35.0 / 25.1, of 32x32 37.7 / 33.9; 10,000 of 15x15
  // 51 / 42, 100,000 228 / 194)
  if (lane_per_column && method == kInitMoments) {
    if (max_side <= 8) return launch_streamed<8, 1>(method, px, sizes, offsets, n, max_side, max_pixels, out, st);
    if (max_side <= 16) return launch_streamed<16, 1>(method, px, sizes, offsets, n, max_side, max_pixels, out, st);
    return launch_streamed<32, 1>(method, px, sizes, offsets, n, max_side, max_pixels, out, st);
  }
  // float pixels: groups of 4 lanes (2 or 4 columns each) up to 16 pixels a side, 16 beyond
  if (max_side <= 8) return launch_streamed<4, 2>(method, px, sizes, offsets, n, max_side, max_pixels, out, st);
  if (max_side <= 16) return launch_streamed<4, 4>(method, px, sizes, offsets, n, max_side, max_pixels, out, st);
  return launch_streamed<16, 2>(method, px, sizes, offsets, n, max_side, max_pixels, out, st);
}

}  // namespace sf
