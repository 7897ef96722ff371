// spotfit_matrix.hip -- gfx950 kernel of the batched implicit-amplitude
// Levenberg-Marquardt Gaussian-spot fit, separable form, its pixel sums on the
// matrix cores.
//
// With f(r, c) = ey(r) ex(c) (Eq. 10 and its axis-aligned elliptical form) every
// sum over a spot's pixels that an evaluation needs (Eqs. 5-9) is an entry of
//   R = E^T (G V),   GX = V^T V,   GY = E^T E
// for the spot's pixel matrix G, the column vectors V = [ex, dx ex, dx^2 ex, 1]
// and the row vectors E = [ey, dy ey, dy^2 ey, 1]: products of 4-wide matrices,
// which v_mfma_f64_4x4x4_4b multiplies for four spots at once.  One pass of a
// wavefront evaluates four spots, 16 lanes each; the contraction over columns
// and rows happens inside the matrix instructions, so no lane adds up a total.
//
// Mapping of a pass.  Lane = v + 4 blk + 16 k: block blk is the pass's spot.
//   columns  lane group k owns the T = ceil(w / 4) columns T k .. T k + T - 1,
//            read as windows of 4 pixels (V = 0 for columns that are not its own)
//   rows     lane v reads row 4 a + v of row tile a (a row below the spot reads
//            the last row; its E is 0)
//   A operand of tile (a, b): pixel (4 a + v, column b of group k);
//   B operand: V of that column for vector v.  The product's row i = lane / 16,
//   column j = v is the B layout again, so S = G V feeds E^T S directly.
// The sums of a spot depend on its own shape alone, in the same order whatever
// the batch, the launch shape or the spots beside it: a spot has the same bits
// in every launch of this kernel.
//
// A wavefront holds NS spots, one owned by each of its first NS lanes: a step
// evaluates all of them in passes of four (spots of one shape: new ones first, so
// that the sums of g and g^2 are formed in few passes, and the next pass's pixels
// are loaded as this one's are used; spots of any shapes: by size, so that few
// passes go over the tiles of a large one), then every owner takes its spot's scalar
// steps (Eqs. 6, 8, the normal equations, the damped solve, the decisions of the
// Fit2DGaussian loop) from the totals in LDS.  NS is the launch's trade between
// the length of a step and the lanes that share its scalar part: 4 slots (every
// lane of a block owns its slot; the entries of the normal equations are shared
// out) for the shortest steps, 64 for the least work per spot.
//
// What bounds it: the vector pipe, which the double-precision matrix
// instructions share (a 4x4x4_4b issues every 16 cycles and no vector
// instruction beside it, measured), and, with few wavefronts, the chain of one
// wavefront's own instructions (4.8 cycles each alone, measured).  One pass over
// spots of one shape is 144 vector and 28 matrix instructions at 16x16 px,
// against ~270 for the same four spots in the lane-owned mapping, whose rows each
// cost broadcasts, weights and totals beside their two multiply-adds per pixel;
// at 32x32 px 375 and 88 against ~1050.  With 64 slots the scalar part is a
// quarter of a step.  Measured on one MI355X against the lane-owned, narrow and
// wide mappings these launches took before: 1M spots of 15x15 0.860 ms (1.037),
// 500k of 32x32 1.41 (2.14), 2M of seven sizes from 7 to 32 px in one launch 3.13
// (4.60), 200,000 floats of 17x17 0.584 (0.885), 10,000 of 21x21 0.069 (0.168),
// 10,007 of 7..32 px 0.079 (0.589), 1,024 of 11x11 0.0179 (0.0480).  Passes of
// mixed shapes in straight-line code for their largest spot's tiles, ordered by
// size, against a branch per tile in the order of the slots: 3.20 (3.47) and
// 0.082 (0.110).  Not faster: the next pass's pixels loaded ahead in passes of
// mixed shapes (3.34), 44 or 48 slots at three wavefronts per SIMD (15x15 0.877,
// 0.917), the sums of g and g^2 taken from the products of a new spot's first
// pass (0.870), a solve of three rows for wavefronts without elliptical spots
// (no case moved by more than its runs differ).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

// Nothing is fused that the source does not fuse: the compiler does so only within
// a basic block, which is not the same in every build of the kernel.
#pragma clang fp contract(off)

#include "spotfit.h"
#include "spotfit_internal.h"
#include "lanegroup.h"
#include "spotfit_lm.h"
#include "separable.h"

namespace sf {
namespace mtx {

using namespace lm;
using namespace sep;

// Totals of one evaluation, per spot: R (5), GX (8), GY (8), and of a new
// spot's first evaluation the sums of g and g^2; kChi: chi^2 summed directly.
enum Tot : int {
  kFG = 0, kBx, kBsx, kBy, kBsy,                          // sum g f, and its dx, dx^2, dy, dy^2
  kSxx, kXq1, kXq2, kSx, kXq3, kX1, kXq4, kX2,            // sum dx^m ex^2 (m = 0..4), dx^m ex
  kSyy, kYq1, kYq2, kSy, kYq3, kY1, kYq4, kY2,
  kG, kGG, kChi, kTotals
};

// A mode of the loop beside those of spotfit_lm.h: the best point is evaluated
// again for its normal equations, for a retry with more damping.
constexpr int kRegrad = 5;

// 10^k for |k| <= kP10, as pow10i gives it (exact powers, correctly rounded reciprocals).
constexpr int kP10 = 22;
__device__ const double kPow10[2 * kP10 + 1] = {
    1e-22, 1e-21, 1e-20, 1e-19, 1e-18, 1e-17, 1e-16, 1e-15, 1e-14, 1e-13, 1e-12, 1e-11,
    1e-10, 1e-9,  1e-8,  1e-7,  1e-6,  1e-5,  1e-4,  1e-3,  1e-2,  1e-1,  1e0,   1e1,
    1e2,   1e3,   1e4,   1e5,   1e6,   1e7,   1e8,   1e9,   1e10,  1e11,  1e12,  1e13,
    1e14,  1e15,  1e16,  1e17,  1e18,  1e19,  1e20,  1e21,  1e22};

// The spots of a launch.  Position p is spot p, or, with the class lists of a
// mixed-size batch, entry p of the lists from the largest class down.  A launch
// that holds every spot at once (take null) gives wavefront b the positions
// per b .. per b + per - 1.  Otherwise the positions go out in chunks of C from
// kMatrixCounters counters, wavefront b drawing from counter b % kMatrixCounters:
// atomics on one address from all over the chip pass one by one (about 50 ns
// each), so one counter for 2,000 wavefronts held up 1M spots of 15x15 px by
// themselves (1.1 ms with 21,000 draws, 1.6 ms with 31,000).  Counter g hands
// out the chunks g, g + kMatrixCounters, ..: every counter's share has the same
// mix of spots, also of a sorted list.
struct MatrixQueue {
  const int32_t* counts;  // spots per class, or null: no lists
  const int32_t* lists;
  int64_t cap;
  int32_t* take;
  int32_t count, first;  // positions; chunks per counter given out at the start
  int32_t per;           // positions of a wavefront that takes no more
  __device__ __forceinline__ int32_t spot(int32_t p) const {
    if ((uint32_t)p >= (uint32_t)count) return -1;
    if (!counts) return p;
    const int32_t n2 = counts[2], n1 = counts[1];
    if (p < n2) return lists[2 * cap + p];
    if (p < n2 + n1) return lists[cap + (p - n2)];
    return lists[p - n2 - n1];
  }
};
// Positions per chunk with NS slots per wavefront.
constexpr int chunk_of(int ns) { return ns < 16 ? ns : 16; }

// Bits of Shared::geo above the width and height.
enum : uint32_t { kGeoNew = 1u << 16, kGeoEll = 1u << 17 };

// LDS of one wavefront: per slot (a slot is a spot in flight) the totals of its
// last evaluation, its candidate, and where its pixels are.
template <int NS>
struct Shared {
  double tot[kTotals][NS + 1];  // one pad column: the 16 lanes of a spot write different banks
  double x[NS], y[NS], sx[NS], sy[NS], hx[NS], hy[NS];  // candidate; h = -1 / (2 sigma^2)
  double ra[NS], rb[NS];  // amplitudes of a point whose residuals are summed
  int64_t off[NS];
  uint32_t geo[NS];  // w | h << 8 | flags
  int order[NS];     // the slots to evaluate, new spots first
  double p10[2 * kP10 + 1];
  // normal equations at the best point (of 4 slots: before the contraction of a
  // symmetric spot), for a retry with more damping; a wavefront of more slots
  // evaluates the best point again instead
  static constexpr bool kKeepA = NS <= 16;
  double A[kKeepA ? 14 : 1][kKeepA ? NS : 1];
};

__device__ __forceinline__ double mfma4(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// The damped step (A + lam diag A) d = bv (Eq. 14) by an LDL^T factorisation, as
// solve4, with every rounding written out so that each build of the kernel takes
// the same bits; NaN when a pivot is not positive.
__device__ __forceinline__ void damped_step(const double (&A)[10], const double (&bv)[4], double lam,
                                            double (&d)[4]) {
  const double d0 = __builtin_fma(lam, A[0], A[0]), m11 = __builtin_fma(lam, A[4], A[4]);
  const double m22 = __builtin_fma(lam, A[7], A[7]), m33 = __builtin_fma(lam, A[9], A[9]);
  const double i0 = rcp_nr(d0);
  const double l10 = A[1] * i0, l20 = A[2] * i0, l30 = A[3] * i0;
  const double d1 = __builtin_fma(-l10, A[1], m11);
  const double i1 = rcp_nr(d1);
  const double u21 = __builtin_fma(-l20, A[1], A[5]), u31 = __builtin_fma(-l30, A[1], A[6]);
  const double l21 = u21 * i1, l31 = u31 * i1;
  const double d2 = __builtin_fma(-l21, u21, __builtin_fma(-l20, A[2], m22));
  const double i2 = rcp_nr(d2);
  const double u32 = __builtin_fma(-l31, u21, __builtin_fma(-l30, A[2], A[8]));
  const double l32 = u32 * i2;
  const double d3 =
      __builtin_fma(-l32, u32, __builtin_fma(-l31, u31, __builtin_fma(-l30, A[3], m33)));
  const double i3 = rcp_nr(d3);
  const double z1 = __builtin_fma(-l10, bv[0], bv[1]);
  const double z2 = __builtin_fma(-l21, z1, __builtin_fma(-l20, bv[0], bv[2]));
  const double z3 =
      __builtin_fma(-l32, z2, __builtin_fma(-l31, z1, __builtin_fma(-l30, bv[0], bv[3])));
  const double x3 = z3 * i3;
  const double x2 = __builtin_fma(-l32, x3, z2 * i2);
  const double x1 = __builtin_fma(-l31, x3, __builtin_fma(-l21, x2, z1 * i1));
  const double x0 =
      __builtin_fma(-l30, x3, __builtin_fma(-l20, x2, __builtin_fma(-l10, x1, bv[0] * i0)));
  const bool ok = d0 > 0.0 && d1 > 0.0 && d2 > 0.0 && d3 > 0.0 && __builtin_isfinite(x0) &&
                  __builtin_isfinite(x1) && __builtin_isfinite(x2) && __builtin_isfinite(x3);
  const double nanv = __builtin_nan("");
  d[0] = ok ? x0 : nanv;
  d[1] = ok ? x1 : nanv;
  d[2] = ok ? x2 : nanv;
  d[3] = ok ? x3 : nanv;
}

// Four consecutive pixels as stored (element alignment).
template <int DT>
struct Raw;
template <>
struct Raw<SPOTFIT_U16> {
  typedef uint32_t vec __attribute__((ext_vector_type(2), aligned(2)));
  static constexpr int kSize = 2;
  uint32_t v[2];
  __device__ __forceinline__ void load(const char* p) {
    const vec t = *reinterpret_cast<const vec*>(p);
    v[0] = t[0];
    v[1] = t[1];
  }
  template <int B>
  __device__ __forceinline__ double get() const {
    return double(B & 1 ? v[B / 2] >> 16 : v[B / 2] & 0xffffu);
  }
  // the same pixels, opaque: converted anew, so that the doubles of a row are
  // not kept from one use of it to the next
  __device__ __forceinline__ Raw fresh() const {
    Raw r = *this;
    asm("" : "+v"(r.v[0]), "+v"(r.v[1]));
    return r;
  }
  // drop the first n < 4 pixels
  __device__ __forceinline__ void shift(int n) {
    const uint64_t t = ((uint64_t)v[1] << 32 | v[0]) >> (16 * n);
    v[0] = (uint32_t)t;
    v[1] = (uint32_t)(t >> 32);
  }
};
template <>
struct Raw<SPOTFIT_F32> {
  typedef float vec __attribute__((ext_vector_type(4), aligned(4)));
  static constexpr int kSize = 4;
  float v[4];
  __device__ __forceinline__ void load(const char* p) {
    const vec t = *reinterpret_cast<const vec*>(p);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = t[i];
  }
  template <int B>
  __device__ __forceinline__ double get() const {
    return double(v[B]);
  }
  __device__ __forceinline__ Raw fresh() const {
    Raw r = *this;
    asm("" : "+v"(r.v[0]), "+v"(r.v[1]), "+v"(r.v[2]), "+v"(r.v[3]));
    return r;
  }
  __device__ __forceinline__ void shift(int n) {
    const bool two = (n & 2) != 0, one = (n & 1) != 0;
    v[0] = two ? v[2] : v[0];
    v[1] = two ? v[3] : v[1];
    v[0] = one ? v[1] : v[0];
    v[1] = one ? v[2] : v[1];
    v[2] = one ? v[3] : v[2];
  }
};

template <int N, int I = 0, typename F>
__device__ __forceinline__ void unrolled(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    unrolled<N, I + 1>(f);
  }
}

// Tiles of a shape's larger side.
__device__ __forceinline__ int tiles_of(uint32_t geo) {
  const int w = geo & 0xff, h = (geo >> 8) & 0xff;
  return ((w > h ? w : h) + 3) >> 2;
}

// Where a lane reads its pixels of a spot: CH windows of 4 columns.  A window
// that reaches past its row's end goes on in the next row, still inside the
// spot (its columns there have V = 0); on the last row it starts `over` pixels
// earlier instead and Raw::shift puts it back, so no lane reads outside the spot.
template <int CH, int DT>
struct Window {
  uint32_t row, step, last[CH];  // byte offsets: the lane's first row, 4 rows, the last row
  int w, h, start[CH], own[CH], over[CH];  // shape; first column, the group's own columns of it

  __device__ __forceinline__ void set(uint32_t geo, int v, int k) {
    w = geo & 0xff;
    h = (geo >> 8) & 0xff;
    const int T = (w + 3) >> 2;
    const uint32_t pitch = uint32_t(w) * Raw<DT>::kSize;
#pragma unroll
    for (int q = 0; q < CH; ++q) {
      const int first = T * k + 4 * q;
      const int n = T - 4 * q < w - first ? T - 4 * q : w - first;
      own[q] = n < 0 ? 0 : n < 4 ? n : 4;
      start[q] = n > 0 ? first : 0;
      over[q] = start[q] + 4 > w ? start[q] + 4 - w : 0;
      last[q] = pitch * uint32_t(h - 1) - uint32_t(over[q]) * Raw<DT>::kSize;
    }
    row = pitch * uint32_t(v);
    step = pitch * 4u;
  }
};

// The smallest and the largest of a per-block value (the same on the 16 lanes
// of a block) over the wavefront's four blocks.
__device__ __forceinline__ int min_over_blocks(int v) {
  const int a = __builtin_amdgcn_readlane(v, 0), b = __builtin_amdgcn_readlane(v, 4);
  const int c = __builtin_amdgcn_readlane(v, 8), d = __builtin_amdgcn_readlane(v, 12);
  const int e = a < b ? a : b, f = c < d ? c : d;
  return e < f ? e : f;
}
__device__ __forceinline__ int max_over_blocks(int v) {
  const int a = __builtin_amdgcn_readlane(v, 0), b = __builtin_amdgcn_readlane(v, 4);
  const int c = __builtin_amdgcn_readlane(v, 8), d = __builtin_amdgcn_readlane(v, 12);
  const int e = a > b ? a : b, f = c > d ? c : d;
  return e > f ? e : f;
}

// Total over the 16 lanes of a block, in a fixed order, on each of them.
__device__ __forceinline__ double block_sum(double v) {
  v += dpp_mov<0xB1>(v);
  v += dpp_mov<0x4E>(v);
  v = pair<1>(v, v);
  return pair<0>(v, v);
}

// A lane's place in a pass, and what it holds of every matrix of one.
struct Lane {
  int v, blk, k;          // lane = v + 4 blk + 16 k
  double c0, c1, c2, c3;  // vector v's weight of ex: 1, dx, dx^2, and 1 in place of ex
  int tr, tg;             // the total that entry (row k, column v) of R and of a Gram matrix is, or -1
  __device__ __forceinline__ explicit Lane(int lane) {
    v = lane & 3;
    blk = (lane >> 2) & 3;
    k = lane >> 4;
    c0 = v == 0 ? 1.0 : 0.0;
    c1 = v == 1 ? 1.0 : 0.0;
    c2 = v == 2 ? 1.0 : 0.0;
    c3 = v == 3 ? 1.0 : 0.0;
    tr = k == 0 ? (v < 3 ? kFG + v : -1) : v == 0 ? (k == 1 ? kBy : k == 2 ? kBsy : -1) : -1;
    static_assert(kXq1 == kSxx + 1 && kXq2 == kSxx + 2 && kSx == kSxx + 3, "row 0 of a Gram matrix");
    tg = k == 0   ? kSxx + v
         : k == 1 ? (v == 2 ? kXq3 : v == 3 ? kX1 : -1)
         : k == 2 ? (v == 2 ? kXq4 : v == 3 ? kX2 : -1)
                  : -1;
  }
};

// V of one column, E of one row: vector v's entry for profile factor f at
// distance d from the candidate's centre.
__device__ __forceinline__ double vector_entry(const Lane& ln, double f, double d) {
  return __builtin_fma(f, __builtin_fma(__builtin_fma(ln.c2, d, ln.c1), d, ln.c0), ln.c3);
}

// The profile factors of a pass: lane v of a quad has column start + v of each
// window of its group, and row 4 (4 q + v) + k.
template <int Q, int CH, int DT>
__device__ __forceinline__ void factors(const Lane& ln, const Window<CH, DT>& win, double x, double y,
                                        double hx, double hy, double& ex, double& ey) {
  const double dxc = double(win.start[Q] + ln.v) - x;
  const int row = 16 * Q + 4 * ln.v + ln.k;
  const double dyr = double(row) - y;
  double arg[2] = {dxc * dxc * hx, dyr * dyr * hy}, fac[2];
  exp_neg_n<2>(arg, fac);
  ex = ln.v < win.own[Q] ? fac[0] : 0.0;
  ey = row < win.h ? fac[1] : 0.0;
}
// One of the two, where a spot has more windows of columns than quads of row
// tiles or the other way round.
template <int Q, int CH, int DT>
__device__ __forceinline__ double column_factor(const Lane& ln, const Window<CH, DT>& win, double x, double hx) {
  const double dxc = double(win.start[Q] + ln.v) - x;
  double arg[1] = {dxc * dxc * hx}, fac[1];
  exp_neg_n<1>(arg, fac);
  return ln.v < win.own[Q] ? fac[0] : 0.0;
}
template <int Q, int CH, int DT>
__device__ __forceinline__ double row_factor(const Lane& ln, const Window<CH, DT>& win, double y, double hy) {
  const int row = 16 * Q + 4 * ln.v + ln.k;
  const double dyr = double(row) - y;
  double arg[1] = {dyr * dyr * hy}, fac[1];
  exp_neg_n<1>(arg, fac);
  return row < win.h ? fac[0] : 0.0;
}

// The entry of R, GX and GY that this lane holds, to the slot's totals.
template <int NS>
__device__ __forceinline__ void put_totals(const Lane& ln, Shared<NS>& L, int slot, double R, double GX,
                                           double GY) {
  if (ln.tr >= 0) L.tot[ln.tr][slot] = R;
  if (ln.tg >= 0) {
    L.tot[ln.tg][slot] = GX;
    L.tot[ln.tg + (kSyy - kSxx)][slot] = GY;
  }
}

// Residuals r = alpha f + beta - g of row tile AT, window Q (B columns): their
// squares added to cs, one sum per column of the lane.  aex: alpha ex.  KIND: how
// rows below the spot are left out (1M floats of 15x15 1.26 ms with selects
// everywhere, 1.21 so; 36,600 of 32x32 251 us, 239).
enum class Rows {
  kAll,     // there are none in this tile
  kBranch,  // by a branch
  kSelect,  // by a select of each sum, two instructions a pixel
};
template <int AT, int B, Rows KIND, int DT>
__device__ __forceinline__ void residual_row(const Lane& ln, const Raw<DT>& px, const double (&aex)[4],
                                             double eyq, double beta, int h, double (&cs)[4]) {
  // row 4 AT + v is with lane AT % 4 of the quad of row group v
  const int src = (AT & 3) | (ln.blk << 2) | (ln.v << 4);
  const int2 u = __builtin_bit_cast(int2, eyq);
  const int2 r2 = make_int2(__builtin_amdgcn_ds_bpermute(src << 2, u.x),
                            __builtin_amdgcn_ds_bpermute(src << 2, u.y));
  const double e = __builtin_bit_cast(double, r2);
  const bool rowin = 4 * AT + ln.v < h;
  auto add = [&] {
    unrolled<B>([&](auto bi) {
      constexpr int t = decltype(bi)::value;
      const double res = __builtin_fma(aex[t], e, beta - px.template get<t>());
      cs[t] = KIND != Rows::kSelect || rowin ? __builtin_fma(res, res, cs[t]) : cs[t];
    });
  };
  if constexpr (KIND == Rows::kBranch) {
    if (rowin) add();
  } else {
    add();
  }
}

// Sums of g and g^2 over a spot's own pixels, from its lanes' partial sums.
template <int NS>
__device__ __forceinline__ void put_pixel_sums(const Lane& ln, Shared<NS>& L, int slot, bool fresh,
                                               double sg, double sgg) {
  sg = block_sum(sg);
  sgg = block_sum(sgg);
  if (ln.v == 0 && ln.k == 0 && fresh) {
    L.tot[kG][slot] = sg;
    L.tot[kGG][slot] = sgg;
  }
}

template <int NS>
__device__ __forceinline__ Amplitudes slot_amplitudes(const Shared<NS>& L, int slot, int w, int h) {
  return amplitudes(double(w * h), L.tot[kSx][slot], L.tot[kSxx][slot], L.tot[kSy][slot],
                    L.tot[kSyy][slot], L.tot[kFG][slot], L.tot[kG][slot]);
}

// Evaluates the cnt > 0 slots of L.order, the first cnt_new of them new spots,
// at their candidates, four a pass (Eqs. 2, 5-7, 10), into L.tot.  Every slot
// has the shape of geo0, with TB columns per lane group and TR row tiles or, if
// RECT, at most TR row tiles: those below the spots are branched over (uneven
// spots of one shape in the passes for mixed shapes, over the tiles of their
// larger side both ways, / so: 1M of 16-bit 8x32 2.72 ms / 1.30, 16x6 1.21 / 0.84;
// of float 32x8 4.42 / 2.07, 16x6 1.67 / 1.24; lane-owned 3.61, 1.00, 3.50, 1.01).  Float
// data: with chi^2 summed over the pixels.  ANY (two tiles each way): slots of any
// shapes up to 8 x 8.
//
// The pixels of a pass stay in registers, and the next pass's take their places
// as they are used; of floats above 16 px, whose 40 to 64 registers would push
// the owners' state out of the registers, kRows row tiles are in flight instead,
// read once for the products and once for the residuals (200,000 of 17x17:
// 826 us held, 683 read twice).
template <int NS, int DT, int TB, int TR, bool RECT, bool ANY = false>
__device__ __forceinline__ void evaluate_uniform(const void* data, Shared<NS>& L, int cnt, int cnt_new,
                                                 uint32_t geo0) {
  constexpr int CH = (TB + 3) / 4, CR = (TR + 3) / 4;  // windows of columns, quads of row tiles
  constexpr bool kFloat = DT != SPOTFIT_U16, kRing = kFloat && (CH > 1 || CR > 1);
  constexpr int kRows = kRing ? 4 : TR;
  // opaque: a lane's constants are formed once a step here, not held in
  // registers over the rest of it
  int lane = __lane_id();
  asm volatile("" : "+v"(lane));
  const Lane ln(lane);
  static_assert(!ANY || (TB == 2 && TR == 2), "every row and column is checked");
  Window<CH, DT> win, win_next;
  if constexpr (!ANY) win.set(geo0, ln.v, ln.k);
  Window<CH, DT>& ahead = ANY ? win_next : win;  // of the pixels to load
  const int rows = int((geo0 >> 8 & 0xffu) + 3) >> 2;  // row tiles of the spots
  auto in = [&](int at) { return !RECT || at < rows; };
  Raw<DT> px[kRows][CH];
  auto slot_at = [&](int p) { return L.order[p + ln.blk < cnt ? p + ln.blk : cnt - 1]; };
  const char* base[CH];
  auto aim = [&](int sl) {  // at the first rows of a slot's windows
    if constexpr (ANY) ahead.set(L.geo[sl], ln.v, ln.k);
    const char* p = static_cast<const char*>(data) + L.off[sl] * Raw<DT>::kSize;
#pragma unroll
    for (int q = 0; q < CH; ++q) base[q] = p + ahead.start[q] * Raw<DT>::kSize;
  };
  uint32_t rb;
  auto rewind = [&] {
    rb = ahead.row;
    if constexpr (CH > 1) asm volatile("" : "+v"(rb));  // its rows' offsets do not fit the registers
  };
  auto load_next = [&](Raw<DT> (&to)[CH]) {
#pragma unroll
    for (int q = 0; q < CH; ++q) to[q].load(base[q] + (rb < ahead.last[q] ? rb : ahead.last[q]));
    rb += ahead.step;
  };
  // the last row tile holds the last row (of two: either): windows cut off there
  // come back
  auto put_back = [&](auto ai, Raw<DT> (&row)[CH]) {
    constexpr int at = decltype(ai)::value;
    if constexpr (RECT || at == TR - 1 || TR == 2) {
      if (RECT && at != rows - 1) return;
#pragma unroll
      for (int q = 0; q < CH; ++q) row[q].shift(4 * at + ln.v >= win.h - 1 ? win.over[q] : 0);
    }
  };
  // after item i of a ring pass (TR row tiles for the products, then for the
  // residuals): the item that takes its place
  auto refill = [&](auto ii) {
    constexpr int i = decltype(ii)::value + kRows;
    if constexpr (i < 2 * TR) {
      if constexpr (i == TR) rewind();
      load_next(px[i % kRows]);
    }
  };
  // RECT: row tile a is in place a % kRows both times; after the products (then
  // the residuals) of tile at, the next tile of that place, or the first one again
  auto refill_rect = [&](auto ai, bool again) {
    constexpr int at = decltype(ai)::value;
    const bool more = at + kRows < rows;
    if (!more && !again) return;
    rb = win.row + (more ? uint32_t(at + kRows) : uint32_t(at % kRows)) * win.step;
    asm volatile("" : "+v"(rb));
    load_next(px[at % kRows]);
  };
  auto add_row = [&](auto ai, const Raw<DT> (&row)[CH], double& sg, double& sgg) {
    constexpr int at = decltype(ai)::value;
    const bool rowin = (!RECT && at < TR - 1 && TR > 2) || 4 * at + ln.v < win.h;
    unrolled<TB>([&](auto bi) {
      constexpr int t = decltype(bi)::value;
      const double g = row[t / 4].template get<t % 4>();
      // a group owns at least T - 3 columns
      const double gm = rowin && (t < TB - 3 || t % 4 < win.own[t / 4]) ? g : 0.0;
      sg += gm;
      sgg = __builtin_fma(gm, gm, sgg);
    });
    __builtin_amdgcn_sched_barrier(0);
  };
  int slot = slot_at(0);
  if constexpr (!kRing) {
    aim(slot);
    rb = ahead.row;
    unrolled<TR>([&](auto ai) {
      if (in(decltype(ai)::value)) load_next(px[decltype(ai)::value]);
    });
  }

#pragma unroll 1
  for (int p = 0; p < cnt; p += 4) {
    const double x = L.x[slot], y = L.y[slot], hx = L.hx[slot], hy = L.hy[slot];
    const int cslot = slot;
    if constexpr (ANY) win = win_next;
    if constexpr (RECT) {
      // formed anew in each pass: the masks of all its rows and columns, held over the
      // passes, take the scalar registers of the whole kernel
      asm volatile("" : "+v"(win.h));
#pragma unroll
      for (int q = 0; q < CH; ++q) asm volatile("" : "+v"(win.own[q]), "+v"(win.over[q]));
    }
    if constexpr (kRing) {
      aim(slot);
      if (p < cnt_new) {
        double sg = 0.0, sgg = 0.0;
        rewind();
        unrolled<TR>([&](auto ai) {
          if (!in(decltype(ai)::value)) return;
          Raw<DT> row[CH];
          load_next(row);
          put_back(ai, row);
          add_row(ai, row, sg, sgg);
        });
        put_pixel_sums(ln, L, cslot, p + ln.blk < cnt_new, sg, sgg);
      }
      rewind();
      unrolled<kRows>([&](auto ai) {
        if (in(decltype(ai)::value)) load_next(px[decltype(ai)::value]);
      });
    }
    // the next pass (or this one's last slot again): its rows are loaded as this
    // pass's are used
    slot = slot_at(p + 4);
    if constexpr (!kRing) {
      aim(slot);
      rewind();
    }
    double exq[CH], eyq[CR], V[TB], E[TR];
    double R = 0.0, GX = 0.0, GY = 0.0;
    unrolled<(CH > CR ? CH : CR)>([&](auto qi) {
      constexpr int q = decltype(qi)::value;
      if constexpr (q < CH && q < CR) {
        factors<q>(ln, win, x, y, hx, hy, exq[q], eyq[q]);
      } else if constexpr (q < CH) {
        exq[q] = column_factor<q>(ln, win, x, hx);
      } else {
        eyq[q] = rows > 4 * q ? row_factor<q>(ln, win, y, hy) : 0.0;
      }
    });
    const double dy0 = double(ln.k) - y;
    unrolled<(TB > TR ? TB : TR)>([&](auto ti) {
      constexpr int t = decltype(ti)::value;
      if constexpr (t < TB) {
        const double dx = (double(win.start[t / 4]) - x) + double(t % 4);
        V[t] = vector_entry(ln, lg::gbcast<4, t % 4>(exq[t / 4]), dx);
      }
      if constexpr (t < TR) E[t] = vector_entry(ln, lg::gbcast<4, t % 4>(eyq[t / 4]), dy0 + double(4 * t));
      if constexpr (t < TB) GX = mfma4(V[t], V[t], GX);
      if constexpr (t < TR) GY = mfma4(E[t], E[t], GY);
      // (of three: without the first one the loads of the next pass came after the
      // products, 2 % at 9..12 px)
      if constexpr (t % 4 == 3 || (TB == 3 && t == 0)) __builtin_amdgcn_sched_barrier(0);
    });
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!kRing) {
      unrolled<TR>([&](auto ai) { put_back(ai, px[decltype(ai)::value]); });
      if (p < cnt_new) {
        double sg = 0.0, sgg = 0.0;
        unrolled<TR>([&](auto ai) {
          constexpr int at = decltype(ai)::value;
          if (!in(at)) return;
          Raw<DT> row[CH];
#pragma unroll
          for (int q = 0; q < CH; ++q) row[q] = px[at][q].fresh();
          add_row(ai, row, sg, sgg);
        });
        put_pixel_sums(ln, L, cslot, p + ln.blk < cnt_new, sg, sgg);
      }
    }
    unrolled<TR>([&](auto ai) {
      constexpr int at = decltype(ai)::value;
      if (!in(at)) return;
      if constexpr (kRing) put_back(ai, px[at % kRows]);
      double S = 0.0;
      unrolled<TB>([&](auto bi) {
        constexpr int t = decltype(bi)::value;
        S = mfma4(px[at % kRows][t / 4].template get<t % 4>(), V[t], S);
      });
      R = mfma4(E[at], S, R);
      if constexpr (kRing && RECT) refill_rect(ai, true);
      else if constexpr (kRing) refill(ai);
      else if constexpr (!kFloat) load_next(px[at]);
      __builtin_amdgcn_sched_barrier(0);  // bounds the tiles in flight (registers)
    });
    put_totals(ln, L, cslot, R, GX, GY);
    if constexpr (kFloat) {
      wave_lds_sync();
      const Amplitudes am = slot_amplitudes(L, cslot, win.w, win.h);
      double aex[CH][4], cs[CH][4], c2s = 0.0;
      unrolled<TB>([&](auto bi) {
        constexpr int t = decltype(bi)::value;
        aex[t / 4][t % 4] = am.a * lg::gbcast<4, t % 4>(exq[t / 4]);
        cs[t / 4][t % 4] = 0.0;
      });
      unrolled<TR>([&](auto ai) {
        constexpr int at = decltype(ai)::value, i = kRing && !RECT ? TR + at : at;
        constexpr Rows kRowsOut = RECT || at == TR - 1 || TR == 2 ? Rows::kBranch : Rows::kAll;
        if (!in(at)) return;
        if constexpr (kRing) put_back(ai, px[i % kRows]);
        unrolled<CH>([&](auto qi) {
          constexpr int q = decltype(qi)::value, B = TB - 4 * q < 4 ? TB - 4 * q : 4;
          residual_row<at, B, kRowsOut>(ln, px[i % kRows][q].fresh(), aex[q], eyq[at / 4], am.b, win.h, cs[q]);
        });
        if constexpr (kRing && RECT) refill_rect(ai, false);
        else if constexpr (kRing) refill(std::integral_constant<int, i>{});
        else load_next(px[at]);
        __builtin_amdgcn_sched_barrier(0);
      });
      unrolled<TB>([&](auto bi) {
        constexpr int t = decltype(bi)::value;
        c2s += t % 4 < win.own[t / 4] ? cs[t / 4][t % 4] : 0.0;
      });
      c2s = block_sum(c2s);
      if (ln.v == 0 && ln.k == 0) L.tot[kChi][cslot] = c2s;
    }
  }
}

// chi^2 summed over the pixels (Eq. 2), r = alpha f + beta - g, for the cnt > 0
// slots of L.order at their points L.x .. L.hy with the amplitudes L.ra, L.rb:
// 16-bit data, where a decision lies within the closed form's error.
template <int NS, int CH>
__device__ __forceinline__ void sum_residuals(const void* data, Shared<NS>& L, int cnt) {
  constexpr int NT = 4 * CH, DT = SPOTFIT_U16;
  int lane = __lane_id();
  asm volatile("" : "+v"(lane));
  const Lane ln(lane);
#pragma unroll 1
  for (int p = 0; p < cnt; p += 4) {
    const int slot = L.order[p + ln.blk < cnt ? p + ln.blk : cnt - 1];
    const double x = L.x[slot], y = L.y[slot], hx = L.hx[slot], hy = L.hy[slot];
    const double alpha = L.ra[slot], beta = L.rb[slot];
    Window<CH, DT> win;
    win.set(L.geo[slot], ln.v, ln.k);
    const char* base = static_cast<const char*>(data) + L.off[slot] * Raw<DT>::kSize;
    const int Tm = max_over_blocks((win.w + 3) >> 2), Hm = max_over_blocks((win.h + 3) >> 2);
    double exq[CH], eyq[CH], c2s = 0.0;
    unrolled<CH>([&](auto qi) {
      constexpr int q = decltype(qi)::value;
      exq[q] = eyq[q] = 0.0;
      if (q == 0 || Tm > 4 * q || Hm > 4 * q) factors<q>(ln, win, x, y, hx, hy, exq[q], eyq[q]);
    });
    unrolled<CH>([&](auto qi) {
      constexpr int q = decltype(qi)::value;
      if (q == 0 || Tm > 4 * q) {
        double aex[4], cs[4];
        unrolled<4>([&](auto bi) {
          constexpr int t = decltype(bi)::value;
          aex[t] = alpha * lg::gbcast<4, t>(exq[q]);
          cs[t] = 0.0;
        });
        Raw<DT> px[NT];
        uint32_t rb = win.row;
        unrolled<NT>([&](auto ai) {
          constexpr int at = decltype(ai)::value;
          if (at < Hm) px[at].load(base + win.start[q] * Raw<DT>::kSize + (rb < win.last[q] ? rb : win.last[q]));
          rb += win.step;
        });
        unrolled<NT>([&](auto ai) {
          constexpr int at = decltype(ai)::value;
          if (at < Hm) {
            px[at].shift(4 * at + ln.v >= win.h - 1 ? win.over[q] : 0);
            residual_row<at, 4, Rows::kBranch>(ln, px[at], aex, eyq[at / 4], beta, win.h, cs);
          }
        });
        unrolled<4>([&](auto bi) {
          constexpr int t = decltype(bi)::value;
          c2s += t < win.own[q] ? cs[t] : 0.0;
        });
      }
    });
    c2s = block_sum(c2s);
    if (ln.v == 0 && ln.k == 0) L.tot[kChi][slot] = c2s;
  }
}

// put_back of the row tiles AT, AT - 1, .. `first`: the tiles before hold no
// slot's last row, and a pass has nothing to put back there (with the lane's
// place formed once a step instead of in each pass: 372 -> 301 vector
// instructions a pass at 5 tiles, 2M spots of seven sizes from 7 to 32 px 3199 us
// -> 3130, 10,007 of 7..32 px 81.6 -> 79.1).
template <int AT, int N, typename R, typename F>
__device__ __forceinline__ void put_back_from(R (&px)[N], int first, F& put_back) {
  put_back(std::integral_constant<int, AT>{}, px[AT]);
  if constexpr (AT > 0)
    if (first < AT) put_back_from<AT - 1>(px, first, put_back);
}

struct Candidate {
  double x, y, hx, hy;
};

// One pass over four slots of any shapes (this lane's block has `slot`, of shape
// geo) at their candidates, into L.tot.  load: read their pixels first, at `off`,
// into px, shifted into place; else px holds them.  sums: some slot (fresh) is a
// new spot.  Every slot has at most TB columns per lane group and TR row tiles;
// the tiles that a smaller one does not have add zeros to its sums, so it has
// the same bits in every company.
//
// A wavefront of 4 slots keeps px from step to step, so a step neither reads
// memory nor waits for it.  A lone wavefront per SIMD is bound by that chain of
// latencies: 32 markers of 13x13 px 38.6 us a replayed frame (40.6 with the
// pixels read at each step), 1,024 of 11x11 18.0 (19.5), 4,000 raw spots of
// 9..21 px 41.0 (47.3).  Of more slots, wide floats go through a ring of row tiles as
// in evaluate_uniform.
template <int NS, int CH, int DT, int TB, int TR>
__device__ __forceinline__ void evaluate_pass(const void* data, const Lane& ln, Shared<NS>& L, int slot,
                                              Raw<DT> (&px)[4 * CH][CH], const Candidate& c, int64_t off,
                                              uint32_t geo, bool load, bool sums, bool fresh) {
  constexpr int CQ = (TB + 3) / 4, CR = (TR + 3) / 4;
  constexpr bool kFloat = DT != SPOTFIT_U16, kRing = NS > 4 && kFloat && CQ > 1;
  constexpr int kRows = kRing ? 4 : TR;
  Window<CQ, DT> win;
  win.set(geo, ln.v, ln.k);
  const char* base = static_cast<const char*>(data) + off * Raw<DT>::kSize;
  uint32_t rb = win.row;
  auto load_next = [&](Raw<DT> (&to)[CH]) {
#pragma unroll
    for (int q = 0; q < CQ; ++q)
      to[q].load(base + win.start[q] * Raw<DT>::kSize + (rb < win.last[q] ? rb : win.last[q]));
    rb += win.step;
  };
  // windows cut off by a spot's end come back
  auto put_back = [&](auto ai, Raw<DT> (&row)[CH]) {
    constexpr int at = decltype(ai)::value;
#pragma unroll
    for (int q = 0; q < CQ; ++q) row[q].shift(4 * at + ln.v >= win.h - 1 ? win.over[q] : 0);
  };
  auto refill = [&](auto ii) {  // after item i of the ring
    constexpr int i = decltype(ii)::value + kRows;
    if constexpr (i < 2 * TR) {
      if constexpr (i == TR) rb = win.row;
      load_next(px[i % kRows]);
    }
  };
  auto add_row = [&](auto ai, const Raw<DT> (&row)[CH], double& sg, double& sgg) {
    constexpr int at = decltype(ai)::value;
    const bool rowin = 4 * at + ln.v < win.h;
    unrolled<TB>([&](auto bi) {
      constexpr int t = decltype(bi)::value;
      const double g = row[t / 4].template get<t % 4>();
      const double gm = rowin && t % 4 < win.own[t / 4] ? g : 0.0;
      sg += gm;
      sgg = __builtin_fma(gm, gm, sgg);
    });
    __builtin_amdgcn_sched_barrier(0);
  };
  // a slot's last row is in this row tile or a later one
  const int last_tile = load && !kRing ? min_over_blocks((win.h - 1) >> 2) : 0;
  if constexpr (kRing) {
    if (sums) {
      double sg = 0.0, sgg = 0.0;
      unrolled<TR>([&](auto ai) {
        Raw<DT> row[CH];
        load_next(row);
        put_back(ai, row);
        add_row(ai, row, sg, sgg);
      });
      put_pixel_sums(ln, L, slot, fresh, sg, sgg);
      rb = win.row;
    }
  }
  if (load) unrolled<kRows>([&](auto ai) { load_next(px[decltype(ai)::value]); });
  double exq[CQ], eyq[CR], V[TB], E[TR];
  double R = 0.0, GX = 0.0, GY = 0.0;
  unrolled<(CQ > CR ? CQ : CR)>([&](auto qi) {
    constexpr int q = decltype(qi)::value;
    if constexpr (q < CQ && q < CR)
      factors<q>(ln, win, c.x, c.y, c.hx, c.hy, exq[q], eyq[q]);
    else if constexpr (q < CQ)
      exq[q] = column_factor<q>(ln, win, c.x, c.hx);
    else
      eyq[q] = row_factor<q>(ln, win, c.y, c.hy);
  });
  const double dy0 = double(ln.k) - c.y;
  unrolled<(TB > TR ? TB : TR)>([&](auto ti) {
    constexpr int t = decltype(ti)::value;
    if constexpr (t < TB) {
      const double dx = (double(win.start[t / 4]) - c.x) + double(t % 4);
      V[t] = vector_entry(ln, lg::gbcast<4, t % 4>(exq[t / 4]), dx);
      GX = mfma4(V[t], V[t], GX);
    }
    if constexpr (t < TR) {
      E[t] = vector_entry(ln, lg::gbcast<4, t % 4>(eyq[t / 4]), dy0 + double(4 * t));
      GY = mfma4(E[t], E[t], GY);
    }
  });
  if constexpr (!kRing) {
    if (load) put_back_from<TR - 1>(px, last_tile, put_back);
    if (sums) {
      double sg = 0.0, sgg = 0.0;
      unrolled<TR>([&](auto ai) {
        constexpr int at = decltype(ai)::value;
        Raw<DT> row[CH];
#pragma unroll
        for (int q = 0; q < CQ; ++q) row[q] = px[at][q].fresh();
        add_row(ai, row, sg, sgg);
      });
      put_pixel_sums(ln, L, slot, fresh, sg, sgg);
    }
  }
  unrolled<TR>([&](auto ai) {
    constexpr int at = decltype(ai)::value;
    if constexpr (kRing) put_back(ai, px[at % kRows]);
    Raw<DT> row[CQ];
#pragma unroll
    for (int q = 0; q < CQ; ++q) row[q] = px[at % kRows][q].fresh();
    double S = 0.0;
    unrolled<TB>([&](auto bi) {
      constexpr int t = decltype(bi)::value;
      S = mfma4(row[t / 4].template get<t % 4>(), V[t], S);
    });
    R = mfma4(E[at], S, R);
    if constexpr (kRing) refill(ai);
    if constexpr (kRing || at % 2 == 1) __builtin_amdgcn_sched_barrier(0);
  });
  put_totals(ln, L, slot, R, GX, GY);
  if constexpr (kFloat) {
    wave_lds_sync();
    const Amplitudes am = slot_amplitudes(L, slot, win.w, win.h);
    double aex[CQ][4], cs[CQ][4], c2s = 0.0;
    auto scale = [&](auto qi) {
      constexpr int q = decltype(qi)::value, B = TB - 4 * q < 4 ? TB - 4 * q : 4;
      unrolled<B>([&](auto bi) {
        constexpr int t = decltype(bi)::value;
        aex[q][t] = am.a * lg::gbcast<4, t>(exq[q]);
        cs[q][t] = 0.0;
      });
    };
    // of 4 wide slots the row tiles stay one run of code: a lone wavefront waits
    // for its own instructions (32 spots of 17x17 23.6 us so, 24.1 with branches)
    constexpr Rows kRowsOut = NS == 4 && CQ > 1 ? Rows::kSelect : Rows::kBranch;
    auto window = [&](auto ai, auto qi, const Raw<DT>& g) {
      constexpr int q = decltype(qi)::value, B = TB - 4 * q < 4 ? TB - 4 * q : 4;
      residual_row<decltype(ai)::value, B, kRowsOut>(ln, g.fresh(), aex[q], eyq[decltype(ai)::value / 4], am.b,
                                                     win.h, cs[q]);
    };
    auto add_up = [&](auto qi) {
      constexpr int q = decltype(qi)::value, B = TB - 4 * q < 4 ? TB - 4 * q : 4;
      unrolled<B>([&](auto bi) {
        constexpr int t = decltype(bi)::value;
        c2s += t < win.own[q] ? cs[q][t] : 0.0;
      });
    };
    if constexpr (kRing) {  // row by row, as the ring goes
      unrolled<CQ>(scale);
      unrolled<TR>([&](auto ai) {
        constexpr int i = TR + decltype(ai)::value;
        put_back(ai, px[i % kRows]);
        unrolled<CQ>([&](auto qi) { window(ai, qi, px[i % kRows][decltype(qi)::value]); });
        refill(std::integral_constant<int, i>{});
        __builtin_amdgcn_sched_barrier(0);
      });
      unrolled<CQ>(add_up);
    } else {  // window by window: fewer registers
      unrolled<CQ>([&](auto qi) {
        scale(qi);
        unrolled<TR>([&](auto ai) {
          window(ai, qi, px[decltype(ai)::value][decltype(qi)::value]);
          __builtin_amdgcn_sched_barrier(0);
        });
        add_up(qi);
      });
    }
    c2s = block_sum(c2s);
    if (ln.v == 0 && ln.k == 0) L.tot[kChi][slot] = c2s;
  }
}

// The pass with the tiles of the largest of its four slots.  UNEVEN: with four row
// tiles, or four columns per lane group, where no spot has more and more the other way.
template <int NS, int CH, int DT, bool UNEVEN>
__device__ __forceinline__ void evaluate_four(const void* data, const Lane& ln, Shared<NS>& L, int slot,
                                              Raw<DT> (&px)[4 * CH][CH], const Candidate& c, int64_t off,
                                              uint32_t geo, bool load, bool sums, bool fresh) {
  const int tiles = max_over_blocks(tiles_of(geo));
  const int cols = UNEVEN ? max_over_blocks((int(geo & 0xff) + 3) >> 2) : tiles;
  const int rows = UNEVEN ? max_over_blocks((int(geo >> 8 & 0xff) + 3) >> 2) : tiles;
  unrolled<4 * CH - 1>([&](auto ti) {
    constexpr int TB = decltype(ti)::value + 2;
    if (tiles != TB && !(TB == 2 && tiles < 2)) return;
    if constexpr (UNEVEN && TB > 4) {
      if (rows <= 4)
        return evaluate_pass<NS, CH, DT, TB, 4>(data, ln, L, slot, px, c, off, geo, load, sums, fresh);
      if (cols <= 4)
        return evaluate_pass<NS, CH, DT, 4, TB>(data, ln, L, slot, px, c, off, geo, load, sums, fresh);
    }
    evaluate_pass<NS, CH, DT, TB, TB>(data, ln, L, slot, px, c, off, geo, load, sums, fresh);
  });
}

// chi^2 summed over the pixels (Eq. 2) of a wavefront of 4 slots, 16-bit data, on
// every lane of a block: of its slot (shape geo) at c, with the pixels that its
// lanes hold.  As sum_residuals, which reads the pixels again and takes its sums
// through LDS: with few spots a launch is as long as its longest chain of steps
// (4,000 raw spots of 9..21 px 38.9 us -> 37.5, one served frame of 110 63.4 ->
// 61.0, 1,024 of 11x11 18.3 -> 17.9).
template <int CH, int DT, int TB>
__device__ __forceinline__ double block_residuals_of(const Lane& ln, const Raw<DT> (&px)[4 * CH][CH],
                                                     const Candidate& c, uint32_t geo, double alpha,
                                                     double beta) {
  constexpr int CQ = (TB + 3) / 4;
  Window<CQ, DT> win;
  win.set(geo, ln.v, ln.k);
  double exq[CQ], eyq[CQ], c2s = 0.0;
  unrolled<CQ>([&](auto qi) {
    constexpr int q = decltype(qi)::value;
    factors<q>(ln, win, c.x, c.y, c.hx, c.hy, exq[q], eyq[q]);
  });
  unrolled<CQ>([&](auto qi) {
    constexpr int q = decltype(qi)::value, B = TB - 4 * q < 4 ? TB - 4 * q : 4;
    double aex[4], cs[4];
    unrolled<B>([&](auto bi) {
      constexpr int t = decltype(bi)::value;
      aex[t] = alpha * lg::gbcast<4, t>(exq[q]);
      cs[t] = 0.0;
    });
    unrolled<TB>([&](auto ai) {
      constexpr int at = decltype(ai)::value;
      residual_row<at, B, Rows::kBranch>(ln, px[at][q].fresh(), aex, eyq[at / 4], beta, win.h, cs);
    });
    unrolled<B>([&](auto bi) {
      constexpr int t = decltype(bi)::value;
      c2s += t < win.own[q] ? cs[t] : 0.0;
    });
  });
  return block_sum(c2s);
}
template <int CH, int DT>
__device__ __forceinline__ double block_residuals(const Raw<DT> (&px)[4 * CH][CH], const Candidate& c,
                                                  uint32_t geo, double alpha, double beta) {
  int lane = __lane_id();
  asm volatile("" : "+v"(lane));
  const Lane ln(lane);
  const int tiles = max_over_blocks(tiles_of(geo));
  double c2 = 0.0;
  unrolled<4 * CH - 1>([&](auto ti) {
    constexpr int TB = decltype(ti)::value + 2;
    if (tiles == TB || (TB == 2 && tiles < 2)) c2 = block_residuals_of<CH, DT, TB>(ln, px, c, geo, alpha, beta);
  });
  return c2;
}

// Evaluates the cnt > 0 slots of L.order, of any shapes, four a pass.
template <int NS, int CH, int DT>
__device__ __forceinline__ void evaluate_any(const void* data, Shared<NS>& L, int cnt) {
  int lane = __lane_id();
  asm volatile("" : "+v"(lane));
  const Lane ln(lane);
#pragma unroll 1
  for (int p = 0; p < cnt; p += 4) {
    const int slot = L.order[p + ln.blk < cnt ? p + ln.blk : cnt - 1];
    const uint32_t geo = L.geo[slot];
    const bool fresh = (geo & kGeoNew) != 0;
    Raw<DT> px[4 * CH][CH];
    evaluate_four<NS, CH, DT, false>(data, ln, L, slot, px, Candidate{L.x[slot], L.y[slot], L.hx[slot], L.hy[slot]},
                              L.off[slot], geo, true, __builtin_amdgcn_ballot_w64(fresh) != 0, fresh);
  }
}

// The kernel's arguments, read anew where they are used (scalar loads from the
// argument segment) instead of held in scalar registers over the whole fit,
// where they do not fit.
typedef const __attribute__((address_space(4))) KArgs* ArgPtr;
template <bool ANEW = true>
__device__ __forceinline__ ArgPtr args() {
  ArgPtr p = (ArgPtr)__builtin_amdgcn_kernarg_segment_ptr();
  if constexpr (ANEW) asm volatile("" : "+s"(p));
  return p;
}

// Results of spot s.
__device__ __forceinline__ void write_out(ArgPtr ka, int64_t s, const double (&p)[4], double a, double b,
                                          double chi, int it, int status, int n_grad, int n_trial) {
  float* po = ka->params_out + 6 * s;
#pragma unroll
  for (int q = 0; q < 4; ++q) po[q] = float(p[q]);
  po[4] = float(a);
  po[5] = float(b);
  ka->chi2_out[s] = float(chi);
  ka->iters_out[s] = it;
  ka->status_out[s] = status;
  int32_t* ev = ka->evals_out;
  if (ev) {
    ev[2 * s] = n_grad;
    ev[2 * s + 1] = n_trial;
  }
}

// Normal equations.  Parameter j of (x, y, sx, sy) has df_j = dx^ox dy^oy w_j f.
__device__ __forceinline__ constexpr int order_x(int j) { return j == 0 ? 1 : j == 2 ? 2 : 0; }
__device__ __forceinline__ constexpr int order_y(int j) { return j == 1 ? 1 : j == 3 ? 2 : 0; }

// Eq. 7 sums of one parameter and its Eq. 8 amplitude derivatives.
struct Param {
  double dF, dFG, da, db, aS, aF, W, Z;
};
// X, Y: sums dx^ox ex, dy^oy ey; Xq, Yq: of ex^2, ey^2; B: sum g dx^ox dy^oy f.
__device__ __forceinline__ Param param(const Amplitudes& am, double Nn, double Gs, double FG, double X,
                                       double Y, double Xq, double Yq, double B, double wt) {
  Param r;
  r.dF = X * Y * wt;
  const double Sfd = Xq * Yq * wt;
  r.dFG = B * wt;
  const double dFF = 2.0 * Sfd;
  const double gam = __builtin_fma(Nn, dFF, -(2.0 * am.F * r.dF));
  r.da = __builtin_fma(Nn, r.dFG, -__builtin_fma(Gs, r.dF, am.a * gam)) * am.iD;
  r.db = __builtin_fma(Gs, dFF, -__builtin_fma(FG, r.dF, __builtin_fma(am.F, r.dFG, am.b * gam))) * am.iD;
  r.aS = am.a * Sfd;
  r.aF = am.a * r.dF;
  r.W = __builtin_fma(r.da, am.FF, __builtin_fma(r.db, am.F, r.aS));
  r.Z = __builtin_fma(r.da, am.F, __builtin_fma(r.db, Nn, r.aF));
  return r;
}
// Right-hand side J_j^T (g - h).
__device__ __forceinline__ double param_rhs(const Amplitudes& am, double Nn, double Gs, double FG,
                                            const Param& q) {
  // sum f r and sum r (0 up to rounding, Eq. 4)
  const double sfr = __builtin_fma(am.a, am.FF, __builtin_fma(am.b, am.F, -FG));
  const double sr = __builtin_fma(am.a, am.F, __builtin_fma(am.b, Nn, -Gs));
  return -__builtin_fma(q.da, sfr,
                        __builtin_fma(am.a, __builtin_fma(am.b, q.dF, q.aS) - q.dFG, q.db * sr));
}
// Entry (i, j) of J^T J, with J_j = da_j f + a df_j + db_j (Eq. 9, second factor):
//   da_i W_j + db_i Z_j + a (da_j Sfd_i + db_j dF_i) + a^2 sum df_i df_j
// with W_j = da_j FF + a Sfd_j + db_j F and Z_j = da_j F + a dF_j + N db_j.
// Xq, Yq: sums dx^(ox_i + ox_j) ex^2, dy^(oy_i + oy_j) ey^2; wt = w_i w_j.
__device__ __forceinline__ double normal_entry(const Param& pi, const Param& pj, double a2, double Xq,
                                               double Yq, double wt) {
  return __builtin_fma(pi.da, pj.W,
                       __builtin_fma(pi.db, pj.Z,
                                     __builtin_fma(pj.da, pi.aS, __builtin_fma(pj.db, pi.aF, a2 * (Xq * Yq * wt)))));
}
// Symmetric spots, sigma = sx = sy: contracted along d/dsigma = d/dsx + d/dsy,
// padded with identity (A: 00 01 02 03 11 12 13 22 23 33).
__device__ __forceinline__ void contract(double (&A)[10], double (&bv)[4]) {
  A[2] += A[3];
  A[3] = 0.0;
  A[5] += A[6];
  A[6] = 0.0;
  A[7] += __builtin_fma(2.0, A[8], A[9]);
  A[8] = 0.0;
  A[9] = 1.0;
  bv[2] += bv[3];
  bv[3] = 0.0;
}

// Of 4 slots: the entries of a slot's normal equations, one per lane of its
// block (row k, column v), into L.A.
__device__ __forceinline__ void spread_normal(const Lane& ln, Shared<4>& L, int slot, const Amplitudes& am,
                                              double Nn, double Gs, double FG, double sx, double sy) {
  const double isx = rcp_nr(sx), isy = rcp_nr(sy);
  auto weight = [&](int j) {
    const double r = j & 1 ? isy : isx;
    const double r2 = r * r;
    return j < 2 ? r2 : r2 * r;
  };
  auto at = [&](int order, int zero, int one, int two) {
    return L.tot[order == 0 ? zero : order == 1 ? one : two][slot];
  };
  auto of = [&](int j, double wt) {
    const int ox = order_x(j), oy = order_y(j);
    return param(am, Nn, Gs, FG, at(ox, kSx, kX1, kX2), at(oy, kSy, kY1, kY2), at(ox, kSxx, kXq1, kXq2),
                 at(oy, kSyy, kYq1, kYq2), L.tot[j == 0 ? kBx : j == 1 ? kBy : j == 2 ? kBsx : kBsy][slot], wt);
  };
  const int i = ln.k, j = ln.v;
  const double wi = weight(i), wj = weight(j);
  const Param pi = of(i, wi), pj = of(j, wj);
  const int ox = order_x(i) + order_x(j), oy = order_y(i) + order_y(j);
  const double Xq = L.tot[ox == 0 ? kSxx : ox == 1 ? kXq1 : ox == 2 ? kXq2 : ox == 3 ? kXq3 : kXq4][slot];
  const double Yq = L.tot[oy == 0 ? kSyy : oy == 1 ? kYq1 : oy == 2 ? kYq2 : oy == 3 ? kYq3 : kYq4][slot];
  const double entry = normal_entry(pi, pj, am.a * am.a, Xq, Yq, wi * wj);
  const double rhs = param_rhs(am, Nn, Gs, FG, pj);
  // entry (i, j), i <= j, of the upper triangle is number i (7 - i) / 2 + j
  if (i <= j) L.A[i * (7 - i) / 2 + j][slot] = entry;
  if (i == 0) L.A[10 + j][slot] = rhs;
}

template <int NS, int CH, int DT, bool LONE>
__device__ __forceinline__ void fit_matrix(const MatrixQueue& mq, Shared<NS>& L) {
  constexpr int HM = 16 * CH;
  constexpr bool kKeepA = Shared<NS>::kKeepA;
  const int lane = __lane_id();
  // Slots and their owners: lane l < NS owns slot l; of 4 slots, all 16 lanes of
  // a block own its slot, each taking the same steps, so that they can share out
  // the normal equations.  lead: the owner that speaks for its slot.
  constexpr bool kBlocks = NS == 4;
  const int own = kBlocks ? (lane >> 2) & 3 : lane;
  const bool owner = lane < NS || kBlocks;
  const bool lead = kBlocks ? (lane & 0x33) == 0 : owner;
  // rank of the lane's slot among those whose lead's bit is set in m
  auto rank_of = [&](uint64_t m) {
    if constexpr (kBlocks) return __builtin_popcountll(m & ((1ull << (4 * own)) - 1));
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
  };

  // a wavefront of 4 slots is there for short steps: it does not wait for its
  // arguments again
  const auto args = [] { return mtx::args<!kBlocks>(); };
  const void* data = args()->data;

  // ---- the owner's state (its candidate is in L; of 4 slots: in registers) ----
  int32_t s = -1;
  double pc[4] = {0.0, 0.0, 1.0, 1.0};  // candidate
  Candidate cand{};
  int64_t off = 0;
  uint32_t geo = 0;
  Raw<DT> px[4 * CH][CH];
  int k = 0, it = 0, mode = kNew, n_grad = 0, n_trial = 0;
  bool small = false;
  double best[4] = {0.0, 0.0, 0.0, 0.0};  // point at the start of the iteration
  double chi_best = 0.0, a_best = 0.0, b_best = 0.0, chib_err = 0.0;

  // The candidate pc, for the next evaluation.
  auto publish = [&](bool fresh) {
    cand = Candidate{pc[0], pc[1], -0.5 * rcp_nr(pc[2] * pc[2]), -0.5 * rcp_nr(pc[3] * pc[3])};
    if constexpr (!kBlocks) {
      L.x[own] = cand.x;
      L.y[own] = cand.y;
      L.sx[own] = pc[2];
      L.sy[own] = pc[3];
      L.hx[own] = cand.hx;
      L.hy[own] = cand.hy;
      L.geo[own] = geo;
      if (fresh) L.off[own] = off;
    }
  };
  // Taking a spot, in two steps so that its loads are in flight over other work:
  // look up queue position pos, then start the spot (an unusable one ends here).
  struct Next {
    spotfit_shape_t sh;
    int64_t off;
    float i0, i1, i2, i3;
  };
  auto look_up = [&](int32_t pos, Next& nx) {
    s = mq.spot(pos);
    if (s < 0) return;
    const ArgPtr ka = args();
    nx.sh = ka->sizes[s];
    nx.off = ka->offsets[s];
    const float* in = ka->init + 4 * (int64_t)s;
    nx.i0 = in[0];
    nx.i1 = in[1];
    nx.i2 = in[2];
    nx.i3 = in[3];
  };
  auto begin = [&](const Next& nx) {
    const ArgPtr ka = args();
    const spotfit_shape_t nsh = nx.sh;
    const int64_t noff = nx.off;
    const float4 nin = make_float4(nx.i0, nx.i1, nx.i2, nx.i3);
    const bool ell = nsh.model == SPOTFIT_ELL;
    const int max_side = ka->opt.max_side < HM ? ka->opt.max_side : HM;
    const bool bad = nsh.w < 3 || nsh.h < 3 || nsh.w * nsh.h > ka->opt.max_pixels || nsh.w > max_side ||
                     nsh.h > max_side || (nsh.model != SPOTFIT_SYM && !ell) || !__builtin_isfinite(nin.x) ||
                     !__builtin_isfinite(nin.y) || !__builtin_isfinite(nin.z) || !(nin.z > 0.f) ||
                     (ell && (!__builtin_isfinite(nin.w) || !(nin.w > 0.f)));
    if (bad) {
      const double nan = __builtin_nan("");
      const double p4[4] = {nan, nan, nan, nan};
      if (lead) write_out(ka, s, p4, nan, nan, nan, 0, SPOTFIT_BAD_INPUT, 0, 0);
      s = -1;
      return;
    }
    pc[0] = nin.x;
    pc[1] = nin.y;
    pc[2] = nin.z;
    pc[3] = ell ? nin.w : nin.z;
    off = noff;
    geo = uint32_t(nsh.w) | uint32_t(nsh.h) << 8 | kGeoNew | (ell ? kGeoEll : 0u);
    publish(true);
    k = ka->opt.lambda0_exp10;
    it = 0;
    mode = kNew;
    n_grad = n_trial = 0;
  };

  constexpr int C = chunk_of(NS);
  const int counter = blockIdx.x % kMatrixCounters;
  int32_t* const take = mq.take ? mq.take + counter * kMatrixCounterWords : nullptr;
  // position r of the wavefront's chunks q, q + 1, .. (of its counter)
  auto position = [&](int q, int r) { return ((q + r / C) * kMatrixCounters + counter) * C + r % C; };
  bool left = mq.take != nullptr;  // the counter may hold more positions
  int pool = 0, pool_end = 0;      // what is left of the last chunk drawn
  {
    Next nx;
    const int wave = blockIdx.x / kMatrixCounters;
    if (owner)
      look_up(left ? position(wave * (NS / C), own) : own < mq.per ? (int32_t)blockIdx.x * mq.per + own : -1, nx);
    if (lane < 2 * kP10 + 1) L.p10[lane] = kPow10[lane];
    if (s >= 0) begin(nx);
  }

  while (left || __builtin_amdgcn_ballot_w64(s >= 0) != 0) {
    // ================= the slots to evaluate, new spots first =================
    const bool act = s >= 0;
    const bool fresh = act && mode == kNew;
    const uint64_t m_act = __builtin_amdgcn_ballot_w64(act && lead);
    const uint64_t m_new = __builtin_amdgcn_ballot_w64(fresh && lead);
    const int cnt = __builtin_popcountll(m_act);
    int w = geo & 0xff, h = (geo >> 8) & 0xff;
    if (cnt > 0) {
      const int lead0 = __builtin_ctzll(m_act);
      if constexpr (kBlocks) {
        // block b evaluates slot b, from registers; a block without a spot goes
        // along on the first one's pixels
        const int2 o = __builtin_bit_cast(int2, off);
        const int2 o0 = make_int2(__builtin_amdgcn_readlane(o.x, lead0), __builtin_amdgcn_readlane(o.y, lead0));
        const uint32_t geo0 = (uint32_t)__builtin_amdgcn_readlane((int)geo, lead0);
        int l = lane;
        // where its registers are short: formed once a step, not held
        if constexpr (CH == 1 || DT != SPOTFIT_U16) asm volatile("" : "+v"(l));
        evaluate_four<NS, CH, DT, LONE>(data, Lane(l), L, own, px, cand,
                                        act ? off : __builtin_bit_cast(int64_t, o0), act ? geo : geo0,
                                        m_new != 0, m_new != 0, fresh);
      } else {
        wave_lds_sync();
        geo = L.geo[owner ? own : 0];
        w = geo & 0xff;
        h = (geo >> 8) & 0xff;
        const uint32_t geo0 = (uint32_t)__builtin_amdgcn_readlane((int)geo, lead0) & 0xffffu;
        const int T = ((geo0 & 0xff) + 3) >> 2, Tr = ((geo0 >> 8) + 3) >> 2;
        // (16 slots, which batches of 8,000 to 32,000 spots take, have neither of the
        // two kinds of passes below: their code made every step 2 % longer)
        constexpr bool kMany = NS > 16;
        const bool uni = (kMany || T == Tr) && __builtin_amdgcn_ballot_w64(act && (geo & 0xffffu) != geo0) == 0;
        // small spots of any shapes go through passes of two tiles, the next one's
        // pixels ahead: 1M of 4..8 px 805 us of 16-bit pixels (910 in passes by size),
        // 994 of floats (1150)
        const bool small = kMany && !uni && __builtin_amdgcn_ballot_w64(act && tiles_of(geo) > 2) == 0;
        int rank = 0;
        if (uni || small) {  // new spots first, so that few passes form their sums of g and g^2
          rank = fresh ? rank_of(m_new) : rank_of(m_act & ~m_new) + __builtin_popcountll(m_new);
        } else {  // by size, so that few passes go over the tiles of a large spot
          const int tiles = tiles_of(geo);
          int before = 0;
#pragma unroll
          for (int t = 4 * CH; t >= 1; --t) {
            const uint64_t m = __builtin_amdgcn_ballot_w64(act && tiles == t);
            if (tiles == t) rank = before + rank_of(m);
            before += __builtin_popcountll(m);
          }
        }
        if (act) L.order[rank] = own;
        wave_lds_sync();
        const int cnt_new = __builtin_popcountll(m_new);
        if (__builtin_expect(small, 0)) {
          if constexpr (kMany) evaluate_uniform<NS, DT, 2, 2, false, true>(data, L, cnt, cnt_new, geo0);
        } else if (uni) {
          unrolled<4 * CH - 1>([&](auto ti) {
            constexpr int TB = decltype(ti)::value + 2;
            if (T != TB && !(TB == 2 && T < 2)) return;
            if (!kMany || __builtin_expect(Tr == TB || (TB == 2 && Tr < 2), 1))
              evaluate_uniform<NS, DT, TB, TB, false>(data, L, cnt, cnt_new, geo0);
            else if constexpr (kMany)
              evaluate_uniform<NS, DT, TB, 4 * CH, true>(data, L, cnt, cnt_new, geo0);
          });
        } else {
          evaluate_any<NS, CH, DT>(data, L, cnt);
        }
      }
      wave_lds_sync();
    }

    // ================= the owner's scalar steps =================
    const bool sym = !(geo & kGeoEll);
    const double Nn = double(w * h);
    double A[10], bv[4];
    double Sx, Sxx, Sy, Syy, FG, Gs, chi = 0.0, chi_err = 0.0;
    Amplitudes am{};
    bool do_grad = false, do_solve = false, near_self = false, near_best = false;
    if (act) {
      const ArgPtr ka = args();
      if constexpr (!kBlocks) {
        pc[0] = L.x[own];
        pc[1] = L.y[own];
        pc[2] = L.sx[own];
        pc[3] = L.sy[own];
      }
      Sx = L.tot[kSx][own];
      Sxx = L.tot[kSxx][own];
      Sy = L.tot[kSy][own];
      Syy = L.tot[kSyy][own];
      FG = L.tot[kFG][own];
      Gs = L.tot[kG][own];
      am = amplitudes(Nn, Sx, Sxx, Sy, Syy, FG, Gs);
      if constexpr (DT == SPOTFIT_U16) {
        const double Vs = __builtin_fma(Nn, L.tot[kGG][own], -(Gs * Gs));  // every step exact
        chi_closed(Vs, am, Nn, FG, Gs, w, h, chi, chi_err);
        // a decision closer to its threshold than the closed form's error bound
        // is taken with chi^2 summed over the pixels (the best point's too when
        // that comparison involves it), so that it is the one that sum takes
        if (mode != kRegrad && chi_err > 0.0) {
          near_self = fabs(chi - ka->opt.max_error_per_px * Nn) <= chi_err;
          if (mode != kNew) {
            const double e2 = chi_err + chib_err;
            near_best = fabs(chi - chi_best * ka->opt.one_minus_tau) <= e2 ||
                        fabs(chi - chi_best * ka->opt.one_plus_tau) <= e2 ||
                        fabs(chi - chi_best * ka->opt.one_minus_min_delta) <= e2;
          }
        }
      } else {
        chi = L.tot[kChi][own];
      }
    }
    if constexpr (DT == SPOTFIT_U16 && kBlocks) {
      bool want = near_self || near_best;
      bool of_best = false;  // first the candidates' sums, then the best points'
#pragma unroll 1
      while (__builtin_amdgcn_ballot_w64(want) != 0) {
        Candidate at = cand;
        double alpha = am.a, beta = am.b;
        if (of_best) {
          at = Candidate{best[0], best[1], -0.5 * rcp_nr(best[2] * best[2]), -0.5 * rcp_nr(best[3] * best[3])};
          alpha = a_best;
          beta = b_best;
        }
        const double c2 = block_residuals<CH, DT>(px, at, geo, alpha, beta);
        if (want) {
          if (of_best) {
            chi_best = c2;
            chib_err = 0.0;
          } else {
            chi = c2;
            chi_err = 0.0;
          }
        }
        want = !of_best && near_best && chib_err > 0.0;
        of_best = true;
      }
    } else if constexpr (DT == SPOTFIT_U16) {
      bool want = near_self || near_best;
      if (__builtin_amdgcn_ballot_w64(want) != 0) {
        bool of_best = false;  // first the candidates' sums, then the best points'
#pragma unroll 1
        for (int round = 0; round < 2; ++round) {
          const uint64_t m = __builtin_amdgcn_ballot_w64(want && lead);
          if (m == 0) break;
          wave_lds_sync();
          if (want) {
            L.order[rank_of(m)] = own;
            L.ra[own] = of_best ? a_best : am.a;
            L.rb[own] = of_best ? b_best : am.b;
            if (of_best) {
              L.x[own] = best[0];
              L.y[own] = best[1];
              L.hx[own] = -0.5 * rcp_nr(best[2] * best[2]);
              L.hy[own] = -0.5 * rcp_nr(best[3] * best[3]);
            }
          }
          wave_lds_sync();
          sum_residuals<NS, CH>(data, L, __builtin_popcountll(m));
          wave_lds_sync();
          if (want) {
            const double c2 = L.tot[kChi][own];
            if (of_best) {
              chi_best = c2;
              chib_err = 0.0;
            } else {
              chi = c2;
              chi_err = 0.0;
            }
          }
          want = near_best && chib_err > 0.0;
          of_best = true;
        }
      }
    }
    if (act) {
      const ArgPtr ka = args();
      const double a = am.a, b = am.b, Tme = ka->opt.max_error_per_px * Nn;
      const bool okD = am.D > 0.0 && __builtin_isfinite(am.D);
      if (!okD || !__builtin_isfinite(chi) || !__builtin_isfinite(a) || !__builtin_isfinite(b))
        chi = __builtin_nan("");
      if (mode == kTrialFirst || mode == kTrialRetry) ++n_trial;

      // ----------------- decisions (Fit2DGaussian loop) -----------------
      bool start = false, done = false, out_best = false;
      int status = SPOTFIT_MAX_ITER;
      if (mode == kRegrad) {
        // the best point's normal equations once more, for the retry from it
        mode = kTrialRetry;
        do_grad = do_solve = true;
      } else if (mode == kNew) {
        start = true;
      } else {
        if (mode == kTrialFirst && chi < chi_best * ka->opt.one_minus_tau) --k;  // improved: less damping
        const bool worse = chi_best * ka->opt.one_plus_tau < chi;
        if (!small && worse && k < ka->opt.lambda_max_exp10) {
          ++k;  // more damping, retry from best
          if constexpr (kKeepA) {
            mode = kTrialRetry;
            do_solve = true;
          } else {
            mode = kRegrad;
#pragma unroll
            for (int q = 0; q < 4; ++q) pc[q] = best[q];
          }
        } else if (worse || __builtin_isnan(chi)) {
          status = SPOTFIT_NOT_CONVERGED;
          out_best = true;
          done = true;
        } else if (chi < Tme) {
          status = SPOTFIT_MAX_ERROR;
          done = true;
        } else if (chi_best * ka->opt.one_minus_min_delta < chi) {
          status = SPOTFIT_MIN_DELTA;
          done = true;
        } else if (small) {
          status = SPOTFIT_MIN_STEP;
          done = true;
        } else {
          start = true;
        }
      }
      if (start) {  // a new iteration at the accepted point pc
        if (it >= ka->opt.max_iter) {
          done = true;
        } else {
          ++it;
          ++n_grad;
          if (__builtin_isnan(chi)) {
            status = SPOTFIT_NOT_CONVERGED;
            done = true;
          } else if (chi < Tme) {
            status = SPOTFIT_MAX_ERROR;
            done = true;
          } else {
            chi_best = chi;
            chib_err = chi_err;
            a_best = a;
            b_best = b;
#pragma unroll
            for (int q = 0; q < 4; ++q) best[q] = pc[q];
            mode = kTrialFirst;
            do_grad = true;
            do_solve = true;
          }
        }
      }
      if (done) {
        double p4[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) p4[q] = out_best ? best[q] : pc[q];
        if (lead) write_out(ka, s, p4, out_best ? a_best : a, out_best ? b_best : b, out_best ? chi_best : chi, it,
                  status, n_grad, n_trial);
        s = -1;
      }
    }

    // spots for the owners without one: the counter's answer, then their
    // descriptions, come in over the normal equations and the solve
    const uint64_t m_free = left ? __builtin_amdgcn_ballot_w64(lead && s < 0) : 0;
    const int need = __builtin_popcountll(m_free), have = pool_end - pool;
    const bool taking = m_free != 0 && owner && s < 0;
    int drawn_l0 = 0;
    Next nx;
    if (need > have && lane == 0) drawn_l0 = atomicAdd(take, (need - have + C - 1) / C);

    // ----------------- normal equations at pc (Eqs. 7-9, 11) -----------------
    if constexpr (kBlocks) {
      if (do_grad) {
        int l = lane;
        asm volatile("" : "+v"(l));  // the lane's rows of totals are looked up here, not held
        spread_normal(Lane(l), L, own, am, Nn, Gs, FG, pc[2], pc[3]);
      }
      wave_lds_sync();
    } else if (do_grad) {
      const double X[3] = {Sx, L.tot[kX1][own], L.tot[kX2][own]};
      const double Xq[5] = {Sxx, L.tot[kXq1][own], L.tot[kXq2][own], L.tot[kXq3][own], L.tot[kXq4][own]};
      const double Y[3] = {Sy, L.tot[kY1][own], L.tot[kY2][own]};
      const double Yq[5] = {Syy, L.tot[kYq1][own], L.tot[kYq2][own], L.tot[kYq3][own], L.tot[kYq4][own]};
      // sum g d_j f / w_j for x, y, sx, sy
      const double Bj[4] = {L.tot[kBx][own], L.tot[kBy][own], L.tot[kBsx][own], L.tot[kBsy][own]};
      const double isx = rcp_nr(pc[2]), isy = rcp_nr(pc[3]);
      const double wt[4] = {isx * isx, isy * isy, isx * isx * isx, isy * isy * isy};
      Param pp[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        pp[j] = param(am, Nn, Gs, FG, X[order_x(j)], Y[order_y(j)], Xq[order_x(j)], Yq[order_y(j)], Bj[j], wt[j]);
        bv[j] = param_rhs(am, Nn, Gs, FG, pp[j]);
      }
      const double a2 = am.a * am.a;
#pragma unroll
      for (int t = 0; t < 10; ++t) {
        const int i = t < 4 ? 0 : t < 7 ? 1 : t < 9 ? 2 : 3;
        const int j = t < 4 ? t : t < 7 ? t - 3 : t < 9 ? t - 5 : 3;
        A[t] = normal_entry(pp[i], pp[j], a2, Xq[order_x(i) + order_x(j)], Yq[order_y(i) + order_y(j)],
                            wt[i] * wt[j]);
      }
      if (sym) contract(A, bv);
      if constexpr (kKeepA) {
#pragma unroll
        for (int q = 0; q < 10; ++q) L.A[q][own] = A[q];
#pragma unroll
        for (int q = 0; q < 4; ++q) L.A[10 + q][own] = bv[q];
      }
    }

    {
      if (m_free) {
        const int rank = rank_of(m_free);
        int32_t pos = pool + rank;
        pool += need;
        if (need > have) {
          const int q = mq.first + __builtin_amdgcn_readfirstlane(drawn_l0);
          if (rank >= have) pos = position(q, rank - have);
          pool = position(q, need - have - 1) + 1;
          pool_end = position(q, (need - have - 1) / C * C) + C;
        }
        left = pool < mq.count;  // positions only grow
        if (taking) look_up(pos, nx);
      }

      // ----------------- damped step (Eq. 14) and limit() -----------------
      if (do_solve) {
        const ArgPtr ka = args();
        if constexpr (kKeepA) {
          if (kBlocks || !do_grad) {
#pragma unroll
            for (int q = 0; q < 10; ++q) A[q] = L.A[q][own];
#pragma unroll
            for (int q = 0; q < 4; ++q) bv[q] = L.A[10 + q][own];
            if (kBlocks && sym) contract(A, bv);
          }
        }
        double d[4];
        const double lam = k >= -kP10 && k <= kP10 ? L.p10[k + kP10] : pow10i(k);
        damped_step(A, bv, lam, d);
        const double smin = ka->opt.sigma_min, smax = ka->opt.sigma_max_frac * double(w > h ? w : h);
        const double rel = ka->opt.min_step_rel;
        const double p2 = clampn(best[2] + d[2], smin, smax);
        pc[0] = clampn(best[0] + d[0], -0.5, double(w) - 0.5);
        pc[1] = clampn(best[1] + d[1], -0.5, double(h) - 0.5);
        pc[2] = p2;
        pc[3] = sym ? p2 : clampn(best[3] + d[3], smin, smax);
        // MinStep: every step below min_step_rel of its parameter, the centre
        // measured from the centre of the ROI
        small = fabs(d[0]) < rel * fabs(best[0] - 0.5 * double(w - 1)) &&
                fabs(d[1]) < rel * fabs(best[1] - 0.5 * double(h - 1)) &&
                fabs(d[2]) < rel * fabs(best[2]) && (sym || fabs(d[3]) < rel * fabs(best[3]));
      }
      if (act) {
        geo &= ~kGeoNew;
        publish(false);
      }
    }
    if (taking && s >= 0) begin(nx);
  }
}

// LONE: a wavefront has a SIMD for itself, and its registers: wide floats of 4 slots,
// whose pixels take 64 of them, spill none there, and have room for the passes of
// uneven spots (which cost the others 2 to 6 %).  32 floats of 30x12 32.4 us without
// it, 24.5 so (26.0 with a lane per column), of 32x32 32.7, 32.4 (30.2).  A batch that
// needs two wavefronts per SIMD is slower so (10,000 of 32x32 76 us, 118).
template <int NS, int CH, int DT, bool LONE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(LONE ? 1 : CH == 1 && (NS == 4 || (NS == 16 && DT == SPOTFIT_U16)) ? 3 : 2))) void fit_matrix_kernel(
    KArgs /* read through args() */, MatrixQueue mq) {
  __shared__ Shared<NS> lds;
  fit_matrix<NS, CH, DT, LONE>(mq, lds);
}

__global__ void matrix_queue_reset_kernel(int32_t* take) {
  if (threadIdx.x < kMatrixCounters) take[threadIdx.x * kMatrixCounterWords] = 0;
}

template <int NS, int CH>
static const void* symbol(int dtype) {
  return dtype == SPOTFIT_U16 ? reinterpret_cast<const void*>(&fit_matrix_kernel<NS, CH, SPOTFIT_U16, false>)
                              : reinterpret_cast<const void*>(&fit_matrix_kernel<NS, CH, SPOTFIT_F32, false>);
}

template <int NS, int CH>
static hipError_t launch(const KArgs& ka, const MatrixQueue& mq, int grid, hipStream_t st) {
  if (ka.dtype == SPOTFIT_U16)
    hipLaunchKernelGGL((fit_matrix_kernel<NS, CH, SPOTFIT_U16, false>), dim3(grid), dim3(64), 0, st, ka, mq);
  else
    hipLaunchKernelGGL((fit_matrix_kernel<NS, CH, SPOTFIT_F32, false>), dim3(grid), dim3(64), 0, st, ka, mq);
  return hipGetLastError();
}

}  // namespace mtx

#define SF_MATRIX_SHAPES(X) \
  X(4, 1) X(16, 1) X(32, 1) X(64, 1) X(4, 2) X(16, 2) X(32, 2) X(64, 2)

const void* matrix_kernel_symbol(int slots, bool wide, int dtype) {
#define SF_MXSYM(NS, CH) \
  if (slots == NS && wide == (CH == 2)) return mtx::symbol<NS, CH>(dtype);
  SF_MATRIX_SHAPES(SF_MXSYM)
#undef SF_MXSYM
  return nullptr;
}

hipError_t launch_matrix_kernel(int slots, bool wide, const KArgs& ka, const MixedWs* ws, int resident,
                                int spread, bool lone, hipStream_t st) {
  const int64_t need = (ka.n + slots - 1) / slots;
  int grid = (int)(need < resident ? need : resident);
  mtx::MatrixQueue mq{};
  mq.count = (int32_t)ka.n;
  if (ws) {
    mq.counts = ws->counters;
    mq.lists = ws->lists;
    mq.cap = ws->cap;
  }
  if (need > grid && grid >= kMatrixCounters) {
    grid -= grid % kMatrixCounters;  // every counter the same wavefronts
    mq.take = ka.queue;
    mq.first = grid / kMatrixCounters * (slots / mtx::chunk_of(slots));
    hipLaunchKernelGGL(mtx::matrix_queue_reset_kernel, dim3(1), dim3(64), 0, st, mq.take);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  } else {
    // of 4 slots and spots of several shapes, as few spots per wavefront as come
    // with `spread` wavefronts: a small spot's steps then don't wait for a large
    // one's tiles, nor either for the other's close decisions (a frame of 110
    // spots of 9..21 px with a wavefront per spot 57.0 us, with four spots each
    // 61.0; of one shape it does not pay: 32 spots of 13x13 31.3 and 30.5, 1,024
    // of 11x11 19.3 and 17.9)
    mq.per = slots;
    if (slots == 4 && spread > 0)
      for (mq.per = 1; mq.per < 4 && (ka.n + mq.per - 1) / mq.per > spread;) mq.per *= 2;
    grid = (int)((ka.n + mq.per - 1) / mq.per);
  }
  if (lone && slots == 4 && wide && ka.dtype == SPOTFIT_F32 && !mq.take) {
    hipLaunchKernelGGL((mtx::fit_matrix_kernel<4, 2, SPOTFIT_F32, true>), dim3(grid), dim3(64), 0, st, ka, mq);
    return hipGetLastError();
  }
#define SF_MXLAUNCH(NS, CH) \
  if (slots == NS && wide == (CH == 2)) return mtx::launch<NS, CH>(ka, mq, grid, st);
  SF_MATRIX_SHAPES(SF_MXLAUNCH)
#undef SF_MXLAUNCH
  return hipErrorInvalidValue;
}

}  // namespace sf
