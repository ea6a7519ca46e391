// wts_soft.h -- what the Soft-DTW kernels share: Soft-DTW forward (Eq. 3-5;
// wts_soft.hip and, for batches of few strips, wts_soft_team.hip) and its
// gradient (Eq. 6; wts_soft_bwd.hip, a workgroup a strip, and wts_soft_wave.hip,
// one wave a strip; wts_soft_link.h joins the strips) for gfx950.
//
// Units.  The cumulative costs are kept scaled, R' = R * k with
// k = log2(e) / gamma, so the soft-min of Eq. 3 becomes
//   min'(a, b, c) = m - log2(2^(m-a) + 2^(m-b) + 2^(m-c)),  m = min(a, b, c),
// evaluated with float64 differences and the hardware base-2 exponential and
// logarithm (v_exp_f32 / v_log_f32).  Every cost delta enters as delta * k:
// the kernels take the series multiplied by sqrt(k) when they load them, so
// the squared differences come out scaled with no multiply per cell (the
// gradient's sums are scaled back once per row).  The Soft-DTW value is
// r'(M-1, N-1) / k.
//
// Forward.  Same skewed wavefront sweep as the DTW kernels (one wave per strip
// of 64*RHO rows, strips of a pair chained through device memory).  It keeps
// every strip's bottom row and, every 16 sweep steps, the sweep state of each
// lane (its RHO cumulative costs at the previous column and the diagonal
// input from the row above): enough to replay any 16-step tile.
//
// Backward.  E of Eq. 6 follows from Eq. 5 by the chain rule:
//   e(i, j) = sum over the successors s of (i, j) of e(s) * w_s(i, j),
// where w_s(i, j) = 2^(m_s - r'(i, j)) / sum_s is the normalised weight of
// (i, j) in the soft-min of its successor s, and e(M-1, N-1) = 1 (the cell
// that closes the path).  The kernel walks each strip's tiles from the last
// column to the first: a tile is replayed forward, leaving the normalised
// weights of the up and left predecessors of every cell (float32), and then
// swept backwards in "push" form (by other waves of the workgroup, or by the
// same wave) -- each finished cell splits its e over its three predecessors with
// its own weights, the diagonal taking what the other two do not, so that the
// split conserves e up to the rounding of one float32 subtraction -- and no cell ever needs a
// neighbour's weights.  e lies in [0, 1] and travels in float32 (registers,
// lane shifts, LDS and the push rows between strips).  The pushes of a
// strip's top row feed the strip above, so strips are pipelined from the
// bottom up.  Per row l of the barycenter the kernel accumulates, in
// float64, sum_j e(l, j) and sum_j e(l, j) y_j, and the gradient is
//   d Soft-DTW / d b_l = 2 (b_l * sum_j e(l, j) - sum_j e(l, j) y_j).
#pragma once
#include <type_traits>

#include "wts_device.h"
#include "wts_kernels.h"

namespace wts {

namespace {

__device__ __forceinline__ float shl1_f32(float v, float old) {
  // DPP wave_shl:1 -- lane k receives v from lane k+1; lane 63 receives `old`.
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old),
                                                               __builtin_bit_cast(int, v), 0x130,
                                                               0xf, 0xf, false));
}

constexpr int kRing = 128;   // Y columns in LDS (>= 16 + 63 for a tile, power of 2)
// The ring holds kRing + 16 slots: slots kRing .. kRing + 15 mirror slots
// 0 .. 15, so the 16 steps of a group read consecutive slots yb .. yb + 15
// from one base (immediate LDS offsets, no wrap-around per step).
__device__ __forceinline__ void ring_put(double* row, int slot, double v) {
  row[slot] = v;
  if (slot < 16) row[slot + kRing] = v;
}
constexpr int kTile = 16;    // sweep steps per checkpoint / replay tile

// Def. 3's squared cost in the scaled units of these kernels, k |x - y|^2,
// in d + 1 operations per cell: the rows carry x' = sk (x - mu) and
// |x'|^2, the columns y' = sk (y - mu) as -2 y' and |y'|^2, and
// k |x - y|^2 = |x'|^2 + |y'|^2 + x' . (-2 y').  mu, the first row of the
// pair's row series, keeps the three terms of the order of the series'
// spread, so cancellation costs no more than a few roundings of that size.
template <int D>
__device__ __forceinline__ double sq_cost(const double (&x)[D], double xx, const double (&ym2)[D],
                                          double yy) {
  double s = xx + yy;
#pragma unroll
  for (int c = 0; c < D; ++c) s = __builtin_fma(x[c], ym2[c], s);
  return s;
}
template <int D>
__device__ __forceinline__ double sq_norm(const double (&v)[D]) {
  double q = v[0] * v[0];
#pragma unroll
  for (int c = 1; c < D; ++c) q = __builtin_fma(v[c], v[c], q);
  return q;
}
// One column into the Y ring: -2 y' per channel and |y'|^2.
template <int D>
__device__ __forceinline__ void ring_col(double (*ys)[kRing + 16], double* yq, int slot,
                                         const double (&yc)[D]) {
#pragma unroll
  for (int c = 0; c < D; ++c) ring_put(ys[c], slot, -2.0 * yc[c]);
  ring_put(yq, slot, sq_norm<D>(yc));
}

// Soft-min of the three predecessors in scaled units.  Returns the soft-min
// value and the three (unnormalised) base-2 exponentials.
struct SoftMin {
  double v;
  float ed, eu, el, s;
};
__device__ __forceinline__ SoftMin softmin3(double dg, double up, double lf) {
  const double m = __builtin_fmin(__builtin_fmin(dg, up), lf);
  SoftMin o;
  o.ed = __builtin_amdgcn_exp2f((float)(m - dg));
  o.eu = __builtin_amdgcn_exp2f((float)(m - up));
  o.el = __builtin_amdgcn_exp2f((float)(m - lf));
  o.s = (o.ed + o.eu) + o.el;
  o.v = m - (double)__builtin_amdgcn_logf(o.s);
  return o;
}

// Sakoe-Chiba band (the bandwidth of Table I, a fraction w of the longer
// length): cell (i, j) of an M x N pair lies in the band iff
//   |i (N-1) - j (M-1)| <= B,   B = R min(M-1, N-1),
//   R = max(ceil(w max(M, N)), ceil(max(M-1, N-1) / min(M-1, N-1))),
// a band of radius R around the diagonal from (0, 0) to (M-1, N-1) along
// the longer side; the lower bound on R keeps a predecessor in the band for
// every cell of the band but (0, 0).  Returns B, or +inf (every cell) when
// w = 0 or a side has length 1.  The test is done in float64, exact for
// M, N < 2^26 (checked at plan time).
__device__ __forceinline__ double band_halfwidth(int M, int N, double w) {
  if (!(w > 0.0) || M == 1 || N == 1) return __builtin_huge_val();
  const int64_t am = M - 1, bn = N - 1;
  const int64_t mn = am < bn ? am : bn, mx = am < bn ? bn : am;
  int64_t R = (int64_t)__builtin_ceil(w * (double)(M > N ? M : N));
  const int64_t Rmin = (mx + mn - 1) / mn;
  if (R < Rmin) R = Rmin;
  return (double)(R * mn);
}

// Columns of the band over rows i_first .. i_last (the band's left edge is
// non-decreasing in i, so the range runs from row i_first's left edge to row
// i_last's right edge), in exact integer arithmetic: a 16-step group whose
// cells all lie outside it can skip its cell arithmetic.
__device__ __forceinline__ void band_strip_cols(int M, int N, double w, int i_first, int i_last,
                                                int* jlo, int* jhi) {
  *jlo = 0;
  *jhi = N - 1;
  if (!(w > 0.0) || M == 1 || N == 1) return;
  const int64_t am = M - 1, bn = N - 1;
  const int64_t B = (int64_t)band_halfwidth(M, N, w);
  // left edge of row i: ceil((i bn - B) / am); right edge: floor((i bn + B) / am)
  auto floor_div = [](int64_t x, int64_t y) { return x / y - ((x % y != 0) && (x < 0)); };
  const int64_t lo = -floor_div(B - (int64_t)i_first * bn, am);
  const int64_t hi = floor_div((int64_t)i_last * bn + B, am);
  if (lo > 0) *jlo = (int)(lo < bn ? lo : bn);
  if (hi < bn) *jhi = (int)(hi > 0 ? hi : 0);
}

// softmin3 for a cell that may lie outside the band: there every input may
// be +inf, so the shift m is replaced by 0 to keep the arithmetic free of
// inf - inf (the caller discards the result of such a cell).
__device__ __forceinline__ SoftMin softmin3_band(double dg, double up, double lf, bool inb) {
  double m = __builtin_fmin(__builtin_fmin(dg, up), lf);
  m = inb ? m : 0.0;
  SoftMin o;
  o.ed = __builtin_amdgcn_exp2f((float)(m - dg));
  o.eu = __builtin_amdgcn_exp2f((float)(m - up));
  o.el = __builtin_amdgcn_exp2f((float)(m - lf));
  o.s = (o.ed + o.eu) + o.el;
  o.v = m - (double)__builtin_amdgcn_logf(o.s);
  return o;
}

#define WTS_SOFT_D_SWITCH(d, CALL) \
  switch (d) {                     \
    case 1: return CALL(1);        \
    case 2: return CALL(2);        \
    case 3: return CALL(3);        \
    case 4: return CALL(4);        \
    case 5: return CALL(5);        \
    case 6: return CALL(6);        \
    case 7: return CALL(7);        \
    case 8: return CALL(8);        \
    default: return hipErrorInvalidValue; \
  }

}  // namespace

}  // namespace wts
