// FP64 per-(Gaussian, plane) geometry: Eq. 9 transform, Eq. 11 factor,
// Eq. 12/13 culling and boxes, and the in-plane conic of Eq. 8 restricted
// to the probe plane x3 = 0, plus its adjoint.
//
// Derivation (probe frame of one plane, R = [e1 e2 n], m = R^-1 (mu - o)):
//   d^2(x) = |M (x|0 - m)|^2 with M = L^T R, columns b1, b2, b3.
//   G = M^-T = L^-1 R^-T has columns g_k = L^-1 (row k of R^-1); the
//   probe-frame covariance is Sigma'_jk = g_j . g_k, so the Eq. 13 box
//   half-widths are sqrt(chi^2 Sigma'_kk) (the cofactor-over-determinant of
//   the probe-frame precision) and the plane misses the ellipsoid iff
//   r^2 = m3^2 / Sigma'_33 > chi^2.
//   Restricted to x3 = 0 the quadratic is |R_B (x - c)|^2 + r^2 where
//   R_B = [[T11, T12], [0, T22]] is the Cholesky factor of B^T B, B = [b1 b2]:
//   T11 = |b1|, T12 = b1.b2 / T11, T22 = |b1 x b2| / T11 = |det M| |g3| / T11
//   (b1 x b2 = det(M) g3), and the centre is the conditional mean
//   c = m12 - m3 (Sigma'_13, Sigma'_23) / Sigma'_33.
// Everything is evaluated in double precision from the float32 inputs and
// rounded once into the float32 record.
#pragma once

#include "ug_internal.h"

namespace ug {

// Reciprocal and square root of the positive, normal values of the record
// construction (double) and its adjoint (float): the hardware's estimate y and
// one correction.  With e = 1 - x y, the reciprocal is y (1 + e + e^2 + ...):
// two terms for doubles (third order, Halley's form), one for floats
// (Newton's); with e = 1 - x y^2 the reciprocal root is y (1 + e / 2 + 3 e^2 /
// 8 + ...), and the root is Newton's step from x times it.  Within an ulp or
// two; the record is rounded to float right after.
// The exact division and square root take two to four times the
// instructions, and both kernels are bound by their arithmetic.
__device__ __forceinline__ double recip(double x) {
  const double y = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, y, 1.0);
  return fma(y, fma(e, e, e), y);
}
__device__ __forceinline__ float recip(float x) {
  const float y = __builtin_amdgcn_rcpf(x);
  return fmaf(fmaf(-x, y, 1.f), y, y);
}

// root = sqrt(x), inv = 1 / sqrt(x).
__device__ __forceinline__ void root_pair(double x, double& root, double& inv) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  inv = fma(y * e, fma(0.375, e, 0.5), y);
  const double g = x * inv;
  root = fma(fma(-g, g, x), 0.5 * inv, g);
}
__device__ __forceinline__ void root_pair(float x, float& root, float& inv) {
  const float y = __builtin_amdgcn_rsqf(x);
  inv = fmaf(0.5f * y, fmaf(-x * y, y, 1.f), y);
  const float g = x * inv;
  root = fmaf(fmaf(-g, g, x), 0.5f * inv, g);
}

// max and min of two doubles in one instruction (the other operand for a NaN;
// fmax and fmin also quiet each operand first).
__device__ __forceinline__ double max64(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double min64(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// sqrt(x) of x >= 0, kept within [1e-150, 1e150] (no cut-off: x is infinite).
__device__ __forceinline__ double root(double x) {
  double r, i;
  root_pair(min64(max64(x, 1e-300), 1e300), r, i);
  return r;
}

// Gaussian parameters in scalar type T (double for the record construction,
// float for its adjoint, whose tolerance is far looser).
template <typename T>
struct GaussT {
  T mu[3];
  T l[6];  // raw (l11, l21, l31, l22, l32, l33)
  T a, c;
  T L11, L21, L31, L22, L32, L33;
  T iL11, iL22, iL33;  // reciprocals of the diagonal
  T alpha, log2a;
  bool finite;
};
using GaussIn = GaussT<double>;

template <typename T>
struct ConicT {
  T m1, m2, m3;
  T g1[3], g2[3], g3[3];
  T b1[3], b2[3];
  T S11, S22, S33, S13, S23, iS;  // iS = 1 / S33
  T T11, T12, T22, detL, n3;  // n3 = sqrt(S33)
  T iT11, in3;                // reciprocals of T11, n3
  T c1, c2, r2;
};
using Conic = ConicT<double>;

// Plane pose in scalar type T.
template <typename T>
struct PlaneT {
  T o[3], rinv[9], e1[3], e2[3], absdet, sx, sy;
};

// What the record construction reads of a plane: the pose, the pixel index of
// its in-plane origin, the reciprocal spacings and the size.
struct PlaneRec {
  PlaneT<double> pose;
  double cu, cv, isx, isy;
  int W, H;
};

template <typename T>
__device__ __forceinline__ PlaneT<T> plane_as(const PlaneConst& P) {
  PlaneT<T> q;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    q.o[k] = (T)P.o[k];
    q.e1[k] = (T)P.e1[k];
    q.e2[k] = (T)P.e2[k];
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) q.rinv[k] = (T)P.rinv[k];
  q.absdet = (T)P.absdet;
  q.sx = (T)P.sx;
  q.sy = (T)P.sy;
  return q;
}

// A Gaussian's stored parameters as loaded (split from their set-up so a
// kernel can issue the loads early, beside other loads it waits for).
struct GaussRaw {
  float mu[3], l[6], a, c;
};

__device__ __forceinline__ GaussRaw load_gauss_raw(const ug_gaussians& g, int i) {
  GaussRaw r;
#pragma unroll
  for (int k = 0; k < 3; ++k) r.mu[k] = g.means[3 * i + k];
#pragma unroll
  for (int k = 0; k < 6; ++k) r.l[k] = g.lraw[6 * i + k];
  r.a = g.opacity[i];
  r.c = g.intensity[i];
  return r;
}

// exact: divisions for the reciprocals (the float cull's and the box support's
// decisions rest on them).
template <typename T>
__device__ __forceinline__ void gauss_setup(const GaussRaw& r, T beta, GaussT<T>& G, bool exact = false) {
  bool fin = true;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    G.mu[k] = (T)r.mu[k];
    fin = fin && __builtin_isfinite(G.mu[k]);
  }
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    G.l[k] = (T)r.l[k];
    fin = fin && __builtin_isfinite(G.l[k]);
  }
  G.a = (T)r.a;
  G.c = (T)r.c;
  fin = fin && __builtin_isfinite(G.a) && __builtin_isfinite(G.c);
  G.finite = fin;
  // Eq. 11: diagonal entries squared plus beta.
  G.L11 = G.l[0] * G.l[0] + beta;
  G.L21 = G.l[1];
  G.L31 = G.l[2];
  G.L22 = G.l[3] * G.l[3] + beta;
  G.L32 = G.l[4];
  G.L33 = G.l[5] * G.l[5] + beta;
  G.iL11 = exact ? (T)1 / G.L11 : recip(G.L11);
  G.iL22 = exact ? (T)1 / G.L22 : recip(G.L22);
  G.iL33 = exact ? (T)1 / G.L33 : recip(G.L33);
  // alpha = sigmoid(a); log2(alpha) = -softplus(-a) / ln 2, stable for any
  // a.  In single precision for both types: the records hold it in float
  // (e0 and emin), so a double evaluation would only cost time.
  const float na = -(float)G.a;
  const float sp = fmaxf(na, 0.f) + log1pf(expf(-fabsf(na)));
  G.log2a = (T)(-sp * (float)(1.0 / kLn2));
  G.alpha = (T)(1.f / (1.f + expf(na)));
}

template <typename T>
__device__ __forceinline__ void load_gauss(const ug_gaussians& g, int i, T beta, GaussT<T>& G, bool exact = false) {
  gauss_setup(load_gauss_raw(g, i), beta, G, exact);
}

// Forward substitution y = L^-1 q.
template <typename T>
__device__ __forceinline__ void fsub(const GaussT<T>& G, T q0, T q1, T q2, T* y) {
  y[0] = q0 * G.iL11;
  y[1] = (q1 - G.L21 * y[0]) * G.iL22;
  y[2] = (q2 - G.L31 * y[0] - G.L32 * y[1]) * G.iL33;
}

// Back substitution h = L^-T d.
template <typename T>
__device__ __forceinline__ void bsub(const GaussT<T>& G, const T* d, T* h) {
  h[2] = d[2] * G.iL33;
  h[1] = (d[1] - G.L32 * h[2]) * G.iL22;
  h[0] = (d[0] - G.L21 * h[1] - G.L31 * h[2]) * G.iL11;
}

// Phase 1 of Section 4.4: probe coordinates of the mean and the distance of
// the plane from the ellipsoid.  Returns false if the plane misses the
// chi^2 ellipsoid (|m3| > sqrt(chi^2 Sigma'_33), i.e. r^2 > chi^2).
template <typename T>
__device__ __forceinline__ bool conic_cull(const GaussT<T>& G, const PlaneT<T>& P, T chi2, ConicT<T>& k) {
  const T d0 = G.mu[0] - P.o[0], d1 = G.mu[1] - P.o[1], d2 = G.mu[2] - P.o[2];
  k.m3 = P.rinv[6] * d0 + P.rinv[7] * d1 + P.rinv[8] * d2;
  fsub(G, P.rinv[6], P.rinv[7], P.rinv[8], k.g3);
  k.S33 = k.g3[0] * k.g3[0] + k.g3[1] * k.g3[1] + k.g3[2] * k.g3[2];
  return k.m3 * k.m3 <= chi2 * k.S33;  // false for NaN as well
}

// The rest of the conic, after conic_cull accepted the pair.
template <typename T>
__device__ __forceinline__ void conic_full(const GaussT<T>& G, const PlaneT<T>& P, ConicT<T>& k) {
  const T d0 = G.mu[0] - P.o[0], d1 = G.mu[1] - P.o[1], d2 = G.mu[2] - P.o[2];
  k.m1 = P.rinv[0] * d0 + P.rinv[1] * d1 + P.rinv[2] * d2;
  k.m2 = P.rinv[3] * d0 + P.rinv[4] * d1 + P.rinv[5] * d2;
  fsub(G, P.rinv[0], P.rinv[1], P.rinv[2], k.g1);
  fsub(G, P.rinv[3], P.rinv[4], P.rinv[5], k.g2);
  const T iS = recip(k.S33);
  k.iS = iS;
  k.r2 = k.m3 * k.m3 * iS;
  k.S11 = k.g1[0] * k.g1[0] + k.g1[1] * k.g1[1] + k.g1[2] * k.g1[2];
  k.S22 = k.g2[0] * k.g2[0] + k.g2[1] * k.g2[1] + k.g2[2] * k.g2[2];
  k.S13 = k.g1[0] * k.g3[0] + k.g1[1] * k.g3[1] + k.g1[2] * k.g3[2];
  k.S23 = k.g2[0] * k.g3[0] + k.g2[1] * k.g3[1] + k.g2[2] * k.g3[2];
  // b_k = L^T e_k
  k.b1[0] = G.L11 * P.e1[0] + G.L21 * P.e1[1] + G.L31 * P.e1[2];
  k.b1[1] = G.L22 * P.e1[1] + G.L32 * P.e1[2];
  k.b1[2] = G.L33 * P.e1[2];
  k.b2[0] = G.L11 * P.e2[0] + G.L21 * P.e2[1] + G.L31 * P.e2[2];
  k.b2[1] = G.L22 * P.e2[1] + G.L32 * P.e2[2];
  k.b2[2] = G.L33 * P.e2[2];
  root_pair(k.b1[0] * k.b1[0] + k.b1[1] * k.b1[1] + k.b1[2] * k.b1[2], k.T11, k.iT11);
  const T iT11 = k.iT11;
  k.T12 = (k.b1[0] * k.b2[0] + k.b1[1] * k.b2[1] + k.b1[2] * k.b2[2]) * iT11;
  k.detL = G.L11 * G.L22 * G.L33;
  root_pair(k.S33, k.n3, k.in3);
  k.T22 = k.detL * P.absdet * k.n3 * iT11;
  k.c1 = k.m1 - k.m3 * k.S13 * iS;
  k.c2 = k.m2 - k.m3 * k.S23 * iS;
}

__device__ __forceinline__ double cross_norm2(const double* a, const double* b) {
  const double x = a[1] * b[2] - a[2] * b[1];
  const double y = a[2] * b[0] - a[0] * b[2];
  const double z = a[0] * b[1] - a[1] * b[0];
  return x * x + y * y + z * z;
}

// Inclusive pixel-index range covered by [centre - half, centre + half],
// padded so float rounding never drops a pixel the record's own test keeps.
__device__ __forceinline__ bool pixel_range(double centre, double half, int32_t size, int& lo, int& hi) {
  const double pad = 1e-3 + 1e-5 * half;
  double a = centre - half - pad, b = centre + half + pad;
  if (!(a <= b)) return false;  // NaN
  if (b < 0.0 || a > (double)(size - 1)) return false;
  lo = (int)ceil(max64(a, 0.0));
  hi = (int)floor(min64(b, (double)(size - 1)));
  return lo <= hi;
}

struct Footprint {
  RecAcc acc;
  RecGeo geo;
  uint32_t keys;              // keys emitted
  uint32_t counted;           // keys reported and held against the capacity (the PAPER rectangle's tiles)
  RowSpans spans;             // by rows: as in Rec
};

// Column ranges of the record's ellipse over bands of pixel rows.  The
// ellipse is (t11 du + t12 dv)^2 + (t22 dv)^2 <= e0 - emin (du, dv relative
// to the record's centre); its right edge is concave in dv and its left edge
// convex, so the extreme columns over a row band sit at the clamped
// stationary points.  The per-record constants are float (relative error
// ~1e-7, far inside the 1e-5 relative padding); the per-band remainders,
// where cancellation happens near the ellipse's top and bottom, are double,
// with their square roots in float.  Contraction is off, so every kernel
// that calls these gets the same answer bit for bit.
struct BandPrep {
  double thr, t12, t22, inv_t11, u0, v0, vext, dvr;
  bool inf;
};

__device__ __forceinline__ bool band_prep(const RecAcc& ra, int ub, int vb, BandPrep& b) {
#pragma clang fp contract(off)
  b.thr = (double)ra.e0 - (double)ra.emin;  // exact
  if (!(b.thr >= 0.0)) return false;
  b.inf = __builtin_isinf(b.thr);
  if (b.inf) return true;
  b.t12 = ra.t12;
  b.t22 = ra.t22;
  b.inv_t11 = (double)(1.0f / ra.t11);
  b.u0 = (double)ub + (double)ra.fu;
  b.v0 = (double)vb + (double)ra.fv;
  const float sq = __builtin_amdgcn_sqrtf((float)b.thr);
  b.vext = (double)(sq / ra.t22) * (1.0 + 1e-6) + 1e-3;
  const float S = __builtin_amdgcn_sqrtf(ra.t12 * ra.t12 + ra.t22 * ra.t22);
  b.dvr = (double)(-ra.t12 * sq / (ra.t22 * S));  // row offset of the rightmost point; the leftmost is -dvr
  return true;
}

// Column range [ua, uz] of the ellipse over pixel rows [ya, yb], clipped to
// [umin, umax] and padded so float rounding in the accumulation never keeps
// a pixel outside it; false if empty.
__device__ __forceinline__ bool band_cols(const BandPrep& b, int ya, int yb, int umin, int umax, int& ua, int& uz) {
#pragma clang fp contract(off)
  if (b.inf) {
    ua = umin;
    uz = umax;
    return umin <= umax;
  }
  const double lo = max64((double)ya - b.v0, -b.vext), hi = min64((double)yb - b.v0, b.vext);
  if (!(lo <= hi)) return false;
  const double dvr = min64(max64(b.dvr, lo), hi);
  const double dvl = min64(max64(-b.dvr, lo), hi);
  const double qr = max64(b.thr - b.t22 * b.t22 * dvr * dvr, 0.0);
  const double ql = max64(b.thr - b.t22 * b.t22 * dvl * dvl, 0.0);
  const double ur = b.u0 + (-b.t12 * dvr + (double)__builtin_amdgcn_sqrtf((float)qr)) * b.inv_t11;
  const double ul = b.u0 + (-b.t12 * dvl - (double)__builtin_amdgcn_sqrtf((float)ql)) * b.inv_t11;
  const double pad = 1e-3 + 1e-5 * (ur - ul);
  const double a = max64(ul - pad, (double)umin), c = min64(ur + pad, (double)umax);
  if (!(a <= c)) return false;
  ua = (int)ceil(a);
  uz = (int)floor(c);
  return ua <= uz;
}

// The same column ranges for the sub-block masks of the emission, in single
// precision relative to the record's centre and widened further (a mask may
// name a sub-block too many, whose pairs add exact zeros; it must not miss
// one).  At row offset dv the ellipse spans -(t12 / t11) dv -/+
// sqrt(d - t22^2 dv^2) / t11, with its right end at dvr and its left at -dvr.
// The plane's own columns relative to the centre are exact in single precision
// up to kFarColumns pixels from it; a record farther away (a plane that is
// tiny against the Gaussian) takes every sub-block of its tiles.
constexpr int kFarColumns = 1 << 23;
struct BandMask {
  float t22, a, i11, d, dvr, fu, fv;
  int ub, vb;
  bool all;  // no cut-off, a constant that is not finite, or a far centre
};

__device__ __forceinline__ bool band_mask_prep(const RecAcc& ra, int ub, int vb, BandMask& b) {
  const float d = ra.e0 - ra.emin;
  b.i11 = __builtin_amdgcn_rcpf(ra.t11);
  b.t22 = ra.t22;
  b.a = ra.t12 * b.i11;
  b.d = d * 1.0001f;
  const float iS = __builtin_amdgcn_rcpf(fmaf(ra.t12, ra.t12, ra.t22 * ra.t22));
  b.dvr = -ra.t12 * __builtin_amdgcn_sqrtf(d * iS) * __builtin_amdgcn_rcpf(ra.t22);
  b.fu = ra.fu;
  b.fv = ra.fv;
  b.ub = ub;
  b.vb = vb;
  b.all = !(d < 1e30f && fabsf(b.a) < 1e12f && fabsf(b.dvr) < 1e12f && b.i11 < 1e12f && ra.t22 < 1e12f &&
            ub >= -kFarColumns && ub <= kFarColumns);
  return d >= 0.f;
}

// Sub-block columns [ca, cz] (of 8 pixels) the ellipse may reach in the rows
// [lo, hi] below the centre's pixel row, cut to the pixel columns [umin, umax]
// (>= 0); ca > cz if none.
__device__ __forceinline__ void band_mask_cols(const BandMask& b, float lo, float hi, int umin, int umax, int& ca,
                                               int& cz) {
  const float pv = fmaf(2e-6f, fmaxf(fabsf(lo), fabsf(hi)), 2e-3f);
  const float vr = __builtin_amdgcn_fmed3f(b.dvr, lo - pv, hi + pv);
  const float vl = __builtin_amdgcn_fmed3f(-b.dvr, lo - pv, hi + pv);
  const float tr = b.t22 * vr, tl = b.t22 * vl;
  const float qr = fmaf(-tr, tr, b.d), ql = fmaf(-tl, tl, b.d);
  const float ur = fmaf(-b.a, vr, __builtin_amdgcn_sqrtf(fmaxf(qr, 0.f)) * b.i11);
  const float ul = fmaf(-b.a, vl, -__builtin_amdgcn_sqrtf(fmaxf(ql, 0.f)) * b.i11);
  const float pu = fmaf(1e-5f, fmaxf(fabsf(ur), fabsf(ul)), 3e-3f);
  // columns relative to the centre's pixel, cut before the conversion
  const float fl = fmaxf(ceilf(ul + b.fu - pu), (float)(umin - b.ub));
  const float fr = fminf(floorf(ur + b.fu + pu), (float)(umax - b.ub));
  const bool any = qr >= 0.f && fl <= fr;  // qr < 0: the rows lie beside the ellipse
  ca = any ? ((int)fl + b.ub) >> 3 : 1;
  cz = any ? ((int)fr + b.ub) >> 3 : 0;
  static_assert(kSubBlock == 8, "shift");
  if (b.all) {
    ca = umin >> 3;
    cz = umax >> 3;
  }
}

// Mask of the sub-blocks of tile column tx that the bands' columns reach (K =
// TW / 8 column blocks per band, NB bands).
template <int NB, int K>
__device__ __forceinline__ uint32_t tile_mask(const int (&ca)[NB], const int (&cz)[NB], int tx) {
  const int x0 = tx * K;
  uint32_t m = 0;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int lo = max(ca[b] - x0, 0), n = max(min(cz[b] - x0, K - 1) - lo + 1, 0);
    m |= ((1u << n) - 1u) << (lo + b * K);
  }
  return m;
}

// Tile index of pixel index px >= 0 for a tile size T that is a power of two
// (8, 16 or 32): a shift, where an integer division by the runtime T would
// cost a few dozen instructions.
__device__ __forceinline__ int tile_of(int px, int T) { return px >> (31 - __builtin_clz((unsigned)T)); }

// Tiles [tx0, tx1] of tile row ty that a record binned by rows covers: those under
// the column range of the ellipse over the whole tile row; false if none.
__device__ __forceinline__ bool rows_span(const BandPrep& bp, int ty, int TW, int TH, int H, int umin, int umax,
                                          int& tx0, int& tx1) {
  const int ya = ty * TH, yb = min(ya + TH - 1, H - 1);
  int ua, uz;
  if (!band_cols(bp, ya, yb, umin, umax, ua, uz)) return false;
  tx0 = tile_of(ua, TW);
  tx1 = tile_of(uz, TW);
  return true;
}

// Key count of a record binned by rows over its tile rectangle (rows_span summed
// over its tile rows), and the spans of its first tile rows (RowSpans).
__device__ __forceinline__ uint32_t rows_count(const RecAcc& ra, const RecGeo& geo, int W, int H, int TW, int TH,
                                               RowSpans& spans) {
  spans = RowSpans{0u, 0u};
  const int bits = span_bits(geo.tx1 - geo.tx0);
  const int umin = geo.tx0 * TW;
  const int umax = min(geo.tx1 * TW + TW - 1, W - 1);
  BandPrep bp;
  if (!band_prep(ra, geo.ub, geo.vb, bp)) return 0;
  uint32_t keys = 0;
  int at = 0;
  for (int ty = geo.ty0; ty <= geo.ty1; ++ty) {
    int tx0, tx1;
    if (rows_span(bp, ty, TW, TH, H, umin, umax, tx0, tx1)) {
      keys += (uint32_t)(tx1 - tx0 + 1);
    } else {
      tx0 = geo.tx0 + 1;
      tx1 = geo.tx0;
    }
    if (at + bits <= 32) {
      spans.first |= (uint32_t)(tx0 - geo.tx0) << at;
      spans.last |= (uint32_t)(tx1 - geo.tx0) << at;
      at += bits;
    }
  }
  return keys;
}

// The float record of an accepted pair: the in-plane factor scaled to pixel
// units, the conic centre (u0, v0) split into an integer base pixel and a
// fraction, the exponent offset and cut-off, the intensity.
__device__ __forceinline__ void record_conic(const GaussIn& G, const PlaneT<double>& P, const Conic& k, double chi2,
                                             double u0, double v0, Footprint& f) {
  const double ks = sqrt(kHalfLog2e);
  double ubd = floor(u0 + 0.5), vbd = floor(v0 + 0.5);
  ubd = min64(max64(ubd, -1.0e9), 1.0e9);
  vbd = min64(max64(vbd, -1.0e9), 1.0e9);
  f.acc.t11 = (float)(ks * k.T11 * P.sx);
  f.acc.t12 = (float)(ks * k.T12 * P.sy);
  f.acc.t22 = (float)(ks * k.T22 * P.sy);
  f.acc.fu = (float)(u0 - ubd);
  f.acc.fv = (float)(v0 - vbd);
  f.acc.e0 = (float)(G.log2a - kHalfLog2e * k.r2);
  f.acc.emin = (float)(G.log2a - kHalfLog2e * chi2);
  f.acc.c = (float)G.c;
  f.geo.ub = (int32_t)ubd;
  f.geo.vb = (int32_t)vbd;
}

// Pixels [lo, hi] (clipped to the image) whose index lies in
// [centre - half, centre + half], edges included, with no padding; false if
// none.
__device__ __forceinline__ bool box_pixels(double centre, double half, int32_t size, int& lo, int& hi) {
  double a = centre - half, b = centre + half;
  if (!(a <= b)) return false;  // NaN
  if (b < 0.0 || a > (double)(size - 1)) return false;
  a = a > 0.0 ? ceil(a) : 0.0;
  b = b < (double)(size - 1) ? floor(b) : (double)(size - 1);
  lo = (int)a;
  hi = (int)b;
  return lo <= hi;
}

// Record of a pair under the paper-literal Phase-2 support (the plane meets
// the Eq. 13 box, decided by the caller): the rectangle fields hold the
// pixels whose centres lie in the in-plane part of the box, b_{1:2} = m_{1:2}
// -/+ sqrt(chi^2 Sigma'_kk), and the cut-off is -inf, so every pixel of the
// rectangle takes its Eq. 8 weight.  Pixel u's centre is at
// (u - cu) sx in the plane, hence the index interval below.  No keys.
__device__ __forceinline__ bool make_box_record(const GaussIn& G, const PlaneRec& Q, const Conic& k, double chi2,
                                                Footprint& f) {
  const PlaneT<double>& P = Q.pose;
  // exact divisions, here and in the Gaussian's factor (load_gauss): a pixel
  // centre on the box's edge decides here
  int ulo, uhi, vlo, vhi;
  if (!box_pixels(k.m1 / P.sx + Q.cu, sqrt(chi2 * k.S11) / P.sx, Q.W, ulo, uhi)) return false;
  if (!box_pixels(k.m2 / P.sy + Q.cv, sqrt(chi2 * k.S22) / P.sy, Q.H, vlo, vhi)) return false;
  record_conic(G, P, k, chi2, k.c1 / P.sx + Q.cu, k.c2 / P.sy + Q.cv, f);
  f.acc.emin = -INFINITY;
  f.geo.tx0 = (uint16_t)ulo;
  f.geo.tx1 = (uint16_t)uhi;
  f.geo.ty0 = (uint16_t)vlo;
  f.geo.ty1 = (uint16_t)vhi;
  f.keys = f.counted = 0;
  return true;
}

// Record, tile rectangle and key count of an accepted pair (conic_full done).
// Returns false if the footprint misses the image.  by_rows: keys only for
// the tiles the ellipse reaches.  PAPER rectangles hold a fair share of tiles
// it does not (their mask would be empty): at 1M Gaussians and 256 planes of
// 256^2 69M tiles of 16 x 16, 41M of them reached; counting them here costs
// the record kernel less than emitting, sorting and skipping the rest.
__device__ __forceinline__ bool make_footprint(const GaussIn& G, const PlaneRec& Q, const Conic& k, double chi2,
                                               int box_mode, bool by_rows, int TW, int TH, Footprint& f) {
  const double isx = Q.isx, isy = Q.isy;
  const double u0 = k.c1 * isx + Q.cu;
  const double v0 = k.c2 * isy + Q.cv;
  int ulo, uhi, vlo, vhi;
  if (box_mode == UG_BOX_PAPER) {
    // Eq. 13: b_{1:2} = m_{1:2} -/+ sqrt(chi^2 Sigma'_kk).
    if (!pixel_range(k.m1 * isx + Q.cu, root(chi2 * k.S11) * isx, Q.W, ulo, uhi)) return false;
    if (!pixel_range(k.m2 * isy + Q.cv, root(chi2 * k.S22) * isy, Q.H, vlo, vhi)) return false;
  } else {
    // Box of the ellipse cut by the plane: conditional variances
    // Sigma'_kk - Sigma'_k3^2 / Sigma'_33 = |g_k x g3|^2 / |g3|^2.
    const double q = max64(chi2 - k.r2, 0.0);
    if (!pixel_range(u0, root(q * cross_norm2(k.g1, k.g3) * k.iS) * isx, Q.W, ulo, uhi)) return false;
    if (!pixel_range(v0, root(q * cross_norm2(k.g2, k.g3) * k.iS) * isy, Q.H, vlo, vhi)) return false;
  }
  record_conic(G, Q.pose, k, chi2, u0, v0, f);
  f.geo.tx0 = (uint16_t)tile_of(ulo, TW);
  f.geo.tx1 = (uint16_t)tile_of(uhi, TW);
  f.geo.ty0 = (uint16_t)tile_of(vlo, TH);
  f.geo.ty1 = (uint16_t)tile_of(vhi, TH);
  f.counted = (uint32_t)(f.geo.tx1 - f.geo.tx0 + 1) * (uint32_t)(f.geo.ty1 - f.geo.ty0 + 1);
  f.keys = by_rows ? rows_count(f.acc, f.geo, Q.W, Q.H, TW, TH, f.spans) : f.counted;
  if (box_mode == UG_BOX_ROWS) f.counted = f.keys;
  return f.counted > 0;
}

// Adjoint of make_footprint's float record with respect to the Gaussian's
// raw parameters, holding the cut-off set fixed.  dr = (dt11, dt12, dt22,
// dfu, dfv, de0, dc).  Accumulates into dmu[3], dL[6] (L11, L21, L31, L22,
// L32, L33), da, dc.
template <typename T>
__device__ __forceinline__ void footprint_adjoint(const GaussT<T>& G, const PlaneT<T>& P, const ConicT<T>& k,
                                                  const float* dr, T* dmu, T* dL, T& da, T& dc) {
  const T ks = (T)0.84932180028801904272;  // sqrt(log2(e) / 2)
  const T dT11 = ks * P.sx * (T)dr[0];
  const T dT12 = ks * P.sy * (T)dr[1];
  const T dT22 = ks * P.sy * (T)dr[2];
  const T dc1 = (T)dr[3] * recip(P.sx);
  const T dc2 = (T)dr[4] * recip(P.sy);
  const T de0 = (T)dr[5];
  dc += (T)dr[6];
  // e0 = log2(sigmoid(a)) - kHalfLog2e r^2
  da += de0 * ((T)1 - G.alpha) * (T)(1.0 / kLn2);
  const T dr2 = -(T)kHalfLog2e * de0;
  // T22 = detM n3 / T11, T12 = b1.b2 / T11, T11 = |b1|
  const T iT11 = k.iT11;
  const T detM = k.detL * P.absdet;
  const T dT11t = dT11 - (dT12 * k.T12 + dT22 * k.T22) * iT11;
  const T ddetL = dT22 * P.absdet * k.n3 * iT11;
  const T dn3 = dT22 * detM * iT11;
  T db1[3], db2[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    db1[j] = (dT11t * k.b1[j] + dT12 * k.b2[j]) * iT11;
    db2[j] = dT12 * k.b1[j] * iT11;
  }
  // c1 = m1 - m3 S13/S33, c2 = m2 - m3 S23/S33, r2 = m3^2 / S33
  const T iS = k.iS;
  T dm[3];
  dm[0] = dc1;
  dm[1] = dc2;
  dm[2] = (-dc1 * k.S13 - dc2 * k.S23 + dr2 * (T)2 * k.m3) * iS;
  const T dS13 = -dc1 * k.m3 * iS;
  const T dS23 = -dc2 * k.m3 * iS;
  const T dS33 = (dc1 * k.m3 * k.S13 + dc2 * k.m3 * k.S23 - dr2 * k.m3 * k.m3) * iS * iS;
  const T in3 = k.in3;
  T dg1[3], dg2[3], dg3[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    dg1[j] = dS13 * k.g3[j];
    dg2[j] = dS23 * k.g3[j];
    dg3[j] = dS13 * k.g1[j] + dS23 * k.g2[j] + (T)2 * dS33 * k.g3[j] + dn3 * k.g3[j] * in3;
  }
  // g = L^-1 q  ->  dL_ij -= h_i g_j with h = L^-T dg (lower triangle)
  T h[3];
  bsub(G, dg1, h);
  dL[0] -= h[0] * k.g1[0]; dL[1] -= h[1] * k.g1[0]; dL[2] -= h[2] * k.g1[0];
  dL[3] -= h[1] * k.g1[1]; dL[4] -= h[2] * k.g1[1]; dL[5] -= h[2] * k.g1[2];
  bsub(G, dg2, h);
  dL[0] -= h[0] * k.g2[0]; dL[1] -= h[1] * k.g2[0]; dL[2] -= h[2] * k.g2[0];
  dL[3] -= h[1] * k.g2[1]; dL[4] -= h[2] * k.g2[1]; dL[5] -= h[2] * k.g2[2];
  bsub(G, dg3, h);
  dL[0] -= h[0] * k.g3[0]; dL[1] -= h[1] * k.g3[0]; dL[2] -= h[2] * k.g3[0];
  dL[3] -= h[1] * k.g3[1]; dL[4] -= h[2] * k.g3[1]; dL[5] -= h[2] * k.g3[2];
  // b_j = sum_i L_ij e_i  ->  dL_ij += e_i db_j
  dL[0] += P.e1[0] * db1[0] + P.e2[0] * db2[0];
  dL[1] += P.e1[1] * db1[0] + P.e2[1] * db2[0];
  dL[2] += P.e1[2] * db1[0] + P.e2[2] * db2[0];
  dL[3] += P.e1[1] * db1[1] + P.e2[1] * db2[1];
  dL[4] += P.e1[2] * db1[1] + P.e2[2] * db2[1];
  dL[5] += P.e1[2] * db1[2] + P.e2[2] * db2[2];
  // detL = L11 L22 L33
  dL[0] += ddetL * G.L22 * G.L33;
  dL[3] += ddetL * G.L11 * G.L33;
  dL[5] += ddetL * G.L11 * G.L22;
  // m = R^-1 (mu - o)  ->  dmu = R^-T dm
#pragma unroll
  for (int j = 0; j < 3; ++j) dmu[j] += P.rinv[j] * dm[0] + P.rinv[3 + j] * dm[1] + P.rinv[6 + j] * dm[2];
}

}  // namespace ug
