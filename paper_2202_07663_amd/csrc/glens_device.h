// Per-particle decode and per-sub-pixel forward / adjoint math of the lens model.
//
// Forward model (Gu et al. 2022, Sec. 2.1.1): deflection by an elliptical power law (EPL,
// deflection through the Gauss hypergeometric series of Tessore & Metcalf 2015) or its
// slope-2 case the SIE, plus external shear; ray trace beta = x - alpha;
// elliptical Sersic source plus Cartesian shapelets at beta; elliptical Sersic lens light
// at x.
//
// Everything is written in complex image-plane variables that are smooth in the
// eccentricities (eps1, eps2), so the gradient has no 0/0 at a round lens:
//   z = (x - x_c) + i (y - y_c),  eps = eps1 + i eps2,  w = z - eps conj(z),
//   B = theta_E sqrt(1 - |eps|^2),  X = conj(eps) w^2 / |w|^2,
//   alpha = B^t |w|^-t w S_t(X),  S_t(X) = sum_n c_n(t) (-X)^n,
//   c_0 = 1,  c_n = c_{n-1} (2n - 2 + t) / (2n + 2 - t),  t = gamma_epl - 1.
// This is the paper's (q, phi) form rewritten: with q = (1-|eps|)/(1+|eps|),
// q x_l + i y_l = ((1+q)/2) e^{-i phi} w, the elliptical radius R = |w| / (1 + |eps|), the
// prefactor 2b/(1+q) (b/R)^(t-1) = B^t |w|^(1-t) and (1-q)/(1+q) e^{-2i phi} = conj(eps).
// For t = 1 the series sums to S_1(X) = atan(sqrt X) / sqrt X, the SIE closed form.
//
// Precision: sub-pixel positions, the deflection and the ray trace run in FP64 (on CDNA4 a
// double FMA issues at the rate of an unpacked float FMA), so the source offset
// beta - x_s keeps full FP32 relative precision even where the source has a cusp; the light
// profiles and all derivative terms run in FP32 on offsets from their centres.
//
// Sersic light uses the rotation-free quadratic form of the elliptical radius,
//   q x_l^2 + y_l^2 / q = [(1+|e|^2-2e1) dx^2 - 4 e2 dx dy + (1+|e|^2+2e1) dy^2] / (1-|e|^2),
// which is the same quantity without the position angle.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>

#include "glens_types.h"

#define GL_HD __host__ __device__ __forceinline__

namespace glens {

constexpr float kInvSqrtPi = 0.56418958354775628f;

// System of a Group that owns block b of a grouped launch.
__device__ __forceinline__ int find_sys(const Group& g, int b) {
  int i = 0;
  while (i + 1 < g.nsys && b >= g.block0[i + 1]) ++i;
  return i;
}

// Single-precision hardware transcendentals in base 2 (about 1 ulp), for normal, finite
// arguments; callers fold log2(e) into their per-particle constants.
__device__ __forceinline__ float exp2_f32(float x) { return __builtin_amdgcn_exp2f(x); }
__host__ inline float exp2_f32(float x) { return exp2f(x); }
__device__ __forceinline__ float log2_f32(float x) { return __builtin_amdgcn_logf(x); }
__host__ inline float log2_f32(float x) { return log2f(x); }
__device__ __forceinline__ float rcp_f32(float x) { return __builtin_amdgcn_rcpf(x); }
__host__ inline float rcp_f32(float x) { return 1.0f / x; }
__device__ __forceinline__ float rsq_f32(float x) { return __builtin_amdgcn_rsqf(x); }
__host__ inline float rsq_f32(float x) { return 1.0f / sqrtf(x); }
__device__ __forceinline__ float clamp_f32(float x, float most) {
  return __builtin_amdgcn_fmed3f(x, -most, most);
}
__host__ inline float clamp_f32(float x, float most) { return fminf(fmaxf(x, -most), most); }
constexpr float kLn2f = 0.69314718055994531f;
constexpr float kLog2e = 1.44269504088896341f;

// ------------------------------------------------------------------------------------------
// Per-particle decode (prologue). Double precision: it runs once per particle.
// ------------------------------------------------------------------------------------------

// Rescale |eps| onto eps_max when above it; returns the clamp Jacobian (symmetric).
GL_HD void clamp_eps(double e1, double e2, double emax, double& c1, double& c2, double& j11,
                     double& j12, double& j22) {
  const double r = sqrt(e1 * e1 + e2 * e2);
  if (r > emax) {
    const double s = emax / r, u1 = e1 / r, u2 = e2 / r;
    c1 = e1 * s;
    c2 = e2 * s;
    j11 = s * (1.0 - u1 * u1);
    j12 = -s * u1 * u2;
    j22 = s * (1.0 - u2 * u2);
  } else {
    c1 = e1;
    c2 = e2;
    j11 = 1.0;
    j12 = 0.0;
    j22 = 1.0;
  }
}

// r_n = sqrt(2^n / n!) for n = 0 .. kMaxNmax; r_n1 r_n2 scales coefficient (n1, n2).
constexpr double kHermR[kMaxNmax + 1] = {
    1.0, 1.4142135623730951, 1.4142135623730951, 1.1547005383792515, 0.816496580927726,
    0.5163977794943222, 0.29814239699997197, 0.15936381457791915, 0.07968190728895957};
GL_HD inline double hermite_scale(int n1, int n2) { return kHermR[n1] * kHermR[n2]; }

GL_HD void decode_light(const float* th, LightC& L) {
  const double re = th[0], n = th[1];
  double e1, e2, j11, j12, j22;
  clamp_eps(th[2], th[3], kLightEpsMax, e1, e2, j11, j12, j22);
  const double ee = e1 * e1 + e2 * e2, den = 1.0 / (1.0 - ee);
  L.i0 = th[6];
  L.qa = float((1.0 + ee - 2.0 * e1) * den);
  L.qb = float(-4.0 * e2 * den);
  L.qc = float((1.0 + ee + 2.0 * e1) * den);
  L.qbh = float(-2.0 * e2 * den);
  L.kq = float(-(1.9992 * n - 0.3271) / n);
  L.inv2n = float(0.5 / n);
  L.l2re_n = float(log2(re) / n);
  L.bn = float(1.9992 * n - 0.3271);
  L.bnl = float((1.9992 * n - 0.3271) * 1.4426950408889634);
  L.n = float(n);
  L.re = float(re);
  L.e1 = float(e1);
  L.e2 = float(e2);
  L.inv1me2 = float(den);
  L.kqi = float(-(1.9992 * n - 0.3271) / n * double(th[6]));
  L.j11 = float(j11);
  L.j12 = float(j12);
  L.j22 = float(j22);
}

// Number of parameters of the mass model (lens mass + external shear) in the gl.h layout.
GL_HD int mass_param_count(int mass, int shear) { return 5 + (mass == 1) + 2 * shear; }

// Mass constants of one parameter vector (layout of gl.h): everything but the series
// coefficients, whose term counts it sets.
GL_HD void decode_mass(const float* th, int mass, int shear, MassC& c) {
  int p = 0;
  const double theta_e = th[p++];
  const double t = (mass == 1) ? double(th[p++]) - 1.0 : 1.0;
  double e1, e2, j11, j12, j22;
  clamp_eps(th[p], th[p + 1], kMassEpsMax, e1, e2, j11, j12, j22);
  p += 2;
  c.xc = th[p++];
  c.yc = th[p++];
  if (shear) {
    c.g1 = th[p++];
    c.g2 = th[p++];
  } else {
    c.g1 = 0.0;
    c.g2 = 0.0;
  }
  c.omg1 = 1.0 - c.g1;
  c.opg1 = 1.0 + c.g1;
  c.ome1 = 1.0 - e1;
  c.ope1 = 1.0 + e1;
  c.e12 = 2.0 * e1;
  c.e22 = 2.0 * e2;
  const double ee = e1 * e1 + e2 * e2, eabs = sqrt(ee);
  const double B = theta_e * sqrt(1.0 - ee);
  c.t = t;
  c.e1 = e1;
  c.e2 = e2;
  c.ee = ee;
  c.tlnb = t * log(B);
  // theta_E < 0: the SIE from kSieClosedMin on has an image (alpha is odd in B there) and no
  // gradient; elsewhere the power B^t does not exist and log L is -inf
  c.bmass = B < 0.0 && !(mass == 0 && eabs >= kSieClosedMin) ? NAN : B;
  c.w2floor = 1e-12 * (1.0 + eabs) * (1.0 + eabs);
  c.epsabs = eabs;
  c.theta_e = float(theta_e);
  c.hp = float(1.0 - 0.5 * t);
  c.hm = float(-0.5 * t);
  c.omt = float(1.0 - t);
  const bool sx = eabs < kSxClosedMin;
  c.icr = (1.0 - ee) * (sx ? 1.0 : e1);
  c.ici = sx ? 0.0 : -e2 * (1.0 - ee);
  c.e1f = float(e1);
  c.e2f = float(e2);
  c.eef = float(ee);
  c.w2floorf = float(c.w2floor);
  c.tlnb2 = float(c.tlnb * 1.4426950408889634);
  c.hb = B < 0.0 ? NAN : float(0.5 * B);
  // kappa is in proportion to constants rounded to FP32 (EPL: 2^(hm log2|w|^2 + tlnb2), on the
  // ring |w| = B), and ha and hq are rounded with them
  const double l2b2 = 2.0 * log(B) * 1.4426950408889634;
  c.l2b2 = float(l2b2);
  const double sc = mass == 1 ? 1.0 + 0.6931471805599453 * (c.hm * l2b2 + c.tlnb2) : 1.0 + (c.hb - 0.5 * B) * rcp_f32(c.hb);
  const double ha = c.hp * (1.0 + ee) * sc, hq = c.hp * (1.0 - ee) * sc;
  c.ha = float(ha);
  c.hal = float(ha - c.ha);
  c.hq = float(hq);
  c.hql = float(hq - c.hq);
  c.tf = float(t);
  c.lnb = float(log(B));
  c.xcf = float(c.xc);
  c.ycf = float(c.yc);
  c.iebr = eabs >= kSxClosedMin ? float(e1 / ee) : 0.f;
  c.iebi = eabs >= kSxClosedMin ? float(e2 / ee) : 0.f;
  c.tfac = float(t / (2.0 * (1.0 - ee)));
  c.mj11 = float(j11);
  c.mj12 = float(j12);
  c.mj22 = float(j22);
  // series: terms until the tail bound |eps|^N / (1 - |eps|) drops below the tolerance
  // (FP64 value series), and below the looser derivative tolerance (adjoint series)
  c.sie_closed = (mass == 0 && eabs >= kSieClosedMin) ? 1 : 0;
  int nt = 1, ntd = 1;
  if (eabs > 1e-30) {
    nt = int(ceil(log((c.sie_closed ? kSeriesTolSie : kSeriesTol) * (1.0 - eabs)) / log(eabs)));
    nt = nt < 1 ? 1 : (nt > kMaxTerms ? kMaxTerms : nt);
    ntd = int(ceil(log(kSeriesTolDeriv * (1.0 - eabs)) / log(eabs))) + 1;
    ntd = ntd < 1 ? 1 : (ntd > nt ? nt : ntd);
  }
  c.nterms = nt;
  c.nterms_d = ntd;
  // SIE closed form: s = sqrt(conj(eps)), S_1(X) = atan(s u) / (s u), u = w / |w|
  if (c.sie_closed) {
    const double ang = -0.5 * atan2(e2, e1), rs = sqrt(eabs);
    c.sr = rs * cos(ang);
    c.si = rs * sin(ang);
  } else {
    c.sr = c.si = 0.0;
  }
}

// Series ratio c_n / c_{n-1} = (2n - 2 + t) / (2n + 2 - t) and the increment of
// d log c_n / dt, 1 / (2n - 2 + t) + 1 / (2n + 2 - t), for n >= 1.
GL_HD void series_step(int n, double t, double& ratio, double& dlog) {
  const double a = 2.0 * n - 2.0 + t, b = 2.0 * n + 2.0 - t;
  ratio = a / b;
  dlog = 1.0 / a + 1.0 / b;
}

// Stores term n of the value series (c_n), of the derivative series n c_n (at n - 1) and
// of dc_n / dt = c_n sum_k dlog_k, given the running product and sum.
GL_HD void series_store(const MassC& m, PConst& c, int n, double cn, double dsum) {
  c.c[n] = n < m.nterms ? cn : 0.0;
  c.dc[n] = n < m.nterms_d ? float(cn * dsum) : 0.f;
  if (n > 0) c.nc[n - 1] = n < m.nterms_d ? float(n * cn) : 0.f;
  if (n == kMaxTerms - 1) c.nc[kMaxTerms - 1] = 0.f;
}

// ------------------------------------------------------------------------------------------
// The floored sub-pixel. The elliptical mass radius R is kept >= 1e-6 arcsec (R^2 >= 1e-12);
// below that the deflection is the formula with R frozen at 1e-6, a function of the remaining
// variables whose derivatives the per-lane FP32 adjoint does not carry (the frozen radius on
// |w| is 1e-12 (1 + |eps|)^2, which depends on eps, and the SIE's closed form with a frozen
// radius is not its series with one). The prologue finds that sub-pixel (at most one per
// particle) and evaluates the frozen-radius deflection and its derivatives exactly, by
// forward-mode dual numbers in FP64 over (t, eps1, eps2, x_c, y_c).
// ------------------------------------------------------------------------------------------
struct D5 {
  double v;
  double d[5];
};
GL_HD D5 d5(double v, int k = -1) {
  D5 r;
  r.v = v;
#pragma unroll
  for (int i = 0; i < 5; ++i) r.d[i] = i == k ? 1.0 : 0.0;
  return r;
}
GL_HD D5 operator+(const D5& a, const D5& b) {
  D5 r;
  r.v = a.v + b.v;
  for (int i = 0; i < 5; ++i) r.d[i] = a.d[i] + b.d[i];
  return r;
}
GL_HD D5 operator-(const D5& a, const D5& b) {
  D5 r;
  r.v = a.v - b.v;
  for (int i = 0; i < 5; ++i) r.d[i] = a.d[i] - b.d[i];
  return r;
}
GL_HD D5 operator*(const D5& a, const D5& b) {
  D5 r;
  r.v = a.v * b.v;
  for (int i = 0; i < 5; ++i) r.d[i] = a.d[i] * b.v + a.v * b.d[i];
  return r;
}
GL_HD D5 operator*(double s, const D5& a) {
  D5 r;
  r.v = s * a.v;
  for (int i = 0; i < 5; ++i) r.d[i] = s * a.d[i];
  return r;
}
GL_HD D5 operator/(const D5& a, const D5& b) {
  D5 r;
  r.v = a.v / b.v;
  for (int i = 0; i < 5; ++i) r.d[i] = (a.d[i] - r.v * b.d[i]) / b.v;
  return r;
}
// f(a) given f(a.v) and f'(a.v)
GL_HD D5 d5_chain(const D5& a, double f, double df) {
  D5 r;
  r.v = f;
  for (int i = 0; i < 5; ++i) r.d[i] = df * a.d[i];
  return r;
}
GL_HD D5 d5_exp(const D5& a) { const double e = exp(a.v); return d5_chain(a, e, e); }
GL_HD D5 d5_log(const D5& a) { return d5_chain(a, log(a.v), 1.0 / a.v); }
GL_HD D5 d5_sqrt(const D5& a) { const double r = sqrt(a.v); return d5_chain(a, r, 0.5 / r); }
GL_HD D5 d5_atan(const D5& a) { return d5_chain(a, atan(a.v), 1.0 / (1.0 + a.v * a.v)); }
GL_HD D5 d5_atanh(const D5& a) { return d5_chain(a, atanh(a.v), 1.0 / (1.0 - a.v * a.v)); }
GL_HD D5 d5_cos(const D5& a) { return d5_chain(a, cos(a.v), -sin(a.v)); }
GL_HD D5 d5_sin(const D5& a) { return d5_chain(a, sin(a.v), cos(a.v)); }
GL_HD D5 d5_atan2(const D5& y, const D5& x) {
  D5 r;
  r.v = atan2(y.v, x.v);
  const double n = x.v * x.v + y.v * y.v;
  for (int i = 0; i < 5; ++i) r.d[i] = (x.v * y.d[i] - y.v * x.d[i]) / n;
  return r;
}

// Centre of sub-pixel column (or row) n of the system's grid: x0 + n dxs, one rounding.
GL_HD double subpix_coord(double x0, int n, double dxs) { return fma(double(n), dxs, x0); }

// Deflection at image position (x, y) with the elliptical radius frozen at its floor
// R_f = 1e-6 arcsec, as dual numbers over (t, eps1, eps2, x_c, y_c).
//   EPL (and the SIE's series): alpha = A w S_t(X) with A = (theta_E sqrt(q) / R_f)^t,
//     q = (1 - |eps|)/(1 + |eps|), w = z - eps conj(z), X = conj(eps) w^2 / |w_f|^2,
//     |w_f| = R_f (1 + |eps|): the series form in which |w| only enters through R;
//   SIE: the closed form with the radius frozen, in the lens frame (rotation by
//     phi = atan2(eps2, eps1) / 2): alpha_l = b / q' (atan(q' x_l / R_f), atanh(q' y_l / R_f)),
//     b = theta_E sqrt(q), q' = sqrt(1 - q^2); at |eps| = 0 the SIS limit b z / R_f.
// |eps| has no derivative at eps = 0: there the eps-derivatives of |eps| are taken as 0.
GL_HD void floored_deflection(const MassC& c, int mass, double x, double y, D5& ar, D5& ai) {
  const double rf = 1e-6;
  const D5 e1 = d5(c.e1, 1), e2 = d5(c.e2, 2);
  const D5 zr = d5(x) - d5(c.xc, 3), zi = d5(y) - d5(c.yc, 4);
  const D5 ee = e1 * e1 + e2 * e2;
  const D5 ea = ee.v > 0.0 ? d5_sqrt(ee) : d5(0.0);
  const D5 one = d5(1.0);
  const D5 q = (one - ea) / (one + ea);
  const double the = double(c.theta_e);
  if (mass == 1) {
    const D5 t = d5(c.t, 0);
    const D5 A = d5_exp(t * (d5(log(the / rf)) + 0.5 * d5_log(q)));
    const D5 wr = zr - e1 * zr - e2 * zi, wi = zi - e2 * zr + e1 * zi;
    const D5 wf2 = (rf * rf) * ((one + ea) * (one + ea));
    const D5 w2r = wr * wr - wi * wi, w2i = 2.0 * (wr * wi);
    const D5 Xr = (e1 * w2r + e2 * w2i) / wf2, Xi = (e1 * w2i - e2 * w2r) / wf2;
    D5 Sr = one, Si = d5(0.0), cn = one, pr = one, pi = d5(0.0);
    for (int n = 1; n < c.nterms; ++n) {
      cn = cn * (d5(2.0 * n - 2.0) + t) / (d5(2.0 * n + 2.0) - t);
      const D5 nr = d5(0.0) - (pr * Xr - pi * Xi), ni = d5(0.0) - (pr * Xi + pi * Xr);
      pr = nr;
      pi = ni;
      Sr = Sr + cn * pr;
      Si = Si + cn * pi;
    }
    ar = A * (wr * Sr - wi * Si);
    ai = A * (wr * Si + wi * Sr);
    return;
  }
  const D5 b = the * d5_sqrt(q);
  if (ea.v == 0.0) {  // circular: the SIS with its radius frozen
    ar = (1.0 / rf) * (b * zr);
    ai = (1.0 / rf) * (b * zi);
    return;
  }
  const D5 phi = 0.5 * d5_atan2(e2, e1);
  const D5 cp = d5_cos(phi), sp = d5_sin(phi);
  const D5 xl = cp * zr + sp * zi, yl = sp * (d5(0.0) - zr) + cp * zi;
  const D5 qp = d5_sqrt(one - q * q);
  const D5 axl = b / qp * d5_atan((1.0 / rf) * (qp * xl));
  const D5 ayl = b / qp * d5_atanh((1.0 / rf) * (qp * yl));
  ar = cp * axl - sp * ayl;
  ai = sp * axl + cp * ayl;
}

// Finds the floored sub-pixel of one particle (fills c.fl_*; after decode_mass). Only the
// sub-pixel nearest the lens centre can have R below the floor. xs: the source centre.
GL_HD void decode_floor(const SysDesc& s, const float* xs, const MassC& m, PConst& c) {
  c.fl_i = c.fl_j = c.fl_pix = c.fl_sub = -1;
  c.fl_a[0] = c.fl_a[1] = 0.0;
  const double fj = rint((m.xc - s.x0) / s.dxs), fi = rint((m.yc - s.y0) / s.dxs);
  if (!(fj >= 0.0 && fj < double(s.W * s.k) && fi >= 0.0 && fi < double(s.H * s.k))) return;
  const int jj = int(fj), ii = int(fi);
  const double x = subpix_coord(s.x0, jj, s.dxs), y = subpix_coord(s.y0, ii, s.dxs);
  const double zr = x - m.xc, zi = y - m.yc;
  const double wr = zr - m.e1 * zr - m.e2 * zi, wi = zi - m.e2 * zr + m.e1 * zi;
  if (!(wr * wr + wi * wi < m.w2floor)) return;
  D5 ar, ai;
  floored_deflection(m, s.mass, x, y, ar, ai);
  c.fl_i = ii;
  c.fl_j = jj;
  c.fl_pix = (ii / s.k) * s.W + jj / s.k;
  c.fl_sub = (ii % s.k) * s.k + jj % s.k;
  c.fl_s[0] = float(x - ar.v - (m.g1 * x + m.g2 * y) - double(xs[0]));
  c.fl_s[1] = float(y - ai.v - (m.g2 * x - m.g1 * y) - double(xs[1]));
  c.fl_a[0] = ar.v;
  c.fl_a[1] = ai.v;
  for (int k = 0; k < 5; ++k) {
    c.fl_d[k][0] = ar.d[k];
    c.fl_d[k][1] = ai.d[k];
  }
}

// Orders (n1, n2) of shapelet coefficient q: q runs over n = n1 + n2 = 0, 1, ... and, within
// one n, over n2 = 0 .. n.
GL_HD void shapelet_orders(int q, int& n1, int& n2) {
  int n = 0;
  while ((n + 1) * (n + 2) / 2 <= q) ++n;
  n2 = q - n * (n + 1) / 2;
  n1 = n - n2;
}

// Light constants (lens light, source Sersic, shapelet coefficients) of one vector, spread
// over the lanes of the prologue: lane 1 the lens light, lane 2 the source, lane 3 the
// shapelet scale, lanes 3 .. 3 + M - 1 one shapelet coefficient each (M = (n_max + 1)
// (n_max + 2) / 2 <= 45). Every field is written by exactly one lane.
GL_HD void decode_lights_lane(const float* th, int mass, int shear, int lens_light, int nmax,
                              PConst& c, int lane) {
  const int pl = mass_param_count(mass, shear);        // lens light
  const int ps = pl + (lens_light ? 7 : 0);            // source Sersic
  const int pb = ps + 7;                               // shapelet scale, then coefficients
  // the two profiles side by side: one pass over the decode's code for both lanes
  if (lane == 2 || (lane == 1 && lens_light)) {
    const float* p = th + (lane == 1 ? pl : ps);
    decode_light(p, lane == 1 ? c.lens : c.src);
    double* xs = lane == 1 ? &c.lxs : &c.sxs;
    xs[0] = p[4];
    xs[1] = p[5];
  } else if (lane == 1) {
    c.lxs = c.lys = 0.0;
  }
  if (nmax < 0) return;
  const int q = lane - 3, M = (nmax + 1) * (nmax + 2) / 2;
  if (q < 0 || q >= M) return;
  const double beta = th[pb];
  if (q == 0) {
    c.beta = float(beta);
    c.inv_beta = float(1.0 / beta);
    c.rt2_ib = float(1.4142135623730951 / beta);
  }
  const double f = 0.56418958354775628 / beta;  // 1 / (beta sqrt(pi))
  int n1, n2;
  shapelet_orders(q, n1, n2);
  c.shp[q] = float(double(th[pb + 1 + q]) * (f * hermite_scale(n1, n2)));
}

// ------------------------------------------------------------------------------------------
// Double-precision helpers for the ray trace, for the argument ranges met there (normal,
// finite, positive arguments). Written from the mathematics:
//   rcp: hardware estimate (relative error about 2^-23) refined by one Newton step
//        r <- r + r (1 - x r), which squares the error (about 1e-14);
//   the power B^t |w|^-t: per-particle tables (pow_from_table, after these helpers).
// The targets sit below the 1e-10 relative tolerance of the deflection series: the ray
// trace needs |alpha| to ~1e-9 arcsec, far below FP32 resolution but far above FP64's.
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ double rcp_f64(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  return fma(fma(-x, r, 1.0), r, r);
}
__host__ inline double rcp_f64(double x) { return 1.0 / x; }
// 1 / sqrt(x): hardware estimate and one Newton step, as rcp
__device__ __forceinline__ double rsq_f64(double x) {
  const double r = __builtin_amdgcn_rsq(x);
  return fma(0.5 * r, fma(-x * r, r, 1.0), r);
}
__host__ inline double rsq_f64(double x) { return 1.0 / sqrt(x); }

constexpr double kLn2 = 0.6931471805599453;  // nearest double to ln 2

// The power tables (PConst::pw): entry i < kPowExp is B^t 2^(-t e/2) for e = i - kPowExp/2 ...
GL_HD double pow_exponent_entry(double t, double log2B, int i) {
  return exp2(t * (log2B - 0.5 * (i - kPowExp / 2)));
}
// ... and kPowExp + 8 j + k the Taylor coefficient k (zero above kPowDeg) of m^(-t/2) about
// m_j = 1 + (j + 1/2)/16: a_0 = m_j^(-t/2), a_k = a_(k-1) (-t/2 - k + 1) / (k m_j). Segment j (no
// segment: nothing).
GL_HD void pow_segments_lane(double t, int j, double* pw) {
  if (j < 0 || j >= kPowSeg) return;
  double* seg = pw + kPowExp + 8 * j;
  const double mj = 1.0 + (j + 0.5) / kPowSeg;
  double a = exp2(-0.5 * t * log2(mj));
  seg[0] = a;
  for (int q = 1; q < 8; ++q) {
    if (q <= kPowDeg) a *= (-0.5 * t - (q - 1)) / (q * mj);
    seg[q] = q <= kPowDeg ? a : 0.0;
  }
}

// The power tables shared by `nl` lanes (this one is lane l of them): the exponent entries
// round-robin, and the sixteen segments' Taylor coefficients one segment per lane on the last
// kPowSeg lanes.
GL_HD void pow_tables_lane(double t, double log2B, int l, int nl, double* pw) {
  for (int i = l; i < kPowExp; i += nl) pw[i] = pow_exponent_entry(t, log2B, i);
  pow_segments_lane(t, l - (nl - kPowSeg), pw);
}

// A = B^t |w|^-t = B^t (|w|^2)^(-t/2) from the particle's power tables (staged in LDS): with
// |w|^2 = 2^e m, m in [1, 2), the four leading mantissa bits pick the sixteenth j of [1, 2)
// and the remaining ones give x = m - m_j exactly, so that A = T[e] P_j(x) (about 3e-11
// relative; no logarithm or exponential). |w|^2 is at least the 1e-12 floor, so e >= -40; an
// exponent beyond the table (|w| above 2^31 arcsec) is clamped.
GL_HD double pow_from_table(const double* __restrict__ pw, double w2) {
  const uint64_t b = __builtin_bit_cast(uint64_t, w2);
  const int e = int((b >> 52) & 0x7ffu) - 1023;
  const int j = int((b >> 48) & 15u);
  const double m = __builtin_bit_cast(double, (b & 0x0000ffffffffffffull) | 0x3ff0000000000000ull);
  const double x = m - (1.0 + 0.5 / kPowSeg);
  const double* a = pw + kPowExp + 8 * j;
  double p = fma(a[6], x, a[5]);
  p = fma(p, x, a[4]);
  p = fma(p, x, a[3]);
  p = fma(p, x, a[2]);
  p = fma(p, x, a[1]);
  p = fma(p, x, a[0]);
  const int ie = e + kPowExp / 2;
  return pw[min(max(ie, 0), kPowExp - 1)] * p;
}

// ------------------------------------------------------------------------------------------
// Sub-pixel math
// ------------------------------------------------------------------------------------------

struct Cx {
  float r, i;
};
GL_HD Cx cmul(Cx a, Cx b) { return {a.r * b.r - a.i * b.i, a.r * b.i + a.i * b.r}; }
GL_HD Cx cadd(Cx a, Cx b) { return {a.r + b.r, a.i + b.i}; }
GL_HD Cx csub(Cx a, Cx b) { return {a.r - b.r, a.i - b.i}; }
GL_HD Cx cscale(Cx a, float s) { return {a.r * s, a.i * s}; }
GL_HD Cx cconj(Cx a) { return {a.r, -a.i}; }
GL_HD Cx cmuli(Cx a) { return {-a.i, a.r}; }  // i a
GL_HD float cdot(Cx g, Cx v) { return g.r * v.r + g.i * v.i; }  // real dot product

// EPL / SIE deflection plus shear at image position x, in FP64: beta - x_s with beta = x - alpha
// - alpha_ext. The row's y enters through RayRow, so that w takes one FMA per component. Both
// masses take the series. The SIE is t = 1: A = B / |w| takes a reciprocal square root instead of
// the power table, and the series goes on to kSeriesTolSie (its c_n = 1 / (2n + 1) leave a tail
// below 1e-12 of alpha also at the longest, |eps| = 0.6), so that an offset beta - x_s of 1e-6
// arcsec still has FP32 precision, as with the closed form. That, a complex arctangent, costs
// three times the instructions of the longest series kept and is left to the sampler's launches
// (glens_chain.h).
// The radius is not floored here (|w|^2 is above its floor and |X| = |eps|): at the particle's
// floored sub-pixel, if it has one, the result is not finite or not used, and the caller takes
// the prologue's c.fl_s instead.
// pw: the particle's power tables c.pw (staged in LDS); yy: c.ee, in vector registers (an FMA
// reads one scalar operand, and that is the series coefficient).
struct RayRow {
  double wr, wi;       // w = (1 - e1) x + wr, -e2 x + wi
  double ax, ay;       // -g2 y - x_s, (1 + g1) y - y_s
};
__device__ __forceinline__ RayRow ray_row(const PConst& c, double y) {
  const double zi = y - c.yc;
  return {fma(-c.e2, zi, -c.ome1 * c.xc), fma(c.ope1, zi, c.e2 * c.xc), fma(-c.g2, y, -c.sxs),
          fma(c.opg1, y, -c.sys)};
}
template <int MASS>
__device__ __forceinline__ void ray_trace(const PConst& c, const double* __restrict__ cs,
                                          const double* __restrict__ pw, double yy, double x,
                                          const RayRow& row, float& sdx, float& sdy) {
  const double wr = fma(c.ome1, x, row.wr), wi = fma(-c.e2, x, row.wi);
  const double wi2 = wi * wi;
  const double w2 = fma(wr, wr, wi2);
  const double rw = MASS == 0 ? rsq_f64(w2) : 0.0;
  const double inv = MASS == 0 ? rw * rw : rcp_f64(w2);
  const double pr = fma(wr, wr, -wi2), pi = wr * wi;  // w^2 = pr + 2 i pi
  const double Xr = inv * fma(c.e1, pr, c.e22 * pi), Xi = inv * fma(c.e12, pi, -c.e2 * pr);
  // The coefficients are real, so the series is evaluated at the complex point y = -X by
  // synthetic division by the real quadratic (v - y)(v - conj y) = v^2 - 2 Re(y) v + |y|^2
  // (Knuth, TAOCP vol. 2, sec. 4.6.4): b_n = c_n + 2 Re(y) b_(n+1) - |y|^2 b_(n+2) from the
  // top down to n = 0, and the sum is b_0 - Re(y) b_1 + i Im(y) b_1. That is two real FMAs
  // per term where complex Horner takes four. |y| = |eps| < 1, so rounding errors made
  // early are damped as the recurrence runs down. Terms are taken two per trip (so that the
  // two carried values need no register moves); coefficients past the series length are
  // zero, so rounding the length up to an even number is exact.
  const double r2 = -2.0 * Xr;
  double b1 = 0.0, b2 = 0.0;  // b_(n+1), b_(n+2)
  const int nt2 = (c.nterms + 1) & ~1;
  for (int n0 = nt2 - 2; n0 >= 0; n0 -= 2) {  // leaves b_n0 in b1 and b_(n0+1) in b2
    b2 = fma(r2, b1, fma(-yy, b2, cs[n0 + 1]));
    b1 = fma(r2, b2, fma(-yy, b1, cs[n0]));
  }
  const double Sr = fma(Xr, b2, b1), Sm = Xi * b2;  // S = Sr - i Sm
  const double A = MASS == 0 ? c.bmass * rw : pow_from_table(pw, w2);
  const double tr = fma(wr, Sr, wi * Sm), ti = fma(wi, Sr, -wr * Sm);
  // beta - x_s = x - alpha - alpha_ext - x_s
  sdx = float(fma(-A, tr, fma(x, c.omg1, row.ax)));
  sdy = float(fma(-A, ti, fma(x, -c.g2, row.ay)));
}

// The mass terms of one sub-pixel, added to acc (FP32): z the offset from the lens centre, alpha
// the deflection, g = d s / d beta weighted by the pixel adjoint. alpha comes from the kept
// beta - x_s of the forward pass's FP64 ray trace (an FP32 ray trace would move it by ~3e-7
// arcsec, which shows at 2e-3 in the gradient of a vector far from the posterior); the rest
// only enters derivatives, whose tolerance (a relative 1e-3 on the gradient) is far above FP32
// rounding. With w = z - eps conj(z), A = B^t |w|^-t and alpha = A w S_t(X), X = conj(eps) w^2 /
// |w|^2, no series is summed for the derivatives in z and eps:
//   * alpha_z = kappa = (1 - t/2) A, a real number: the series obeys
//       X (1 + X) dS/dX = (1 - t/2)(1 - S) - (t/2) X S
//     (equal coefficients of (-X)^n for every n), which turns A ((1 - t/2) S + X S_X +
//     X ((t/2) S + X S_X)), the derivative of the closed form, into (1 - t/2) A;
//   * alpha has degree 1 - t in z, so z alpha_z + conj(z) alpha_zb = (1 - t) alpha gives
//       Gamma = alpha_zb = ((1 - t) alpha - kappa z) z / |z|^2   (SIE: -kappa z^2 / |z|^2);
//   * d alpha/d eps = -tfac conj(eps) alpha - conj(z) aw,
//     d alpha/d conj(eps) = -tfac eps alpha - z awb + W, with tfac = t / (2 (1 - |eps|^2)),
//     aw = d alpha/dw, awb = d alpha/d conj(w) at fixed eps and W = A w u2 dS/dX (A depends on
//     |eps|^2, X on conj(eps)). kappa = aw - conj(eps) awb and Gamma = awb - eps aw, so
//     (1 - |eps|^2)(aw, awb) = (kappa + conj(eps) Gamma, Gamma + eps kappa), and conj(eps) W = w aw -
//     (1 - t/2) alpha. With h = g . (d alpha/dx) + i g . (d alpha/dy) = kappa g + gb Gamma, the two
//     components G = g.(d alpha/d eps_1) + i g.(d alpha/d eps_2) are
//       (1 - |eps|^2) G = -t eps Re(gb alpha) - z (h + eps conj(h)) + (1 - |eps|^2) gb W;
//     times conj(eps), with w = z - eps conj(z) and Re(conj(z) h) = (1 - t) Re(gb alpha),
//       conj(eps)(1 - |eps|^2) G = kappa w (gb - conj(eps) g)
//         - (1 - t/2)((1 + |eps|^2) Re(gb alpha) + i (1 - |eps|^2) Im(gb alpha)).
//     These terms cancel like |eps|, so the difference is taken per sub-pixel (of sums over a tile,
//     the differences had twice the error) and the sums are divided at the end. For |eps| <
//     kSxClosedMin W is summed by the derivative series instead, in the form above it;
//   * d alpha / dt = alpha (ln B - ln|w|^2 / 2) + A w S_t by its series (EPL), with the
//     coefficients times -2 / ln 2 so that the sum runs over base-2 logarithms.
// Series are summed by synthetic division at y = -X (ray_trace), four terms per trip (the length
// rounded up, the padding coefficients are zero); |y|^2 = |eps|^2 is a constant of the particle.
// dcs / ncs: the particle's c.dc (scaled) / c.nc staged in LDS.
// GENERAL = false: the particle has no floored sub-pixel and |eps| >= kSxClosedMin. At a floored
// sub-pixel everything is kept finite and the caller passes g = 0.
template <int MASS, bool GENERAL>
__device__ __forceinline__ void mass_adjoint(const PConst& c, const float* __restrict__ ncs,
                                             const float* __restrict__ dcs, float zr, float zi,
                                             float ar, float ai, Cx g, float* acc) {
  const float e1 = c.e1f, e2 = c.e2f;
  const float wr = fmaf(-e2, zi, fmaf(-e1, zr, zr)), wi = fmaf(-e2, zr, fmaf(e1, zi, zi));
  const float wr2 = wr * wr, zr2 = zr * zr;
  float w2 = fmaf(wi, wi, wr2), z2 = fmaf(zi, zi, zr2);
  if (GENERAL) {
    w2 = fmaxf(w2, c.w2floorf);
    z2 = fmaxf(z2, kR2Floor);
  }
  const float iz2 = rcp_f32(z2);
  const float ga = fmaf(g.i, ai, g.r * ar);  // Re(gb alpha)
  float kap, A = 0.f, l2w2 = 0.f, Gr, Gi;
  if (MASS == 1) {
    l2w2 = log2_f32(w2);
    A = exp2_f32(fmaf(c.hm, l2w2, c.tlnb2));
    kap = c.hp * A;
    const float vr = fmaf(c.omt, ar, -kap * zr), vi = fmaf(c.omt, ai, -kap * zi);
    const float ur = zr * iz2, ui = zi * iz2;
    Gr = fmaf(vr, ur, -vi * ui);
    Gi = fmaf(vr, ui, vi * ur);
  } else {
    kap = c.hb * rsq_f32(w2);
    A = 2.0f * kap;
    const float f = -kap * iz2;
    Gr = f * fmaf(-zi, zi, zr2);
    Gi = (2.0f * f) * (zr * zi);
  }
  const float kr = kap * g.r, ki = kap * g.i;
  const float hxr = fmaf(g.i, Gi, fmaf(g.r, Gr, kr));
  const float hxi = fmaf(-g.i, Gr, fmaf(g.r, Gi, ki));
  acc[A_M_ALPHA] += ga;
  acc[A_M_X] += hxr;
  acc[A_M_Y] += hxi;
  acc[A_M_G1] = fmaf(-g.i, zi, fmaf(g.r, zr, acc[A_M_G1]));
  acc[A_M_G2] = fmaf(g.i, zr, fmaf(g.r, zi, acc[A_M_G2]));
  const bool sx = GENERAL && c.epsabs < kSxClosedMin;
  float u2r = 0.f, u2i = 0.f, Xr = 0.f, Xi = 0.f;
  if (MASS == 1 || GENERAL) {
    const float iw2 = rcp_f32(w2);
    u2r = fmaf(-wi, wi, wr2) * iw2;
    u2i = 2.0f * wr * wi * iw2;
    Xr = e1 * u2r + e2 * u2i;
    Xi = e1 * u2i - e2 * u2r;
  }
  const float r2 = -2.0f * Xr, yy = c.eef;
  const float gwr = fmaf(g.i, wi, g.r * wr), gwi = fmaf(g.r, wi, -g.i * wr);  // gb w
  const int nd4 = (c.nterms_d + 3) & ~3;
  if (MASS == 1) {
    float t1 = 0.f, t2 = 0.f;
    for (int n0 = nd4 - 4; n0 >= 0; n0 -= 4) {
#pragma unroll
      for (int q = 3; q >= 0; --q) {
        const float t0 = fmaf(r2, t1, fmaf(-yy, t2, dcs[n0 + q]));
        t2 = t1;
        t1 = t0;
      }
    }
    // Re(gb w S_t), S_t = t1 + conj(X) t2
    const float p = fmaf(gwr, t1, t2 * fmaf(gwi, Xi, gwr * Xr));
    acc[A_M_T] = fmaf(A, p, fmaf(l2w2 - c.l2b2, ga, acc[A_M_T]));
  }
  if (sx) {  // gb W
    float d1 = 0.f, d2 = 0.f;
    for (int n0 = nd4 - 4; n0 >= 0; n0 -= 4) {
#pragma unroll
      for (int q = 3; q >= 0; --q) {
        const float d0 = fmaf(r2, d1, fmaf(-yy, d2, ncs[n0 + q]));
        d2 = d1;
        d1 = d0;
      }
    }
    const Cx SX = {-fmaf(Xr, d2, d1), Xi * d2};  // dS/dX = -dS/dy
    A *= 1.0f - c.eef;
    const Cx W = cmul(Cx{A * gwr, A * gwi}, cmul(Cx{u2r, u2i}, SX));
    const float sr = fmaf(e1, hxr, fmaf(e2, hxi, hxr)), si = fmaf(e2, hxr, fmaf(-e1, hxi, hxi));
    acc[A_M_E1] += fmaf(zi, si, fmaf(-zr, sr, W.r));
    acc[A_M_E2] += fmaf(-zi, sr, fmaf(-zr, si, W.i));
  } else {
    // kappa (gb - conj(eps) g), Im(gb alpha)
    const float ur = fmaf(-e1, kr, fmaf(-e2, ki, kr)), ui = fmaf(e2, kr, fmaf(-e1, ki, -ki));
    const float gi = fmaf(-g.i, ar, g.r * ai);
    acc[A_M_E1] += fmaf(wr, ur, fmaf(-wi, ui, fmaf(-c.hal, ga, -c.ha * ga)));
    acc[A_M_E2] += fmaf(wr, ui, fmaf(wi, ur, fmaf(-c.hql, gi, -c.hq * gi)));
  }
}

// Elliptical Sersic intensity at offset (dx, dy) from its centre.
GL_HD float sersic_fwd(const LightC& L, float dx, float dy) {
  // R^2 = dx (qa dx + qb dy) + qc dy^2
  float q = fmaf(dx, fmaf(L.qb, dy, L.qa * dx), L.qc * dy * dy);
  q = q < kR2Floor ? kR2Floor : q;  // a select, not fmaxf: a NaN offset stays NaN
  // rho = (R / R_eff)^(1/n) = 2^(log2(R^2) / (2n) - log2(R_eff) / n);  I = I0 e^(b_n (1 - rho))
  const float rho = exp2_f32(fmaf(log2_f32(q), L.inv2n, -L.l2re_n));
  return L.i0 * exp2_f32(fmaf(-L.bnl, rho, L.bnl));
}

// Accumulator terms (weight sb) of the lens light or the source, and s of LightSlot. With the
// half gradient (px, py) = (qa dx + qb dy / 2, qb dx / 2 + qc dy) of R^2 = dx px + dy py,
// dI/d(dx, dy) = s (px, py), s = I0 (-b_n / n) E rho / R^2. The sums over the ellipticity terms
// are combinations of s dx^2, s dx dy and s dy^2 (s R^2 itself is one), so only these three are
// kept, and I0 multiplies the sums instead of their terms. E rho - E is kept as a sum of its own:
// of the two sums, the difference had up to 1.4 times its error at rho near 1.
__device__ __forceinline__ float sersic_adj(const LightC& L, float dx, float dy, float px,
                                            float py, float sb, float* acc) {
  const float q0 = fmaf(dx, px, dy * py);
  const float q = fmaxf(q0, kR2Floor);  // a NaN offset has made log L non-finite already
  const float l2rho = fmaf(log2_f32(q), L.inv2n, -L.l2re_n);
  const float rho = exp2_f32(l2rho);
  const float sE = sb * exp2_f32(fmaf(-L.bnl, rho, L.bnl)), sEr = sE * rho;
  const float s = q0 < kR2Floor ? 0.0f : sEr * L.kqi * rcp_f32(q);
  acc[L_E] += sE;
  acc[L_RHO] += sEr;
  acc[L_RHO1] += sEr - sE;
  acc[L_RHOLN] = fmaf(sEr, l2rho, acc[L_RHOLN]);
  const float sx = s * dx, sy = s * dy;
  acc[L_XX] = fmaf(sx, dx, acc[L_XX]);
  acc[L_XY] = fmaf(sx, dy, acc[L_XY]);
  acc[L_YY] = fmaf(sy, dy, acc[L_YY]);
  return s;
}

// Scaled Hermite polynomials g_n(u) = H_n(u) / 2^n (H_n the physicists' polynomials):
// g_0 = 1, g_1 = u, g_(n+1) = u g_n - (n/2) g_(n-1), two operations per step, and
// g_n' = n g_(n-1). The Hermite functions are phi_n = (2^n n! sqrt(pi))^(-1/2) H_n e^(-u^2/2)
// = pi^(-1/4) r_n g_n e^(-u^2/2) with r_n = sqrt(2^n / n!); the coefficients carry r_n1 r_n2
// (hermite_scale) so that the sums run over the g_n directly.
// Started from h0 instead of 1 the recurrence gives h0 g_n(u) (it is linear).
template <int NMAX>
GL_HD void hermite(float u, float* h, float h0 = 1.0f) {
  h[0] = h0;
  if (NMAX >= 1) h[1] = h0 * u;
#pragma unroll
  for (int n = 1; n < NMAX; ++n) h[n + 1] = fmaf(u, h[n], -(0.5f * n) * h[n - 1]);
}

// Index of coefficient (n1, n2) in the order n = 0..NMAX, n1 = n..0, n2 = n - n1.
__host__ __device__ constexpr int shp_index(int n1, int n2) {
  return (n1 + n2) * (n1 + n2 + 1) / 2 + n2;
}

// Shapelet intensity at offset (sdx, sdy) from the source centre:
// G(u, v) sum_k c'_k g_n1(u) g_n2(v), c'_k = c_k r_n1 r_n2 / (beta sqrt(pi)),
// G = exp(-(u^2+v^2)/2), summed as U = sum_n1 g_n1(u) T_n1 with
// T_n1 = sum_n2 c'_(n1,n2) g_n2(v).
template <int NMAX>
GL_HD float shapelet_fwd(const PConst& c, float sdx, float sdy, const float* shp) {
  const float u = sdx * c.inv_beta, v = sdy * c.inv_beta;
  float hu[NMAX + 1], hv[NMAX + 1];
  hermite<NMAX>(u, hu);
  hermite<NMAX>(v, hv);
  // g_0 = 1: every sum starts from its n = 0 term (no addition of a zero, which the
  // compiler must keep for signed zeros)
  float U = 0.f;
#pragma unroll
  for (int n1 = 0; n1 <= NMAX; ++n1) {
    float T = shp[shp_index(n1, 0)];
#pragma unroll
    for (int n2 = 1; n2 <= NMAX - n1; ++n2) T = fmaf(shp[shp_index(n1, n2)], hv[n2], T);
    U = n1 == 0 ? T : fmaf(hu[n1], T, U);
  }
  return exp2_f32(-0.5f * kLog2e * (u * u + v * v)) * U;
}

// Factors 2^(-n/2) that take a coefficient of g_n1(u) g_n2(v), n = n1 + n2, to one of
// He_n1(x) He_n2(y) (shapelet_adj).
constexpr float kHeScale[kMaxNmax + 1] = {1.0f, 0.70710678118654752f, 0.5f, 0.35355339059327376f,
                                          0.25f, 0.17677669529663688f, 0.125f,
                                          0.08838834764831844f, 0.0625f};

// Shapelet accumulator terms and the weighted derivatives sb dI/d(beta_x, beta_y). They run
// over the probabilists' polynomials He_n(x) = 2^(n/2) g_n(u), x = sqrt(2) u:
// He_(n+1) = x He_n - n He_(n-1) and He_n' = n He_(n-1), so that the products n He_(n-1) serve
// the recurrence and the derivative sums. he: the coefficients c'_k 2^(-n/2).
//   dI/dx = G (sum_n1 n1 He_(n1-1)(x) T_n1 - x U / 2),
//   dI/dy = G (sum_n1 He_n1(x) Tv_n1 - y U / 2),  Tv_n1 = sum_n2 he_(n1,n2) n2 He_(n2-1)(y),
//   dI/dc_k = G He_n1(x) He_n2(y) / (sqrt(n1! n2!) beta sqrt(pi)) (the factor is applied when
//   the accumulators are mapped onto the gradient, and so is -1 / beta of the beta sum).
// The x-polynomials are taken times sg = sb G, so every sum over them carries the weight:
// U, Ux and Uy below are sb G times the sums above, and sb I = U.
template <int NMAX>
GL_HD void shapelet_adj(const PConst& c, float sdx, float sdy, const float* he, float sb,
                        float* acc, float& gbx, float& gby) {
  const float ib = c.rt2_ib;
  // sg is zero from |y| = 32 on (e^-256), and stays so: the y-polynomials, which do not carry it,
  // would overflow where the forward pass's g_n(v) are still finite (NaN from 0 x infinity)
  const float x = sdx * ib, y = clamp_f32(sdy * ib, 32.0f);
  const float sg = sb * exp2_f32(-0.25f * kLog2e * fmaf(x, x, y * y));
  float hx[NMAX + 2], hy[NMAX + 2];  // He_n, hx times sg
  float ex[NMAX + 2], ey[NMAX + 2];  // n He_(n-1), ex times sg
  hx[0] = sg;
  hy[0] = 1.f;
  ex[0] = ey[0] = 0.f;
#pragma unroll
  for (int n = 0; n < NMAX; ++n) {
    ex[n + 1] = n == 0 ? hx[0] : float(n + 1) * hx[n];
    ey[n + 1] = n == 0 ? 1.f : float(n + 1) * hy[n];
    hx[n + 1] = n == 0 ? x * hx[0] : fmaf(x, hx[n], -ex[n]);
    hy[n + 1] = n == 0 ? y : fmaf(y, hy[n], -ey[n]);
  }
  float U = 0.f, Ux = 0.f, Uy = 0.f;
#pragma unroll
  for (int n1 = 0; n1 <= NMAX; ++n1) {
    // He_0 = 1: T and Tv start from their first terms (no addition of a zero)
    float T = he[shp_index(n1, 0)], Tv = 0.f;
#pragma unroll
    for (int n2 = 1; n2 <= NMAX - n1; ++n2) {
      const float ck = he[shp_index(n1, n2)];
      T = fmaf(ck, hy[n2], T);
      Tv = n2 == 1 ? ck : fmaf(ck, ey[n2], Tv);
    }
    U = n1 == 0 ? hx[0] * T : fmaf(hx[n1], T, U);
    if (n1 < NMAX) Uy = n1 == 0 ? hx[0] * Tv : fmaf(hx[n1], Tv, Uy);
    if (n1 > 0) Ux = n1 == 1 ? ex[1] * T : fmaf(ex[n1], T, Ux);
  }
#pragma unroll
  for (int n1 = 0; n1 <= NMAX; ++n1) {
    acc[A_SHP_C + shp_index(n1, 0)] += hx[n1];
#pragma unroll
    for (int n2 = 1; n2 <= NMAX - n1; ++n2)
      acc[A_SHP_C + shp_index(n1, n2)] = fmaf(hx[n1], hy[n2], acc[A_SHP_C + shp_index(n1, n2)]);
  }
  const float Uh = 0.5f * U;
  const float Ix = fmaf(-x, Uh, Ux), Iy = fmaf(-y, Uh, Uy);  // sb dI/dx, sb dI/dy
  acc[A_SHP_BETA] += fmaf(y, Iy, fmaf(x, Ix, U));
  gbx = Ix * ib;
  gby = Iy * ib;
}

// d(source Sersic + shapelets)/d(beta) at offset (sdx, sdy) from the source centre, in FP64
// (the floored sub-pixel's weight g of the mass terms, formed once per particle):
//   Sersic: dI/dR^2 = -I b_n rho / (2 n R^2), rho = (R / R_eff)^(1/n), dR^2 = 2 (px, py);
//   shapelets: as shapelet_adj, with g_n' = n g_(n-1).
GL_HD void source_light_grad(const PConst& c, int nmax, double sdx, double sdy, double& gx,
                             double& gy) {
  const LightC& L = c.src;
  const double px = L.qa * sdx + 0.5 * double(L.qb) * sdy;
  const double py = L.qc * sdy + 0.5 * double(L.qb) * sdx;
  const double r2 = sdx * px + sdy * py;
  gx = gy = 0.0;
  if (r2 >= kR2FloorD) {
    const double n = L.n, rho = exp(log(r2) / (2.0 * n) - log(double(L.re)) / n);
    const double I = double(L.i0) * exp(double(L.bn) * (1.0 - rho));
    const double dIdr2 = -I * double(L.bn) * rho / (2.0 * n * r2);
    gx = 2.0 * dIdr2 * px;
    gy = 2.0 * dIdr2 * py;
  }
  if (nmax < 0) return;
  const double ib = c.inv_beta, u = sdx * ib, v = sdy * ib;
  double hu[kMaxNmax + 1], hv[kMaxNmax + 1];
  hu[0] = hv[0] = 1.0;
  hu[1] = u;
  hv[1] = v;
  for (int k = 1; k < nmax; ++k) {
    hu[k + 1] = u * hu[k] - 0.5 * k * hu[k - 1];
    hv[k + 1] = v * hv[k] - 0.5 * k * hv[k - 1];
  }
  double U = 0.0, Uu = 0.0, Uv = 0.0;
  for (int n1 = 0; n1 <= nmax; ++n1)
    for (int n2 = 0; n1 + n2 <= nmax; ++n2) {
      const double ck = c.shp[shp_index(n1, n2)];
      U += ck * hu[n1] * hv[n2];
      if (n1 > 0) Uu += ck * n1 * hu[n1 - 1] * hv[n2];
      if (n2 > 0) Uv += ck * n2 * hu[n1] * hv[n2 - 1];
    }
  const double G = exp(-0.5 * (u * u + v * v));
  gx += G * (Uu - u * U) * ib;
  gy += G * (Uv - v * U) * ib;
}

// ------------------------------------------------------------------------------------------
// Accumulators -> d logL / d theta in the parameter order of gl.h. Returns d.
// ------------------------------------------------------------------------------------------
// offsets: the centre slots hold s dx, s dy (lens light) instead of the gradient itself (source).
GL_HD void light_grad(const LightC& L, const double* a, bool offsets, float* g) {
  const double i0 = L.i0, bnn = L.bn / double(L.n);
  g[0] = float(i0 * a[L_RHO] * (bnn / L.re));                                  // R_eff
  g[1] = float(i0 * (bnn * kLn2 * a[L_RHOLN] - 1.9992 * a[L_RHO1]));          // n
  // sum s R^2 and the two eccentricity sums
  const double xx = a[L_XX], xy = a[L_XY], yy = a[L_YY];
  const double r2q = xx + yy + L.qa * xx + L.qb * xy + L.qc * yy;
  const double ge1 = L.inv1me2 * (L.e1 * r2q + yy - xx);
  const double ge2 = L.inv1me2 * (L.e2 * r2q - 2.0 * xy);
  g[2] = float(L.j11 * ge1 + L.j12 * ge2);                                     // eps1
  g[3] = float(L.j12 * ge1 + L.j22 * ge2);                                     // eps2
  const double dx = a[L_DX], dy = a[L_DY];
  g[4] = float(offsets ? -(L.qa * dx + L.qbh * dy) : -dx);                     // x
  g[5] = float(offsets ? -(L.qbh * dx + L.qc * dy) : -dy);                     // y
  g[6] = float(a[L_E]);                                                        // I0
}

// Sums of g . d alpha/d(theta) over the sub-pixels, from the accumulators a (mass_adjoint).
struct MassSums {
  double alpha, t, e1, e2, x, y, g1, g2;
};
GL_HD MassSums mass_sums(const PConst& c, const double* a) {
  MassSums m;
  const double e1 = c.e1, e2 = c.e2, ee = e1 * e1 + e2 * e2, oo = 1.0 / (1.0 - ee);
  const double ii = 1.0 / (c.icr * c.icr + c.ici * c.ici);
  // -2 tfac Re(gb alpha), where it is not in the sums
  const double k = c.epsabs < kSxClosedMin ? -c.t * oo * a[A_M_ALPHA] : 0.0;
  m.alpha = a[A_M_ALPHA];
  m.t = -0.5 * kLn2 * a[A_M_T];
  m.e1 = (a[A_M_E1] * c.icr + a[A_M_E2] * c.ici) * ii + k * e1;
  m.e2 = (a[A_M_E2] * c.icr - a[A_M_E1] * c.ici) * ii + k * e2;
  m.x = a[A_M_X];
  m.y = a[A_M_Y];
  const double gr = a[A_SRC + L_DX], gi = a[A_SRC + L_DY];  // sum g
  m.g1 = a[A_M_G1] + c.xc * gr - c.yc * gi;
  m.g2 = a[A_M_G2] + c.yc * gr + c.xc * gi;
  return m;
}

// The mass's part of the gradient, in the order of gl.h.
GL_HD void mass_grad(const MassC& c, const MassSums& m, int mass, int shear, float* gr) {
  int j = 0;
  gr[j++] = float(-double(c.t) / c.theta_e * m.alpha);
  if (mass == 1) gr[j++] = float(-m.t);
  gr[j++] = float(-(c.mj11 * m.e1 + c.mj12 * m.e2));
  gr[j++] = float(-(c.mj12 * m.e1 + c.mj22 * m.e2));
  gr[j++] = float(m.x);
  gr[j++] = float(m.y);
  if (shear) {
    gr[j++] = float(-m.g1);
    gr[j++] = float(-m.g2);
  }
}

// 1 / beta as the adjoint's sub-pixels have it (shapelet_adj): its FP32 rounding enters their
// Gaussians and these factors alike, and the two errors partly cancel (they do in G / beta at r =
// beta).
GL_HD double adjoint_inv_beta(const PConst& c) { return 0.7071067811865476 * c.rt2_ib; }

// Gradient component of shapelet coefficient q (0 <= q < M).
GL_HD float shapelet_coef_grad(const PConst& c, const double* a, int q) {
  int n1, n2;
  shapelet_orders(q, n1, n2);
  return float(a[A_SHP_C + q] * (adjoint_inv_beta(c) * kInvSqrtPi) *
               (hermite_scale(n1, n2) * double(kHeScale[n1 + n2])));
}

}  // namespace glens
