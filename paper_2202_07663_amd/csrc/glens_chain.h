// The sub-pixel passes of the sampler's chains: the ray trace with the SIE's closed form, and the
// adjoint with every sum of the gradient taken per sub-pixel.
//
// A chain's position reaches the pipeline rounded to FP32, and a rounding that falls the other
// way moves log p~ of a sharp posterior by up to 1e-5 of itself (measured on the 60 x 60 system:
// gradients that differ by 1e-7 flip some 100 of 64 x 51 rounded coordinates within three
// leapfrog steps, and the log p~ reached differ by 1e-6). So that a seed keeps giving the chains
// that it gave, the HMC launches keep this arithmetic, term for term; the batched likelihood
// calls, the fit and the variational fit take the shorter sums of glens_device.h (mass_adjoint).
// What that costs, one leapfrog step (these kernels, and the kick, move and decode fused into one
// launch) beside one gradient call of the batched kernels, in us: 60 x 60 EPL with n_max 6,
// 62.2 / 58.2 at 64 chains, 127 / 111 at 256, 180 / 165 at 512, 307 / 284 at 1024; with n_max 8,
// whose adjoint spills here, 97.6 / 62.2 at 64 and 288 / 195 at 512; an SIE with n_max 3, 52.5 / 53.1
// at 64 and 165 / 131 at 512. The two are alike where a launch leaves the chip partly idle and the
// adjoint does not spill; elsewhere the same chains are what is paid for.
#pragma once

#include <hip/hip_runtime.h>

#include "glens_device.h"
#include "glens_sums.h"

namespace glens {
namespace chain {

// EPL / SIE deflection plus shear at image position (x, y), in FP64: returns beta - x_s with
// beta = x - alpha - alpha_ext.
// at_floor: this is the particle's floored sub-pixel (c.fl_*); the SIE then takes the
// frozen-radius closed form the prologue evaluated (the EPL's value there is this formula's).
// cs / pw: the particle's series coefficients c.c and power tables c.pw (staged in LDS).
template <int MASS>
GL_HD void ray_trace(const PConst& c, const double* __restrict__ cs,
                     const double* __restrict__ pw, double x, double y, bool at_floor,
                     float& sdx, float& sdy) {
  const double zr = x - c.xc, zi = y - c.yc;
  const double e1 = c.e1, e2 = c.e2;
  const double wr = zr - e1 * zr - e2 * zi, wi = zi - e2 * zr + e1 * zi;
  const double w2 = fmax(wr * wr + wi * wi, c.w2floor);
  const double inv_w2 = rcp_f64(w2);
  const double u2r = (wr * wr - wi * wi) * inv_w2, u2i = 2.0 * wr * wi * inv_w2;
  const double Xr = e1 * u2r + e2 * u2i, Xi = e1 * u2i - e2 * u2r;
  double Sr, Si, A;
  if (MASS == 0 && c.sie_closed) {
    // S_1(X) = atan(zeta) / zeta, zeta = s w / |w|; atan of |zeta| < 1 in closed form
    const double rinv = sqrt(inv_w2);
    const double ur = wr * rinv, ui = wi * rinv;
    const double a = c.sr * ur - c.si * ui, b = c.sr * ui + c.si * ur;
    const double aa = a * a;
    const double atr = 0.5 * atan(2.0 * a / (1.0 - c.epsabs));
    const double ati = 0.25 * log(((1.0 + b) * (1.0 + b) + aa) / ((1.0 - b) * (1.0 - b) + aa));
    const double ie = 1.0 / c.epsabs;  // S = atan(zeta) conj(zeta) / |eps|
    Sr = (atr * a + ati * b) * ie;
    Si = (ati * a - atr * b) * ie;
    A = c.bmass * rinv;
  } else {
    // The coefficients are real, so the series is evaluated at the complex point y = -X by
    // synthetic division by the real quadratic (v - y)(v - conj y) = v^2 - 2 Re(y) v + |y|^2
    // (Knuth, TAOCP vol. 2, sec. 4.6.4): b_n = c_n + 2 Re(y) b_(n+1) - |y|^2 b_(n+2) from the
    // top down to n = 0, and the sum is b_0 - Re(y) b_1 + i Im(y) b_1. That is two real FMAs
    // per term where complex Horner takes four. |y| = |eps| < 1, so rounding errors made
    // early are damped as the recurrence runs down. Terms are taken two per trip (so that the
    // two carried values need no register moves); coefficients past the series length are
    // zero, so rounding the length up to an even number is exact.
    const double yr = -Xr, yi = -Xi;
    const double r2 = 2.0 * yr, yy = fma(yr, yr, yi * yi);
    double b1 = 0.0, b2 = 0.0;  // b_(n+1), b_(n+2)
    const int nt2 = (c.nterms + 1) & ~1;
    for (int n0 = nt2 - 2; n0 >= 0; n0 -= 2) {  // leaves b_n0 in b1 and b_(n0+1) in b2
      b2 = fma(r2, b1, fma(-yy, b2, cs[n0 + 1]));
      b1 = fma(r2, b2, fma(-yy, b1, cs[n0]));
    }
    Sr = fma(-yr, b2, b1);
    Si = yi * b2;
    A = pow_from_table(pw, w2);
  }
  double ar = A * (wr * Sr - wi * Si), ai = A * (wr * Si + wi * Sr);
  if (MASS == 0 && at_floor) {
    ar = c.fl_a[0];
    ai = c.fl_a[1];
  }
  // beta - x_s = x - alpha - alpha_ext - x_s
  sdx = float(x - ar - (c.g1 * x + c.g2 * y) - c.sxs);
  sdy = float(y - ai - (c.g2 * x - c.g1 * y) - c.sys);
}

template <int MASS, int LL, int NMAX>
__device__ __forceinline__ float surface_brightness(const PConst& c, const double* cs,
                                                    const double* s_pw, double x, double y,
                                                    bool at_floor, const float* shp,
                                                    float2& sd) {
  chain::ray_trace<MASS>(c, cs, s_pw, x, y, at_floor, sd.x, sd.y);
  float v = sersic_fwd(c.src, sd.x, sd.y);
  if (NMAX >= 0) v += shapelet_fwd<(NMAX < 0 ? 0 : NMAX)>(c, sd.x, sd.y, shp);
  if (LL) v += sersic_fwd(c.lens, float(x - c.lxs), float(y - c.lys));
  return v;
}

// MASS: 0 SIE, 1 EPL; LL: lens light on (1) or off (0); NMAX: shapelet order (-1: none).
// Every system of one launch has the same (MASS, LL, NMAX).
// The pixels [p0, p1) of one particle's model image. The restrict qualifiers tell the compiler
// that the image stores do not write the particle's constants, which then stay scalar loads.
template <int MASS, int LL, int NMAX>
// beta (or null): where beta - x_s of each sub-pixel is kept for the adjoint, [k^2][H][W].
__device__ __forceinline__ void forward_pixels(const SysDesc& s, const PConst* __restrict__ c,
                                               const double* cs, const double* s_pw,
                                               float* __restrict__ out,
                                               float2* __restrict__ beta, int p0, int p1) {
  const int W = s.W, k = s.k;
  // shapelet coefficients held in vector registers for the whole loop (an empty asm with a
  // vector-register operand): the scalar registers, which the compiler had filled, keep the
  // other constants instead of reloading them every sub-pixel
  constexpr int M = NMAX < 0 ? 1 : (NMAX + 1) * (NMAX + 2) / 2;
  float shp[M];
#pragma unroll
  for (int q = 0; q < M; ++q) {
    shp[q] = NMAX < 0 ? 0.f : c->shp[q];
    asm("" : "+v"(shp[q]));
  }
  for (int pix = p0 + threadIdx.x; pix < p1; pix += blockDim.x) {
    const int i = pix / W, j = pix - i * W;
    float sum = 0.f;
    for (int a = 0; a < k; ++a) {
      const double y = subpix_coord(s.y0, i * k + a, s.dxs);
      for (int b = 0; b < k; ++b) {
        const double x = subpix_coord(s.x0, j * k + b, s.dxs);
        // the SIE's floored sub-pixel takes the prologue's frozen-radius deflection
        const bool at_floor = MASS == 0 && i * k + a == c->fl_i && j * k + b == c->fl_j;
        float2 sd;
        sum += surface_brightness<MASS, LL, NMAX>(*c, cs, s_pw, x, y, at_floor, shp, sd);
        if (beta) {  // streamed past the caches: read once, by the adjoint, much later
          float* bp = reinterpret_cast<float*>(beta + (a * k + b) * (s.H * W) + pix);
          __builtin_nontemporal_store(sd.x, bp);
          __builtin_nontemporal_store(sd.y, bp + 1);
        }
      }
    }
    out[pix] = sum * s.inv_k2;
  }
}

// Accumulator slots (per particle, summed over sub-pixels).
enum AccSlot {
  A_M_ALPHA = 0,  // sum g.alpha                      -> theta_E (and SIE)
  A_M_T = 1,      // sum g.(d alpha / d t)             -> gamma_epl
  A_M_E1 = 2, A_M_E2 = 3,   // sum g.(d alpha / d eps_k) (clamped eps)
  A_M_X = 4, A_M_Y = 5,     // sum g.(d alpha / d x), g.(d alpha / d y)
  A_M_G1 = 6, A_M_G2 = 7,   // sum g.(x, -y), g.(y, x)
  A_LENS = 8,     // 8 slots, see LightSlot
  A_SRC = 16,     // 8 slots; the centre slots also collect the shapelet beta-gradient
  A_SHP_BETA = 24,
  A_SHP_C = 25,   // kMaxShp slots
};
enum LightSlot { L_E = 0, L_RHO = 1, L_RHO1 = 2, L_RHOLN = 3, L_Q1 = 4, L_Q2 = 5, L_DX = 6, L_DY = 7 };
static_assert(A_SHP_C + kMaxShp <= kNAcc, "accumulator slots");

// The lens quantities of one sub-pixel that the adjoint uses (FP32).
struct MassState {
  float sdx, sdy;     // beta - x_s (source offset)
  Cx z, w, u2, X;     // z, w, w^2/|w|^2, X = conj(eps) u2
  float lnw2;         // ln |w|^2 (floored)
  float A;            // B^t |w|^-t
  Cx S, XSX, U2SX, St;  // S_t(X), X dS/dX, u2 dS/dX, dS/dt
  Cx alpha;
};

// The lens quantities the adjoint needs, in FP32: z, w, u2, X, ln|w|^2, A, S, X dS/dX,
// u2 dS/dX, dS/dt, alpha. (sdx, sdy) is beta - x_s of the forward pass's FP64 ray trace (SysDesc::beta): the
// light profiles and their derivatives are evaluated there (an FP32 ray trace moves it by
// ~3e-7 arcsec, which shows at 2e-3 in the gradient of a vector far from the posterior). The
// rest only enters the Jacobian d(beta)/d(theta) and the local derivatives, whose tolerance
// (a relative 1e-3 on the gradient) is far above FP32 rounding:
//   alpha = x - alpha_ext - x_s - (beta - x_s), formed from the kept offset (FP64 up to the
//         last subtraction), and S = alpha / (A w), so the value series is not run again
//         (a sub-pixel whose |w|^2 hit the floor, where alpha carries no S, sums it);
//   dS/dX by the closed form of the identity below for |eps| >= kSxClosedMin (its numerator
//         cancels like |eps|, costing at most a relative 1e-6 / 0.02), by its series below;
//   dS/dt (EPL) by its series; the series run over the FP32-resolution length nterms_d;
//   log and exp are the hardware ones.
// |w|^2 is kept at or above the floor so that every quantity stays finite; the particle's
// floored sub-pixel itself (c.fl_*) takes its mass terms from the prologue's exact
// derivatives instead (the caller passes a zero weight here).
// ncs / dcs: the particle's c.nc / c.dc (staged in LDS). SXS = false: the caller has checked
// that |eps| >= kSxClosedMin, so dS/dX takes the closed form without a test.
template <int MASS, bool SXS = true>
__device__ __forceinline__ void mass_jacobian_f32(const PConst& c, const float* __restrict__ ncs,
                                                  const float* __restrict__ dcs, double x,
                                                  double y, float sdx, float sdy, MassState& m) {
  const float zr = float(x) - c.xcf, zi = float(y) - c.ycf;
  const float e1 = c.e1f, e2 = c.e2f;
  const float wr = zr - e1 * zr - e2 * zi, wi = zi - e2 * zr + e1 * zi;
  const float w2 = fmaxf(wr * wr + wi * wi, c.w2floorf);
  const float inv_w2 = rcp_f32(w2);
  const float u2r = (wr * wr - wi * wi) * inv_w2, u2i = 2.0f * wr * wi * inv_w2;
  const float Xr = e1 * u2r + e2 * u2i, Xi = e1 * u2i - e2 * u2r;
  const float l2w2 = log2_f32(w2);
  m.sdx = sdx;
  m.sdy = sdy;
  m.z = {zr, zi};
  m.w = {wr, wi};
  m.u2 = {u2r, u2i};
  m.X = {Xr, Xi};
  m.lnw2 = kLn2f * l2w2;
  // A = B^t |w|^-t = 2^(t log2 B - (t/2) log2 |w|^2) (SIE: t = 1)
  const float A = exp2_f32(fmaf(-0.5f * c.tf, l2w2, c.tlnb2));
  const float ar = float(x - (c.g1 * x + c.g2 * y) - c.sxs) - sdx;
  const float ai = float(y - (c.g2 * x - c.g1 * y) - c.sys) - sdy;
  // series by synthetic division at y = -X (ray_trace): dS/dt (EPL) and, for small |eps|,
  // dS/dy
  const float yr = -Xr, yi = -Xi, r2 = 2.0f * yr, yy = yr * yr + yi * yi;
  const bool sx_series = SXS && c.epsabs < kSxClosedMin;
  // four terms per trip, the length rounded up to a multiple of four (the padding
  // coefficients are zero): the LDS reads of a trip go out together, which at this kernel's
  // three waves per SIMD was measured faster than two terms per trip. dS/dt (EPL) here, dS/dy
  // (small |eps| only) below in a loop of its own, so that the common path carries no state
  // of the other.
  const int nd4 = (c.nterms_d + 3) & ~3;
  float t1 = 0.f, t2 = 0.f;
  if (MASS == 1) {
    for (int n0 = nd4 - 4; n0 >= 0; n0 -= 4) {
#pragma unroll
      for (int q = 3; q >= 0; --q) {
        const float t0 = fmaf(r2, t1, fmaf(-yy, t2, dcs[n0 + q]));
        t2 = t1;
        t1 = t0;
      }
    }
  }
  // S = alpha conj(w) / (A |w|^2)
  const float r = rcp_f32(A * w2);
  const float Sr = (ar * wr + ai * wi) * r;
  const float Si = (ai * wr - ar * wi) * r;
  if (sx_series) {
    float d1 = 0.f, d2 = 0.f;
    for (int n0 = nd4 - 4; n0 >= 0; n0 -= 4) {
#pragma unroll
      for (int q = 3; q >= 0; --q) {
        const float d0 = fmaf(r2, d1, fmaf(-yy, d2, ncs[n0 + q]));
        d2 = d1;
        d1 = d0;
      }
    }
    const Cx SX = {-fmaf(-yr, d2, d1), -yi * d2};  // dS/dX = -dS/dy
    m.XSX = cmul(m.X, SX);
    m.U2SX = cmul(m.u2, SX);
  } else {
    // S = sum c_n (-X)^n with c_n / c_(n-1) = (2n - 2 + t) / (2n + 2 - t) obeys
    //   X (1 + X) dS/dX = (1 - t/2)(1 - S) - (t/2) X S
    // (as series: the coefficient of (-X)^n on both sides agrees for every n; for the SIE,
    // t = 1, it is S_X = (1/(1+X) - S) / (2X), which the closed form atan(zeta)/zeta obeys),
    // so X dS/dX is the right side over 1 + X, and u2 dS/dX = X dS/dX / conj(eps), as
    // X = conj(eps) u2. The numerator cancels like |X| = |eps|, so this is used for
    // |eps| >= kSxClosedMin only.
    const float xsr = Xr * Sr - Xi * Si, xsi = Xr * Si + Xi * Sr;
    const float numr = c.hp * (1.0f - Sr) + c.hm * xsr;
    const float numi = -c.hp * Si + c.hm * xsi;
    const float opr = 1.0f + Xr, inv = rcp_f32(opr * opr + Xi * Xi);
    m.XSX = {(numr * opr + numi * Xi) * inv, (numi * opr - numr * Xi) * inv};
    m.U2SX = cmul(m.XSX, Cx{c.iebr, c.iebi});
  }
  m.St = MASS == 1 ? Cx{fmaf(-yr, t2, t1), yi * t2} : Cx{0.f, 0.f};
  m.A = A;
  m.S = {Sr, Si};
  m.alpha = {ar, ai};
}

// Adds the mass-parameter terms g . d alpha/d(theta) to acc, with g = d s / d beta (already
// weighted by the pixel adjoint); beta = x - alpha - alpha_ext, so the signs are applied at
// the mapping. For a complex derivative D, g . D = Re(gb D) with gb = conj(g), and every
// derivative is contracted with gb as soon as it is formed:
//   with aw = d alpha/dw = A P1 and awb = d alpha/d conj(w) = A u2 P2 (eps fixed),
//   U = gb aw, V = gb awb;
//   d alpha/dz = aw - conj(eps) awb, d alpha/d conj(z) = awb - eps aw, and with x = z +
//   conj z, y = i (z - conj z):
//     g . d alpha/dx = Re((1 - eps) U + (1 - conj eps) V) = (1 - e1) Sp + e2 Dm,
//     g . d alpha/dy = -Im((1 + eps) U - (1 + conj eps) V) = -(1 + e1) Dm - e2 Sp,
//   Sp = Re U + Re V, Dm = Im U - Im V;
//   d alpha/d eps = -tfac conj(eps) alpha - conj(z) aw,
//   d alpha/d conj(eps) = -tfac eps alpha - z awb + A w u2 S_X (A depends on |eps|^2, X on
//   conj(eps)); with eps = e1 + i e2 and W = gb A w u2 S_X:
//     g . d alpha/de1 = -2 tfac e1 Re(gb alpha) - Re(z) Sp - Im(z) Dm + Re W,
//     g . d alpha/de2 = -2 tfac e2 Re(gb alpha) + Re(z) Dm - Im(z) Sp + Im W;
//   d alpha/dt = alpha (ln B - ln|w|^2 / 2) + A w S_t.
template <int MASS>
GL_HD void mass_adjoint(const PConst& c, const MassState& m, float x, float y, Cx g, float* acc) {
  const Cx XSX = m.XSX;
  const Cx P1 = cadd(cscale(m.S, c.hp), XSX);  // (1 - t/2) S + X S_X
  const Cx P2 = csub(cscale(m.S, c.hm), XSX);  // -(t/2) S - X S_X
  const Cx gA = {g.r * m.A, -g.i * m.A};  // A gb
  const Cx U = cmul(gA, P1);
  const Cx V = cmul(gA, cmul(m.u2, P2));
  const float Sp = U.r + V.r, Dm = U.i - V.i;
  const float e1 = c.e1f, e2 = c.e2f;
  const float ga = cdot(g, m.alpha);  // Re(gb alpha)
  const Cx gAw = cmul(gA, m.w);
  const Cx W = cmul(gAw, m.U2SX);
  acc[A_M_ALPHA] += ga;
  if (MASS == 1) {
    const float lt = fmaf(-0.5f, m.lnw2, c.lnb);  // ln B - ln|w|^2 / 2
    acc[A_M_T] += fmaf(lt, ga, gAw.r * m.St.r - gAw.i * m.St.i);
  }
  const float k = -2.0f * c.tfac;
  acc[A_M_E1] += fmaf(k * e1, ga, W.r - m.z.r * Sp - m.z.i * Dm);
  acc[A_M_E2] += fmaf(k * e2, ga, W.i + m.z.r * Dm - m.z.i * Sp);
  acc[A_M_X] += fmaf(1.0f - e1, Sp, e2 * Dm);
  acc[A_M_Y] -= fmaf(1.0f + e1, Dm, e2 * Sp);
  acc[A_M_G1] += g.r * x - g.i * y;
  acc[A_M_G2] += g.r * y + g.i * x;
}

// Accumulator terms (weight sb) and the weighted sb dI/d(dx, dy). With the half gradient of
// R^2, (px, py) = (qa dx + qb dy / 2, qb dx / 2 + qc dy), R^2 = dx px + dy py and
// dR^2/d(dx, dy) = 2 (px, py); dI/dR^2 = -I b_n rho / (2 n R^2), so
// 2 sb dI/dR^2 = sb I rho (-b_n / n) / R^2 =: sIQ2 and sb dI/d(dx, dy) = sIQ2 (px, py).
// Slots: L_E: sb E; L_RHO: sb I rho; L_RHO1: sb I (rho - 1); L_RHOLN: sb I rho log2(rho)
// (ln 2 is applied at the mapping); L_Q1, L_Q2: the two eccentricity terms times
// 2 sb dI/dR^2 (the 1/2 is applied at the mapping).
GL_HD void sersic_adj(const LightC& L, float dx, float dy, float sb, float* acc, float& gdx,
                      float& gdy) {
  const float px = fmaf(L.qa, dx, L.qbh * dy), py = fmaf(L.qc, dy, L.qbh * dx);
  float q = fmaf(dx, px, dy * py);
  const bool fl = q < kR2Floor;
  q = fl ? kR2Floor : q;
  const float l2rho = fmaf(log2_f32(q), L.inv2n, -L.l2re_n);
  const float rho = exp2_f32(l2rho);
  const float sE = sb * exp2_f32(fmaf(-L.bnl, rho, L.bnl));
  const float sI = L.i0 * sE, sIr = sI * rho;
  const float sIQ2 = fl ? 0.0f : sIr * L.kq * rcp_f32(q);
  gdx = sIQ2 * px;
  gdy = sIQ2 * py;
  const float r2q = fmaf(dx, dx, fmaf(dy, dy, q));
  acc[L_E] += sE;
  acc[L_RHO] += sIr;
  acc[L_RHO1] += sIr - sI;
  acc[L_RHOLN] = fmaf(sIr, l2rho, acc[L_RHOLN]);
  acc[L_Q1] = fmaf(sIQ2, fmaf(L.e1, r2q, fmaf(dy, dy, -dx * dx)), acc[L_Q1]);
  acc[L_Q2] = fmaf(sIQ2, fmaf(L.e2, r2q, -2.0f * dx * dy), acc[L_Q2]);
}

// Shapelet accumulator terms and the weighted derivatives sb dI/d(beta_x, beta_y), using
// g_n' = n g_(n-1) for the scaled Hermite polynomials:
//   dI/du = G (sum_n1 n1 g_(n1-1)(u) T_n1 - u U),
//   dI/dv = G (sum_n1 g_n1(u) Tv_n1 - v U),  Tv_n1 = sum_n2 c'_(n1,n2) n2 g_(n2-1)(v),
//   dI/dc_k = G g_n1(u) g_n2(v) r_n1 r_n2 / (beta sqrt(pi)) (the factor r_n1 r_n2 /
//   (beta sqrt(pi)) is applied when the accumulators are mapped onto the gradient).
// The u-polynomials are taken times sg = sb G, so every sum over them carries the weight:
// U, Uu and Uv below are sb G times the sums above, and sb I = U.
template <int NMAX>
GL_HD void shapelet_adj(const PConst& c, float sdx, float sdy, const float* shp, float sb,
                        float* acc, float& gbx, float& gby) {
  const float ib = c.inv_beta;
  const float u = sdx * ib, v = sdy * ib;
  const float sg = sb * exp2_f32(-0.5f * kLog2e * (u * u + v * v));
  float hu[NMAX + 1], hv[NMAX + 1];
  hermite<NMAX>(u, hu, sg);
  hermite<NMAX>(v, hv);
  float U = 0.f, Uu = 0.f, Uv = 0.f;
#pragma unroll
  for (int n1 = 0; n1 <= NMAX; ++n1) {
    // g_0(v) = 1: T starts from its n2 = 0 term (no addition of a zero)
    float T = shp[shp_index(n1, 0)], Tv = 0.f;
#pragma unroll
    for (int n2 = 1; n2 <= NMAX - n1; ++n2) {
      const float ck = shp[shp_index(n1, n2)];
      T = fmaf(ck, hv[n2], T);
      Tv = n2 == 1 ? ck : fmaf(ck, float(n2) * hv[n2 - 1], Tv);
    }
    U = n1 == 0 ? hu[0] * T : fmaf(hu[n1], T, U);
    if (n1 < NMAX) Uv = n1 == 0 ? hu[0] * Tv : fmaf(hu[n1], Tv, Uv);
    if (n1 > 0) Uu = n1 == 1 ? hu[0] * T : fmaf(float(n1) * hu[n1 - 1], T, Uu);
  }
#pragma unroll
  for (int n1 = 0; n1 <= NMAX; ++n1)
#pragma unroll
    for (int n2 = 0; n2 <= NMAX - n1; ++n2)
      acc[A_SHP_C + shp_index(n1, n2)] = fmaf(hu[n1], hv[n2], acc[A_SHP_C + shp_index(n1, n2)]);
  const float Iu = Uu - u * U, Iv = Uv - v * U;  // sb dI/du, sb dI/dv
  acc[A_SHP_BETA] += (-U - u * Iu - v * Iv) * ib;
  gbx = Iu * ib;
  gby = Iv * ib;
}

// ------------------------------------------------------------------------------------------
// Accumulators -> d logL / d theta in the parameter order of gl.h.
// ------------------------------------------------------------------------------------------
GL_HD void light_grad(const LightC& L, const double* a, float* g) {
  g[0] = float(a[L_RHO] * L.bn / (double(L.n) * L.re));                 // R_eff
  g[1] = float(-1.9992 * a[L_RHO1] + L.bn / double(L.n) * kLn2 * a[L_RHOLN]);  // n
  const double ge1 = L.inv1me2 * a[L_Q1], ge2 = L.inv1me2 * a[L_Q2];
  g[2] = float(L.j11 * ge1 + L.j12 * ge2);                               // eps1
  g[3] = float(L.j12 * ge1 + L.j22 * ge2);                               // eps2
  g[4] = float(-a[L_DX]);                                                // x
  g[5] = float(-a[L_DY]);                                                // y
  g[6] = float(a[L_E]);                                                  // I0
}

GL_HD MassSums mass_sums(const double* a) {
  return {a[A_M_ALPHA], a[A_M_T], a[A_M_E1], a[A_M_E2], a[A_M_X], a[A_M_Y], a[A_M_G1], a[A_M_G2]};
}

// Gradient component of shapelet coefficient q (0 <= q < M).
GL_HD float shapelet_coef_grad(const PConst& c, const double* a, int q) {
  int n1, n2;
  shapelet_orders(q, n1, n2);
  return float(a[A_SHP_C + q] * (double(c.inv_beta) * kInvSqrtPi) * hermite_scale(n1, n2));
}

// The sub-pixels of pixels [p0, p1) of one particle into the per-lane accumulators.
// GENERAL = false: the particle has no floored sub-pixel and |eps| >= kSxClosedMin.
template <int MASS, int LL, int NMAX, bool GENERAL>
__device__ __forceinline__ void adj_pixels(const SysDesc& s, const PConst& c,
                                           const float* s_nc, const float* s_dc,
                                           const float* shp, const float2* beta,
                                           const float* sbar, int p0, int p1, float* acc) {
  const int HW = s.H * s.W, W = s.W, k = s.k;
  const int fl_i = c.fl_i, fl_j = c.fl_j;
  for (int pix = p0 + threadIdx.x; pix < p1; pix += blockDim.x) {
    const int i = pix / W, j = pix - i * W;
    const float sb = sbar[pix];
    for (int a = 0; a < k; ++a) {
      const double y = subpix_coord(s.y0, i * k + a, s.dxs);
      for (int b = 0; b < k; ++b) {
        const double x = subpix_coord(s.x0, j * k + b, s.dxs);
        MassState m;
        const float* bp = reinterpret_cast<const float*>(beta + (a * k + b) * HW + pix);
        chain::mass_jacobian_f32<MASS, GENERAL>(c, s_nc, s_dc, x, y, __builtin_nontemporal_load(bp),
                                         __builtin_nontemporal_load(bp + 1), m);
        // gx, gy: sb d(source light)/d(beta)
        float gx, gy;
        chain::sersic_adj(c.src, m.sdx, m.sdy, sb, acc + A_SRC, gx, gy);
        if (NMAX >= 0) {
          float hx, hy;
          chain::shapelet_adj<(NMAX < 0 ? 0 : NMAX)>(c, m.sdx, m.sdy, shp, sb, acc, hx, hy);
          gx += hx;
          gy += hy;
        }
        acc[A_SRC + L_DX] += gx;
        acc[A_SRC + L_DY] += gy;
        if (LL) {
          float lx, ly;
          chain::sersic_adj(c.lens, float(x - c.lxs), float(y - c.lys), sb, acc + A_LENS, lx, ly);
          acc[A_LENS + L_DX] += lx;
          acc[A_LENS + L_DY] += ly;
        }
        // the floored sub-pixel's mass terms are added by finalize from the prologue's
        // exact derivatives
        const bool at_floor = GENERAL && i * k + a == fl_i && j * k + b == fl_j;
        chain::mass_adjoint<MASS>(c, m, float(x), float(y),
                           at_floor ? Cx{0.f, 0.f} : Cx{gx, gy}, acc);
      }
    }
  }
}

template <int NMAX>
constexpr int n_slots() {
  return NMAX < 0 ? A_SHP_BETA : A_SHP_C + (NMAX + 1) * (NMAX + 2) / 2;
}

}  // namespace chain
}  // namespace glens
