// Per-particle stages of the likelihood pipeline that run as one block per particle: the decode
// (prologue; one wave, or four where the batch leaves the chip idle: launch_prologue) and the
// gradient finalize (one wave). The pipeline's prologue_kernel and finalize_kernel wrap them, and
// so do kernels that fuse them with a sampler's per-chain step (the HMC kick and drift), which
// saves a launch and its fixed cost per step at small batches.
#pragma once

#include <hip/hip_runtime.h>

#include "glens_chain.h"
#include "glens_device.h"
#include "glens_fit_device.h"

namespace glens {

// Orders the LDS accesses of one wave's lanes (LDS serves a wave in order, so nothing is waited
// for): the barrier of code that one wave of a block runs alone.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// ------------------------------------------------------------------------------------------
// prologue: one block of WAVES = 1 or 4 waves per particle. Bound by latency (one chain of FP64
// logarithms, square roots and divisions, its code fetched once per wave), so four waves take one
// part each, and decode for themselves what it needs of the mass (passed through the particle's
// constants in memory it would cost two L2 round trips):
//   0  the mass, and the series: lane n (1 <= n < kMaxTerms) computes the ratio c_n / c_(n-1)
//      and the increment of d log c_n / dt; inclusive scans across the wave (product and sum)
//      give every lane its c_n and d log c_n / dt;
//   1  lanes 1 and 2 the light profiles, lanes 3 .. one shapelet coefficient each;
//   2  the power tables' first half and their polynomial segments;
//   3  the second half; its lane 63 looks for the floored sub-pixel.
// One wave (a kernel that works on the particle with one wave before) takes them in turn.
// z_lds (or null): the particle's unconstrained parameters, in LDS, instead of s.z.
// ------------------------------------------------------------------------------------------
constexpr int kPrologueMaxWaves = 4;
// Waves per particle of a launch over n particles: four while the chip runs them all at once
// (three blocks per CU); beyond, the sum of their work counts, which one wave has less of (60 x 60
// EPL: 64 particles 7.7 us with one wave, 5.5 with four; 512: 11.0 and 8.8, 1024: 11.7 and 12.6
// between events; 4096: 16.6 and 28.2 us).
inline int prologue_waves(int n) { return n <= 768 ? kPrologueMaxWaves : 1; }
template <int WAVES>
__device__ __forceinline__ void prologue_particle(const SysDesc& s, int p,
                                                  const float* z_lds = nullptr) {
  static_assert(WAVES == 1 || WAVES == 4, "one wave for all parts, or one per part");
  static_assert(kPowExp == 128, "one exponent entry per lane of two waves");
  static_assert(kMaxTerms <= 63, "one lane per series term, lane 63 free");
  static_assert(3 + kMaxShp <= 64, "one lane per shapelet coefficient");
  __shared__ float th[kMaxParams];
  const int d = s.d, lane = threadIdx.x & 63;
  const int wave = WAVES == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int j = threadIdx.x; j < d; j += 64 * WAVES) {
    const size_t i = (size_t)p * d + j;
    if (s.z) {
      th[j] = bijector_fwd(s.prior[j], z_lds ? z_lds[j] : s.z[i]);
      s.theta_out[i] = th[j];
    } else {
      th[j] = s.theta[i];
    }
  }
  __syncthreads();
  PConst& c = s.pc[p];
  const float* xs = th + mass_param_count(s.mass, s.shear) + (s.lens_light ? 7 : 0) + 4;
  if (WAVES == 4 && wave == 1) {
    decode_lights_lane(th, s.mass, s.shear, s.lens_light, s.nmax, c, lane);
    return;
  }
  MassC m;
  decode_mass(th, s.mass, s.shear, m);
  if (WAVES == 4 && wave >= 2) {
    const int i = lane + 64 * (wave - 2);
    const double log2B = log2(m.bmass);
    c.pw[i] = pow_exponent_entry(m.t, log2B, i);
    if (wave == 2)
      pow_segments_lane(m.t, lane - (64 - kPowSeg), c.pw);
    else if (lane == 63)
      decode_floor(s, xs, m, c);
    return;
  }
  if (lane == 0) static_cast<MassC&>(c) = m;
  if (WAVES == 1) decode_lights_lane(th, s.mass, s.shear, s.lens_light, s.nmax, c, lane);
  double cn = 1.0, dsum = 0.0;  // lane n: c_n / c_(n-1) and its d log / dt increment (n >= 1)
  if (lane > 0 && lane < kMaxTerms) series_step(lane, m.t, cn, dsum);
  for (int o = 1; o < 64; o <<= 1) {  // inclusive scans: c_n and d log c_n / dt on lane n
    const double pc = __shfl_up(cn, o, 64), pd = __shfl_up(dsum, o, 64);
    if (lane >= o) {
      cn *= pc;
      dsum += pd;
    }
  }
  if (WAVES == 1) {
    if (lane == 63)
      decode_floor(s, xs, m, c);
    else
      pow_tables_lane(m.t, log2(m.bmass), lane, 63, c.pw);
  }
  if (lane < kMaxTerms) series_store(m, c, lane, cn, dsum);
}

// ------------------------------------------------------------------------------------------
// finalize: one wave per particle (the first of its block); lanes sum the tiles' partial
// accumulators (in tile order); lane 0 maps the mass's sums to the parameter gradient, lanes 1
// and 2 the light profiles' (one pass over the code for both), the other lanes one shapelet
// coefficient each; a vector whose log L or gradient is not finite gets log L = -inf and a zero
// gradient. Returns the gradient's components (in LDS, before that check), and whether it
// passed, to every lane. Bound by latency: 5.9 -> 4.3 us (60 x 60, 64 vectors of 15 tiles, whose
// partial sums were loaded one after the other past the eighth).
// CHAIN: the accumulators are those of the sampler's adjoint (glens_chain.h).
// ------------------------------------------------------------------------------------------
struct FinalGrad {
  const float* g;
  bool ok;
  double logl;
};
template <bool CHAIN>
__device__ __forceinline__ FinalGrad finalize_particle(const SysDesc& s, int p) {
  __shared__ double a[kNAcc];
  __shared__ float gr[kMaxParams];
  const PConst& c = s.pc[p];
  const int lane = threadIdx.x, nmax = s.nmax;
  const int lens0 = CHAIN ? int(chain::A_LENS) : lens_slot(nmax);
  const int src0 = CHAIN ? int(chain::A_SRC) : int(A_SRC);
  const int ns = CHAIN ? int(chain::A_SHP_BETA) + (nmax < 0 ? 0 : 1 + (nmax + 1) * (nmax + 2) / 2)
                       : lens0 + (s.lens_light ? kLightSlots : 0);
  const int tiles = CHAIN ? s.tiles : s.adj_tiles;
  const double logl = s.logl[p];
  const LightC L = lane == 1 ? c.lens : c.src;  // on its way while the sums are taken
  const double* acc = s.acc + (size_t)p * tiles * kNAcc;
  for (int q = lane; q < ns; q += 64) {
    double v = 0.0;
    for (int t0 = 0; t0 < tiles; t0 += 16) {  // sixteen loads in flight, added in tile order
      double b[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) b[u] = t0 + u < tiles ? acc[(t0 + u) * kNAcc + q] : 0.0;
#pragma unroll
      for (int u = 0; u < 16; ++u) v += b[u];
    }
    a[q] = v;
  }
  wave_sync();
  // the layout of gl.h: mass, lens light, source, shapelet scale and coefficients
  const int jl = mass_param_count(s.mass, s.shear), js = jl + (s.lens_light ? 7 : 0), jb = js + 7;
  const int M = nmax < 0 ? 0 : (nmax + 1) * (nmax + 2) / 2, d = jb + (nmax < 0 ? 0 : 1 + M);
  if (lane == 2 || (lane == 1 && s.lens_light)) {
    const double* al = a + (lane == 1 ? lens0 : src0);
    float* g = gr + (lane == 1 ? jl : js);
    if (CHAIN)
      chain::light_grad(L, al, g);
    else
      light_grad(L, al, lane == 1, g);
  }
  for (int q = lane - 3; q >= 0 && q < M; q += 61)
    gr[jb + 1 + q] = CHAIN ? chain::shapelet_coef_grad(c, a, q) : shapelet_coef_grad(c, a, q);
  if (lane == 0) {
    if (nmax >= 0)
      gr[jb] = CHAIN ? float(a[chain::A_SHP_BETA]) : float(-adjoint_inv_beta(c) * a[A_SHP_BETA]);
    MassSums ms = CHAIN ? chain::mass_sums(a) : mass_sums(c, a);
    if (c.fl_i >= 0) {
      // the floored sub-pixel: g = sbar d(source light)/d(beta) there (FP64), contracted with
      // the prologue's exact deflection derivatives; shear terms as the main loop forms them
      const int k = s.k, HW = s.H * s.W;
      const double sb = s.sbar[(size_t)p * HW + c.fl_pix];
      const float2 bs = s.beta[((size_t)p * k * k + c.fl_sub) * HW + c.fl_pix];
      double gx, gy;
      source_light_grad(c, nmax, bs.x, bs.y, gx, gy);
      gx *= sb;
      gy *= sb;
      ms.alpha += gx * c.fl_a[0] + gy * c.fl_a[1];
      ms.t += gx * c.fl_d[0][0] + gy * c.fl_d[0][1];
      ms.e1 += gx * c.fl_d[1][0] + gy * c.fl_d[1][1];
      ms.e2 += gx * c.fl_d[2][0] + gy * c.fl_d[2][1];
      ms.x -= gx * c.fl_d[3][0] + gy * c.fl_d[3][1];  // d/dx = -d/dx_c
      ms.y -= gx * c.fl_d[4][0] + gy * c.fl_d[4][1];
      double x = subpix_coord(s.x0, c.fl_j, s.dxs), y = subpix_coord(s.y0, c.fl_i, s.dxs);
      if (CHAIN) {
        x = float(x);
        y = float(y);
      } else {  // the sums of g in mass_sums hold this sub-pixel's, those of g z do not
        x -= c.xc;
        y -= c.yc;
      }
      ms.g1 += gx * x - gy * y;
      ms.g2 += gx * y + gy * x;
    }
    mass_grad(c, ms, s.mass, s.shear, gr);
  }
  wave_sync();
  int bad = 0;
  for (int q = lane; q < d; q += 64) bad |= !isfinite(gr[q]);
  const bool ok = isfinite(logl) && !__any(bad);
  float* out = s.grad + (size_t)p * s.d;
  for (int q = lane; q < d; q += 64) out[q] = ok ? gr[q] : 0.f;
  if (lane == 0 && !ok) s.logl[p] = -INFINITY;
  return {gr, ok, logl};
}

}  // namespace glens
