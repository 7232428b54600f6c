// HIP kernels of the batched lens likelihood and its adjoint.
//
// One call runs, per lens system and parameter vector ("particle"):
//   prologue       per-particle constants (decode, series coefficients, bijector)
//   subpix_fwd     sub-pixel forward model, k x k mean -> m0[P][H][W]
//   conv           PSF convolution in LDS, per-pixel log-likelihood terms summed in FP64,
//                  and (adjoint) the pixel seed d logL / d m and its correlation with the
//                  PSF -> sbar[P][H][W] = d logL / d (sub-pixel brightness)
//   subpix_adj     sub-pixel adjoint: recompute, local derivatives, per-lane FP32
//                  accumulators, FP64 cross-lane and cross-wave sums -> acc[P][tiles][slot]
//   finalize       sum over tiles and map the accumulators onto d logL / d theta
// Every launch takes a Group of systems that share the kernel configuration, so a
// continuous-batching server can advance many systems in one launch.
#pragma once

#include <hip/hip_runtime.h>

#include "glens_device.h"
#include "glens_fit_device.h"
#include "glens_particle.h"
#include "glens_sums.h"

namespace glens {

constexpr int kConvThreads = 256;
constexpr int kBandMaxThreads = 512;  // banded PSF pass
constexpr int kMfmaMaxThreads = 1024;
constexpr int kConvMaxStrips = 8;  // strips per lane: (H/8 rounded up) * W <= 8 * 256

// prologue: one block per particle (prologue_particle)
template <int WAVES>
__global__ void __launch_bounds__(64 * WAVES) prologue_kernel(Group g) {
  const int si = find_sys(g, blockIdx.x);
  prologue_particle<WAVES>(g.sys[si], blockIdx.x - g.block0[si]);
}

// ------------------------------------------------------------------------------------------
// sub-pixel forward: lanes own pixels, loop over the k x k sub-pixels
// ------------------------------------------------------------------------------------------
// MASS: 0 SIE, 1 EPL; LL: lens light on (1) or off (0); NMAX: shapelet order (-1: none). Every
// system of one launch has the same (MASS, LL, NMAX).
// The pixels [p0, p1) of one particle's model image. The restrict qualifiers tell the compiler
// that the image stores do not write the particle's constants, which then stay scalar loads.
// beta (or null): where beta - x_s of each sub-pixel is kept for the adjoint, [k^2][H][W].
template <int MASS, int LL, int NMAX>
__device__ __forceinline__ void forward_pixels(const SysDesc& s, const PConst* __restrict__ c,
                                               const double* s_pw, float* __restrict__ out,
                                               float2* __restrict__ beta, int p0, int p1) {
  const int W = s.W, HW = s.H * W, k = s.k;
  const int fl_sub = c->fl_sub;
  const double dxs = s.dxs;
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
  double yy = c->ee;
  asm("" : "+v"(yy));
  PixelWalk w(W, p0);
  for (int pix = p0 + threadIdx.x; pix < p1; pix += blockDim.x, w.next()) {
    const double xj = subpix_coord(s.x0, w.j * k, dxs);
    char* bp = reinterpret_cast<char*>(beta);  // uniform: the lane adds its 32-bit offset
    const unsigned off = unsigned(pix) * unsigned(sizeof(float2));
    float sum = 0.f;
    for (int a = 0; a < k; ++a) {
      const double y = subpix_coord(s.y0, w.i * k + a, dxs);
      const RayRow row = ray_row(*c, y);
      const float ly = float(y - c->lys);
      double x = xj;
      for (int b = 0; b < k; ++b, x += dxs, bp += HW * sizeof(float2)) {
        float sdx, sdy;
        ray_trace<MASS>(*c, c->c, s_pw, yy, x, row, sdx, sdy);
        if (a * k + b == fl_sub && pix == c->fl_pix) {  // the first test is wave-uniform
          sdx = c->fl_s[0];
          sdy = c->fl_s[1];
        }
        float v = sersic_fwd(c->src, sdx, sdy);
        if (NMAX >= 0) v += shapelet_fwd<(NMAX < 0 ? 0 : NMAX)>(*c, sdx, sdy, shp);
        if (LL) v += sersic_fwd(c->lens, float(x - c->lxs), ly);
        sum += v;
        if (beta) {  // streamed past the caches: read once, by the adjoint, much later
          float* p = reinterpret_cast<float*>(bp + off);
          __builtin_nontemporal_store(sdx, p);
          __builtin_nontemporal_store(sdy, p + 1);
        }
      }
    }
    out[pix] = sum * s.inv_k2;
  }
}

// Bound by VALU issue at large batches: 175 instructions per sub-pixel at 60 x 60, n_max 6 (193
// with w and beta - x_s formed term by term), 36 of them the FP64 series. The register cap keeps
// six waves per SIMD (five from n_max = 7, whose coefficients alone take 36 or 45 registers):
// left to itself the compiler takes 83 registers and five waves. Measured: 307 -> 281 us (60 x 60,
// 4096 vectors, log L), 147 -> 68 us (53 x 37 SIE + lens light, k = 3, 777 vectors; its closed
// form needed 116 registers and two library transcendentals per sub-pixel).
template <int MASS, int LL, int NMAX>
__global__ void __launch_bounds__(kSubThreads)
__attribute__((amdgpu_waves_per_eu(NMAX >= 7 ? 5 : 6))) subpix_fwd_kernel(Group g) {
  const int si = find_sys(g, blockIdx.x);
  const SysDesc& s = g.sys[si];
  const int lb = blockIdx.x - g.block0[si];
  const int part = lb / s.ftiles, tile = lb - part * s.ftiles;
  const PConst& c = s.pc[part];
  // the EPL's power tables in LDS (lanes read entries of their own); the value series'
  // coefficients stay in the particle's constants, read through the scalar cache: uniform over the
  // workgroup, they enter the series' FMAs as scalar operands
  __shared__ double s_pw[MASS == 1 ? kPowExp + kPowSeg * 8 : 1];
  if (MASS == 1) {
    for (int i = threadIdx.x; i < kPowExp + kPowSeg * 8; i += blockDim.x) s_pw[i] = c.pw[i];
    __syncthreads();
  }
  const int HW = s.H * s.W;
  const int p0 = tile * s.fpix_per_tile;
  const int p1 = min(HW, p0 + s.fpix_per_tile);
  float2* beta = s.mode == 2 && s.beta ? s.beta + (size_t)part * s.k * s.k * HW : nullptr;
  float* out = s.m0 + (size_t)part * HW;
  forward_pixels<MASS, LL, NMAX>(s, &c, s_pw, out, beta, p0, p1);
}

// ------------------------------------------------------------------------------------------
// PSF convolution + likelihood (+ adjoint seed). One workgroup per particle; the image and
// its zero halo live in LDS. Each lane computes kConvRows consecutive rows of one column:
// per tap column it loads kConvRows + K - 1 values and does K * kConvRows FMAs with the taps
// as wave-uniform (scalar) operands.
// ------------------------------------------------------------------------------------------
// The likelihood sums are taken in an order that the block's size does not enter (a block of a
// group takes the size that suits all its systems, and a system's log L is the same bits in any
// company): the pixels in parts that one wave sums whatever the block (64 work items, or a tile
// of the matrix-core pass), then the parts by this sum.
// The total of the n parts in LDS, on every lane of the wave that calls it.
__device__ __forceinline__ double parts_sum(const double* part, int n) {
  double v = 0.0;
  for (int m = threadIdx.x & 63; m < n; m += 64) v += part[m];
  return wave_sum(v);
}

// The padded image sits in LDS column-major (column pitch Hs, odd so that the lanes of a wave,
// which own consecutive columns, hit distinct banks). A lane's strip of kConvRows output rows
// in column j reads, per tap column b, kConvRows + K - 1 consecutive words at immediate
// offsets from one base address.
template <int K>
__device__ __forceinline__ void correlate_strip(const float* __restrict__ buf, int Hs, int i0,
                                                int j, const float* __restrict__ taps,
                                                float* acc) {
  constexpr int R = kConvRows;
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] = 0.f;
#pragma unroll 1
  for (int b = 0; b < K; ++b) {
    const float* colp = buf + (j + b) * Hs + i0;
    float col[R + K - 1];
#pragma unroll
    for (int rr = 0; rr < R + K - 1; ++rr) col[rr] = colp[rr];
#pragma unroll
    for (int a = 0; a < K; ++a) {
      const float kv = taps[a * K + b];
#pragma unroll
      for (int r = 0; r < R; ++r) acc[r] = fmaf(kv, col[r + a], acc[r]);
    }
  }
}

template <int K>
__global__ void __launch_bounds__(kConvThreads) conv_kernel(Group g) {
  extern __shared__ float lds[];
  // parts of 64 consecutive strips, as conv_band_kernel takes them
  __shared__ double part_ll[kConvMaxStrips * kConvThreads / 64];
  __shared__ double part_c2[kConvMaxStrips * kConvThreads / 64];
  const int si = find_sys(g, blockIdx.x);
  const SysDesc& s = g.sys[si];
  const int part = blockIdx.x - g.block0[si];
  constexpr int R = kConvRows, C = (K - 1) / 2;
  const int H = s.H, W = s.W, HW = H * W;
  const int nstrip = (H + R - 1) / R;
  const int Hs = (nstrip * R + K - 1) | 1, Wp = W + K - 1, NP = Hs * Wp;
  const int mode = s.mode;
  float* A = lds;  // padded image; in the adjoint pass it holds the padded pixel seed
  const float* m0 = s.m0 + (size_t)part * HW;
  for (int idx = threadIdx.x; idx < NP; idx += blockDim.x) A[idx] = 0.f;
  __syncthreads();
  for (int idx = threadIdx.x; idx < HW; idx += blockDim.x) {  // coalesced global read
    const int i = idx / W, j = idx - i * W;
    A[(j + C) * Hs + i + C] = m0[idx];
  }
  __syncthreads();
  const float* obs = s.obs;
  const int nitem = nstrip * W;
  // A lane owns at most kConvMaxStrips strips (checked on the host); their pixel seeds stay
  // in registers until every lane has finished reading the image.
  float seed[kConvMaxStrips][R];
#pragma unroll
  for (int t = 0; t < kConvMaxStrips; ++t) {
    const int base = (threadIdx.x & ~63) + t * kConvThreads;
    if (base >= nitem) break;  // the whole wave
    // lanes past the last strip repeat it, without a result
    const int sidx = min(base + int(threadIdx.x & 63), nitem - 1);
    const bool mine = sidx == base + int(threadIdx.x & 63);
    const int st = sidx / W, j = sidx - st * W, i0 = st * R;
    float acc[R];
    correlate_strip<K>(A, Hs, i0, j, s.psf_flip, acc);
    double ll = 0.0, c2 = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = i0 + r;
      seed[t][r] = 0.f;
      if (i >= H || !mine) continue;
      const float m = acc[r];
      if (mode == 0) {
        s.img[(size_t)part * HW + i * W + j] = m;
      } else {
        const float pos = m > 0.f ? m : 0.f;
        const float s2 = s.s2b + pos * s.inv_gt;
        const float res = obs[i * W + j] - m;
        const float is2 = rcp_f32(s2);
        const float chi = res * res * is2;
        c2 += double(chi);
        ll += double(chi + kLn2f * log2_f32(6.283185307179586f * s2));
        const float sp = m > 0.f ? s.inv_gt : 0.f;
        seed[t][r] = res * is2 + 0.5f * sp * (res * res * is2 * is2 - is2);
      }
    }
    if (mode != 0) {
      ll = wave_sum(ll);
      c2 = wave_sum(c2);
      if ((threadIdx.x & 63) == 0) {
        part_ll[base / 64] = ll;
        part_c2[base / 64] = c2;
      }
    }
  }
  if (mode == 0) return;
  __syncthreads();  // the parts are there, and every lane is done with the image
  if (threadIdx.x < 64) {
    const int np = (nitem + 63) / 64;
    const double v = -0.5 * parts_sum(part_ll, np), ctot = parts_sum(part_c2, np);
    if (threadIdx.x == 0) {
      s.logl[part] = isfinite(v) ? v : -INFINITY;
      if (s.chi2) s.chi2[part] = ctot;
    }
  }
  if (mode != 2) return;
  // overwrite the image's interior with the seed
#pragma unroll
  for (int t = 0; t < kConvMaxStrips; ++t) {
    const int sidx = threadIdx.x + t * blockDim.x;
    if (sidx >= nstrip * W) break;
    const int st = sidx / W, j = sidx - st * W, i0 = st * R;
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (i0 + r < H) A[(j + C) * Hs + i0 + r + C] = seed[t][r];
  }
  __syncthreads();
  // d logL / d m0 = correlation of the pixel seed with the (unflipped) PSF
#pragma unroll
  for (int t = 0; t < kConvMaxStrips; ++t) {
    const int sidx = threadIdx.x + t * blockDim.x;
    if (sidx >= nstrip * W) break;
    const int st = sidx / W, j = sidx - st * W, i0 = st * R;
    float acc[R];
    correlate_strip<K>(A, Hs, i0, j, s.psf, acc);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = i0 + r;
      if (i >= H) break;
      s.sbar[(size_t)part * HW + i * W + j] = acc[r] * s.inv_k2;
    }
  }
}

// ------------------------------------------------------------------------------------------
// PSF pass on matrix cores. One workgroup (4 to 16 waves) per particle. Each operand is scaled by a
// power of two (exact) so that its largest magnitude lies in [2^14, 2^15), then split into two
// fp16 parts, x = h + l with h = f16(x) and l = f16(x - h) (the difference is exact in FP32),
// which represents it to about 2^-22 of itself: the scaled padded image sits in LDS as two
// fp16 arrays, and the Toeplitz operands of the PSF are built (scaled and split) once per
// model. Each output tile of 16 rows x N columns takes, for every PSF row a, three
// v_mfma_f32_16x16x32_f16 accumulating in FP32 (hl + lh first, then hh; the dropped l.l term
// is below 2^-22 of the product), and the result is scaled back. Against an FP64 sum this
// keeps pixel errors near 6e-8, as an FP32 sum does. Operand layouts of the instruction (one
// wave; lane l, element e): A[m][k] in lane m + 16 (k / 8), element k % 8; B[k][n] in lane
// n + 16 (k / 8), element k % 8; D[m][n] in lane n + 16 (m / 4), element m % 4. Going from
// PSF row a to a + 1 moves a tile's image rows down by one: lane (m, k / 8) takes the
// fragment of lane (m + 1, k / 8) by a DPP row shift, and only the lanes with m = 15 read LDS.
// Per pixel the likelihood and seed arithmetic is that of conv_kernel.
// ------------------------------------------------------------------------------------------
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// x -> two fp16 parts, stored at p[0], p[stride]
__device__ __forceinline__ void split2_f16(float x, uint16_t* p, int stride) {
  const _Float16 h = static_cast<_Float16>(x);
  p[0] = __builtin_bit_cast(uint16_t, h);
  p[stride] = __builtin_bit_cast(uint16_t, static_cast<_Float16>(x - static_cast<float>(h)));
}

// Exponent s with max_abs 2^s in [2^14, 2^15) (0 for zero or non-finite values).
__device__ __forceinline__ int f16_scale_exp(float max_abs) {
  if (!(max_abs > 0.f) || !(max_abs < INFINITY)) return 0;
  int e;
  frexpf(max_abs, &e);  // max_abs = f 2^e, f in [0.5, 1)
  return 15 - e;
}

// Largest value over the block, returned to every thread.
__device__ __forceinline__ float block_max(float v, float* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
  const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[wave] = v;
  __syncthreads();
  float m = red[0];
  for (int w = 1; w < nw; ++w) m = fmaxf(m, red[w]);
  return m;
}

// Eight consecutive fp16 from LDS at an 8-byte aligned address.
__device__ __forceinline__ f16x8 lds_frag(const uint16_t* p) {
  const uint2 a = reinterpret_cast<const uint2*>(p)[0], b = reinterpret_cast<const uint2*>(p)[1];
  return __builtin_bit_cast(f16x8, make_uint4(a.x, a.y, b.x, b.y));
}

// Lane i of each 16-lane row takes the fragment of lane i + 1 (DPP row_shl:1); lane 15 keeps
// its own.
__device__ __forceinline__ int dpp_row_next(int v) {
  return __builtin_amdgcn_update_dpp(v, v, 0x101, 0xF, 0xF, false);
}
__device__ __forceinline__ f16x8 shift_rows(f16x8 f) {
  int4 v = __builtin_bit_cast(int4, f);
  v.x = dpp_row_next(v.x);
  v.y = dpp_row_next(v.y);
  v.z = dpp_row_next(v.z);
  v.w = dpp_row_next(v.w);
  return __builtin_bit_cast(f16x8, v);
}

__device__ __forceinline__ f32x4 mfma_f16(f16x8 a, f16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// acc[v] = correlation of the scaled LDS image (parts x, x + nel) with the scaled PSF over
// the tiles t0 + v nw, v < G, of one of the block's nw waves. tab: this direction's fragments [K][64][h, l];
// those of row a + 2 are loaded while row a is computed. Each product is issued over the G
// tiles before the next, so consecutive matrix instructions are independent. APART: the products
// with a low part, some 2^-11 of the others, are summed apart, so that a third as many additions
// round at the size of the result.
template <int G, bool APART>
__device__ __forceinline__ void mfma_tiles(const uint16_t* x, int nel, const MfmaGeom& q,
                                           const uint4* __restrict__ tab, int K, int t0, int nw,
                                           f32x4* acc) {
  const int lane = threadIdx.x & 63, mr = lane & 15, g = lane >> 4;
  int off[G];  // this lane's fragment offset in tile v at row a = 0
  f16x8 ah[G], al[G];
  f32x4 low[G];
#pragma unroll
  for (int v = 0; v < G; ++v) {
    const int t = t0 + v * nw;
    const int tr = t / q.TC, tc = t - tr * q.TC;
    off[v] = (tr * 16 + mr) * q.pitch + tc * q.N + 8 * g;
    ah[v] = lds_frag(x + off[v]);
    al[v] = lds_frag(x + off[v] + nel);
    acc[v] = low[v] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // PSF fragments two rows ahead (an L2 round trip is longer than one row's products)
  const uint4* tb = tab + lane * 2;
  uint4 nh = tb[0], nl = tb[1], nnh = nh, nnl = nl;
  if (K > 1) {
    nnh = tb[128];
    nnl = tb[129];
  }
  for (int a = 0; a < K; ++a) {
    const f16x8 bh = __builtin_bit_cast(f16x8, nh);
    const f16x8 bl = __builtin_bit_cast(f16x8, nl);
    nh = nnh;
    nl = nnl;
    if (a + 2 < K) {
      nnh = tb[(a + 2) * 128];
      nnl = tb[(a + 2) * 128 + 1];
    }
    f32x4* lo = APART ? low : acc;
#pragma unroll
    for (int v = 0; v < G; ++v) lo[v] = mfma_f16(ah[v], bl, lo[v]);
#pragma unroll
    for (int v = 0; v < G; ++v) lo[v] = mfma_f16(al[v], bh, lo[v]);
#pragma unroll
    for (int v = 0; v < G; ++v) acc[v] = mfma_f16(ah[v], bh, acc[v]);
    if (a + 1 < K) {
#pragma unroll
      for (int v = 0; v < G; ++v) {
        ah[v] = shift_rows(ah[v]);
        al[v] = shift_rows(al[v]);
      }
      if (mr == 15) {  // the new bottom row of each tile
        const int ro = (a + 1) * q.pitch;
#pragma unroll
        for (int v = 0; v < G; ++v) {
          ah[v] = lds_frag(x + off[v] + ro);
          al[v] = lds_frag(x + off[v] + ro + nel);
        }
      }
    }
  }
  if (APART)
#pragma unroll
    for (int v = 0; v < G; ++v) acc[v] += low[v];
}

// Per-pixel state of the matrix-core PSF kernel. The launch descriptor's fields are copied
// here once: read through the descriptor (a dynamically indexed kernel argument) they were
// loaded again for every pixel.
constexpr int kMfmaGroup = 5;  // most tiles that a wave takes at a time (mfma_pass)
struct MfmaPass {
  const MfmaGeom& q;
  int nw;             // waves of the block
  int unscale;        // exponent that takes the scaled sums back: -(image scale + PSF scale)
  int H, W, mode;
  float s2b, inv_gt, inv_k2;
  const float* obs;   // [H][W]
  float* out;         // this particle's model image (mode 0), or its seed and then sbar
  float mx;           // largest seed magnitude of this lane's pixels
  double ll[kMfmaGroup], c2[kMfmaGroup];  // this lane's likelihood sums of each tile of a group
};

// Pixels of tiles t0 + v nw, v < G: element r of acc[v] is pixel (i0 + r, j).
// Forward (ADJ false): the model image, or the likelihood terms and the seed; adjoint: sbar.
template <int G, bool ADJ>
__device__ __forceinline__ void mfma_pixels(MfmaPass& P, int t0, const f32x4* acc) {
  const int lane = threadIdx.x & 63, n = lane & 15, r0 = 4 * (lane >> 4);
  const int H = P.H, W = P.W;
#pragma unroll
  for (int v = 0; v < G; ++v) {
    const int t = t0 + v * P.nw, tr = t / P.q.TC, tc = t - tr * P.q.TC;
    const int j = tc * P.q.N + n, i0 = tr * 16 + r0;
    if (n >= P.q.N || j >= W) continue;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = i0 + r;
      if (i >= H) break;
      const float m = ldexpf(acc[v][r], P.unscale);
      const int px = i * W + j;
      if (ADJ) {
        P.out[px] = m * P.inv_k2;
      } else if (P.mode == 0) {
        P.out[px] = m;
      } else {
        const float pos = m > 0.f ? m : 0.f;
        const float s2 = P.s2b + pos * P.inv_gt;
        const float res = P.obs[px] - m;
        const float is2 = rcp_f32(s2);
        const float chi = res * res * is2;
        P.c2[v] += double(chi);
        P.ll[v] += double(chi + kLn2f * log2_f32(6.283185307179586f * s2));
        if (P.mode == 2) {
          const float sp = m > 0.f ? P.inv_gt : 0.f;
          const float sd = res * is2 + 0.5f * sp * (res * res * is2 * is2 - is2);
          P.out[px] = sd;
          P.mx = fmaxf(P.mx, fabsf(sd));
        }
      }
    }
  }
}

// This lane's index, hidden from the compiler: what the image's load and the seed's compute from
// it would otherwise be shared, and held in registers throughout the products between them.
__device__ __forceinline__ int own_thread() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// This lane's first kMfmaKeep pixels of src, all loads in flight. Four at a time past the block's
// last pixel are left out (the test is uniform): of an image below 27 x 27 twelve of sixteen.
constexpr int kMfmaKeep = 16;
__device__ __forceinline__ void mfma_load(const float* src, int HW, float* v) {
  const int t = own_thread();
#pragma unroll
  for (int u = 0; u < kMfmaKeep; ++u) v[u] = 0.f;
#pragma unroll
  for (int u0 = 0; u0 < kMfmaKeep; u0 += 4) {
    if (u0 * int(blockDim.x) >= HW) break;
#pragma unroll
    for (int u = u0; u < u0 + 4; ++u) {
      const int idx = t + u * int(blockDim.x);
      if (idx < HW) v[u] = src[idx];
    }
  }
}

// The interior of the padded LDS image: src 2^sx as two fp16 parts (v: mfma_load's).
__device__ __forceinline__ void mfma_fill(const float* src, const float* v, int HW, int W, int C,
                                          int sx, uint16_t* x, int pitch, int nel) {
  const int t = own_thread();
  PixelWalk w(W, t - int(threadIdx.x));
  x += C * pitch + C;
#pragma unroll
  for (int u0 = 0; u0 < kMfmaKeep; u0 += 4) {
    if (u0 * int(blockDim.x) >= HW) break;
#pragma unroll
    for (int u = u0; u < u0 + 4; ++u, w.next())
      if (t + u * int(blockDim.x) < HW)
        split2_f16(ldexpf(v[u], sx), x + w.i * pitch + w.j, nel);
  }
  for (int idx = t + kMfmaKeep * blockDim.x; idx < HW; idx += blockDim.x, w.next())
    split2_f16(ldexpf(src[idx], sx), x + w.i * pitch + w.j, nel);
  __syncthreads();
}

// G tiles of the wave: correlate, then the per-pixel step.
template <int G, bool ADJ, bool APART>
__device__ __forceinline__ void mfma_group(MfmaPass& P, const uint16_t* x, int nel,
                                           const uint4* tab, int K, int t0) {
  f32x4 acc[G];
  mfma_tiles<G, APART>(x, nel, P.q, tab, K, t0, P.nw, acc);
  mfma_pixels<G, ADJ>(P, t0, acc);
}

// The wave's tiles wave, wave + nw, .. in groups of at most five, as even as possible: a group's
// products hide the latency of the PSF fragment loads only when it has several tiles. The forward
// pass of a likelihood leaves its sums of each tile in tile_ll and, if not null, tile_c2 (LDS).
template <bool ADJ, bool APART>
__device__ __forceinline__ void mfma_pass(MfmaPass& P, const uint16_t* x, int nel,
                                          const uint4* tab, int K, double* tile_ll = nullptr,
                                          double* tile_c2 = nullptr) {
  // wave-uniform: kept in scalar registers
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ntw = wave < P.q.T ? (P.q.T - wave + P.nw - 1) / P.nw : 0;
  const int ng = (ntw + kMfmaGroup - 1) / kMfmaGroup;
  for (int gi = 0, u = 0; gi < ng; ++gi) {
    const int n = (ntw - u + ng - gi - 1) / (ng - gi), t0 = wave + u * P.nw;
    if (!ADJ)
#pragma unroll
      for (int v = 0; v < kMfmaGroup; ++v) P.ll[v] = P.c2[v] = 0.0;
    switch (n) {
      case 1: mfma_group<1, ADJ, APART>(P, x, nel, tab, K, t0); break;
      case 2: mfma_group<2, ADJ, APART>(P, x, nel, tab, K, t0); break;
      case 3: mfma_group<3, ADJ, APART>(P, x, nel, tab, K, t0); break;
      case 4: mfma_group<4, ADJ, APART>(P, x, nel, tab, K, t0); break;
      default: mfma_group<5, ADJ, APART>(P, x, nel, tab, K, t0); break;
    }
    if (!ADJ && P.mode != 0) {  // one copy of the sums' code for every group size
      const int lane = threadIdx.x & 63;  // lane 8 v holds tile v's
      const bool holds = lane % 8 == 0 && lane / 8 < n;
      const double tl = wave_sums_f64<kMfmaGroup>(P.ll);
      if (holds) tile_ll[t0 + lane / 8 * P.nw] = tl;
      if (tile_c2) {
        const double tc = wave_sums_f64<kMfmaGroup>(P.c2);
        if (holds) tile_c2[t0 + lane / 8 * P.nw] = tc;
      }
    }
    u += n;
  }
}

// log L and chi^2 of one particle from its bands' partial sums.
__device__ __forceinline__ void band_totals(const SysDesc& s, int part) {
  const double* lp = s.lpart + (size_t)part * kConvMaxBands * 2;
  double tot = 0.0, ctot = 0.0;
  for (int q = 0; q < s.bands; ++q) {
    tot += lp[2 * q];
    ctot += lp[2 * q + 1];
  }
  const double v = -0.5 * tot;
  s.logl[part] = isfinite(v) ? v : -INFINITY;
  if (s.chi2) s.chi2[part] = ctot;
}

// One block per particle. Its size (launch_conv_mfma) is what fills a CU: four waves per SIMD at
// the 128 registers allowed here, from 256 threads where four blocks fit, 512 or 1024 where the
// image leaves room in LDS for fewer or the batch has too few particles for more; a tile's sums
// do not depend on the wave that takes it. LDS holds the image's two fp16 parts only: with the
// pixels and the seed in FP32 beside them one block of 1024 threads fitted at 100 x 100, and its
// phases followed each other with nothing to fill the gaps (2048 vectors: 720 us at 256 threads
// throughout, 443 at 1024, 357 now with two blocks of 512); 80 x 80, 512 vectors (images) 36 ->
// 28 us; 60 x 60: 512 vectors 42 -> 34.5 us, 4096 194 -> 183 us (log L only 118 -> 106; 1.4 to 2 us
// less with one sum per lane of the block, whose order followed the block's size). Bound there by
// the fill and split of the image (about 35 us of the forward half) and by the row shifts and the
// LDS reads of the new rows beside the products (matrix cores 34 us a half): reloading either part
// of the fragments from LDS instead of shifting it measured 278 us for the kernel, both 394; five
// waves per SIMD, at most four or three tiles a group, 180 against 176 at the same clocks; four
// tiles a group at four waves 189.
// ADJ_ONLY: only the adjoint pass, from the seed that the banded forward kernel left in memory (and
// log L from its bands' partial sums), in place of the banded VALU adjoint: 44 -> 32 us (80 x 80, 300
// vectors), 52 -> 33.4 us (500). The operands' two parts are 22 bits or more of a seed's 24, so
// that the sums have to be the better for it: with the low products apart the rms error against 64
// bits is 0.41 to 0.83 of the VALU sums' over the sizes that come here (1.2 to 1.4 of them in one
// accumulator, at the sizes whose strips are summed over two lanes).
template <bool ADJ_ONLY>
__global__ void __launch_bounds__(kMfmaMaxThreads) __attribute__((amdgpu_waves_per_eu(4)))
conv_mfma_kernel(Group g) {
  extern __shared__ __align__(16) uint16_t xlds[];
  __shared__ double tile_ll[kMfmaMaxTiles], tile_c2[kMfmaMaxTiles];
  __shared__ float redf[kMfmaMaxThreads / 64];
  const int si = find_sys(g, blockIdx.x);
  const SysDesc& s = g.sys[si];
  const int part = blockIdx.x - g.block0[si];
  const int H = s.H, W = s.W, HW = H * W, K = s.K, C = (K - 1) / 2, mode = s.mode;
  const MfmaGeom q = mfma_geom(H, W, K);
  const int nel = q.Hq * q.pitch;  // fp16 per part (a multiple of 4)
  for (int i = threadIdx.x; i < nel / 4; i += blockDim.x)
    reinterpret_cast<uint4*>(xlds)[i] = make_uint4(0u, 0u, 0u, 0u);
  // a lane's pixels wait in registers (those of a large image past the sixteenth are read again,
  // from L2) for the image's largest magnitude: in LDS they would take as much room again
  const float* src = (ADJ_ONLY ? s.seed : s.m0) + (size_t)part * HW;
  float v[kMfmaKeep], mx = 0.f;
  mfma_load(src, HW, v);
#pragma unroll
  for (int u = 0; u < kMfmaKeep; ++u) mx = fmaxf(mx, fabsf(v[u]));
  for (int idx = threadIdx.x + kMfmaKeep * blockDim.x; idx < HW; idx += blockDim.x)
    mx = fmaxf(mx, fabsf(src[idx]));
  // the block_max barriers also end the zero fill
  int sx = f16_scale_exp(block_max(mx, redf));
  mfma_fill(src, v, HW, W, C, sx, xlds, q.pitch, nel);
  MfmaPass P{q, int(blockDim.x) >> 6, -(sx + s.psf_mfma_exp), H, W, mode, s.s2b, s.inv_gt,
             s.inv_k2, s.obs, (mode == 0 ? s.img : s.sbar) + (size_t)part * HW, 0.f, {}, {}};
  if (ADJ_ONLY) {
    if (threadIdx.x == 0) band_totals(s, part);
  } else {
    mfma_pass<false, false>(P, xlds, nel, s.psf_mfma, K, tile_ll, s.chi2 ? tile_c2 : nullptr);
    if (mode == 0) return;
    __syncthreads();  // the tiles' sums are there
    if (threadIdx.x < 64) {
      const double l = -0.5 * parts_sum(tile_ll, q.T);
      if (threadIdx.x == 0) s.logl[part] = isfinite(l) ? l : -INFINITY;
      if (s.chi2) {
        const double ctot = parts_sum(tile_c2, q.T);
        if (threadIdx.x == 0) s.chi2[part] = ctot;
      }
    }
    if (mode != 2) return;
    // every wave is done with the image and has written its part of the seed to sbar (the barrier
    // above): the image's interior takes the scaled seed
    sx = f16_scale_exp(block_max(P.mx, redf));
    mfma_load(P.out, HW, v);
    mfma_fill(P.out, v, HW, W, C, sx, xlds, q.pitch, nel);
    P.unscale = -(sx + s.psf_mfma_exp);
  }
  // d logL / d m0 = correlation of the pixel seed with the (unflipped) PSF
  mfma_pass<true, ADJ_ONLY>(P, xlds, nel, s.psf_mfma + 2 * 64 * K, K);
}

// ------------------------------------------------------------------------------------------
// Banded PSF pass for small batches: one workgroup per (particle, band of rows), so that a
// few particles still spread over many CUs. Band b owns output rows [b R_b, (b+1) R_b) and
// loads the rows of its input it needs (C = (K-1)/2 more on either side). Three kernels:
//   conv_band_kernel       the PSF, the likelihood terms (partial sums per band) and the
//                          adjoint seed of each pixel (to a [P][H][W] buffer);
//   conv_band_adj_kernel   the correlation of the seed with the PSF; the first band of a
//                          particle also adds the likelihood partials (band order). Where the
//                          matrix-core kernel takes the system it does this instead,
//                          except for the sampler's chains;
//   conv_band_sum_kernel   the same addition when there is no adjoint pass.
// With band_split = 1 the arithmetic per pixel is that of conv_kernel (only the order of the
// log L sum differs). Very small batches split each strip's K PSF columns over G = 2 or 4
// adjacent lanes (columns g, g + G, ...), whose partial sums are then added by an xor
// butterfly: more lanes in flight and K^2 kConvRows / G FMAs in each lane's chain.
// ------------------------------------------------------------------------------------------
static_assert(kBandMaxThreads % 64 == 0, "whole lane groups of the split PSF columns");
struct Band {
  int part, band, r0, r1, nsr, Hs;
};

// Sums a strip's partial accumulators over the G lanes that share it (adjacent lanes, G a
// power of two <= 4, every lane of the group active); each lane ends with the full sums.
__device__ __forceinline__ void split_sum(float* acc, int G) {
  for (int o = 1; o < G; o <<= 1) {
#pragma unroll
    for (int r = 0; r < kConvRows; ++r) acc[r] += __shfl_xor(acc[r], o, 64);
  }
}

__device__ __forceinline__ Band band_of(const SysDesc& s, int local, int K) {
  Band b;
  b.part = local / s.bands;
  b.band = local - b.part * s.bands;
  b.r0 = b.band * s.band_rows;
  b.r1 = min(s.H, b.r0 + s.band_rows);
  b.nsr = (b.r1 - b.r0 + kConvRows - 1) / kConvRows;
  b.Hs = (b.nsr * kConvRows + K - 1) | 1;
  return b;
}

// Taps of one PSF column in LDS: a multiple of four, so that they are read four at a time.
template <int K>
constexpr int tap_pitch() {
  return (K + 3) & ~3;
}

// Rows [r0 - C, r0 - C + Hs) of src (zero outside the image) into the column-major LDS tile A, and
// the PSF's taps column by column into T (read from there, they need neither 21 scalar loads a
// column nor, where lanes take different columns, as many vector loads from memory). One pass,
// several loads in flight.
template <int K>
__device__ __forceinline__ void load_band(const float* __restrict__ src,
                                          const float* __restrict__ taps, const SysDesc& s,
                                          const Band& b, float* A, float* T) {
  constexpr int C = (K - 1) / 2, U = 4;
  const int H = s.H, W = s.W, Wp = W + K - 1, n = b.Hs * Wp;
  for (int idx = threadIdx.x; idx < K * K; idx += blockDim.x)
    T[(idx % K) * tap_pitch<K>() + idx / K] = taps[idx];
  PixelWalk w(Wp);
  for (int idx = threadIdx.x; idx < n; idx += U * blockDim.x) {
    float v[U];
    int o[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = b.r0 + w.i - C, j = w.j - C;
      o[u] = w.j * b.Hs + w.i;
      v[u] = 0.f;
      if (unsigned(i) < unsigned(H) && unsigned(j) < unsigned(W)) v[u] = src[i * W + j];
      w.next();
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (idx + u * int(blockDim.x) < n) A[o[u]] = v[u];
  }
  __syncthreads();
}

// correlate_strip with the taps in LDS (load_band), columns b0, b0 + bstep, ...; the same sums in
// the same order.
template <int K>
__device__ __forceinline__ void band_strip(const float* __restrict__ A,
                                           const float* __restrict__ T, int Hs, int i0, int j,
                                           float* acc, int b0, int bstep) {
  constexpr int R = kConvRows, Kp = tap_pitch<K>();
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] = 0.f;
#pragma unroll 1
  for (int b = b0; b < K; b += bstep) {
    const float* colp = A + (j + b) * Hs + i0;
    float col[R + K - 1], kv[Kp];
#pragma unroll
    for (int q = 0; q < Kp; q += 4) {
      const float4 t = *reinterpret_cast<const float4*>(T + b * Kp + q);
      kv[q] = t.x;
      kv[q + 1] = t.y;
      kv[q + 2] = t.z;
      kv[q + 3] = t.w;
    }
#pragma unroll
    for (int rr = 0; rr < R + K - 1; ++rr) col[rr] = colp[rr];
#pragma unroll
    for (int a = 0; a < K; ++a) {
#pragma unroll
      for (int r = 0; r < R; ++r) acc[r] = fmaf(kv[a], col[r + a], acc[r]);
    }
  }
}

// Bound by VALU issue where the batch fills the chip, by latency below. Bands and block size
// follow the waves on the fullest CU (conv_bands); the taps come from LDS. Measured: 47.5 -> 38.9 us
// (80 x 80, K = 21, 300 vectors; products alone 21.5), 56.7 -> 50.4 us (500), 13.0 -> 11.6 us (60 x 60,
// 64 vectors, columns over four lanes).
template <int K>
__global__ void __launch_bounds__(kBandMaxThreads) conv_band_kernel(Group g) {
  extern __shared__ __align__(16) float lds[];
  const int si = find_sys(g, blockIdx.x);
  const SysDesc& s = g.sys[si];
  const Band b = band_of(s, blockIdx.x - g.block0[si], K);
  constexpr int R = kConvRows;
  const int W = s.W, HW = s.H * W, mode = s.mode;
  float* T = lds + band_tile_floats(s.band_rows, W, K);
  load_band<K>(s.m0 + (size_t)b.part * HW, s.psf_flip, s, b, lds, T);
  // work items (strip, column, PSF-column share); the G lanes of one strip are adjacent, and 64
  // and the item count are multiples of G, so they run the loop together. Lanes past the last
  // item repeat it, without a result.
  const int G = s.band_split, gs = G >> 1;  // G = 1, 2, 4: log2 G = G / 2
  const int nitem = b.nsr * W * G, lane = threadIdx.x & 63, np = (nitem + 63) / 64;
  double* parts = reinterpret_cast<double*>(T + K * tap_pitch<K>());  // log L terms, then chi^2
  for (int base = threadIdx.x & ~63; base < nitem; base += blockDim.x) {
    const int sidx = min(base + lane, nitem - 1);
    const int item = sidx >> gs, g0 = (base + lane) & (G - 1);
    const int st = item / W, j = item - st * W, i0 = st * R;
    float acc[R];
    band_strip<K>(lds, T, b.Hs, i0, j, acc, g0, G);
    split_sum(acc, G);
    const bool mine = g0 == 0 && base + lane < nitem;
    double ll = 0.0, c2 = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = b.r0 + i0 + r;
      if (i >= b.r1 || !mine) break;
      const float m = acc[r];
      const size_t o = (size_t)b.part * HW + i * W + j;
      if (mode == 0) {
        s.img[o] = m;
        continue;
      }
      const float pos = m > 0.f ? m : 0.f;
      const float s2 = s.s2b + pos * s.inv_gt;
      const float res = s.obs[i * W + j] - m;
      const float is2 = rcp_f32(s2);
      const float chi = res * res * is2;
      c2 += double(chi);
      ll += double(chi + kLn2f * log2_f32(6.283185307179586f * s2));
      if (mode == 2) {
        const float sp = m > 0.f ? s.inv_gt : 0.f;
        s.seed[o] = res * is2 + 0.5f * sp * (res * res * is2 * is2 - is2);
      }
    }
    if (mode != 0) {
      ll = wave_sum(ll);
      c2 = wave_sum(c2);
      if (lane == 0) {
        parts[base / 64] = ll;
        parts[np + base / 64] = c2;
      }
    }
  }
  if (mode == 0) return;
  __syncthreads();  // the parts are there
  if (threadIdx.x < 64) {
    const double tot = parts_sum(parts, np), ctot = parts_sum(parts + np, np);
    if (threadIdx.x == 0) {
      double* lp = s.lpart + ((size_t)b.part * kConvMaxBands + b.band) * 2;
      lp[0] = tot;
      lp[1] = ctot;
    }
  }
}

template <int K>
__global__ void __launch_bounds__(kBandMaxThreads) conv_band_adj_kernel(Group g) {
  extern __shared__ __align__(16) float lds[];
  const int si = find_sys(g, blockIdx.x);
  const SysDesc& s = g.sys[si];
  const Band b = band_of(s, blockIdx.x - g.block0[si], K);
  constexpr int R = kConvRows;
  const int W = s.W, HW = s.H * W;
  if (b.band == 0 && threadIdx.x == 0) band_totals(s, b.part);
  float* T = lds + band_tile_floats(s.band_rows, W, K);
  load_band<K>(s.seed + (size_t)b.part * HW, s.psf, s, b, lds, T);
  const int G = s.band_split, gs = G >> 1;  // G = 1, 2, 4: log2 G = G / 2
  for (int sidx = threadIdx.x; sidx < b.nsr * W * G; sidx += blockDim.x) {
    const int item = sidx >> gs, g0 = sidx & (G - 1);
    const int st = item / W, j = item - st * W, i0 = st * R;
    float acc[R];
    band_strip<K>(lds, T, b.Hs, i0, j, acc, g0, G);
    split_sum(acc, G);
    if (g0 != 0) continue;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = b.r0 + i0 + r;
      if (i >= b.r1) break;
      s.sbar[(size_t)b.part * HW + i * W + j] = acc[r] * s.inv_k2;
    }
  }
}

__global__ void __launch_bounds__(64) conv_band_sum_kernel(Group g) {
  const int si = find_sys(g, blockIdx.x);
  const SysDesc& s = g.sys[si];
  const int p = (blockIdx.x - g.block0[si]) * blockDim.x + threadIdx.x;
  if (p < s.P) band_totals(s, p);
}

// ------------------------------------------------------------------------------------------
// sub-pixel adjoint
// ------------------------------------------------------------------------------------------
// The sub-pixels of pixels [p0, p1) of one particle into the per-lane accumulators.
// GENERAL = false: the particle has no floored sub-pixel and |eps| >= kSxClosedMin.
template <int MASS, int LL, int NMAX, bool GENERAL>
__device__ __forceinline__ void adj_pixels(const SysDesc& s, const PConst& c,
                                           const float* s_nc, const float* s_dc,
                                           const float* he, const float2* beta,
                                           const float* sbar, int p0, int p1, float* acc) {
  const int HW = s.H * s.W, W = s.W, k = s.k;
  const int fl_i = c.fl_i, fl_j = c.fl_j;
  const double dxs = s.dxs;
  PixelWalk w(W, p0);
  for (int pix = p0 + threadIdx.x; pix < p1; pix += blockDim.x, w.next()) {
    const int i = w.i, j = w.j;
    const float sb = sbar[pix];
    const double xj = subpix_coord(s.x0, j * k, dxs);
    const char* bp = reinterpret_cast<const char*>(beta);  // uniform, as in the forward pass
    const unsigned off = unsigned(pix) * unsigned(sizeof(float2));
    for (int a = 0; a < k; ++a) {
      const double y = subpix_coord(s.y0, i * k + a, dxs);
      const float zi = float(y - c.yc), ly = float(y - c.lys);
      // alpha = x - alpha_ext - x_s - (beta - x_s): its part of this row
      const double cx = -c.g2 * y - c.sxs, cy = c.opg1 * y - c.sys;
      const float lpx = c.lens.qbh * ly, lpy = c.lens.qc * ly;
      double x = xj;
      for (int b = 0; b < k; ++b, x += dxs, bp += HW * sizeof(float2)) {
        const float* p = reinterpret_cast<const float*>(bp + off);
        const float sdx = __builtin_nontemporal_load(p);
        const float sdy = __builtin_nontemporal_load(p + 1);
        // g: sb d(source light)/d(beta)
        const float px = fmaf(c.src.qa, sdx, c.src.qbh * sdy);
        const float py = fmaf(c.src.qc, sdy, c.src.qbh * sdx);
        const float sv = sersic_adj(c.src, sdx, sdy, px, py, sb, acc + A_SRC);
        Cx g;
        if (NMAX >= 0) {
          shapelet_adj<(NMAX < 0 ? 0 : NMAX)>(c, sdx, sdy, he, sb, acc, g.r, g.i);
          g = {fmaf(sv, px, g.r), fmaf(sv, py, g.i)};
        } else {
          g = {sv * px, sv * py};
        }
        acc[A_SRC + L_DX] += g.r;
        acc[A_SRC + L_DY] += g.i;
        if (LL) {
          const float lx = float(x - c.lxs);
          const float lv = sersic_adj(c.lens, lx, ly, fmaf(c.lens.qa, lx, lpx),
                                      fmaf(c.lens.qbh, lx, lpy), sb, acc + lens_slot(NMAX));
          acc[lens_slot(NMAX) + L_DX] = fmaf(lv, lx, acc[lens_slot(NMAX) + L_DX]);
          acc[lens_slot(NMAX) + L_DY] = fmaf(lv, ly, acc[lens_slot(NMAX) + L_DY]);
        }
        // the floored sub-pixel's mass terms are added by finalize from the prologue's
        // exact derivatives
        if (GENERAL && i * k + a == fl_i && j * k + b == fl_j) g = {0.f, 0.f};
        mass_adjoint<MASS, GENERAL>(c, s_nc, s_dc, float(x - c.xc), zi,
                                    float(fma(x, c.omg1, cx)) - sdx,
                                    float(fma(x, -c.g2, cy)) - sdy, g, acc);
      }
    }
  }
}

// Bound by VALU issue (one instruction per CU and cycle; packed FP32 is not used), so what counts
// is instructions per sub-pixel: 391 with every sum of the gradient taken per sub-pixel, 341 with
// the sums of mass_adjoint, sersic_adj and shapelet_adj (330 with the eccentricity's and the Sersic
// index's as combinations of other sums, which cancel). Measured, each with every sum per sub-pixel,
// with those combinations, and now: 546, 480, 487 us (60 x 60, n_max 6, 4096 vectors), 67, 50, 55
// (80 x 80 without shapelets, 300), 121, 93, 99 (53 x 37 SIE, k = 3, n_max 3, 777). At n_max = 8 the
// accumulators and coefficients (over 120 registers) do not fit three waves per SIMD (168 registers:
// 76 spilled in the loop); two waves hide the latencies of this instruction mix as well: 1517, 876,
// 890 us (100 x 100, 2048 vectors); without lens light three waves fit, but two were faster (427 us
// against 500). n_max = 7 keeps three (110, 100, 102 us at 47 x 35, k = 4, 317 vectors; with two 111).
template <int MASS, int LL, int NMAX>
__global__ void __launch_bounds__(kSubThreads)
__attribute__((amdgpu_waves_per_eu(NMAX >= 8 ? 2 : 3)))
subpix_adj_kernel(Group g) {
  constexpr int NS = lens_slot(NMAX) + (LL ? kLightSlots : 0);
  __shared__ double red[kSubThreads / 64][NS];
  const int si = find_sys(g, blockIdx.x);
  const SysDesc& s = g.sys[si];
  const int lb = blockIdx.x - g.block0[si];
  const int part = lb / s.adj_tiles, tile = lb - part * s.adj_tiles;
  const PConst& c = s.pc[part];
  __shared__ float s_nc[kMaxTerms], s_dc[kMaxTerms];
  stage_series(c, -2.8853900817779268f, s_nc, s_dc);  // mass_adjoint's -2 / ln 2
  // beta - x_s from the forward pass (kept there for gradient calls)
  const float2* beta = s.beta + (size_t)part * s.k * s.k * s.H * s.W;
  const int HW = s.H * s.W;
  const int p0 = tile * s.adj_pix_per_tile;
  const int p1 = min(HW, p0 + s.adj_pix_per_tile);
  const float* sbar = s.sbar + (size_t)part * HW;
  float acc[NS];
#pragma unroll
  for (int q = 0; q < NS; ++q) acc[q] = 0.f;
  // shapelet coefficients in vector registers (as in the forward pass), scaled for the He_n
  constexpr int M = NMAX < 0 ? 1 : (NMAX + 1) * (NMAX + 2) / 2;
  float shp[M];
#pragma unroll
  for (int n = 0; n <= (NMAX < 0 ? 0 : NMAX); ++n)
#pragma unroll
    for (int n2 = 0; n2 <= n; ++n2) {
      const int q = shp_index(n - n2, n2);
      shp[q] = NMAX < 0 ? 0.f : c.shp[q] * kHeScale[n];
      asm("" : "+v"(shp[q]));
    }
  // the common case (no floored sub-pixel, |eps| >= kSxClosedMin) runs a loop without those
  // tests
  if (c.fl_i < 0 && !(c.epsabs < kSxClosedMin))
    adj_pixels<MASS, LL, NMAX, false>(s, c, s_nc, s_dc, shp, beta, sbar, p0, p1, acc);
  else
    adj_pixels<MASS, LL, NMAX, true>(s, c, s_nc, s_dc, shp, beta, sbar, p0, p1, acc);
  block_sums<NS>(acc, red, s.acc + ((size_t)part * s.adj_tiles + tile) * kNAcc);
}

// finalize: one 64-lane block per particle (finalize_particle)
__global__ void __launch_bounds__(64) finalize_kernel(Group g) {
  const int si = find_sys(g, blockIdx.x);
  finalize_particle<false>(g.sys[si], blockIdx.x - g.block0[si]);
}

}  // namespace glens
