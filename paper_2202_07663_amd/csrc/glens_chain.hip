// The sub-pixel kernels of the sampler's launches (glens_chain.h).
#include <hip/hip_runtime.h>

#include <utility>

#include "glens_chain.h"
#include "glens_host.h"

namespace glens {

template <int MASS, int LL, int NMAX>
__global__ void __launch_bounds__(kSubThreads) chain_fwd_kernel(Group g) {
  const int si = find_sys(g, blockIdx.x);
  const SysDesc& s = g.sys[si];
  const int lb = blockIdx.x - g.block0[si];
  const int part = lb / s.ftiles, tile = lb - part * s.ftiles;
  const PConst& c = s.pc[part];
  // the power tables in LDS (lanes read entries of their own); the value series' coefficients
  // stay in the particle's constants, read through the scalar cache: uniform over the
  // workgroup, they enter the series' FMAs as scalar operands
  __shared__ double s_pw[kPowExp + kPowSeg * 8];
  for (int i = threadIdx.x; i < kPowExp + kPowSeg * 8; i += blockDim.x) s_pw[i] = c.pw[i];
  __syncthreads();
  const int HW = s.H * s.W;
  const int p0 = tile * s.fpix_per_tile;
  const int p1 = min(HW, p0 + s.fpix_per_tile);
  float2* beta = s.mode == 2 && s.beta ? s.beta + (size_t)part * s.k * s.k * HW : nullptr;
  chain::forward_pixels<MASS, LL, NMAX>(s, &c, c.c, s_pw, s.m0 + (size_t)part * HW, beta, p0, p1);
}

template <int MASS, int LL, int NMAX>
__global__ void __launch_bounds__(kSubThreads) __attribute__((amdgpu_waves_per_eu(3)))
chain_adj_kernel(Group g) {
  constexpr int NS = chain::n_slots<NMAX>();
  __shared__ double red[kSubThreads / 64][NS];
  const int si = find_sys(g, blockIdx.x);
  const SysDesc& s = g.sys[si];
  const int lb = blockIdx.x - g.block0[si];
  const int part = lb / s.tiles, tile = lb - part * s.tiles;
  const PConst& c = s.pc[part];
  __shared__ float s_nc[kMaxTerms], s_dc[kMaxTerms];
  stage_series(c, 1.0f, s_nc, s_dc);
  const float2* beta = s.beta + (size_t)part * s.k * s.k * s.H * s.W;
  const int HW = s.H * s.W;
  const int p0 = tile * s.pix_per_tile;
  const int p1 = min(HW, p0 + s.pix_per_tile);
  const float* sbar = s.sbar + (size_t)part * HW;
  float acc[NS];
#pragma unroll
  for (int q = 0; q < NS; ++q) acc[q] = 0.f;
  constexpr int M = NMAX < 0 ? 1 : (NMAX + 1) * (NMAX + 2) / 2;
  float shp[M];
#pragma unroll
  for (int q = 0; q < M; ++q) {
    shp[q] = NMAX < 0 ? 0.f : c.shp[q];
    asm("" : "+v"(shp[q]));
  }
  if (c.fl_i < 0 && !(c.epsabs < kSxClosedMin))
    chain::adj_pixels<MASS, LL, NMAX, false>(s, c, s_nc, s_dc, shp, beta, sbar, p0, p1, acc);
  else
    chain::adj_pixels<MASS, LL, NMAX, true>(s, c, s_nc, s_dc, shp, beta, sbar, p0, p1, acc);
  block_sums<NS>(acc, red, s.acc + ((size_t)part * s.tiles + tile) * kNAcc);
}

using GroupKernel = void (*)(Group);

template <int MASS, int LL, int... N>
static void fill_chain(GroupKernel* f, GroupKernel* a, std::integer_sequence<int, N...>) {
  ((f[(MASS * 2 + LL) * 16 + N] = chain_fwd_kernel<MASS, LL, N - 1>), ...);
  ((a[(MASS * 2 + LL) * 16 + N] = chain_adj_kernel<MASS, LL, N - 1>), ...);
}

// indexed by subpix_key
struct ChainTable {
  GroupKernel fwd[64] = {};
  GroupKernel adj[64] = {};
  ChainTable() {
    fill_chain<0, 0>(fwd, adj, std::make_integer_sequence<int, kMaxNmax + 2>{});
    fill_chain<0, 1>(fwd, adj, std::make_integer_sequence<int, kMaxNmax + 2>{});
    fill_chain<1, 0>(fwd, adj, std::make_integer_sequence<int, kMaxNmax + 2>{});
    fill_chain<1, 1>(fwd, adj, std::make_integer_sequence<int, kMaxNmax + 2>{});
  }
};
static const ChainTable& chain_table() {
  static const ChainTable t;
  return t;
}

static int launch(GroupKernel k, const Group& g, hipStream_t st) {
  if (g.block0[g.nsys] <= 0) return GL_OK;
  hipLaunchKernelGGL(k, dim3(g.block0[g.nsys]), dim3(kSubThreads), 0, st, g);
  GL_HIP(hipGetLastError());
  return GL_OK;
}
int launch_chain_fwd(int key, const Group& g, hipStream_t st) {
  return launch(chain_table().fwd[key], g, st);
}
int launch_chain_adj(int key, const Group& g, hipStream_t st) {
  return launch(chain_table().adj[key], g, st);
}

}  // namespace glens
