// What the sub-pixel kernels share: their walk over the pixels, the staged derivative series and
// the FP64 sums of the adjoint's per-lane accumulators.
#pragma once

#include <hip/hip_runtime.h>

#include "glens_device.h"

namespace glens {

constexpr int kSubThreads = 256;

// Row and column of the pixels p0 + threadIdx.x + n blockDim.x of a W-column image, stepped
// without a division per pixel. The first row and the step come from a float reciprocal: with
// fewer than 2^15 pixels and W <= 158 columns (p + 1/2) / W is 1/316 or more from an integer,
// and its rounding error below 1e-4, so that the integer part is exact.
struct PixelWalk {
  int i, j, di, dj, W;
  __device__ __forceinline__ PixelWalk(int W_, int p0 = 0) : W(W_) {
    const float inv = rcp_f32(float(W));
    const int p = p0 + int(threadIdx.x);
    i = int((float(p) + 0.5f) * inv);
    j = p - i * W;
    di = int((float(blockDim.x) + 0.5f) * inv);
    dj = int(blockDim.x) - di * W;
  }
  __device__ __forceinline__ void next() {
    i += di;
    j += dj;
    if (j >= W) {
      j -= W;
      ++i;
    }
  }
};

// Copies the particle's derivative-series coefficients to LDS (read uniformly by every lane),
// those of dS/dt times `scale`.
__device__ __forceinline__ void stage_series(const PConst& c, float scale, float* s_nc,
                                             float* s_dc) {
  for (int n = threadIdx.x; n < kMaxTerms; n += blockDim.x) {
    s_nc[n] = c.nc[n];
    s_dc[n] = c.dc[n] * scale;
  }
  __syncthreads();
}

// Sum over a wave's lanes, on every lane (the pairing of wave_sums).
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

constexpr int halved(int n) { return n > 1 ? n / 2 : 1; }

// One step of the transposed butterfly below for a lane holding NV values (all indices
// compile-time, so the values stay in registers).
template <int NV>
__device__ __forceinline__ void wave_sum_step(double* v, int off, int lane) {
  if constexpr (NV > 1) {
    const bool up = lane & off;
#pragma unroll
    for (int i = 0; i < NV / 2; ++i) {
      const double send = up ? v[i] : v[i + NV / 2];
      const double keep = up ? v[i + NV / 2] : v[i];
      v[i] = keep + __shfl_xor(send, off, 64);
    }
  } else {
    v[0] += __shfl_xor(v[0], off, 64);
  }
}

// Wave sums of NS per-lane FP32 values, in FP64, written to out[0 .. NS). A transposed
// butterfly: with the values padded to N (a power of two), at the step with lane offset o a
// lane keeps one half of its values, sends the other half to lane ^ o and adds what it
// receives, so each step halves the values a lane holds. Every sum pairs lanes in the same
// order as a separate xor butterfly per value would, with about N shuffles instead of
// 6 NS. The first step shuffles the FP32 values and adds them in FP64. More than 64 values go in
// two parts (64 and the rest, padded to its own power of two: with 68 padded to 128 the sums cost
// as much as two sub-pixels).
template <int NS>
__device__ __forceinline__ void wave_sums(const float* acc, double* out) {
  if constexpr (NS > 64) {
    wave_sums<64>(acc, out);
    wave_sums<NS - 64>(acc + 64, out + 64);
  } else {
    constexpr int N = NS <= 4 ? 4 : (NS <= 8 ? 8 : (NS <= 16 ? 16 : (NS <= 32 ? 32 : 64)));
    const int lane = threadIdx.x & 63;
    double v[N / 2];
    {
      const bool up = lane & 32;
#pragma unroll
      for (int i = 0; i < N / 2; ++i) {
        const float lo = i < NS ? acc[i] : 0.f, hi = i + N / 2 < NS ? acc[i + N / 2] : 0.f;
        const float send = up ? lo : hi;
        v[i] = double(up ? hi : lo) + double(__shfl_xor(send, 32, 64));
      }
    }
    constexpr int n1 = N / 2, n2 = halved(n1), n3 = halved(n2), n4 = halved(n3), n5 = halved(n4);
    wave_sum_step<n1>(v, 16, lane);
    wave_sum_step<n2>(v, 8, lane);
    wave_sum_step<n3>(v, 4, lane);
    wave_sum_step<n4>(v, 2, lane);
    wave_sum_step<n5>(v, 1, lane);
    // the 64 / N lanes from q 64 / N on hold value q
    constexpr int per = 64 / N;
    if (lane % per == 0 && lane / per < NS) out[lane / per] = v[0];
  }
}

// Wave sums of the NS per-lane values v (at most 8), value q in the lanes from 64 q / N on: the
// transposed butterfly again, with the pairing of wave_sum for each value.
template <int NS>
__device__ __forceinline__ double wave_sums_f64(const double* v) {
  static_assert(NS <= 8, "three steps halve the values");
  constexpr int N = NS == 1 ? 1 : (NS == 2 ? 2 : (NS <= 4 ? 4 : 8));
  const int lane = threadIdx.x & 63;
  double w[N];
#pragma unroll
  for (int i = 0; i < N; ++i) w[i] = i < NS ? v[i] : 0.0;
  constexpr int n1 = halved(N), n2 = halved(n1), n3 = halved(n2);
  wave_sum_step<N>(w, 32, lane);
  wave_sum_step<n1>(w, 16, lane);
  wave_sum_step<n2>(w, 8, lane);
  wave_sum_step<n3>(w, 4, lane);
  wave_sum_step<1>(w, 2, lane);
  wave_sum_step<1>(w, 1, lane);
  return w[0];
}

// FP64 sums of the block's accumulators, across each wave, then across the waves, to out[0 .. NS).
template <int NS>
__device__ __forceinline__ void block_sums(const float* acc, double (*red)[NS], double* out) {
  const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  wave_sums<NS>(acc, red[wave]);
  __syncthreads();
  for (int q = threadIdx.x; q < NS; q += blockDim.x) {
    double v = 0.0;
    for (int w = 0; w < nw; ++w) v += red[w][q];
    out[q] = v;
  }
}

}  // namespace glens
