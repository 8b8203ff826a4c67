// Device-side building blocks of the quantisers (see quant.hip), shared with
// the quantisation-aware fitting kernels (bin.hip, adam.hip).
#pragma once

#include <hip/hip_fp16.h>

#include "gs2d_internal.h"

namespace gs2d {

constexpr int QB = 256;  // threads per block of the extremes kernels
// Threads that reduce the block extremes to the quantisers' parameters: a
// whole number of rows of 12.
constexpr int Q_ROWS = 21;
static_assert(Q_ROWS * 12 <= QB, "a block holds the reducing threads");

__device__ inline float comp(const float *__restrict__ chol, const float *__restrict__ rgb, int n,
                             int c) {
  return c < 3 ? chol[3 * n + c] : rgb[3 * n + c - 3];
}

// Minimum and maximum of six values per thread over a block of QB threads
// into out[12] = {min, max} x 6.
__device__ inline void block_extremes(float (&mn)[6], float (&mx)[6], float *__restrict__ out) {
  __shared__ float red[QB / 64][12];
#pragma unroll
  for (int c = 0; c < 6; ++c)
    for (int o = 32; o > 0; o >>= 1) {
      mn[c] = fminf(mn[c], __shfl_xor(mn[c], o, 64));
      mx[c] = fmaxf(mx[c], __shfl_xor(mx[c], o, 64));
    }
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      red[threadIdx.x >> 6][2 * c] = mn[c];
      red[threadIdx.x >> 6][2 * c + 1] = mx[c];
    }
  __syncthreads();
  if (threadIdx.x < 12) {
    float v = red[0][threadIdx.x];
    for (int w = 1; w < QB / 64; ++w)
      v = (threadIdx.x & 1) ? fmaxf(v, red[w][threadIdx.x]) : fminf(v, red[w][threadIdx.x]);
    out[threadIdx.x] = v;
  }
}

// lo, hi, inv and step of the six components, by a block of at least
// 12 Q_ROWS threads from the n_parts x 12 block extremes.  Every block that
// quantises forms them for itself: as a kernel of their own they were one
// block's chain of n_parts loads (13.7 us at 30,000 Gaussians).  Ends with a
// barrier.
struct QParams {
  float red[Q_ROWS][12];
  float lo[6], hi[6], inv[6], step[6];
};

__device__ inline void quant_params(int n_parts, const float *__restrict__ part, int bits_chol,
                                    int bits_rgb, QParams &Q) {
  const int t = threadIdx.x, i = t % 12, r = t / 12;
  if (t < 12 * Q_ROWS) {
    float v = part[min(r, n_parts - 1) * 12 + i];
#pragma unroll 4
    for (int b = r + Q_ROWS; b < n_parts; b += Q_ROWS) {
      const float x = part[b * 12 + i];
      v = (i & 1) ? fmaxf(v, x) : fminf(v, x);
    }
    Q.red[r][i] = v;
  }
  __syncthreads();
  if (t < 12) {
    float v = Q.red[0][t];
#pragma unroll
    for (int b = 1; b < Q_ROWS; ++b)
      v = (t & 1) ? fmaxf(v, Q.red[b][t]) : fminf(v, Q.red[b][t]);
    if (t & 1) Q.hi[t >> 1] = v;
    else Q.lo[t >> 1] = v;
  }
  __syncthreads();
  if (t < 6) {
    const float L = (float)((1 << (t < 3 ? bits_chol : bits_rgb)) - 1);
    const float rng = f32_sub(Q.hi[t], Q.lo[t]);
    Q.inv[t] = rng == 0.f ? 0.f : __fdiv_rn(L, rng);
    Q.step[t] = rng == 0.f ? 0.f : __fdiv_rn(rng, L);
  }
  __syncthreads();
}

// Code of x in component c (L = 2^bits - 1) and its dequantised value.
__device__ inline float quant_code(const QParams &Q, int c, float L, float x) {
  return fminf(fmaxf(rintf(f32_mul(f32_sub(x, Q.lo[c]), Q.inv[c])), 0.f), L);
}
__device__ inline float quant_value(const QParams &Q, int c, float code) {
  return f32_add(Q.lo[c], f32_mul(code, Q.step[c]));
}

}  // namespace gs2d
