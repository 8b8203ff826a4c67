// Post-training quantisation of a frame's Gaussians and the frame's bit
// count (the compression pipeline, Sec. 3.3.A / 3.3.B).  Distinct
// quantisers per attribute:
//   mean       IEEE binary16, round to nearest even (16 bits per coordinate);
//   Cholesky,  per component a uniform min-max quantiser with b bits over
//   colour     the frame's range: with lo, hi the component's extremes,
//              L = 2^b - 1, inv = L / (hi - lo) (0 if hi == lo),
//              step = (hi - lo) / L:
//                code = clamp(rint((x - lo) * inv), 0, L);  x^ = lo + code step
//              evaluated in FP32 in exactly this order without contraction,
//              so the codes are reproducible integer decisions.
// Bits of vanilla entropy coding: an ideal static coder for the frame's own
// code statistics, N * H per quantised component (H the empirical entropy,
// FP64), 16 bits per coordinate for the means, and lo, hi of every
// component (FP32) as side information.
//
// Two launches: the extremes of blocks of Gaussians, and the encoder.  Its
// first blocks (one thread per Gaussian) write binary16 means, codes and
// dequantised values; its last six each take one component's whole code
// histogram in LDS and its entropy, and the last of those to finish adds up
// the frame.  The codes are evaluated again for the histogram rather than
// counted by global atomics on a few bins, which took 125 of 147 us at 30,000
// Gaussians and 6 bits.
#include <algorithm>

#include "quant_common.h"

namespace gs2d {
namespace {

constexpr int QE = 1024;         // threads per block of the encoder
constexpr int Q_MAX_BLOCKS = 1024;
constexpr int Q_MAX_BITS = 12;

struct QLayout {
  size_t part, done, total;
  int blocks;
};

QLayout q_layout(int N) {
  QLayout q;
  q.blocks = std::min((N + QB - 1) / QB, Q_MAX_BLOCKS);
  size_t o = 0;
  auto take = [&o](size_t b) {
    const size_t at = o;
    o = (o + b + 255) & ~(size_t)255;
    return at;
  };
  q.part = take((size_t)q.blocks * 12 * 4);  // per block: 6 x (min, max)
  q.done = take(4);                          // components whose entropy is written
  q.total = o;
  return q;
}

__global__ void __launch_bounds__(QB)
k_q_extremes(int N, const float *__restrict__ chol, const float *__restrict__ rgb,
             float *__restrict__ part, int *__restrict__ done) {
  float mn[6], mx[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) mn[c] = INFINITY, mx[c] = -INFINITY;
  for (int n = blockIdx.x * QB + threadIdx.x; n < N; n += gridDim.x * QB) {
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      const float x = comp(chol, rgb, n, c);
      mn[c] = fminf(mn[c], x);
      mx[c] = fmaxf(mx[c], x);
    }
  }
  block_extremes(mn, mx, part + blockIdx.x * 12);
  if (blockIdx.x == 0 && threadIdx.x == 0) *done = 0;
}

// N * H of component c's codes, in FP64.
__device__ void component_bits(int N, int c, int nbits, const QParams &Q,
                               const float *__restrict__ chol, const float *__restrict__ rgb,
                               uint32_t *__restrict__ hist, double *__restrict__ red,
                               double *__restrict__ bits) {
  const int tid = threadIdx.x, nb = 1 << nbits;
  const float L = (float)(nb - 1);
  for (int i = tid; i < nb; i += QE) hist[i] = 0;
  __syncthreads();
#pragma unroll 4
  for (int n = tid; n < N; n += QE) {
    const int code = (int)quant_code(Q, c, L, comp(chol, rgb, n, c));
    // a component that is constant over the wavefront: one count for all
    const unsigned long long live = __ballot(true);
    const int first = __builtin_amdgcn_readfirstlane(code);
    if (__ballot(code == first) == live) {
      if ((int)__ffsll((long long)live) - 1 == (tid & 63))
        atomicAdd(&hist[code], (uint32_t)__popcll(live));
    } else {
      atomicAdd(&hist[code], 1u);
    }
  }
  __syncthreads();
  const double inv_n = 1.0 / (double)N;
  double s = 0.0;
  for (int i = tid; i < nb; i += QE) {
    const uint32_t k = hist[i];
    if (k) {
      const double p = (double)k * inv_n;
      s -= p * log2(p);
    }
  }
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((tid & 63) == 0) red[tid >> 6] = s;
  __syncthreads();
  if (tid == 0) {
    double t = 0.0;
    for (int w = 0; w < QE / 64; ++w) t += red[w];
    bits[c] = t * (double)N;
  }
}

// Blocks [0, n_enc): the Gaussians; with bits, blocks n_enc + c: component c.
// bits[6] = 32 N (binary16 means) + sum of the six components + side info.
__global__ void __launch_bounds__(QE)
k_q_encode(int N, int n_enc, int n_parts, const float *__restrict__ xy,
           const float *__restrict__ chol, const float *__restrict__ rgb, int bits_chol,
           int bits_rgb, const float *__restrict__ part, float *__restrict__ q_xy,
           float *__restrict__ q_chol, float *__restrict__ q_rgb, uint16_t *__restrict__ codes,
           float *__restrict__ ranges, double *__restrict__ bits, int *__restrict__ done) {
  __shared__ QParams Q;
  __shared__ uint32_t hist[1 << Q_MAX_BITS];
  __shared__ double red[QE / 64];
  quant_params(n_parts, part, bits_chol, bits_rgb, Q);
  const int tid = threadIdx.x;
  if ((int)blockIdx.x >= n_enc) {
    const int c = (int)blockIdx.x - n_enc;
    component_bits(N, c, c < 3 ? bits_chol : bits_rgb, Q, chol, rgb, hist, red, bits);
    if (tid != 0) return;
    // the components' values are released before they are counted and read
    // back by the block that counts the last one
    __threadfence();
    if (atomicAdd(done, 1) != 5) return;
    __threadfence();
    double t = 32.0 * (double)N + 6.0 * 64.0;
    for (int k = 0; k < 6; ++k)
      t += __hip_atomic_load(bits + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    bits[6] = t;
    return;
  }
  if (ranges && blockIdx.x == 0 && tid < 12) ranges[tid] = (tid & 1) ? Q.hi[tid >> 1] : Q.lo[tid >> 1];
  for (int n = blockIdx.x * QE + tid; n < N; n += n_enc * QE) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const __half h = __float2half_rn(xy[2 * n + k]);
      q_xy[2 * n + k] = __half2float(h);
      if (codes) codes[8 * n + k] = __half_as_ushort(h);
    }
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      const float L = (float)((1 << (c < 3 ? bits_chol : bits_rgb)) - 1);
      const float code = quant_code(Q, c, L, comp(chol, rgb, n, c));
      const float xh = quant_value(Q, c, code);
      if (c < 3) q_chol[3 * n + c] = xh;
      else q_rgb[3 * n + c - 3] = xh;
      if (codes) codes[8 * n + 2 + c] = (uint16_t)code;
    }
  }
}

}  // namespace

hipError_t launch_quant_extremes(int N, const float *chol, const float *rgb, void *qws,
                                 hipStream_t st) {
  const QLayout q = q_layout(N);
  hipLaunchKernelGGL(k_q_extremes, dim3(q.blocks), dim3(QB), 0, st, N, chol, rgb,
                     at<float>(qws, q.part), at<int>(qws, q.done));
  return hipGetLastError();
}

float *quant_parts(int N, void *qws, int *n_parts) {
  const QLayout q = q_layout(N);
  *n_parts = q.blocks;
  return at<float>(qws, q.part);
}

hipError_t launch_quantise(int N, const float *xy, const float *chol, const float *rgb,
                           int bits_chol, int bits_rgb, float *q_xy, float *q_chol, float *q_rgb,
                           uint16_t *codes, float *ranges, double *bits, void *qws,
                           hipStream_t st) {
  const QLayout q = q_layout(N);
  const hipError_t e = launch_quant_extremes(N, chol, rgb, qws, st);
  if (e != hipSuccess) return e;
  const int n_enc = std::min((N + QE - 1) / QE, Q_MAX_BLOCKS);
  auto encode = [&](int enc, int count) {
    hipLaunchKernelGGL(k_q_encode, dim3(enc + count), dim3(QE), 0, st, N, enc, q.blocks, xy, chol,
                       rgb, bits_chol, bits_rgb, at<float>(qws, q.part), q_xy, q_chol, q_rgb, codes,
                       ranges, bits, at<int>(qws, q.done));
  };
  // In place, the components are counted before the encoder writes over them.
  auto overlap = [N](const float *a, const float *b) {
    return a < b + 3 * (size_t)N && b < a + 3 * (size_t)N;
  };
  const bool in_place = overlap(q_chol, chol) || overlap(q_chol, rgb) || overlap(q_rgb, chol) ||
                        overlap(q_rgb, rgb);
  if (bits && in_place) {
    encode(0, 6);
    encode(n_enc, 0);
  } else {
    encode(n_enc, bits ? 6 : 0);
  }
  return hipGetLastError();
}

size_t quantise_workspace_bytes(int N) { return q_layout(N).total; }

}  // namespace gs2d

using namespace gs2d;

extern "C" size_t gs2d_ptq_workspace_bytes(int32_t N) {
  return N < 1 ? 0 : quantise_workspace_bytes(N);
}

extern "C" int gs2d_ptq(int32_t N, const float *xy, const float *chol, const float *rgb,
                        const gs2d_quant_cfg *cfg, float *q_xy, float *q_chol, float *q_rgb,
                        uint16_t *codes, float *ranges, double *bits, void *ws, size_t ws_bytes,
                        void *stream) {
  try {
    if (N < 1 || !xy || !chol || !rgb || !cfg || !q_xy || !q_chol || !q_rgb) return GS2D_EINVAL;
    if (cfg->bits_chol < 1 || cfg->bits_chol > Q_MAX_BITS || cfg->bits_rgb < 1 ||
        cfg->bits_rgb > Q_MAX_BITS)
      return GS2D_EINVAL;
    if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255)) return GS2D_EINVAL;
    if (ws_bytes < quantise_workspace_bytes(N)) return GS2D_ENOSPACE;
    return launch_quantise(N, xy, chol, rgb, cfg->bits_chol, cfg->bits_rgb, q_xy, q_chol, q_rgb,
                           codes, ranges, bits, ws, reinterpret_cast<hipStream_t>(stream)) ==
                   hipSuccess
               ? GS2D_OK
               : GS2D_EHIP;
  } catch (...) {
    return GS2D_EHIP;
  }
}
