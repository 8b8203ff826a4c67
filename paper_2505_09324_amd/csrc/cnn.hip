// Learned initialiser: a small convolutional regressor (Sec. 3.2.B, made
// per-tile) with hand-written training and inference kernels.
//
// Network: input [H][W][8] (RGB, residual vs the previous frame, 2 zero
// channels) -> 4 x (conv3x3 stride 2 pad 1, 64 channels, ReLU) -> conv3x3
// stride 1 head with 73 channels = 9 count logits + 8 slots x 8 parameters,
// one output per 16x16 screen tile.  Activations are channels-last BF16,
// weights BF16 copies of FP32 master weights, accumulation FP32 on MFMA
// (v_mfma_f32_16x16x32_bf16).
//
// Every convolution pass is an implicit GEMM C[M x N] = A[M x K] B[K x N] over
// tiles of pixels; a tile's patch of its input is in LDS (pixel pitch padded so
// that the reads of one MFMA step spread over the banks), the weights are in
// registers, and the next tile's patch is loaded while one is multiplied:
//   forward      M = Cout, N = output pixels, K = (tap, Cin)
//                A = W[co][tap][ci], B = the tap's input pixels; bias, ReLU
//                and the BF16 rounding run in the epilogue
//   grad input   M = Cin, N = input pixels of one stride-parity class,
//                K = (the class's taps, Cout).  With stride 2 an input pixel
//                (y, x) receives output gradients only through the taps
//                with ty = y + 1 (mod 2) and tx = x + 1 (mod 2): 1, 2, 2 or 4
//                of the 9, so the four parity classes are separate GEMMs over
//                the same pixels of dZ and no multiply-by-zero is issued.  The
//                epilogue applies the previous layer's ReLU' and writes its
//                BF16 dZ directly.
//   grad weight  M = Cout, N = (tap, Cin), K = output pixels, split over
//                workgroups whose partials a second kernel sums (plain stores:
//                FP32 atomics from every workgroup cost more than the GEMM).
//                Both operands are channels-last; LDS reads that transpose
//                make fragments of them.  dZ times ones is the bias gradient.
// dZ = dL/d(layer output) masked by ReLU', held as BF16 [pixels][CoutS].
#include <algorithm>
#include <cmath>

#include "gs2d_internal.h"

namespace gs2d {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int NLAYER = 5;
constexpr int HEAD_CH = 73;
constexpr int NSLOT = 8, NPAR = 8;
constexpr int KPAD = 32;     // K of the weight matrices is padded to one MFMA step
constexpr int LP = 64 + 8;   // LDS pitch of a pixel in halves (144 B = 9 x 16 B)

__device__ inline uint16_t f2bf(float x) {  // round to nearest even
  const uint32_t u = __float_as_uint(x);
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

struct ConvDims {
  int Hin, Win, Cin, Hout, Wout, Cout, stride, relu;
  int Mpad;   // rows of the weight matrix (Cout rounded up to 64)
  int Kf;     // forward K = 9 * Cin, padded to a multiple of KPAD
  int CoutS;  // channel stride of dZ (Cout rounded up to 8)
  int Kb;     // row length of the transposed weights = 9 * CoutS, padded to KPAD
};

struct ConvArgs {
  ConvDims d;
  const uint16_t *x;     // layer input [Hin*Win][Cin] bf16 (grad input: its ReLU mask)
  const uint16_t *w;     // [Mpad][Kf] bf16, k = tap * Cin + ci
  const uint16_t *wt;    // [Cin][Kb] bf16, k = tap * CoutS + co (grad input)
  const float *bias;     // [Mpad]
  uint16_t *y;           // forward output [Hout*Wout][Cout] bf16 (hidden layers)
  float *y_planar;       // forward output [Cout][Hout*Wout] fp32 (head)
  const uint16_t *dz;    // dZ of this layer [Hout*Wout][CoutS] bf16
  uint16_t *dz_prev;     // grad input: dZ of the previous layer [Hin*Win][Cin] bf16
};

// Tile of this workgroup out of n (or n: none), grid rounded up to eighths.
// Workgroup b runs on XCD b % 8: each XCD gets a contiguous eighth, so that
// the lines that neighbouring tiles share are fetched into one L2.
__device__ __forceinline__ int xcd_tile(int n) {
  const int t = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  return min(t, n);
}

// Range-checked loads at base + off, base the same for the whole wave: an
// offset of OUTSIDE gives zeros.
typedef unsigned int uint4v __attribute__((ext_vector_type(4)));
constexpr uint32_t OUTSIDE = 0xFFFFFFF0u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *p, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (uint32_t)bytes, 0x00020000);
}
__device__ __forceinline__ uint4 load16(__amdgpu_buffer_rsrc_t b, uint32_t off, uint32_t base) {
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(b, (int)off, (int)base, 0));
}
__device__ __forceinline__ float load4(__amdgpu_buffer_rsrc_t b, uint32_t off, uint32_t base) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(b, (int)off, (int)base, 0));
}

// --------------------------------------------------------------- forward --
// Bias, ReLU and rounding of a wave's 16 x 16 block: lane holds rows row ..
// row + 3 of output pixel `col` (D[4 (lane >> 4) + r][lane & 15]).
__device__ __forceinline__ void store_fwd(const ConvArgs &a, const floatx4 &acc, int row,
                                          long long col, long long P) {
  const ConvDims &d = a.d;
  if (a.y) {
    if (row < d.Cout) {  // Cout is a multiple of 4 for the hidden layers
      uint16_t o[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float v = acc[r] + a.bias[row + r];
        if (d.relu) v = fmaxf(v, 0.f);
        o[r] = f2bf(v);
      }
      *reinterpret_cast<uint2 *>(a.y + col * d.Cout + row) = *reinterpret_cast<uint2 *>(o);
    }
  } else {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (row + r < d.Cout) a.y_planar[(size_t)(row + r) * P + col] = acc[r] + a.bias[row + r];
  }
}

// First layer, from the frame itself.  A workgroup forms a 32 x 4 tile of
// output pixels: it converts the 65 x 9 input pixels that the tile's taps reach
// (RGB and residual as BF16, channels last, 16 bytes per pixel) into LDS,
// writes those the tile owns to x_in (the backward pass reads them), and
// multiplies straight from LDS, one tap of one pixel per 16-byte read; waves 2
// x 2, each 32 channels x 64 pixels with its weights in registers.  The output
// tile goes through LDS so that whole 128-byte pixels are stored.  HBM bound:
// 150 MB at 1920 x 1080 (frame, residual, x_in and the output), 37 us (47 us
// with 64-bit addresses and a border test per load).  As two launches, a
// conversion and an implicit GEMM that read x_in back 2.25 times, it took 17 +
// 37 us; with the output stored from the accumulators (32 bytes of a pixel at a
// time) 57 us.
constexpr int C0_TW = 32, C0_TH = 4, C0_PW = 2 * C0_TW + 1, C0_PH = 2 * C0_TH + 1;
constexpr int C0_N = C0_PW * C0_PH, C0_PER = (C0_N + 255) / 256;
__global__ void __launch_bounds__(256)
k_conv_first(ConvArgs a, const float *__restrict__ frame, const float *__restrict__ prev,
             uint16_t *__restrict__ x_in) {
  __shared__ __attribute__((aligned(16))) union {
    uint4 px[C0_N];
    uint16_t y[C0_TW * C0_TH * LP];
  } sm;
  const ConvDims &d = a.d;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int tiles_x = (d.Wout + C0_TW - 1) / C0_TW;
  const int n_tiles = tiles_x * ((d.Hout + C0_TH - 1) / C0_TH), t = xcd_tile(n_tiles);
  if (t >= n_tiles) return;
  const int ox0 = t % tiles_x * C0_TW, oy0 = t / tiles_x * C0_TH;
  const size_t HW = (size_t)d.Hin * d.Win;
  const int wm = w & 1, wn = w >> 1, r = lane & 15, kg = lane >> 4;
  float f[C0_PER][3], q[C0_PER][3];
  size_t at[C0_PER];
  int own[C0_PER];
  const __amdgpu_buffer_rsrc_t fb = buffer_of(frame, 12 * HW);
  const __amdgpu_buffer_rsrc_t qb = buffer_of(prev, prev ? 12 * HW : 0);
  const int plane = (int)(4 * HW);
#pragma unroll
  for (int j = 0; j < C0_PER; ++j) {
    const int e = tid + 256 * j, py = e / C0_PW, pxx = e - py * C0_PW;
    const int iy = 2 * oy0 - 1 + py, ix = 2 * ox0 - 1 + pxx;
    const bool in = e < C0_N && iy >= 0 && iy < d.Hin && ix >= 0 && ix < d.Win;
    at[j] = (size_t)iy * d.Win + ix;
    own[j] = in && py > 0 && pxx > 0;  // the first row and column belong to the tiles before
    const uint32_t o = in ? (uint32_t)(iy * d.Win + ix) * 4u : OUTSIDE;
#pragma unroll
    for (int c = 0; c < 3; ++c) f[j][c] = load4(fb, o, c * plane);
    if (prev)
#pragma unroll
      for (int c = 0; c < 3; ++c) q[j][c] = load4(qb, o, c * plane);
  }
  uint4 av[3][2];
#pragma unroll
  for (int ks = 0; ks < 3; ++ks)
#pragma unroll
    for (int i = 0; i < 2; ++i)
      av[ks][i] = *reinterpret_cast<const uint4 *>(a.w + (size_t)(32 * wm + 16 * i + r) * d.Kf +
                                                   32 * ks + 8 * kg);
#pragma unroll
  for (int j = 0; j < C0_PER; ++j) {
    uint16_t v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      v[c] = f2bf(f[j][c]);
      v[3 + c] = f2bf(prev ? f[j][c] - q[j][c] : 0.f);
    }
    if (tid + 256 * j < C0_N) sm.px[tid + 256 * j] = *reinterpret_cast<uint4 *>(v);
    if (own[j]) *reinterpret_cast<uint4 *>(x_in + at[j] * 8) = *reinterpret_cast<uint4 *>(v);
  }
  __syncthreads();
  floatx4 acc[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < 3; ++ks) {
    const int tap = 4 * ks + kg, ty = tap / 3, tx = tap - 3 * ty;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int oy = 2 * wn + (j >> 1), ox = 16 * (j & 1) + r;
      uint4 b = make_uint4(0, 0, 0, 0);
      if (tap < 9) b = sm.px[(2 * oy + ty) * C0_PW + 2 * ox + tx];
#pragma unroll
      for (int i = 0; i < 2; ++i)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av[ks][i]),
                                                            __builtin_bit_cast(bf16x8, b),
                                                            acc[i][j], 0, 0, 0);
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = 32 * wm + 16 * i + 4 * kg;
      const int p = 32 * (2 * wn + (j >> 1)) + 16 * (j & 1) + r;
      uint16_t o[4];
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) o[q4] = f2bf(fmaxf(acc[i][j][q4] + a.bias[row + q4], 0.f));
      *reinterpret_cast<uint2 *>(sm.y + p * LP + row) = *reinterpret_cast<uint2 *>(o);
    }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int e = tid + 256 * j, p = e >> 3, c8 = 8 * (e & 7);
    const int oy = oy0 + (p >> 5), ox = ox0 + (p & 31);
    if (oy < d.Hout && ox < d.Wout)
      *reinterpret_cast<uint4 *>(a.y + ((size_t)oy * d.Wout + ox) * 64 + c8) =
          *reinterpret_cast<const uint4 *>(sm.y + p * LP + c8);
  }
}

// Layers with 64 input channels.  A workgroup keeps its 64 rows of the weight
// matrix in registers (16 rows x 576 per wave) and walks over 8 x 8 tiles of
// output pixels.  A tile's input patch goes to LDS once and every tap is read
// from there (pixel pitch 144 bytes: 16-byte reads of pixels at stride 2 spread
// over the banks), while the next tile's patch loads into registers.  K runs
// over (tap, channel) in steps of 32.  Bound by the loads of the patches: 26,
// 11, 6.5 and 8.8 us for the four layers at 1920 x 1080.  As an implicit GEMM
// staged tap by tap, each of its 9 stages waited for memory and every 64
// pixels fetched the 74 KB of weights again: 30, 12, 8.2 and 8.9 us.  Waves of
// 32 rows x 32 pixels halve the LDS reads, but their 144 registers of weights
// leave no room for the patch (31 us; 28 us with the patch loaded straight to
// a second LDS buffer, whose border tests triple the code).
constexpr int CT = 8;  // output tile side
template <int S>
constexpr int CPATCH = (CT - 1) * S + 3;

template <int S>
__global__ void __launch_bounds__(256, 2) k_conv_fwd(ConvArgs a, int tiles_x, int n_tiles) {
  constexpr int PW = CPATCH<S>, CHUNKS = PW * PW * 8, PER = (CHUNKS + 255) / 256;
  __shared__ __attribute__((aligned(16))) uint16_t patch[PW * PW * LP];
  const ConvDims &d = a.d;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int m0 = blockIdx.y * 64;
  const int r = lane & 15, kg = lane >> 4;
  uint4 v[PER];
  auto load = [&](int t) {
    const int iy0 = (t / tiles_x) * CT * S - 1, ix0 = (t % tiles_x) * CT * S - 1;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int e = tid + 256 * j, p = e >> 3, py = p / PW, px = p - py * PW;
      const int iy = iy0 + py, ix = ix0 + px;
      v[j] = make_uint4(0, 0, 0, 0);
      if (e < CHUNKS && iy >= 0 && iy < d.Hin && ix >= 0 && ix < d.Win)
        v[j] = *reinterpret_cast<const uint4 *>(a.x + ((size_t)iy * d.Win + ix) * 64 + 8 * (e & 7));
    }
  };
  load(blockIdx.x);
  uint4 av[18];
#pragma unroll
  for (int k = 0; k < 18; ++k)
    av[k] = *reinterpret_cast<const uint4 *>(a.w + (size_t)(m0 + 16 * w + r) * d.Kf + 32 * k +
                                             8 * kg);
  const long long P = (long long)d.Hout * d.Wout;
  for (int t = blockIdx.x; t < n_tiles; t += gridDim.x) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int e = tid + 256 * j;
      if (e < CHUNKS)
        *reinterpret_cast<uint4 *>(patch + (e >> 3) * LP + 8 * (e & 7)) = v[j];
    }
    __syncthreads();
    if (t + (int)gridDim.x < n_tiles) load(t + gridDim.x);
    floatx4 acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
    // pixel r of 16-pixel block j: row 2 j + (r >> 3)
    const uint16_t *base = patch + ((r >> 3) * S * PW + (r & 7) * S) * LP + 8 * kg;
#pragma unroll
    for (int k = 0; k < 18; ++k) {
      const int tap = k >> 1, ty = tap / 3, tx = tap - 3 * ty;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint4 b = *reinterpret_cast<const uint4 *>(
            base + ((2 * j * S + ty) * PW + tx) * LP + 32 * (k & 1));
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av[k]),
                                                         __builtin_bit_cast(bf16x8, b), acc[j], 0,
                                                         0, 0);
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int oy = (t / tiles_x) * CT + 2 * j + (r >> 3);
      const int ox = (t % tiles_x) * CT + (r & 7);
      if (oy >= d.Hout || ox >= d.Wout) continue;
      store_fwd(a, acc[j], m0 + 16 * w + 4 * kg, (long long)oy * d.Wout + ox, P);
    }
  }
}

// ------------------------------------------------------------ grad input --
// Two BF16 values of `o` where those of `m` are > 0, else 0.
__device__ __forceinline__ uint32_t relu_mask(uint32_t o, uint32_t m) {
  return (__uint_as_float(m << 16) > 0.f ? o & 0xFFFFu : 0u) |
         (__uint_as_float(m & 0xFFFF0000u) > 0.f ? o & 0xFFFF0000u : 0u);
}

// Stride 2.  A workgroup walks over tiles of 8 x 8 pixels of dZ and forms the 16
// x 16 input pixels (8 x 8 of each parity class) whose gradients come from
// those and the next row and column: the 9 x 9 patch of dZ is in LDS, the
// weights in registers (16 rows x 576 per wave).  A wave reads a shifted pixel
// block once for all the taps that use it, 8 reads for 18 MFMAs.  The result
// goes through LDS so that masks are read and pixels written whole.  HBM bound:
// 31 us for the 149 MB of the second layer's at 1920 x 1080, 12 and 7 us for
// the next two.  As a GEMM per parity class, whose staging spent 44 us on
// addresses alone, they took 58, 19 and 9 us.  Three workgroups per compute
// unit instead of two spill registers: 36, 14 and 9 us.
constexpr int BT_W = 9;
__global__ void __launch_bounds__(256, 2) k_conv_bwd_data(ConvArgs a, int tiles_x, int n_tiles) {
  constexpr int N = BT_W * BT_W * 8, PER = (N + 255) / 256;
  __shared__ __attribute__((aligned(16))) uint16_t patch[BT_W * BT_W * LP];
  __shared__ __attribute__((aligned(16))) uint16_t out[256 * LP];
  const ConvDims &d = a.d;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, r = lane & 15, kg = lane >> 4;
  uint4 v[PER];
  auto load = [&](int t) {
    const int oy0 = t / tiles_x * 8, ox0 = t % tiles_x * 8;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int e = tid + 256 * j, p = e >> 3, py = p / BT_W, px = p - py * BT_W;
      v[j] = make_uint4(0, 0, 0, 0);
      if (e < N && oy0 + py < d.Hout && ox0 + px < d.Wout)
        v[j] = *reinterpret_cast<const uint4 *>(
            a.dz + ((size_t)(oy0 + py) * d.Wout + ox0 + px) * 64 + 8 * (e & 7));
    }
  };
  load(blockIdx.x);
  uint4 av[18];
#pragma unroll
  for (int k = 0; k < 18; ++k)
    av[k] = *reinterpret_cast<const uint4 *>(a.wt + (size_t)(16 * w + r) * d.Kb + 32 * k + 8 * kg);
  for (int t = blockIdx.x; t < n_tiles; t += gridDim.x) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int e = tid + 256 * j;
      if (e < N) *reinterpret_cast<uint4 *>(patch + (e >> 3) * LP + 8 * (e & 7)) = v[j];
    }
    __syncthreads();
    // thread's part of the output: pixels (row0 + 2 q, x), channels 8 c .. 8 c + 7
    const int c = tid & 7, x = t % tiles_x * 16 + ((tid >> 3) & 15);
    const int row0 = t / tiles_x * 16 + (tid >> 7);
    uint4 mask[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      mask[q] = make_uint4(0, 0, 0, 0);
      if (x < d.Win && row0 + 2 * q < d.Hin)
        mask[q] = *reinterpret_cast<const uint4 *>(
            a.x + ((size_t)(row0 + 2 * q) * d.Win + x) * 64 + 8 * c);
    }
    if (t + (int)gridDim.x < n_tiles) load(t + gridDim.x);
#pragma unroll 1
    for (int j = 0; j < 4; ++j) {  // 16 pixels of dZ: rows 2 j and 2 j + 1
      const uint16_t *base = patch + ((2 * j + (r >> 3)) * BT_W + (r & 7)) * LP + 8 * kg;
      floatx4 acc[2][2];  // [py][px]
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[i >> 1][i & 1] = floatx4{0.f, 0.f, 0.f, 0.f};
      // in order of falling shift a class meets its taps in their own order
#pragma unroll
      for (int sh = 3; sh >= 0; --sh) {
        const int dy = sh >> 1, dx = sh & 1;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const bf16x8 bv = __builtin_bit_cast(
              bf16x8, *reinterpret_cast<const uint4 *>(base + (dy * BT_W + dx) * LP + 32 * h));
#pragma unroll
          for (int cl = 0; cl < 4; ++cl) {
            const int py = cl >> 1, px = cl & 1;
            if (dy > py || dx > px) continue;  // an even row or column has no shifted tap
            const int ty = py ? (dy ? 0 : 2) : 1, tx = px ? (dx ? 0 : 2) : 1;
            acc[py][px] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, av[2 * (3 * ty + tx) + h]), bv, acc[py][px], 0, 0, 0);
          }
        }
      }
#pragma unroll
      for (int cl = 0; cl < 4; ++cl) {
        const int py = cl >> 1, px = cl & 1;
        uint16_t o[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) o[q] = f2bf(acc[py][px][q]);
        *reinterpret_cast<uint2 *>(
            out + ((2 * (2 * j + (r >> 3)) + py) * 16 + 2 * (r & 7) + px) * LP + 16 * w + 4 * kg) =
            *reinterpret_cast<uint2 *>(o);
      }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (x >= d.Win || row0 + 2 * q >= d.Hin) continue;
      const uint4 o = *reinterpret_cast<const uint4 *>(out + ((tid >> 3) + 32 * q) * LP + 8 * c);
      *reinterpret_cast<uint4 *>(a.dz_prev + ((size_t)(row0 + 2 * q) * d.Win + x) * 64 + 8 * c) =
          make_uint4(relu_mask(o.x, mask[q].x), relu_mask(o.y, mask[q].y),
                     relu_mask(o.z, mask[q].z), relu_mask(o.w, mask[q].w));
    }
  }
}

// Head (stride 1, 80 stored channels): a workgroup forms 8 x 4 input pixels from
// the 10 x 6 patch of dZ, 16 channels per wave.  K = (tap, co) runs in steps of
// 32 across tap borders, so a lane finds the tap of its 8 channels itself.
// Latency bound (255 workgroups at 1920 x 1080): 5.6 us; staged tap by tap,
// with 12 waits for memory instead of one, 15 us.
constexpr int HC = (HEAD_CH + 7) / 8 * 8, HKB = (9 * HC + KPAD - 1) / KPAD * KPAD;
constexpr int HP = HC + 8;  // LDS pitch of a pixel in halves (176 B = 11 x 16 B)
__global__ void __launch_bounds__(256) k_conv_bwd_data_head(ConvArgs a, int tiles_x) {
  constexpr int CH = HC / 8, N = 60 * CH, PER = (N + 255) / 256;
  __shared__ __attribute__((aligned(16))) uint16_t patch[60 * HP + 8];
  __shared__ __attribute__((aligned(16))) uint16_t out[32 * LP];
  const ConvDims &d = a.d;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, r = lane & 15, kg = lane >> 4;
  const int y0 = blockIdx.x / tiles_x * 4, x0 = blockIdx.x % tiles_x * 8;
  uint4 v[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int e = tid + 256 * j, p = e / CH, c = e - p * CH;
    const int y = y0 - 1 + p / 10, x = x0 - 1 + p % 10;
    v[j] = make_uint4(0, 0, 0, 0);
    if (e < N && y >= 0 && y < d.Hout && x >= 0 && x < d.Wout)
      v[j] = *reinterpret_cast<const uint4 *>(a.dz + ((size_t)y * d.Wout + x) * HC + 8 * c);
  }
  uint4 av[HKB / 32];
#pragma unroll
  for (int k = 0; k < HKB / 32; ++k)
    av[k] = *reinterpret_cast<const uint4 *>(a.wt + (size_t)(16 * w + r) * HKB + 32 * k + 8 * kg);
  const int c = tid & 7, y = y0 + (tid >> 6), x = x0 + ((tid >> 3) & 7);
  const bool in = y < d.Hin && x < d.Win;
  const size_t at = ((size_t)y * d.Win + x) * 64 + 8 * c;
  const uint4 mask = in ? *reinterpret_cast<const uint4 *>(a.x + at) : make_uint4(0, 0, 0, 0);
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int e = tid + 256 * j, p = e / CH;
    if (e < N) *reinterpret_cast<uint4 *>(patch + p * HP + 8 * (e - p * CH)) = v[j];
  }
  if (tid == 0) *reinterpret_cast<uint4 *>(patch + 60 * HP) = make_uint4(0, 0, 0, 0);
  __syncthreads();
  floatx4 acc[2];
  acc[0] = acc[1] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < HKB / 32; ++k) {
    const int q = 4 * k + kg, tap = q / CH, co = 8 * (q - tap * CH);
    const int ty = tap / 3, tx = tap - 3 * ty;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      int o = ((2 * j + (r >> 3) + 2 - ty) * 10 + (r & 7) + 2 - tx) * HP + co;
      if (tap >= 9) o = 60 * HP;  // the padding of K
      acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
          __builtin_bit_cast(bf16x8, av[k]),
          __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(patch + o)), acc[j], 0, 0, 0);
    }
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    uint16_t o[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = f2bf(acc[j][q]);
    *reinterpret_cast<uint2 *>(out + (16 * j + r) * LP + 16 * w + 4 * kg) =
        *reinterpret_cast<uint2 *>(o);
  }
  __syncthreads();
  if (!in) return;
  const uint4 o = *reinterpret_cast<const uint4 *>(out + (tid >> 3) * LP + 8 * c);
  *reinterpret_cast<uint4 *>(a.dz_prev + at) =
      make_uint4(relu_mask(o.x, mask.x), relu_mask(o.y, mask.y), relu_mask(o.z, mask.z),
                 relu_mask(o.w, mask.w));
}

// ----------------------------------------------------------- grad weight --
// dW[co][tap][ci] = sum over output pixels of dZ[pixel][co] x[tap's pixel][ci]:
// K runs over pixels, but both operands are channels-last.  They are staged in
// LDS as they lie in memory (a tile of dZ and the patch of x that its taps
// reach) and read with ds_read_b64_tr_b16, which hands each lane 4 pixels of
// one channel: 16 lanes read 4 pixels x 16 channels, every lane from an address
// of its own, so a tap is an offset into the patch.  One MFMA step covers 4
// rows x 8 pixels; lane group kg = lane >> 4 takes row kg, half h pixels 4 h ..
// 4 h + 3.  dZ outside the image is zero; a lane whose output pixel lies outside
// reads x from a zeroed part of LDS instead (0 times infinity would not be 0).
// The pitches put the 8 pixels that 32 lanes read on distinct banks.
//
// HBM and latency bound.  At 1920 x 1080 the 64-channel layers take 36 us (126
// MB with the partials; 40 us when every load tested for the border), the first
// layer 20 us (100 MB and 9 MB of partials), the sums 14 us.  As GEMMs over 64
// x 64 tiles that transposed in registers on their way to LDS, every column
// tile read dZ again and every tap its pixels of x (300 MB through L2 for the
// second layer alone): 44, 18, 12 and 13 us, the first layer 40 us, five sums
// 32 us.
typedef short short4v __attribute__((ext_vector_type(4)));
typedef short short8v __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) short4v lds_short4;
__device__ __forceinline__ bf16x8 read_tr(const uint8_t *lo, const uint8_t *hi) {
  const short4v a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4 *)lo);
  const short4v b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4 *)hi);
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}
__device__ __forceinline__ bf16x8 bf_ones() {
  return __builtin_bit_cast(bf16x8, make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u));
}

// One layer's share of the grad-weight work: splits of `per` tiles, each with
// a partial [M tile][columns + 1][64 rows] in part (the last column is the
// bias gradient: dZ times ones).
struct GwLayer {
  const uint16_t *x, *dz;
  float *part, *dw, *db;
  int Hin, Win, Hout, Wout, Cout, CoutS, Kf;
  int cols, mt, tiles_x, n_tiles, per, splits, work0;
};
struct GwArgs {
  GwLayer L[NLAYER];
  int nwork;  // work items of layers 1 .. 4
};

constexpr int GZ_PIX = 160, GZ_ROW = 8 * GZ_PIX + 128;  // dZ tile: bytes per pixel, per row

// Adds the accumulators of the waves of the second half of the workgroup's K
// range to those of the first, through LDS.
template <int N>
__device__ __forceinline__ void gw_combine(floatx4 (&acc)[N], bool second, float4 *lds, int lane,
                                           int slots) {
  __syncthreads();
  if (second) {
#pragma unroll
    for (int i = 0; i < N; ++i)
      lds[i * slots + lane] = make_float4(acc[i][0], acc[i][1], acc[i][2], acc[i][3]);
  }
  __syncthreads();
  if (!second) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const float4 v = lds[i * slots + lane];
      acc[i] += floatx4{v.x, v.y, v.z, v.w};
    }
  }
}

// Layers with 64 input channels: a workgroup of 8 waves takes 64 rows (co) x 9
// taps x 32 channels over a range of 8 x 8 pixel tiles: waves 2 (32 rows) x 2
// (16 channels) x 2 (upper and lower half of the tile).  Two LDS buffers, and
// the tile after next on its way in registers.
constexpr int GW_LDS = 73728 + 2 * 4096, GW_ZERO = 3328;  // combine buffer; zeroed part
template <int S>
__device__ __forceinline__ void gw_layer(const GwLayer &L, int work, uint8_t *lds) {
  constexpr int PW = 7 * S + 3, PIX = S == 2 ? 80 : 96, ROW = S == 2 ? 1472 : 1152;
  constexpr int BUF = PW * ROW + 8 * GZ_ROW, NX = PW * PW * 4, PER = (NX + 511) / 512;
  static_assert(2 * BUF <= GW_LDS && 2 * ROW + 2 * PIX + 64 <= GW_ZERO, "LDS");
  const int half = work & 1, mt = (work >> 1) % L.mt, split = (work >> 1) / L.mt;
  const int m0 = 64 * mt, t0 = split * L.per, t1 = min(L.n_tiles, t0 + L.per);
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int wm = w & 1, wn = (w >> 1) & 1, g = w >> 2, i16 = lane & 15, kg = lane >> 4;
  struct Stage {
    uint4 x[PER], z;
  };
  const __amdgpu_buffer_rsrc_t xs = buffer_of(L.x, (size_t)L.Hin * L.Win * 128);
  const __amdgpu_buffer_rsrc_t zs = buffer_of(L.dz, (size_t)L.Hout * L.Wout * L.CoutS * 2);
  uint32_t fx[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int e = tid + 512 * j, p = e >> 2;
    fx[j] = e < NX ? (uint32_t)(p / PW * L.Win + p % PW) * 128u + 64u * half + 16u * (e & 3)
                   : OUTSIDE;
  }
  const int zy = tid >> 6, zx = (tid >> 3) & 7;
  const uint32_t fz = m0 + 8 * (tid & 7) < L.CoutS
                          ? (uint32_t)((zy * L.Wout + zx) * L.CoutS + m0 + 8 * (tid & 7)) * 2u
                          : OUTSIDE;
  auto load = [&](Stage &v, int t) {
    const int oy0 = t / L.tiles_x * 8, ox0 = t % L.tiles_x * 8;
    const int iy0 = oy0 * S - 1, ix0 = ox0 * S - 1;
    // unsigned: the second layer's input of the largest frames passes 2^31 bytes
    const uint32_t xbase = (uint32_t)(iy0 * L.Win + ix0) * 128u;
    const uint32_t zbase = (uint32_t)(oy0 * L.Wout + ox0) * (uint32_t)L.CoutS * 2u;
    if (iy0 >= 0 && ix0 >= 0 && iy0 + PW <= L.Hin && ix0 + PW <= L.Win) {  // also within dZ
#pragma unroll
      for (int j = 0; j < PER; ++j) v.x[j] = load16(xs, fx[j], xbase);
      v.z = load16(zs, fz, zbase);
    } else {
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        const int e = tid + 512 * j, p = e >> 2, iy = iy0 + p / PW, ix = ix0 + p % PW;
        const bool in = e < NX && iy >= 0 && iy < L.Hin && ix >= 0 && ix < L.Win;
        v.x[j] = load16(xs, in ? fx[j] + xbase : OUTSIDE, 0);
      }
      const bool in = fz != OUTSIDE && oy0 + zy < L.Hout && ox0 + zx < L.Wout;
      v.z = load16(zs, in ? fz + zbase : OUTSIDE, 0);
    }
  };
  auto put = [&](const Stage &v, uint8_t *buf) {
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int e = tid + 512 * j, p = e >> 2, py = p / PW, px = p - py * PW;
      if (e < NX) *reinterpret_cast<uint4 *>(buf + py * ROW + px * PIX + 16 * (e & 3)) = v.x[j];
    }
    const int p = tid >> 3;
    *reinterpret_cast<uint4 *>(buf + PW * ROW + (p >> 3) * GZ_ROW + (p & 7) * GZ_PIX +
                               16 * (tid & 7)) = v.z;
  };
  floatx4 acc[20];  // [tap][row block], then the bias of the two row blocks
#pragma unroll
  for (int i = 0; i < 20; ++i) acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int row = 4 * g + kg, col = i16 >> 2;
  const bool bias = half == 0 && wn == 0;
  auto tile = [&](const uint8_t *buf, int t) {
    const int oy = t / L.tiles_x * 8 + row, ox = t % L.tiles_x * 8 + col;
    const uint8_t *zb = buf + PW * ROW + row * GZ_ROW + col * GZ_PIX + 64 * wm + 8 * (i16 & 3);
    const uint8_t *xb = buf + row * S * ROW + col * S * PIX, *none = lds + GW_LDS;
    const int c = 32 * wn + 8 * (i16 & 3);
    const uint8_t *x0 = (oy < L.Hout && ox < L.Wout ? xb : none) + c;
    const uint8_t *x1 = (oy < L.Hout && ox + 4 < L.Wout ? xb + 4 * S * PIX : none) + c;
    bf16x8 av[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) av[i] = read_tr(zb + 32 * i, zb + 32 * i + 4 * GZ_PIX);
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      const int o = tap / 3 * ROW + tap % 3 * PIX;
      const bf16x8 bv = read_tr(x0 + o, x1 + o);
#pragma unroll
      for (int i = 0; i < 2; ++i)
        acc[2 * tap + i] =
            __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[i], bv, acc[2 * tap + i], 0, 0, 0);
    }
    if (bias)
#pragma unroll
      for (int i = 0; i < 2; ++i)
        acc[18 + i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[i], bf_ones(), acc[18 + i], 0, 0, 0);
  };
  uint8_t *b0 = lds, *b1 = lds + BUF;
  for (int e = tid; e < GW_ZERO / 4; e += 512) reinterpret_cast<uint32_t *>(lds + GW_LDS)[e] = 0;
  Stage va, vb;
  load(va, t0);
  if (t0 + 1 < t1) load(vb, t0 + 1);
  put(va, b0);
  __syncthreads();
  // a buffer is written between the barrier after its last read and the one
  // before its next
  for (int t = t0; t < t1; t += 2) {
    if (t + 2 < t1) load(va, t + 2);
    tile(b0, t);
    if (t + 1 >= t1) break;
    put(vb, b1);
    __syncthreads();
    if (t + 3 < t1) load(vb, t + 3);
    tile(b1, t + 1);
    if (t + 2 >= t1) break;
    put(va, b0);
    __syncthreads();
  }
  gw_combine(acc, g == 1, reinterpret_cast<float4 *>(lds), tid & 255, 256);
  if (g == 1) return;
  float *part = L.part + ((size_t)split * L.mt + mt) * (L.cols + 1) * 64 + 32 * wm + 4 * kg;
#pragma unroll
  for (int tap = 0; tap < 9; ++tap)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const floatx4 &v = acc[2 * tap + i];
      *reinterpret_cast<float4 *>(part + (64 * tap + 32 * half + 16 * wn + i16) * 64 + 16 * i) =
          make_float4(v[0], v[1], v[2], v[3]);
    }
  if (bias && i16 == 0)
#pragma unroll
    for (int i = 0; i < 2; ++i)
      *reinterpret_cast<float4 *>(part + L.cols * 64 + 16 * i) =
          make_float4(acc[18 + i][0], acc[18 + i][1], acc[18 + i][2], acc[18 + i][3]);
}

// Layers 1 .. 4 in one launch of at most 256 workgroups, one per compute unit,
// of equally many tiles each: a layer alone leaves most units idle (the fourth
// has 135 tiles at 1920 x 1080), and fewer splits mean fewer partials (18 MB).
// The grid is ordered so that the two channel halves of a range of tiles run at
// the same time on one XCD (workgroup b is on XCD b % 8) and share dZ and the
// 128-byte pixels in its L2.
__global__ void __launch_bounds__(512, 2) k_conv_bwd_weight(GwArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[GW_LDS + GW_ZERO];
  const int per_xcd = (int)(gridDim.x >> 3);
  const int work = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
  if (work >= a.nwork) return;
  int l = 1;
  while (l + 1 < NLAYER && work >= a.L[l + 1].work0) ++l;
  if (l == NLAYER - 1) gw_layer<1>(a.L[NLAYER - 1], work - a.L[NLAYER - 1].work0, lds);
  else gw_layer<2>(a.L[l], work - a.L[l].work0, lds);
}

// First layer (8 input channels): 64 rows x 72 columns (tap, ci) over a range
// of 8 x 16 pixel tiles; 16 columns are two taps, which a lane selects by the
// address it reads.  4 waves: 2 (32 rows) x 2 (upper and lower half).
constexpr int G0_ROW = 320, G0_X = 33 * G0_ROW, G0_BUF = G0_X + 16 * GZ_ROW, G0_ZERO = 768;
__global__ void __launch_bounds__(256, 2) k_conv_bwd_weight_first(GwLayer L) {
  __shared__ __attribute__((aligned(16))) uint8_t lds[G0_BUF + G0_ZERO];
  constexpr int NX = 33 * 17, PER = (NX + 255) / 256;
  static_assert(2 * G0_ROW + 2 * 16 + 32 <= G0_ZERO && 12 * 2048 <= G0_BUF, "LDS");
  const int t0 = blockIdx.x * L.per, t1 = min(L.n_tiles, t0 + L.per);
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int wm = w & 1, g = w >> 1, i16 = lane & 15, kg = lane >> 4;
  uint4 vx[PER], vz[4];
  auto load = [&](int t) {
    const int oy0 = t / L.tiles_x * 16, ox0 = t % L.tiles_x * 8;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int e = tid + 256 * j, py = e / 17, px = e - py * 17;
      const int iy = oy0 * 2 - 1 + py, ix = ox0 * 2 - 1 + px;
      vx[j] = make_uint4(0, 0, 0, 0);
      if (e < NX && iy >= 0 && iy < L.Hin && ix >= 0 && ix < L.Win)
        vx[j] = *reinterpret_cast<const uint4 *>(L.x + ((size_t)iy * L.Win + ix) * 8);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int p = (tid >> 3) + 32 * j, oy = oy0 + (p >> 3), ox = ox0 + (p & 7);
      vz[j] = make_uint4(0, 0, 0, 0);
      if (oy < L.Hout && ox < L.Wout)
        vz[j] = *reinterpret_cast<const uint4 *>(L.dz + ((size_t)oy * L.Wout + ox) * 64 + 8 * (tid & 7));
    }
  };
  floatx4 acc[12];  // [column block][row block], then the bias
#pragma unroll
  for (int i = 0; i < 12; ++i) acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};
  int off[5];
#pragma unroll
  for (int n = 0; n < 5; ++n) {
    const int tap = min(8, 2 * n + ((i16 >> 1) & 1));
    off[n] = tap / 3 * G0_ROW + tap % 3 * 16 + 8 * (i16 & 1);
  }
  for (int e = tid; e < G0_ZERO / 4; e += 256) reinterpret_cast<uint32_t *>(lds + G0_BUF)[e] = 0;
  load(t0);
  for (int t = t0; t < t1; ++t) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int e = tid + 256 * j, py = e / 17, px = e - py * 17;
      if (e < NX) *reinterpret_cast<uint4 *>(lds + py * G0_ROW + px * 16) = vx[j];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int p = (tid >> 3) + 32 * j;
      *reinterpret_cast<uint4 *>(lds + G0_X + (p >> 3) * GZ_ROW + (p & 7) * GZ_PIX + 16 * (tid & 7)) =
          vz[j];
    }
    __syncthreads();
    if (t + 1 < t1) load(t + 1);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int row = 8 * g + 4 * s + kg, col = i16 >> 2;
      const int oy = t / L.tiles_x * 16 + row, ox = t % L.tiles_x * 8 + col;
      const uint8_t *zb = lds + G0_X + row * GZ_ROW + col * GZ_PIX + 64 * wm + 8 * (i16 & 3);
      const uint8_t *xb = lds + row * 2 * G0_ROW + col * 32, *none = lds + G0_BUF;
      const uint8_t *x0 = oy < L.Hout && ox < L.Wout ? xb : none;
      const uint8_t *x1 = oy < L.Hout && ox + 4 < L.Wout ? xb + 128 : none;
      bf16x8 av[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) av[i] = read_tr(zb + 32 * i, zb + 32 * i + 4 * GZ_PIX);
#pragma unroll
      for (int n = 0; n < 5; ++n) {
        const bf16x8 bv = read_tr(x0 + off[n], x1 + off[n]);
#pragma unroll
        for (int i = 0; i < 2; ++i)
          acc[2 * n + i] =
              __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[i], bv, acc[2 * n + i], 0, 0, 0);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
        acc[10 + i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[i], bf_ones(), acc[10 + i], 0, 0, 0);
    }
  }
  gw_combine(acc, g == 1, reinterpret_cast<float4 *>(lds), tid & 127, 128);
  if (g == 1) return;
  float *part = L.part + (size_t)blockIdx.x * 73 * 64 + 32 * wm + 4 * kg;
#pragma unroll
  for (int n = 0; n < 6; ++n) {
    const int c = 16 * n + i16;  // block 5 is the bias: its columns are equal
    if (n < 5 ? c < 72 : i16 == 0)
#pragma unroll
      for (int i = 0; i < 2; ++i)
        *reinterpret_cast<float4 *>(part + min(c, 72) * 64 + 16 * i) =
            make_float4(acc[2 * n + i][0], acc[2 * n + i][1], acc[2 * n + i][2], acc[2 * n + i][3]);
  }
}

// The losses from the tiles': out = total, cross entropy, Chamfer.
struct LossSum {
  int n_tiles;
  const float *tile_loss;
  const int *n_cd;
  float *out;
};
__device__ __forceinline__ void sum_losses(const LossSum &L) {
  __shared__ double red[2][4];
  double ce = 0.0, cd = 0.0;
  // 16 loads in flight: the launch waits for this one workgroup
  for (int t0 = threadIdx.x; t0 < L.n_tiles; t0 += 16 * 256) {
    float2 v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j)
      v[j] = *reinterpret_cast<const float2 *>(L.tile_loss +
                                               2 * min(t0 + 256 * j, L.n_tiles - 1));
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const bool in = t0 + 256 * j < L.n_tiles;
      ce += in ? v[j].x : 0.f;
      cd += in ? v[j].y : 0.f;
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    ce += __shfl_xor(ce, o, 64);
    cd += __shfl_xor(cd, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = ce;
    red[1][threadIdx.x >> 6] = cd;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const double c1 = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
    const double c2 = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
    const int n_cd = *L.n_cd;
    L.out[0] = (float)(c1 / L.n_tiles + (n_cd > 0 ? c2 / n_cd : 0.0));
    L.out[1] = (float)(c1 / L.n_tiles);
    L.out[2] = (float)(n_cd > 0 ? c2 / n_cd : 0.0);
  }
}

// Sum of the partials over the splits, added into dW and dbias: one workgroup
// per column (64 rows) of every layer, four lanes' worth of splits each.  The
// first workgroup sums the losses: as a launch of its own that took 4 us of a
// 247 us training step at 1920 x 1080 and 11 of 753 at 3840 x 2160.
__global__ void __launch_bounds__(256) k_gw_reduce(GwArgs a, LossSum loss) {
  __shared__ float red[256];
  if (blockIdx.x == 0) {
    if (loss.out) sum_losses(loss);
    return;
  }
  int b = blockIdx.x - 1, l = 0;
  while (b >= a.L[l].mt * (a.L[l].cols + 1)) b -= a.L[l].mt * (a.L[l].cols + 1), ++l;
  const GwLayer &L = a.L[l];
  const int tid = threadIdx.x, mt = b / (L.cols + 1), c = b - mt * (L.cols + 1);
  const size_t stride = (size_t)L.mt * (L.cols + 1) * 64;
  const float *src = L.part + (size_t)b * 64 + (tid & 63);
  float sum = 0.f;
#pragma unroll 8
  for (int s = tid >> 6; s < L.splits; s += 4) sum += src[s * stride];
  red[tid] = sum;
  __syncthreads();
  const int r = 64 * mt + tid;
  if (tid >= 64 || r >= L.Cout) return;
  sum = (red[tid] + red[tid + 64]) + (red[tid + 128] + red[tid + 192]);
  if (sum != 0.f) atomicAdd(c < L.cols ? &L.dw[(size_t)r * L.Kf + c] : &L.db[r], sum);
}

__device__ inline float sigm(float z) { return 1.f / (1.f + __expf(-z)); }

// x of lane N of this lane's row of 16; sum and largest over the row.
template <int CTRL>
__device__ __forceinline__ float row_dpp(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, true));
}
template <int N>
__device__ __forceinline__ float row_lane(float x) {
  return row_dpp<0x150 + N>(x);
}
// quad_perm [1,0,3,2] and [2,3,0,1], row_half_mirror, row_ror:8
__device__ __forceinline__ float row_sum(float x) {
  x += row_dpp<0xB1>(x);
  x += row_dpp<0x4E>(x);
  x += row_dpp<0x141>(x);
  return x + row_dpp<0x128>(x);
}
__device__ __forceinline__ float row_max(float x) {
  x = fmaxf(x, row_dpp<0xB1>(x));
  x = fmaxf(x, row_dpp<0x4E>(x));
  x = fmaxf(x, row_dpp<0x141>(x));
  return fmaxf(x, row_dpp<0x128>(x));
}

// Prediction s -> nearest target (first minimum), targets N and on.
template <int N>
__device__ __forceinline__ void nearest_target(const float (&Pv)[NPAR], const float (&Qv)[NPAR],
                                               int k, float &bd, float (&Qb)[NPAR]) {
  float Qq[NPAR], dd = 0.f;
#pragma unroll
  for (int j = 0; j < NPAR; ++j) {
    Qq[j] = row_lane<N>(Qv[j]);
    dd += (Pv[j] - Qq[j]) * (Pv[j] - Qq[j]);
  }
  if (N < k && dd < bd) {
    bd = dd;
#pragma unroll
    for (int j = 0; j < NPAR; ++j) Qb[j] = Qq[j];
  }
  if constexpr (N + 1 < NSLOT) nearest_target<N + 1>(Pv, Qv, k, bd, Qb);
}
// Target s -> nearest prediction (first minimum).
template <int N>
__device__ __forceinline__ void nearest_prediction(const float (&Pv)[NPAR],
                                                   const float (&Qv)[NPAR], int k, float &bd,
                                                   int &best) {
  float dd = 0.f;
#pragma unroll
  for (int j = 0; j < NPAR; ++j) {
    const float Ps = row_lane<N>(Pv[j]);
    dd += (Ps - Qv[j]) * (Ps - Qv[j]);
  }
  if (N < k && dd < bd) bd = dd, best = N;
  if constexpr (N + 1 < NSLOT) nearest_prediction<N + 1>(Pv, Qv, k, bd, best);
}
// Adds the targets whose nearest prediction is s to its gradient.
template <int N>
__device__ __forceinline__ void pull_targets(const float (&Pv)[NPAR], const float (&Qv)[NPAR],
                                             int k, int s, int best, float inv_k,
                                             float (&gp)[NPAR]) {
  const int b = __float_as_int(row_lane<N>(__int_as_float(best)));
#pragma unroll
  for (int j = 0; j < NPAR; ++j) {
    const float Qq = row_lane<N>(Qv[j]);
    if (N < k && b == s) gp[j] += 2.f * (Pv[j] - Qq) * inv_k;
  }
  if constexpr (N + 1 < NSLOT) pull_targets<N + 1>(Pv, Qv, k, s, best, inv_k, gp);
}

// Per-tile loss: CE over the 9 count logits + Chamfer between the first k
// slots and the k targets (8-vectors).  16 lanes per tile: lane c < 9 holds
// count logit c, lane s < 8 holds prediction slot s and target s.  The head
// gradient goes out as dZ of the head (BF16 [n_tiles][CoutS]); per-tile loss
// sums to tile_loss (CE, CD).  The 16 lanes are a DPP row, so a value of lane n
// reaches the others as a register move (as LDS permutes, 200 of them per tile,
// the launch took 7.7 us at 1920 x 1080; 5.4 to 6.1 with moves).
__global__ void __launch_bounds__(256)
k_head_loss(int n_tiles, int CoutS, const float *__restrict__ head, const int *__restrict__ tcount,
            const float *__restrict__ tvec, const int *__restrict__ n_cd_dev,
            uint16_t *__restrict__ dz, float *__restrict__ tile_loss) {
  const int gid = blockIdx.x * blockDim.x + threadIdx.x;
  const int t = gid >> 4, l = gid & 15, base = threadIdx.x & 48;  // group's first lane in the wave
  const bool live = t < n_tiles;
  const int tt = live ? t : 0;
  const float inv_tiles = 1.f / (float)n_tiles;
  const int n_cd = max(1, *n_cd_dev);
  const int k = min(max(tcount[tt], 0), NSLOT);
  // cross entropy of the count logits
  const float z = (l < 9) ? head[(size_t)l * n_tiles + tt] : -INFINITY;
  const float mx = row_max(z);
  const float se = row_sum((l < 9) ? __expf(z - mx) : 0.f);
  const float lse = mx + __logf(se);
  const float zk = __shfl(z, base + k, 64);
  const float ce = lse - zk;
  const float gce = (l < 9) ? (__expf(z - lse) - (l == k ? 1.f : 0.f)) * inv_tiles : 0.f;
  // Chamfer: predictions P (sigmoid on the two offsets), targets Q
  const int s = l & 7;
  float Pv[NPAR], Qv[NPAR], raw[2];
#pragma unroll
  for (int j = 0; j < NPAR; ++j) {
    const float r = head[(size_t)(9 + s * NPAR + j) * n_tiles + tt];
    if (j < 2) raw[j] = r;
    Pv[j] = (j < 2) ? sigm(r) : r;
    Qv[j] = tvec[((size_t)tt * NSLOT + s) * NPAR + j];
  }
  const float inv_k = k > 0 ? 1.f / (float)k : 0.f;
  // prediction s -> nearest target (first minimum)
  float bd = INFINITY, Qb[NPAR];
#pragma unroll
  for (int j = 0; j < NPAR; ++j) Qb[j] = 0.f;
  nearest_target<0>(Pv, Qv, k, bd, Qb);
  // target s -> nearest prediction (first minimum)
  float bd2 = INFINITY;
  int best2 = 0;
  nearest_prediction<0>(Pv, Qv, k, bd2, best2);
  const bool own = l < 8 && s < k;
  const float cd = row_sum(own ? (bd + bd2) * inv_k : 0.f);
  float gp[NPAR];
#pragma unroll
  for (int j = 0; j < NPAR; ++j) gp[j] = 2.f * (Pv[j] - Qb[j]) * inv_k;
  pull_targets<0>(Pv, Qv, k, s, best2, inv_k, gp);
  if (!live) return;
  uint16_t *out = dz + (size_t)t * CoutS;
  if (l < 9) out[l] = f2bf(gce);
  if (l < 8) {
    const float sc = 1.f / (float)n_cd;
#pragma unroll
    for (int j = 0; j < NPAR; ++j) {
      float v = own ? gp[j] * sc : 0.f;
      if (j < 2) {
        const float sg = sigm(raw[j]);
        v *= sg * (1.f - sg);
      }
      out[9 + s * NPAR + j] = f2bf(v);
    }
  }
  if (l == 15)
    for (int c = HEAD_CH; c < CoutS; ++c) out[c] = 0;
  if (l == 0) {
    tile_loss[2 * t] = ce;
    tile_loss[2 * t + 1] = cd;
  }
}

}  // namespace

// ------------------------------------------------------------ layout ----
struct CnnLayout {
  int H, W;
  ConvDims L[NLAYER];
  size_t w_off[NLAYER], b_off[NLAYER], n_params;   // FP32 master / grad offsets (floats)
  size_t wb_off[NLAYER], n_wb;                    // bf16 weight offsets (elements)
  size_t wt_off[NLAYER], n_wt;                    // bf16 transposed weights (elements)
  // workspace (bytes)
  size_t x_in, act[NLAYER], head, dz[NLAYER], gpart[NLAYER], tcount, tvec, tile_loss, ncd, total;
  int TX, TY, n_tiles;
  GwArgs gw;  // the grad-weight plan (no pointers)
};

// Grad-weight plan.  Layers 1 .. 4: the fewest tiles per workgroup that give at
// most 256 workgroups (what is resident at once).  Layer 0: GW0_WGS workgroups.
constexpr int GW_WGS = 256, GW0_WGS = 512;
static void gw_plan(const ConvDims *D, GwArgs *A) {
  long long units = 0;
  for (int i = 0; i < NLAYER; ++i) {
    GwLayer &L = A->L[i];
    const ConvDims &d = D[i];
    L = {};
    L.Hin = d.Hin;
    L.Win = d.Win;
    L.Hout = d.Hout;
    L.Wout = d.Wout;
    L.Cout = d.Cout;
    L.CoutS = d.CoutS;
    L.Kf = d.Kf;
    L.cols = 9 * d.Cin;
    L.mt = d.Mpad / 64;
    L.tiles_x = (d.Wout + 7) / 8;
    L.n_tiles = L.tiles_x * (i == 0 ? (d.Hout + 15) / 16 : (d.Hout + 7) / 8);
    if (i > 0) units += 2LL * L.mt * L.n_tiles;
  }
  GwLayer &F = A->L[0];
  F.per = (F.n_tiles + GW0_WGS - 1) / GW0_WGS;
  F.splits = (F.n_tiles + F.per - 1) / F.per;
  for (int per = (int)((units + GW_WGS - 1) / GW_WGS);; ++per) {
    A->nwork = 0;
    for (int i = 1; i < NLAYER; ++i) {
      GwLayer &L = A->L[i];
      L.per = per;
      L.splits = (L.n_tiles + per - 1) / per;
      L.work0 = A->nwork;
      A->nwork += 2 * L.mt * L.splits;
    }
    // a single tile per layer makes 10 work items, so this ends
    if (A->nwork <= GW_WGS) return;
  }
}

static size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

static bool cnn_layout(int H, int W, CnnLayout *C) {
  if (H < 16 || W < 16 || (long long)H * W > (1LL << 26)) return false;
  C->H = H;
  C->W = W;
  int h = H, w = W, cin = 8;
  size_t pw = 0, wb = 0, wt = 0;
  for (int i = 0; i < NLAYER; ++i) {
    ConvDims &d = C->L[i];
    const bool head = (i == NLAYER - 1);
    d.Hin = h;
    d.Win = w;
    d.Cin = cin;
    d.stride = head ? 1 : 2;
    d.Hout = (h + 2 - 3) / d.stride + 1;
    d.Wout = (w + 2 - 3) / d.stride + 1;
    d.Cout = head ? HEAD_CH : 64;
    d.relu = head ? 0 : 1;
    d.Mpad = (d.Cout + 63) / 64 * 64;
    d.Kf = (9 * d.Cin + KPAD - 1) / KPAD * KPAD;
    d.CoutS = (d.Cout + 7) / 8 * 8;
    d.Kb = (9 * d.CoutS + KPAD - 1) / KPAD * KPAD;
    C->w_off[i] = pw;
    pw += (size_t)d.Mpad * d.Kf;
    C->b_off[i] = pw;
    pw += d.Mpad;
    C->wb_off[i] = wb;
    wb += (size_t)d.Mpad * d.Kf;
    C->wt_off[i] = wt;
    wt += (size_t)d.Cin * d.Kb;
    h = d.Hout;
    w = d.Wout;
    cin = d.Cout;
  }
  C->n_params = pw;
  C->n_wb = wb;
  C->n_wt = wt;
  const ConvDims &hd = C->L[NLAYER - 1];
  C->TX = hd.Wout;
  C->TY = hd.Hout;
  C->n_tiles = C->TX * C->TY;
  size_t o = 0;
  auto take = [&o](size_t b) {
    const size_t at = o;
    o = al256(o + b);
    return at;
  };
  C->x_in = take((size_t)H * W * 8 * 2);
  for (int i = 0; i < NLAYER; ++i) {
    const ConvDims &d = C->L[i];
    C->act[i] = (i < NLAYER - 1) ? take((size_t)d.Hout * d.Wout * d.Cout * 2) : 0;
  }
  C->head = take((size_t)HEAD_CH * C->n_tiles * 4);
  gw_plan(C->L, &C->gw);
  for (int i = 0; i < NLAYER; ++i) {  // dZ of every layer's output, BF16
    const ConvDims &d = C->L[i];
    C->dz[i] = take((size_t)d.Hout * d.Wout * d.CoutS * 2);
    const GwLayer &g = C->gw.L[i];
    C->gpart[i] = take((size_t)g.splits * g.mt * (g.cols + 1) * 64 * 4);
  }
  C->tcount = take((size_t)C->n_tiles * 4);
  C->tvec = take((size_t)C->n_tiles * NSLOT * NPAR * 4);
  C->tile_loss = take((size_t)C->n_tiles * 2 * 4);
  C->ncd = take(64);
  C->total = o;
  return true;
}

// Workgroups for n tiles in eighths (xcd_tile).
static unsigned xcd_grid(int n) { return (unsigned)((n + 7) / 8 * 8); }

// 512 workgroups of k_conv_fwd are resident (two per compute unit), shared by
// the M tiles.
static hipError_t launch_conv_fwd(const ConvArgs &a, hipStream_t st) {
  const ConvDims &d = a.d;
  const int tx = (d.Wout + CT - 1) / CT, n = tx * ((d.Hout + CT - 1) / CT), mt = d.Mpad / 64;
  const dim3 g((unsigned)std::min(n, 512 / mt), (unsigned)mt);
  if (d.stride == 2) hipLaunchKernelGGL(k_conv_fwd<2>, g, dim3(256), 0, st, a, tx, n);
  else hipLaunchKernelGGL(k_conv_fwd<1>, g, dim3(256), 0, st, a, tx, n);
  return hipGetLastError();
}

// Grad input: as many resident workgroups walk over the tiles as in the forward
// pass; the head has one tile per workgroup.
static hipError_t launch_conv_bwd_data(const ConvArgs &a, hipStream_t st) {
  const ConvDims &d = a.d;
  const int tx = (d.Wout + 7) / 8;
  if (d.stride == 2) {
    const int n = tx * ((d.Hout + 7) / 8);
    hipLaunchKernelGGL(k_conv_bwd_data, dim3((unsigned)std::min(n, 512)), dim3(256), 0, st, a, tx, n);
  } else {
    hipLaunchKernelGGL(k_conv_bwd_data_head, dim3((unsigned)(tx * ((d.Hout + 3) / 4))), dim3(256), 0,
                       st, a, tx);
  }
  return hipGetLastError();
}

// ---------------------------------------------- weight conversion / Adam --
// Master FP32 weights -> BF16 copies in forward layout and, for the layers
// whose input gradient is needed, the transposed layout W^T[ci][tap][co].
__global__ void __launch_bounds__(256)
k_cnn_weights_to_bf16(ConvDims d, const float *__restrict__ wm, uint16_t *__restrict__ wb,
                      uint16_t *__restrict__ wt) {
  const size_t n = (size_t)d.Mpad * d.Kf;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x) {
    const int co = (int)(i / d.Kf), k = (int)(i % d.Kf);
    const uint16_t b = f2bf(wm[i]);
    wb[i] = b;
    if (wt && co < d.Cout && k < 9 * d.Cin) {
      const int tap = k / d.Cin, ci = k % d.Cin;
      wt[(size_t)ci * d.Kb + tap * d.CoutS + co] = b;
    }
  }
}

// Where each layer's parameters live: FP32 master / gradient offsets
// (weights [Mpad][Kf] then bias [Mpad]) and the BF16 copies.
struct CnnParamMap {
  ConvDims d[NLAYER];
  long long w_off[NLAYER], b_off[NLAYER], wb_off[NLAYER], wt_off[NLAYER];
};

// Adam with decoupled weight decay on the FP32 master weights; each updated
// weight is written to its BF16 copies in the same pass (forward layout, and
// for the layers whose input gradient is needed the transposed one, whose
// padding keeps the zeros of the last full conversion).
__global__ void __launch_bounds__(256)
k_cnn_adam(size_t n, CnnParamMap map, float *__restrict__ p, float *__restrict__ g,
           float *__restrict__ m, float *__restrict__ v, const int32_t *__restrict__ step,
           float lr, float b1, float b2, float eps, float wd, uint16_t *__restrict__ wb,
           uint16_t *__restrict__ wt) {
  float bc1, bc2;
  adam_bias(step[0], b1, b2, &bc1, &bc2);
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x) {
    const float gr = g[i], p0 = p[i];
    g[i] = 0.f;
    const float mm = b1 * m[i] + (1.f - b1) * gr;
    const float vv = b2 * v[i] + (1.f - b2) * gr * gr;
    m[i] = mm;
    v[i] = vv;
    // the decay acts on the weight itself, outside the adaptive scaling
    const float pn = p0 - lr * ((mm / bc1) / (sqrtf(vv / bc2) + eps) + wd * p0);
    p[i] = pn;
    int l = 0;
#pragma unroll
    for (int j = 1; j < NLAYER; ++j)
      if ((long long)i >= map.w_off[j]) l = j;
    if ((long long)i >= map.b_off[l]) continue;  // a bias
    const ConvDims &d = map.d[l];
    const long long e = (long long)i - map.w_off[l];
    const int co = (int)(e / d.Kf), k = (int)(e - (long long)co * d.Kf);
    const uint16_t b = f2bf(pn);
    wb[map.wb_off[l] + e] = b;
    if (l > 0 && co < d.Cout && k < 9 * d.Cin) {
      const int tap = k / d.Cin, ci = k - tap * d.Cin;
      wt[map.wt_off[l] + (long long)ci * d.Kb + tap * d.CoutS + co] = b;
    }
  }
}

// ------------------------------------------------------------- decode ----
// Sum of one int per thread over a block of 256 threads, in every thread.
__device__ inline int block_sum_256(int v, int *red /* [4] */) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  __syncthreads();  // red may still be read from an earlier call
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

// Inclusive prefix sum of one int per thread over a block of 256 threads.
__device__ inline int block_scan_256(int v, int *red /* [4] */) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(v, o, 64);
    if (lane >= o) v += u;
  }
  __syncthreads();
  if (lane == 63) red[w] = v;
  __syncthreads();
  for (int k = 0; k < w; ++k) v += red[k];
  return v;
}

// Per tile: k = argmax of the count logits (first maximum), slots 0..k-1 ->
// Gaussians.  counts[t] = k and bsum[b] = their sum over block b's 256 tiles;
// the write kernel's blocks add up the sums before them, so that the
// Gaussians are placed in tile order without a scan of its own (12 us of one
// block at 8160 tiles).
__global__ void __launch_bounds__(256)
k_decode_counts(int n_tiles, const float *__restrict__ head, int *__restrict__ counts,
                int *__restrict__ bsum, int *__restrict__ flags) {
  __shared__ int red[4];
  const int t = blockIdx.x * 256 + threadIdx.x;
  int best = 0;
  if (t < n_tiles) {
    float bv = head[t];
    for (int c = 1; c < 9; ++c) {
      const float z = head[(size_t)c * n_tiles + t];
      if (z > bv) bv = z, best = c;
    }
    counts[t] = best;
  }
  const int sum = block_sum_256(best, red);
  if (threadIdx.x == 0) {
    bsum[blockIdx.x] = sum;
    if (blockIdx.x == 0) flags[0] = 0;
  }
}

// Slot s of tile t (column tx, row ty) of the head [73][n_tiles] as a
// Gaussian: mu = tile origin + T sigmoid(p0, p1), l1 = exp(clamp(p2, +-4)),
// l2 = p3, l3 = exp(clamp(p4, +-4)), colour (p5, p6, p7); returns whether
// the eight raw parameters are finite.
__device__ inline bool decode_slot(const float *__restrict__ head, int n_tiles, int t, int s,
                                   int tx, int ty, int T, float *__restrict__ xy,
                                   float *__restrict__ chol, float *__restrict__ rgb) {
  float p[NPAR];
  bool ok = true;
  for (int j = 0; j < NPAR; ++j) {
    p[j] = head[(size_t)(9 + s * NPAR + j) * n_tiles + t];
    ok = ok && isfinite(p[j]);
  }
  xy[0] = (float)(tx * T) + (float)T * sigm(p[0]);
  xy[1] = (float)(ty * T) + (float)T * sigm(p[1]);
  chol[0] = __expf(fminf(fmaxf(p[2], -4.f), 4.f));
  chol[1] = p[3];
  chol[2] = __expf(fminf(fmaxf(p[4], -4.f), 4.f));
  rgb[0] = p[5];
  rgb[1] = p[6];
  rgb[2] = p[7];
  return ok;
}

// Eight threads per tile, one per slot; 32 tiles per block.  flags = {a
// non-finite value was written, predicted Gaussians}.
constexpr int DECODE_TILES = 256 / NSLOT;
__global__ void __launch_bounds__(256)
k_decode_write(int n_tiles, int TX, int T, const float *__restrict__ head,
               const int *__restrict__ counts, const int *__restrict__ bsum, int N_out,
               float *__restrict__ xy, float *__restrict__ chol, float *__restrict__ rgb,
               int *__restrict__ flags) {
  __shared__ int red[4];
  const int t0 = blockIdx.x * DECODE_TILES, t1 = min(n_tiles, t0 + DECODE_TILES);
  // Gaussians of the tiles before the block
  int v = 0;
  for (int i = threadIdx.x; i < t0 / 256; i += 256) v += bsum[i];
  const int part = t0 / 256 * 256 + (int)threadIdx.x;
  if (part < t0) v += counts[part];
  const int before = block_sum_256(v, red);
  const int t = t0 + (int)threadIdx.x / NSLOT, s = threadIdx.x % NSLOT;
  const int k = t < n_tiles ? counts[t] : 0;
  const int incl = block_scan_256(s == 0 ? k : 0, red);  // of this tile, at its first thread
  const int o = before + __shfl(incl, (threadIdx.x & 63) & ~(NSLOT - 1), 64) - k;
  if (t == t1 - 1 && s == 0 && t1 == n_tiles) flags[1] = o + k;
  const int n = o + s;
  if (s >= k || n >= N_out) return;
  decode_slot(head, n_tiles, t, s, t % TX, t / TX, T, xy + 2 * n, chol + 3 * n, rgb + 3 * n);
  bool ok = isfinite(xy[2 * n]) && isfinite(xy[2 * n + 1]) && isfinite(chol[3 * n + 1]);
  for (int j = 0; j < 3; ++j) ok = ok && isfinite(rgb[3 * n + j]);
  if (!ok) atomicOr(flags, 1);
}

// Fill slots [n_pred, N) of the output from the plain initialisation, or
// everything when the prediction is unusable (non-finite, or fewer than
// half of N Gaussians).
__global__ void __launch_bounds__(256)
k_decode_merge(int N, const int *__restrict__ flags,
               const float *__restrict__ pxy, const float *__restrict__ pchol,
               const float *__restrict__ prgb, float *__restrict__ xy, float *__restrict__ chol,
               float *__restrict__ rgb, int *__restrict__ used_pred) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  const int np = min(flags[1], N);
  const bool fallback = (flags[0] != 0) || (2 * np < N);
  if (n == 0) *used_pred = fallback ? 0 : np;
  if (n >= N) return;
  if (!fallback && n < np) return;
  const int src = fallback ? n : n - np;
  xy[2 * n] = pxy[2 * src];
  xy[2 * n + 1] = pxy[2 * src + 1];
  for (int j = 0; j < 3; ++j) {
    chol[3 * n + j] = pchol[3 * src + j];
    rgb[3 * n + j] = prgb[3 * src + j];
  }
}

// ------------------------------------------- P-frame re-initialisation ----
// Tiles of a P-frame whose mean squared residual against the previous frame
// exceeds tau are re-initialised from the network's predictions.
//
// k_pf_tiles: a block takes 16 tiles of one tile row, one pixel column per
// thread, so that the frames are read in whole lines; the per-pixel energies
// e = (dr*dr + dg*dg) + db*db wait in LDS for one lane per tile that adds the
// tile's in-frame pixels one at a time in row-major order and divides by
// their count (FP32, each operation rounded once: the selection is a
// decision; the zeros added for pixels outside the frame change nothing).  A
// selected tile's prediction count is the argmax of its count logits (first
// maximum); blk = {tiles selected, predictions, a raw parameter of a used
// slot is not finite}.  The block is bound by that chain of 256 additions
// (one thread per tile reading its pixels from memory in that order took 187
// us at 1920 x 1080).
constexpr int PF_TILES = 16, PF_T = 16;
__global__ void __launch_bounds__(256)
k_pf_tiles(int H, int W, int TX, int n_tiles, const float *__restrict__ frame,
           const float *__restrict__ prev, float tau, const float *__restrict__ head,
           uint8_t *__restrict__ sel, int *__restrict__ pcount, int4 *__restrict__ blk) {
  constexpr int PITCH = PF_T * PF_T + 1;
  __shared__ float e[PF_TILES * PITCH];
  __shared__ int cnt[PF_TILES], on_s[PF_TILES];
  const int tid = threadIdx.x, ty = blockIdx.y, tx0 = blockIdx.x * PF_TILES;
  const size_t HW = (size_t)H * W;
  const int x = tx0 * PF_T + tid, y0 = ty * PF_T;
  float *mine = e + (tid >> 4) * PITCH + (tid & 15);
#pragma unroll 4
  for (int r = 0; r < PF_T; ++r) {
    float v = 0.f;
    if (x < W && y0 + r < H) {
      const size_t p = (size_t)(y0 + r) * W + x;
      const float dr = f32_sub(frame[p], prev[p]);
      const float dg = f32_sub(frame[HW + p], prev[HW + p]);
      const float db = f32_sub(frame[2 * HW + p], prev[2 * HW + p]);
      v = f32_add(f32_add(f32_mul(dr, dr), f32_mul(dg, dg)), f32_mul(db, db));
    }
    mine[r * PF_T] = v;
  }
  __syncthreads();
  int on = 0, k = 0;
  const int tx = tx0 + tid, t = ty * TX + tx;
  if (tid < PF_TILES) {
    if (tx < TX) {
      float acc = 0.f;
#pragma unroll 16
      for (int i = 0; i < PF_T * PF_T; ++i) acc = f32_add(acc, e[tid * PITCH + i]);
      const int w = min(PF_T, W - tx * PF_T), h = min(PF_T, H - y0);
      on = __fdiv_rn(acc, (float)(w * h)) > tau ? 1 : 0;
      if (on) {
        float bv = head[t];
#pragma unroll
        for (int c = 1; c < 9; ++c) {
          const float z = head[(size_t)c * n_tiles + t];
          if (z > bv) bv = z, k = c;
        }
      }
      sel[t] = (uint8_t)on;
      pcount[t] = k;
    }
    cnt[tid] = k;
    on_s[tid] = on;
  }
  __syncthreads();
  // the used slots' raw parameters: 16 threads per tile
  const int ft = tid & (PF_TILES - 1), fk = cnt[ft];
  bool ok = true;
  for (int i = tid / PF_TILES; i < fk * NPAR; i += 256 / PF_TILES)
    ok = ok && isfinite(head[(size_t)(9 + i) * n_tiles + ty * TX + tx0 + ft]);
  const int bad = __syncthreads_or(!ok);
  if (tid == 0) {
    int ns = 0, np = 0;
    for (int i = 0; i < PF_TILES; ++i) {
      ns += on_s[i];
      np += cnt[i];
    }
    blk[blockIdx.y * gridDim.x + blockIdx.x] = make_int4(ns, np, bad, 0);
  }
}

// Block b: the first prediction of each tile of PF_GROUP k_pf_tiles blocks
// (poff, poff[n_tiles] = all predictions), from the sums of the blocks before
// them; and of the warm-started Gaussians [256 b, 256 b + 256) those centred
// in a selected tile (floor(mu / T) in FP32): one bit each and their number.
// Block 0 adds up the selected tiles and the flags: sums = {selected, bad}.
constexpr int PF_GROUP = 16;
__global__ void __launch_bounds__(256)
k_pf_ranks(int N, int TX, int TY, int gx, int n_blk, const float *__restrict__ xy,
           const uint8_t *__restrict__ sel, const int *__restrict__ pcount,
           const int4 *__restrict__ blk, int *__restrict__ poff,
           unsigned long long *__restrict__ freed, int *__restrict__ n_freed,
           int *__restrict__ sums) {
  __shared__ int red[4];
  const int tid = threadIdx.x, b0 = blockIdx.x * PF_GROUP;
  if (b0 < n_blk) {
    int v = 0;
    for (int i = tid; i < b0; i += 256) v += blk[i].y;
    const int before = block_sum_256(v, red);
    // thread = tile: k_pf_tiles block b0 + tid / 16, its tile tid % 16
    const int b = b0 + tid / PF_TILES, ty = b / gx, tx = (b % gx) * PF_TILES + tid % PF_TILES;
    const bool ok = b < n_blk && tx < TX;
    const int k = ok ? pcount[ty * TX + tx] : 0;
    const int incl = before + block_scan_256(k, red);
    if (ok) poff[ty * TX + tx] = incl - k;
    if (ok && ty == TY - 1 && tx == TX - 1) poff[TX * TY] = incl;
  }
  const int n = blockIdx.x * 256 + tid;
  if (blockIdx.x * 256 < N) {
    bool f = false;
    if (n < N) {
      const float gxf = floorf(__fdiv_rn(xy[2 * n], (float)PF_T));
      const float gyf = floorf(__fdiv_rn(xy[2 * n + 1], (float)PF_T));
      if (gxf >= 0.f && gxf < (float)TX && gyf >= 0.f && gyf < (float)TY)
        f = sel[(int)gyf * TX + (int)gxf] != 0;
    }
    const unsigned long long bits = __ballot(f);
    if ((tid & 63) == 0) freed[n >> 6] = bits;
    const int c = block_sum_256(f ? 1 : 0, red);
    if (tid == 0) n_freed[blockIdx.x] = c;
  }
  if (blockIdx.x == 0) {
    int s = 0, bad = 0;
    for (int i = tid; i < n_blk; i += 256) {
      s += blk[i].x;
      bad |= blk[i].z;
    }
    s = block_sum_256(s, red);
    bad = __syncthreads_or(bad);
    if (tid == 0) {
      sums[0] = s;
      sums[1] = bad;
    }
  }
}

// The freed Gaussian of rank r < replaced, in index order, takes prediction
// r: the tile t with poff[t] <= r < poff[t + 1] (binary search), slot r -
// poff[t].  stats = {selected tiles, freed, predicted, replaced = bad ? 0 :
// min(freed, predicted)}.  Its block's first rank comes from the at most 256
// counts of k_pf_ranks (ranks by one block over all Gaussians: 71 us).
__global__ void __launch_bounds__(256)
k_pf_replace(int N, int n_tiles, int TX, const unsigned long long *__restrict__ freed,
             const int *__restrict__ n_freed, const int *__restrict__ sums,
             const int *__restrict__ poff, const float *__restrict__ head, float *__restrict__ xy,
             float *__restrict__ chol, float *__restrict__ rgb, int *__restrict__ stats) {
  __shared__ int red[4];
  const int tid = threadIdx.x, lane = tid & 63, n = blockIdx.x * 256 + tid;
  const int c = tid < (int)gridDim.x ? n_freed[tid] : 0;
  const int total = block_sum_256(c, red);
  const int before = block_sum_256(tid < (int)blockIdx.x ? c : 0, red);
  const int np = poff[n_tiles], replaced = sums[1] ? 0 : min(total, np);
  if (n == 0) {
    stats[0] = sums[0];
    stats[1] = total;
    stats[2] = np;
    stats[3] = replaced;
  }
  if (n >= N) return;
  int r = before;
  for (int w = (n >> 6) & ~3; w < (n >> 6); ++w) r += __popcll(freed[w]);
  const unsigned long long bits = freed[n >> 6];
  r += __popcll(bits & lanemask_lt());
  if (!((bits >> lane) & 1) || r >= replaced) return;
  int lo = 0, hi = n_tiles;  // largest t with poff[t] <= r
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (poff[mid] <= r) lo = mid;
    else hi = mid;
  }
  decode_slot(head, n_tiles, lo, r - poff[lo], lo % TX, lo / TX, PF_T, xy + 2 * n, chol + 3 * n,
              rgb + 3 * n);
}

// Per-tile targets from fitted Gaussians: the Gaussians whose centre lies
// in the tile, at most 8, those with the largest mass
//   m = |l1 * l3| * ((c0*c0 + c1*c1) + c2*c2)   (FP32, this order)
// (ties to the lower index), listed by increasing index.  The order of a
// tile's members does not matter to a choice by (mass, index), so they are
// not sorted: k_target_buckets appends each Gaussian to its tile's bucket,
// which is the tile's own 64 words of the target vectors, or if that is full
// to one list of the frame, and k_cnn_targets reads a bucket into one
// wavefront, one member per lane, before it writes the vectors over it.
// (Sorting the Gaussians by tile and walking each list
// with one thread took 95 us in ten launches at 8160 tiles and 30,000
// Gaussians.)
constexpr int BUCKET = NSLOT * NPAR;
static_assert(BUCKET == 64, "one bucket member per lane");

// The Gaussians past a full bucket: *n entries (tile, Gaussian) in any order.
struct TargetSpill {
  int *n, *tile, *id;
};

// Tile of Gaussian n's centre, -1 outside the frame or for a degenerate one.
__device__ inline int centre_tile(int n, int W, int H, int TX, int T, const float *__restrict__ xy,
                                  const float *__restrict__ chol) {
  const float x = xy[2 * n], y = xy[2 * n + 1];
  const float l1 = chol[3 * n], l3 = chol[3 * n + 2];
  const bool ok = isfinite(x) && isfinite(y) && x >= 0.f && y >= 0.f && x < (float)W &&
                  y < (float)H && isfinite(l1) && isfinite(l3) && l1 != 0.f && l3 != 0.f;
  return ok ? (int)floorf(y / (float)T) * TX + (int)floorf(x / (float)T) : -1;
}

__global__ void __launch_bounds__(256)
k_target_clear(int n_tiles, int *__restrict__ tcount, int *__restrict__ n_cd,
               int *__restrict__ n_spill) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t < n_tiles) tcount[t] = 0;
  if (t == 0) *n_cd = *n_spill = 0;
}

__global__ void __launch_bounds__(256)
k_target_buckets(int N, int W, int H, int TX, int T, const float *__restrict__ xy,
                 const float *__restrict__ chol, int *__restrict__ tcount,
                 int *__restrict__ bucket, TargetSpill spill) {
  const int n = blockIdx.x * 256 + threadIdx.x;
  const int t = n < N ? centre_tile(n, W, H, TX, T, xy, chol) : -1;
  const int c = t >= 0 ? atomicAdd(&tcount[t], 1) : 0;
  if (t >= 0 && c < BUCKET) bucket[(size_t)t * BUCKET + c] = n;
  // the spilled of a wavefront take one run of the list
  const unsigned long long out = __ballot(c >= BUCKET);
  if (out == 0) return;
  int at = 0;
  if ((threadIdx.x & 63) == 0) at = atomicAdd(spill.n, __popcll(out));
  at = __builtin_amdgcn_readfirstlane(at) + __popcll(out & lanemask_lt());
  if (c >= BUCKET) {
    spill.tile[at] = t;
    spill.id[at] = n;
  }
}

__device__ inline float target_mass(int n, const float *__restrict__ chol,
                                    const float *__restrict__ rgb) {
  const float a = fabsf(f32_mul(chol[3 * n], chol[3 * n + 2]));
  const float c0 = rgb[3 * n], c1 = rgb[3 * n + 1], c2 = rgb[3 * n + 2];
  return f32_mul(a, f32_add(f32_add(f32_mul(c0, c0), f32_mul(c1, c1)), f32_mul(c2, c2)));
}

__device__ inline float lane_value(float x, int j) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), j));
}

// The kept members of a tile, by one wavefront: lane s < k holds member s.
struct TargetKept {
  int lane, k, n;
  float m;
  int worst, wn;  // the lightest (of equals the largest index): lane, Gaussian, mass
  float wm;
  __device__ void put(int at, int nj, float mj) {
    if (lane == at) {
      n = nj;
      m = mj;
    }
  }
  __device__ void find_lightest() {
    worst = 0;
    wm = lane_value(m, 0);
    wn = __builtin_amdgcn_readlane(n, 0);
    for (int q = 1; q < NSLOT; ++q) {
      const float qm = lane_value(m, q);
      const int qn = __builtin_amdgcn_readlane(n, q);
      if (qm < wm || (qm == wm && qn > wn)) {
        worst = q;
        wm = qm;
        wn = qn;
      }
    }
  }
  // The definition's step, for members in index order.
  __device__ void insert(int nj, float mj) {
    if (k < NSLOT) {
      put(k++, nj, mj);
    } else {
      find_lightest();
      if (mj > wm) put(worst, nj, mj);
    }
  }
};

// The spilled members of tile t among the kept ones (NSLOT of comparable
// masses); false if one of theirs is a NaN.
__device__ inline bool keep_spilled(TargetKept &K, int t, const TargetSpill &spill,
                                    const float *__restrict__ chol,
                                    const float *__restrict__ rgb) {
  constexpr int BATCH = 8;  // entries per lane in flight
  const int total = *spill.n;
  K.find_lightest();
  for (int b = K.lane; b - K.lane < total; b += 64 * BATCH) {
    unsigned hits = 0;
#pragma unroll
    for (int q = 0; q < BATCH; ++q) {
      const int e = spill.tile[min(b + 64 * q, total - 1)];
      hits |= (b + 64 * q < total && e == t ? 1u : 0u) << q;
    }
    if (__ballot(hits != 0) == 0) continue;
    for (int q = 0; q < BATCH; ++q) {
      bool mem = (hits >> q) & 1;
      if (__ballot(mem) == 0) continue;
      const int n = mem ? spill.id[b + 64 * q] : 0;
      const float m = mem ? target_mass(n, chol, rgb) : 0.f;
      if (__ballot(m != m)) return false;
      while (const unsigned long long in =
                 __ballot(mem && (m > K.wm || (m == K.wm && n < K.wn)))) {
        const int j = __ffsll((long long)in) - 1;
        K.put(K.worst, __builtin_amdgcn_readlane(n, j), lane_value(m, j));
        K.find_lightest();
        if (K.lane == j) mem = false;
      }
    }
  }
  return true;
}

// One wavefront per tile.  With comparable masses every lane counts the members
// of the bucket that come before its own.  A tile of more than 64 members goes
// on with its part of the spilled list, read 512 entries at a time: nearly all
// of a batch's members are lighter than the kept ones and fall out together
// (1280x720 / 65,536 from the content-aware initialisation: 522 us with a pass
// over all Gaussians for each such tile, 26 now; 640x360 / 65,536, 73 members a
// tile: 613 and 63).  A NaN mass, whose place
// depends on the order of insertion, takes the definition itself: the tile's
// Gaussians in index order, inserted one at a time, each replacing the lightest
// kept one (of equals the one with the largest index) if it is heavier.  They
// come from the bucket or, where that is full, from a pass over all Gaussians
// (1920x1080 / 30,000, every 50th colour a NaN: 437 us with that pass for every
// tile with a NaN, 18 from the buckets).  tcount: members in, targets out.
constexpr int TARGET_BLOCK = 1024;
__global__ void __launch_bounds__(TARGET_BLOCK)
k_cnn_targets(int n_tiles, int N, int W, int H, int TX, int T, const float *__restrict__ xy,
              const float *__restrict__ chol, const float *__restrict__ rgb,
              int *__restrict__ tcount, float *__restrict__ tvec, int *__restrict__ n_cd,
              TargetSpill spill) {
  __shared__ int live;
  if (threadIdx.x == 0) live = 0;
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int per = TARGET_BLOCK / 64;
  int found = 0;
  for (int t = blockIdx.x * per + (int)(threadIdx.x >> 6); t < n_tiles; t += gridDim.x * per) {
    const int cnt = __builtin_amdgcn_readfirstlane(tcount[t]);
    float *out = tvec + (size_t)t * BUCKET;
    int n = 0, slot = -1;  // this lane's Gaussian and its place among the targets
    float m = 0.f;
    const int held = min(cnt, BUCKET);  // members in the bucket
    if (lane < held) {
      n = __float_as_int(out[lane]);  // as the stores below see it
      m = target_mass(n, chol, rgb);
    }
    bool in_order = __ballot(m != m) != 0;
    int rank = 0;
    for (int j = 0; j < held; ++j) {
      const float mj = lane_value(m, j);
      const int nj = __builtin_amdgcn_readlane(n, j);
      rank += (mj > m || (mj == m && nj < n)) ? 1 : 0;
    }
    if (cnt <= BUCKET && !in_order) {
      const bool keep = lane < cnt && rank < NSLOT;
      const unsigned long long kept = __ballot(keep);
      if (keep) slot = 0;
      for (int j = 0; j < cnt; ++j) {
        const int nj = __builtin_amdgcn_readlane(n, j);
        if (keep && ((kept >> j) & 1) && nj < n) ++slot;
      }
    } else {
      TargetKept K = {};
      K.lane = lane;
      if (!in_order) {  // the bucket's heaviest, then the spilled members
        for (; K.k < NSLOT; ++K.k) {
          const int j = __ffsll((long long)__ballot(rank == K.k)) - 1;
          K.put(K.k, __builtin_amdgcn_readlane(n, j), lane_value(m, j));
        }
        in_order = !keep_spilled(K, t, spill, chol, rgb);
        if (in_order) K.k = 0;
      }
      if (in_order && cnt <= BUCKET) {
        int place = lane < cnt ? 0 : -1;  // of this lane's member in index order
        for (int j = 0; j < cnt; ++j)
          if (__builtin_amdgcn_readlane(n, j) < n && lane < cnt) ++place;
        for (int i = 0; i < cnt; ++i) {
          const int j = __ffsll((long long)__ballot(place == i)) - 1;
          K.insert(__builtin_amdgcn_readlane(n, j), lane_value(m, j));
        }
      } else if (in_order) {
        for (int b = 0; b < N; b += 64) {
          const bool mem = b + lane < N && centre_tile(b + lane, W, H, TX, T, xy, chol) == t;
          const float mm = mem ? target_mass(b + lane, chol, rgb) : 0.f;
          for (unsigned long long bits = __ballot(mem); bits; bits &= bits - 1) {
            const int j = __ffsll((long long)bits) - 1;
            K.insert(b + j, lane_value(mm, j));
          }
        }
      }
      n = K.n;
      if (lane < K.k) slot = 0;
      for (int q = 0; q < K.k; ++q) {
        const int qn = __builtin_amdgcn_readlane(n, q);
        if (lane < K.k && qn < n) ++slot;
      }
    }
    const int k = min(cnt, NSLOT);
    // the bucket has been read: the vectors take its place, unused slots 0
    if (lane / NPAR >= k) out[lane] = 0.f;
    if (slot >= 0) {
      const int tx = t % TX, ty = t / TX;
      float *q = out + slot * NPAR;
      q[0] = (xy[2 * n] - (float)(tx * T)) / (float)T;
      q[1] = (xy[2 * n + 1] - (float)(ty * T)) / (float)T;
      q[2] = __logf(fabsf(chol[3 * n]));
      q[3] = chol[3 * n + 1];
      q[4] = __logf(fabsf(chol[3 * n + 2]));
      q[5] = rgb[3 * n];
      q[6] = rgb[3 * n + 1];
      q[7] = rgb[3 * n + 2];
    }
    if (lane == 0) {
      tcount[t] = k;
      found += k > 0 ? 1 : 0;
    }
  }
  if (lane == 0 && found) atomicAdd(&live, found);
  __syncthreads();
  if (threadIdx.x == 0 && live) atomicAdd(n_cd, live);
}

// He-normal initial weights from caller-supplied standard normal draws
// (one per parameter slot): W = z * sqrt(2 / (9 * fan_in_channels)) on the
// real (co < Cout, tap < 9, ci < cin_real) entries, 0 elsewhere; bias 0.
__global__ void __launch_bounds__(256)
k_cnn_init(ConvDims d, int cin_real, const float *__restrict__ z, float *__restrict__ w,
           float *__restrict__ b) {
  const size_t n = (size_t)d.Mpad * d.Kf;
  const float sc = sqrtf(2.f / (9.f * (float)cin_real));
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x) {
    const int co = (int)(i / d.Kf), k = (int)(i % d.Kf);
    const int tap = k / d.Cin, ci = k % d.Cin;
    w[i] = (co < d.Cout && tap < 9 && ci < cin_real) ? z[i] * sc : 0.f;
    if (i < (size_t)d.Mpad) b[i] = 0.f;
  }
}

}  // namespace gs2d

using namespace gs2d;

extern "C" {

int gs2d_cnn_init_params(int32_t H, int32_t W, const float *normal_draws, float *master,
                         void *stream) {
  CnnLayout C;
  if (!cnn_layout(H, W, &C) || !normal_draws || !master) return GS2D_EINVAL;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  for (int i = 0; i < NLAYER; ++i) {
    const ConvDims &d = C.L[i];
    const size_t n = (size_t)d.Mpad * d.Kf;
    hipLaunchKernelGGL(k_cnn_init, dim3((unsigned)std::min<size_t>((n + 255) / 256, 2048)),
                       dim3(256), 0, st, d, i == 0 ? 6 : d.Cin, normal_draws + C.w_off[i],
                       master + C.w_off[i], master + C.b_off[i]);
  }
  return hipGetLastError() == hipSuccess ? GS2D_OK : GS2D_EHIP;
}

size_t gs2d_cnn_param_count(int32_t H, int32_t W) {
  CnnLayout C;
  return cnn_layout(H, W, &C) ? C.n_params : 0;
}

size_t gs2d_cnn_workspace_bytes(int32_t H, int32_t W) {
  CnnLayout C;
  return cnn_layout(H, W, &C) ? C.total : 0;
}

size_t gs2d_cnn_bf16_weight_count(int32_t H, int32_t W) {
  CnnLayout C;
  return cnn_layout(H, W, &C) ? C.n_wb + C.n_wt : 0;
}

int gs2d_cnn_layer_info(int32_t H, int32_t W, int32_t layer, int32_t *info /* [12] */) {
  CnnLayout C;
  if (!cnn_layout(H, W, &C) || layer < 0 || layer >= NLAYER || !info) return GS2D_EINVAL;
  const ConvDims &d = C.L[layer];
  const int32_t v[12] = {d.Hin, d.Win, d.Cin, d.Hout, d.Wout, d.Cout, d.stride, d.relu,
                         d.Mpad, d.Kf, (int32_t)C.w_off[layer], (int32_t)C.b_off[layer]};
  for (int i = 0; i < 12; ++i) info[i] = v[i];
  return GS2D_OK;
}

int gs2d_cnn_sync_weights(int32_t H, int32_t W, const float *master, uint16_t *wbf16,
                          void *stream) {
  CnnLayout C;
  if (!cnn_layout(H, W, &C) || !master || !wbf16) return GS2D_EINVAL;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  uint16_t *wt = wbf16 + C.n_wb;
  // the transposed copies are written sparsely: clear their padding first
  if (launch_fill_zero_u32(reinterpret_cast<uint32_t *>(wt), (C.n_wt + 1) / 2, st) != hipSuccess)
    return GS2D_EHIP;
  for (int i = 0; i < NLAYER; ++i) {
    const ConvDims &d = C.L[i];
    const size_t n = (size_t)d.Mpad * d.Kf;
    hipLaunchKernelGGL(k_cnn_weights_to_bf16, dim3((unsigned)std::min<size_t>((n + 255) / 256, 2048)),
                       dim3(256), 0, st, d, master + C.w_off[i], wbf16 + C.wb_off[i],
                       i > 0 ? wt + C.wt_off[i] : nullptr);
  }
  return hipGetLastError() == hipSuccess ? GS2D_OK : GS2D_EHIP;
}

int gs2d_cnn_forward(int32_t H, int32_t W, const float *frame, const float *prev,
                     const float *master, const uint16_t *wbf16, float *head_out, void *ws,
                     size_t ws_bytes, void *stream) {
  CnnLayout C;
  if (!cnn_layout(H, W, &C) || !frame || !master || !wbf16 || !ws) return GS2D_EINVAL;
  if (reinterpret_cast<uintptr_t>(ws) & 255) return GS2D_EINVAL;
  if (ws_bytes < C.total) return GS2D_ENOSPACE;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  uint16_t *x = at<uint16_t>(ws, C.x_in);
  const uint16_t *in = x;
  for (int i = 0; i < NLAYER; ++i) {
    ConvArgs a = {};
    a.d = C.L[i];
    a.x = in;
    a.w = wbf16 + C.wb_off[i];
    a.bias = master + C.b_off[i];
    if (i < NLAYER - 1) {
      a.y = at<uint16_t>(ws, C.act[i]);
      in = a.y;
    } else {
      a.y_planar = at<float>(ws, C.head);
    }
    if (i == 0) {
      const ConvDims &d = a.d;
      hipLaunchKernelGGL(k_conv_first,
                         dim3(xcd_grid((d.Wout + C0_TW - 1) / C0_TW *
                                       ((d.Hout + C0_TH - 1) / C0_TH))),
                         dim3(256), 0, st, a, frame, prev, x);
    } else if (launch_conv_fwd(a, st) != hipSuccess) {
      return GS2D_EHIP;
    }
  }
  if (hipGetLastError() != hipSuccess) return GS2D_EHIP;
  if (head_out &&
      hipMemcpyAsync(head_out, at<float>(ws, C.head), sizeof(float) * HEAD_CH * C.n_tiles,
                     hipMemcpyDeviceToDevice, st) != hipSuccess)
    return GS2D_EHIP;
  return GS2D_OK;
}

int gs2d_cnn_targets(int32_t H, int32_t W, int32_t N, const float *xy, const float *chol,
                     const float *rgb, void *ws, size_t ws_bytes, void *scratch,
                     size_t scratch_bytes, void *stream) {
  CnnLayout C;
  if (!cnn_layout(H, W, &C) || N < 1 || N > 65536 || !xy || !chol || !rgb || !ws || !scratch)
    return GS2D_EINVAL;
  if (ws_bytes < C.total) return GS2D_ENOSPACE;
  // scratch holds the spilled members (tile, Gaussian) and their number; the
  // size asked for is that of the interface, which is larger
  const int G = std::max(1, std::min(SORT_MAX_BLOCKS, (N + 2047) / 2048));
  const size_t need = al256(4 * (size_t)N) * 2 + al256(4 * (size_t)RADIX * G) +
                      al256(4 * ((size_t)C.n_tiles + 1)) + 256;
  if (scratch_bytes < need || (reinterpret_cast<uintptr_t>(scratch) & 255)) return GS2D_ENOSPACE;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  int *tcount = at<int>(ws, C.tcount), *ncd = at<int>(ws, C.ncd);
  float *tvec = at<float>(ws, C.tvec);
  const TargetSpill spill{at<int>(scratch, 2 * al256(4 * (size_t)N)), at<int>(scratch, 0),
                          at<int>(scratch, al256(4 * (size_t)N))};
  hipLaunchKernelGGL(k_target_clear, dim3((C.n_tiles + 255) / 256), dim3(256), 0, st, C.n_tiles,
                     tcount, ncd, spill.n);
  hipLaunchKernelGGL(k_target_buckets, dim3((N + 255) / 256), dim3(256), 0, st, N, W, H, C.TX, 16,
                     xy, chol, tcount, reinterpret_cast<int *>(tvec), spill);
  // at most one block per compute unit: each adds once to the tile counter
  const int per = TARGET_BLOCK / 64;
  hipLaunchKernelGGL(k_cnn_targets, dim3(std::min((C.n_tiles + per - 1) / per, 256)),
                     dim3(TARGET_BLOCK), 0, st, C.n_tiles, N, W, H, C.TX, 16, xy, chol, rgb, tcount,
                     tvec, ncd, spill);
  return hipGetLastError() == hipSuccess ? GS2D_OK : GS2D_EHIP;
}

int gs2d_cnn_tensor_view(int32_t H, int32_t W, int32_t layer, int32_t which, const void *ws,
                         size_t ws_bytes, const void **ptr, int32_t *dims) {
  CnnLayout C;
  if (!cnn_layout(H, W, &C) || layer < 0 || layer >= NLAYER || !ws || !ptr || !dims)
    return GS2D_EINVAL;
  if (ws_bytes < C.total) return GS2D_ENOSPACE;
  const ConvDims &d = C.L[layer];
  const char *b = static_cast<const char *>(ws);
  if (which == 0) {  // the layer's input activations
    *ptr = b + (layer == 0 ? C.x_in : C.act[layer - 1]);
    dims[0] = d.Hin;
    dims[1] = d.Win;
    dims[2] = d.Cin;
  } else if (which == 1) {  // dLoss / d(layer output), ReLU mask applied
    *ptr = b + C.dz[layer];
    dims[0] = d.Hout;
    dims[1] = d.Wout;
    dims[2] = d.CoutS;
  } else {
    return GS2D_EINVAL;
  }
  return GS2D_OK;
}

int gs2d_cnn_read_targets(int32_t H, int32_t W, const void *ws, size_t ws_bytes, int32_t *counts,
                          float *vectors, void *stream) {
  CnnLayout C;
  if (!cnn_layout(H, W, &C) || !ws || !counts || !vectors) return GS2D_EINVAL;
  if (ws_bytes < C.total) return GS2D_ENOSPACE;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const char *b = static_cast<const char *>(ws);
  if (hipMemcpyAsync(counts, b + C.tcount, 4 * (size_t)C.n_tiles, hipMemcpyDeviceToDevice, st) !=
          hipSuccess ||
      hipMemcpyAsync(vectors, b + C.tvec, 4 * (size_t)C.n_tiles * NSLOT * NPAR,
                     hipMemcpyDeviceToDevice, st) != hipSuccess)
    return GS2D_EHIP;
  return GS2D_OK;
}

int gs2d_cnn_backward(int32_t H, int32_t W, const float *master, const uint16_t *wbf16,
                      float *grad, float *loss3, void *ws, size_t ws_bytes, void *stream) {
  CnnLayout C;
  if (!cnn_layout(H, W, &C) || !master || !wbf16 || !grad || !ws) return GS2D_EINVAL;
  if (ws_bytes < C.total) return GS2D_ENOSPACE;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const ConvDims &hd = C.L[NLAYER - 1];
  hipLaunchKernelGGL(k_head_loss, dim3((unsigned)((16LL * C.n_tiles + 255) / 256)), dim3(256), 0,
                     st, C.n_tiles, hd.CoutS, at<const float>(ws, C.head),
                     at<const int>(ws, C.tcount), at<const float>(ws, C.tvec),
                     at<const int>(ws, C.ncd), at<uint16_t>(ws, C.dz[NLAYER - 1]),
                     at<float>(ws, C.tile_loss));
  const uint16_t *wt = wbf16 + C.n_wb;
  GwArgs gw = C.gw;
  int cols = 0;
  for (int i = NLAYER - 1; i >= 0; --i) {
    ConvArgs a = {};
    a.d = C.L[i];
    a.x = (i == 0) ? at<const uint16_t>(ws, C.x_in) : at<const uint16_t>(ws, C.act[i - 1]);
    a.dz = at<const uint16_t>(ws, C.dz[i]);
    GwLayer &g = gw.L[i];
    g.x = a.x;
    g.dz = a.dz;
    g.part = at<float>(ws, C.gpart[i]);
    g.dw = grad + C.w_off[i];
    g.db = grad + C.b_off[i];
    cols += g.mt * (g.cols + 1);
    if (i > 0) {
      a.wt = wt + C.wt_off[i];
      a.dz_prev = at<uint16_t>(ws, C.dz[i - 1]);
      if (launch_conv_bwd_data(a, st) != hipSuccess) return GS2D_EHIP;
    }
  }
  hipLaunchKernelGGL(k_conv_bwd_weight, dim3((unsigned)((gw.nwork + 7) / 8 * 8)), dim3(512), 0, st,
                     gw);
  hipLaunchKernelGGL(k_conv_bwd_weight_first, dim3((unsigned)gw.L[0].splits), dim3(256), 0, st,
                     gw.L[0]);
  hipLaunchKernelGGL(k_gw_reduce, dim3((unsigned)cols + 1), dim3(256), 0, st, gw,
                     LossSum{C.n_tiles, at<const float>(ws, C.tile_loss), at<const int>(ws, C.ncd),
                             loss3});
  return hipGetLastError() == hipSuccess ? GS2D_OK : GS2D_EHIP;
}

int gs2d_cnn_adam(int32_t H, int32_t W, float *master, float *grad, float *m, float *v,
                  int32_t *step, float lr, float weight_decay, uint16_t *wbf16, void *stream) {
  CnnLayout C;
  if (!cnn_layout(H, W, &C) || !master || !grad || !m || !v || !step || !wbf16)
    return GS2D_EINVAL;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  if (launch_step_tick(step, st) != hipSuccess) return GS2D_EHIP;
  CnnParamMap map;
  for (int i = 0; i < NLAYER; ++i) {
    map.d[i] = C.L[i];
    map.w_off[i] = (long long)C.w_off[i];
    map.b_off[i] = (long long)C.b_off[i];
    map.wb_off[i] = (long long)C.wb_off[i];
    map.wt_off[i] = (long long)C.wt_off[i];
  }
  hipLaunchKernelGGL(k_cnn_adam, dim3((unsigned)std::min<size_t>((C.n_params + 255) / 256, 2048)),
                     dim3(256), 0, st, C.n_params, map, master, grad, m, v, step, lr, 0.9f, 0.999f,
                     1e-8f, weight_decay, wbf16, wbf16 + C.n_wb);
  return hipGetLastError() == hipSuccess ? GS2D_OK : GS2D_EHIP;
}

int gs2d_cnn_decode(int32_t H, int32_t W, int32_t N, const float *plain_xy,
                    const float *plain_chol, const float *plain_rgb, float *xy, float *chol,
                    float *rgb, int32_t *n_predicted, void *ws, size_t ws_bytes, void *scratch,
                    size_t scratch_bytes, void *stream) {
  CnnLayout C;
  if (!cnn_layout(H, W, &C) || N < 1 || N > 65536 || !plain_xy || !plain_chol || !plain_rgb ||
      !xy || !chol || !rgb || !n_predicted || !ws || !scratch)
    return GS2D_EINVAL;
  if (ws_bytes < C.total) return GS2D_ENOSPACE;
  const size_t need = al256(4 * ((size_t)C.n_tiles + 1)) * 2 + 256;
  if (scratch_bytes < need || (reinterpret_cast<uintptr_t>(scratch) & 255)) return GS2D_ENOSPACE;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  int *counts = at<int>(scratch, 0);
  int *bsum = at<int>(scratch, al256(4 * ((size_t)C.n_tiles + 1)));
  int *flags = at<int>(scratch, 2 * al256(4 * ((size_t)C.n_tiles + 1)));
  const float *head = at<const float>(ws, C.head);
  hipLaunchKernelGGL(k_decode_counts, dim3((C.n_tiles + 255) / 256), dim3(256), 0, st, C.n_tiles,
                     head, counts, bsum, flags);
  hipLaunchKernelGGL(k_decode_write, dim3((C.n_tiles + DECODE_TILES - 1) / DECODE_TILES), dim3(256),
                     0, st, C.n_tiles, C.TX, 16, head, counts, bsum, N, xy, chol, rgb, flags);
  hipLaunchKernelGGL(k_decode_merge, dim3((N + 255) / 256), dim3(256), 0, st, N, flags, plain_xy,
                     plain_chol, plain_rgb, xy, chol, rgb, n_predicted);
  return hipGetLastError() == hipSuccess ? GS2D_OK : GS2D_EHIP;
}

struct PfLayout {
  size_t sel, pcount, poff, blk, freed, n_freed, sums, total;
  int gx, n_blk;  // k_pf_tiles blocks per tile row and in all
};
static PfLayout pf_layout(const CnnLayout &C, int N) {
  PfLayout L;
  L.gx = (C.TX + PF_TILES - 1) / PF_TILES;
  L.n_blk = L.gx * C.TY;
  size_t o = 0;
  auto take = [&o](size_t b) {
    const size_t at = o;
    o = al256(o + b);
    return at;
  };
  L.sel = take((size_t)C.n_tiles);
  L.pcount = take(4 * (size_t)C.n_tiles);
  L.poff = take(4 * ((size_t)C.n_tiles + 1));
  L.blk = take(16 * (size_t)L.n_blk);
  L.freed = take(8 * ((size_t)(N + 255) / 256 * 4));
  L.n_freed = take(4 * (size_t)((N + 255) / 256));
  L.sums = take(8);
  L.total = o;
  return L;
}

size_t gs2d_cnn_pframe_scratch_bytes(int32_t H, int32_t W, int32_t N) {
  CnnLayout C;
  if (!cnn_layout(H, W, &C) || N < 1 || N > 65536) return 0;
  return pf_layout(C, N).total;
}

int gs2d_cnn_pframe_replace(int32_t H, int32_t W, int32_t N, const float *frame,
                            const float *prev, float tau, const float *head, float *xy,
                            float *chol, float *rgb, int32_t *stats, uint8_t *tile_sel, void *ws,
                            size_t ws_bytes, void *scratch, size_t scratch_bytes, void *stream) {
  CnnLayout C;
  if (!cnn_layout(H, W, &C) || N < 1 || N > 65536 || !frame || !prev || !xy || !chol || !rgb ||
      !stats || !scratch || !(tau >= 0.f) || !std::isfinite(tau))
    return GS2D_EINVAL;
  if (!head) {
    if (!ws) return GS2D_EINVAL;
    if (ws_bytes < C.total) return GS2D_ENOSPACE;
    head = at<const float>(ws, C.head);
  }
  const PfLayout L = pf_layout(C, N);
  if (scratch_bytes < L.total || (reinterpret_cast<uintptr_t>(scratch) & 255))
    return GS2D_ENOSPACE;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  uint8_t *sel = tile_sel ? tile_sel : at<uint8_t>(scratch, L.sel);
  int *pcount = at<int>(scratch, L.pcount), *poff = at<int>(scratch, L.poff);
  int4 *blk = at<int4>(scratch, L.blk);
  auto *freed = at<unsigned long long>(scratch, L.freed);
  int *n_freed = at<int>(scratch, L.n_freed), *sums = at<int>(scratch, L.sums);
  const int nb = (N + 255) / 256, np = (L.n_blk + PF_GROUP - 1) / PF_GROUP;
  hipLaunchKernelGGL(k_pf_tiles, dim3(L.gx, C.TY), dim3(256), 0, st, H, W, C.TX, C.n_tiles, frame,
                     prev, tau, head, sel, pcount, blk);
  hipLaunchKernelGGL(k_pf_ranks, dim3(std::max(nb, np)), dim3(256), 0, st, N, C.TX, C.TY, L.gx,
                     L.n_blk, xy, sel, pcount, blk, poff, freed, n_freed, sums);
  hipLaunchKernelGGL(k_pf_replace, dim3(nb), dim3(256), 0, st, N, C.n_tiles, C.TX, freed, n_freed,
                     sums, poff, head, xy, chol, rgb, stats);
  return hipGetLastError() == hipSuccess ? GS2D_OK : GS2D_EHIP;
}

}  // extern "C"
