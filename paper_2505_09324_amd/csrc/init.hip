// Content-aware ROI initialisation (Sec. 3.2.A) in its synthetic-frame
// form: Gaussian centres are drawn inside the ROI with probability rising
// with the local image gradient, and uniformly outside it.
//
//  1. per pixel: Y = (R+G)+B; central differences (border: twice the
//     one-sided difference); mag = sqrt(gx*gx + gy*gy) in FP32 without
//     contraction; level q = floor(1024 mag).
//  2. sums of q*[roi] (int64), q (int64) and [roi] over groups of 64 pixels
//     in raster order, as inclusive prefixes within a chunk of groups, and
//     the chunks' totals.
//  3. per draw: ROI draws pick the first pixel whose running weight
//     sum_{roi} (q + b + 1) exceeds (pick mod Wt), b = Q // (10 R); outside
//     draws pick the (pick mod O)-th non-ROI pixel.  Scale, jitter and colour
//     follow; all integer decisions are exact.
//
// Two launches and no host read-back.  A draw finds its chunk in a prefix that
// its block forms in LDS, its group in the chunk's 64-pixel prefixes, and its
// pixel by evaluating that group's 64 levels again, one per lane: the
// per-pixel prefix sums (83 MB written, read back and searched at 1920 x 1080)
// are never formed.  Both launches are bound by the latency of their few
// dependent loads; the first also reads the frame once.
#include <cmath>

#include "gs2d_internal.h"

namespace gs2d {

namespace {

constexpr int INIT_BLOCK = 256;        // threads of a drawing block
constexpr int INIT_WAVES = INIT_BLOCK / 64;
constexpr int INIT_LEVELS = 512;       // threads of a level block
constexpr int INIT_GROUP = 64;         // pixels per group: one per lane
constexpr int INIT_BATCH = 32;         // groups whose levels a block forms at a time
constexpr int INIT_MAX_CHUNKS = 1024;  // chunk prefixes a drawing block holds in LDS
constexpr int INIT_DRAWS = 6;          // draws per wavefront: 30,000 in one round of blocks

// A chunk is a whole number of batches, as few as keep the chunks within
// INIT_MAX_CHUNKS (one, 2048 pixels, up to 2 Mpixel frames).
struct InitLayout {
  size_t gqm, gqa, gr, part, total;
  int n_groups, chunk_groups, n_chunks;
};

bool init_layout(int W, int H, InitLayout *L) {
  if (W < 1 || H < 1) return false;
  const long long HW = (long long)W * H;
  if (HW > (1LL << 28)) return false;
  auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
  L->n_groups = (int)((HW + INIT_GROUP - 1) / INIT_GROUP);
  const int batches = (L->n_groups + INIT_BATCH - 1) / INIT_BATCH;
  L->chunk_groups = (batches + INIT_MAX_CHUNKS - 1) / INIT_MAX_CHUNKS * INIT_BATCH;
  L->n_chunks = (L->n_groups + L->chunk_groups - 1) / L->chunk_groups;
  size_t o = 0;
  L->gqm = o;
  o = al(o + (size_t)L->n_groups * 8);
  L->gqa = o;
  o = al(o + (size_t)L->n_groups * 8);
  L->gr = o;
  o = al(o + (size_t)L->n_groups * 4);
  L->part = o;
  o = al(o + (size_t)L->n_chunks * 24);
  L->total = o;
  return true;
}

__device__ inline float luma_sum(const float *__restrict__ T, size_t HW, size_t p) {
  return f32_add(f32_add(T[p], T[HW + p]), T[2 * HW + p]);
}

// Gradient level q of pixel p.  At a border the difference of the pixel and
// its one neighbour is doubled (times 1 elsewhere: exact), so the four lumas
// are loaded without a branch; a frame of one row or column has no
// difference there.  (With the borders as branches the unrolled kernel was
// 22 KB of code run once per launch and bound by fetching it.)
__device__ inline long long level(const float *__restrict__ T, int W, int H, size_t HW,
                                  unsigned p) {
  const unsigned y = p / (unsigned)W, x = p - y * (unsigned)W;
  const bool l = x > 0, r = x + 1 < (unsigned)W, u = y > 0, d = y + 1 < (unsigned)H;
  const float yl = luma_sum(T, HW, l ? p - 1 : p), yr = luma_sum(T, HW, r ? p + 1 : p);
  const float yu = luma_sum(T, HW, u ? p - W : p), yd = luma_sum(T, HW, d ? p + W : p);
  const float gx = W > 1 ? f32_mul(f32_sub(yr, yl), l && r ? 1.0f : 2.0f) : 0.f;
  const float gy = H > 1 ? f32_mul(f32_sub(yd, yu), u && d ? 1.0f : 2.0f) : 0.f;
  const float mag = f32_sqrt(f32_add(f32_mul(gx, gx), f32_mul(gy, gy)));
  return (long long)floorf(f32_mul(mag, 1024.0f));
}

// Sum of v over the wavefront, in every lane.  Levels of ordinary frames are
// far below 2^25, so that 64 of them fit 32 bits and are added with the
// cross-lane moves of the vector unit; otherwise by 64-bit shuffles.
template <int CTRL>
__device__ inline unsigned dpp_add(unsigned x) {
  return x + (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, false);
}
__device__ inline long long wave_sum(long long v) {
  if (__ballot((unsigned long long)v >> 25) == 0) {
    unsigned x = (unsigned)v;
    const auto h = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    x = h[0] + h[1];
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = r[0] + r[1];
    x = dpp_add<0x128>(x);  // row_ror:8
    x = dpp_add<0x141>(x);  // row_half_mirror
    x = dpp_add<0x4E>(x);   // quad_perm [2,3,0,1]
    x = dpp_add<0xB1>(x);   // quad_perm [1,0,3,2]
    return x;
  }
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Block c: the levels of chunk c, reduced to the inclusive prefixes of its
// 64-pixel groups (gqm, gqa, gr) and its totals part[0..2][c] = sum q [roi],
// sum q, sum [roi].
__global__ void __launch_bounds__(INIT_LEVELS)
k_init_groups(int W, int H, int n_groups, int chunk_groups, const float *__restrict__ T,
              const uint8_t *__restrict__ mask, long long *__restrict__ gqm,
              long long *__restrict__ gqa, int *__restrict__ gr, long long *__restrict__ part) {
  __shared__ long long sm[INIT_BATCH], sa[INIT_BATCH];
  __shared__ int sr[INIT_BATCH];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const size_t HW = (size_t)W * H;
  const int g0 = blockIdx.x * chunk_groups, g1 = min(n_groups, g0 + chunk_groups);
  long long run_m = 0, run_a = 0;  // first wavefront: the earlier batches' sums
  int run_r = 0;
  for (int b0 = g0; b0 < g1; b0 += INIT_BATCH) {
    constexpr int PER = INIT_BATCH / (INIT_LEVELS / 64);
#pragma unroll 2
    for (int j = wid * PER; j < (wid + 1) * PER; ++j) {
      const size_t p = (size_t)(b0 + j) * INIT_GROUP + lane;
      const bool ok = p < HW;
      const long long q = ok ? level(T, W, H, HW, (unsigned)p) : 0;
      const unsigned long long in = __ballot(ok && mask[ok ? p : 0] != 0);
      const long long a = wave_sum(q);
      // a group wholly inside or outside the ROI needs no second sum
      const long long m = in == 0 ? 0 : in == ~0ull ? a : wave_sum((in >> lane) & 1 ? q : 0);
      if (lane == 0) {
        sm[j] = m;
        sa[j] = a;
        sr[j] = __popcll(in);
      }
    }
    __syncthreads();
    if (wid == 0) {
      long long m = lane < INIT_BATCH ? sm[lane] : 0, a = lane < INIT_BATCH ? sa[lane] : 0;
      int r = lane < INIT_BATCH ? sr[lane] : 0;
      for (int o = 1; o < INIT_BATCH; o <<= 1) {
        const long long um = __shfl_up(m, o, 64), ua = __shfl_up(a, o, 64);
        const int ur = __shfl_up(r, o, 64);
        if (lane >= o) {
          m += um;
          a += ua;
          r += ur;
        }
      }
      m += run_m;
      a += run_a;
      r += run_r;
      if (lane < INIT_BATCH && b0 + lane < g1) {
        gqm[b0 + lane] = m;
        gqa[b0 + lane] = a;
        gr[b0 + lane] = r;
      }
      run_m = __shfl(m, INIT_BATCH - 1, 64);
      run_a = __shfl(a, INIT_BATCH - 1, 64);
      run_r = __shfl(r, INIT_BATCH - 1, 64);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[blockIdx.x] = run_m;
    part[gridDim.x + blockIdx.x] = run_a;
    part[2 * gridDim.x + blockIdx.x] = run_r;
  }
}

// First index i in [0, n) with f(i) > k; f is non-decreasing and f(n-1) > k.
template <typename F>
__device__ inline int first_above(int n, long long k, F f) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi) / 2;
    if (f(mid) > k)
      hi = mid;
    else
      lo = mid + 1;
  }
  return lo;
}

__device__ inline float clamp_scale(double s) {
  return (float)fmin(fmax(s, 0.5), 16.0);
}

struct DrawArgs {
  int W, H, n_roi, n_out, n_groups, chunk_groups, n_chunks;
  const float *T;
  const uint8_t *mask;
  const long long *gqm, *gqa, *part;
  const int *gr;
  double kappa;
};

// INIT_DRAWS draws per wavefront.  The block first scans the chunk totals
// (INIT_MAX_CHUNKS / INIT_BLOCK per thread): the region totals decide the
// sampling regions, and the chunks' running weights of the ROI draws and of
// the outside draws stay in LDS.  One lane per draw reduces its pick and
// searches the chunks and the groups; then the whole wavefront takes the
// draws' groups one after another, one pixel per lane (their loads are
// independent); last, one lane per draw writes its Gaussian.  With all of it
// done by the wavefront for one draw at a time the 64-bit remainders and
// square roots of 30,000 draws took 40 us.
__global__ void __launch_bounds__(INIT_BLOCK)
k_init_draw(DrawArgs a, const int64_t *__restrict__ pick_roi, const float *__restrict__ jit_roi,
            const int64_t *__restrict__ pick_out, const float *__restrict__ jit_out,
            float *__restrict__ xy, float *__restrict__ chol, float *__restrict__ rgb,
            int *__restrict__ picked) {
  constexpr int PER = INIT_MAX_CHUNKS / INIT_BLOCK;
  // the chunk totals, then the inclusive running weights of the ROI draws
  // and of the outside draws (pixels)
  __shared__ long long f_roi[INIT_MAX_CHUNKS], f_all[INIT_MAX_CHUNKS];
  __shared__ int f_out[INIT_MAX_CHUNKS];
  __shared__ long long red[3][INIT_WAVES];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const long long HW = (long long)a.W * a.H;
  long long v[3][PER], s[3] = {0, 0, 0};
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int c = j * INIT_BLOCK + tid;
    const bool ok = c < a.n_chunks;
    f_roi[c] = ok ? a.part[c] : 0;
    f_all[c] = ok ? a.part[a.n_chunks + c] : 0;
    f_out[c] = ok ? (int)a.part[2 * a.n_chunks + c] : 0;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int c = tid * PER + j;
    v[0][j] = f_roi[c];
    v[1][j] = f_all[c];
    v[2][j] = f_out[c];
#pragma unroll
    for (int k = 0; k < 3; ++k) s[k] += v[k][j];
  }
  long long x[3] = {s[0], s[1], s[2]};
  for (int o = 1; o < 64; o <<= 1)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const long long u = __shfl_up(x[k], o, 64);
      if (lane >= o) x[k] += u;
    }
  if (lane == 63)
#pragma unroll
    for (int k = 0; k < 3; ++k) red[k][wid] = x[k];
  __syncthreads();
  long long run[3], tot[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    run[k] = x[k] - s[k];
    tot[k] = 0;
    for (int w = 0; w < INIT_WAVES; ++w) {
      if (w < wid) run[k] += red[k][w];
      tot[k] += red[k][w];
    }
  }
  // an empty ROI makes the whole frame the ROI; a full one makes the
  // outside draws uniform over the frame
  const bool roi_all = tot[2] == 0, out_all = tot[2] == HW;
  const long long R = roi_all ? HW : tot[2], Q = roi_all ? tot[1] : tot[0];
  const long long O = out_all ? HW : HW - tot[2];
  const long long b = Q / (10 * R), Wt = Q + (b + 1) * R, bb = b + 1;
  const long long chunk_px = (long long)a.chunk_groups * INIT_GROUP;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int c = tid * PER + j;
#pragma unroll
    for (int k = 0; k < 3; ++k) run[k] += v[k][j];
    if (c < a.n_chunks) {
      const long long px = min(HW, (c + 1) * chunk_px);
      f_roi[c] = roi_all ? run[1] + bb * px : run[0] + bb * run[2];
      f_out[c] = (int)(out_all ? px : px - run[2]);
    }
  }
  __syncthreads();
  const long long *gq = roi_all ? a.gqa : a.gqm;
  const int N = a.n_roi + a.n_out;
  const int i0 = (blockIdx.x * INIT_WAVES + wid) * INIT_DRAWS, i = i0 + lane;
  const bool mine = lane < INIT_DRAWS && i < N, roi = i < a.n_roi;
  int g = 0;         // the draw's group
  long long kg = 0;  // what its running weight must exceed there
  if (mine) {
    const long long k = roi ? pick_roi[i] % Wt : pick_out[i - a.n_roi] % O;
    const int c = first_above(a.n_chunks, k,
                              [&](int t) { return roi ? f_roi[t] : (long long)f_out[t]; });
    const long long kc = k - (c == 0 ? 0 : roi ? f_roi[c - 1] : (long long)f_out[c - 1]);
    // running weight at the end of group t of the chunk, from the chunk's start
    const int g0 = c * a.chunk_groups, ng = min(a.chunk_groups, a.n_groups - g0);
    const long long base_px = g0 * (long long)INIT_GROUP;
    auto f_group = [&](int t) {
      const long long px = min(HW, (long long)(g0 + t + 1) * INIT_GROUP) - base_px;
      if (roi) return gq[g0 + t] + bb * (roi_all ? px : (long long)a.gr[g0 + t]);
      return out_all ? px : px - a.gr[g0 + t];
    };
    const int t = first_above(ng, kc, f_group);
    g = g0 + t;
    kg = kc - (t == 0 ? 0 : f_group(t - 1));
  }
  int pick = 0;       // the draw's pixel
  long long wpx = 1;  // and its weight
#pragma unroll 2
  for (int d = 0; d < INIT_DRAWS; ++d) {
    if (i0 + d >= N) break;
    const bool droi = i0 + d < a.n_roi;
    const int dg = __builtin_amdgcn_readlane(g, d);
    const long long dk = __shfl(kg, d, 64);
    const long long pl = (long long)dg * INIT_GROUP + lane;
    const bool ok = pl < HW;
    const size_t ps = ok ? (size_t)pl : 0;
    long long wgt = 0;
    if (droi) {
      if (ok && (roi_all || a.mask[ps])) wgt = level(a.T, a.W, a.H, (size_t)HW, (unsigned)ps) + bb;
    } else {
      wgt = ok && (out_all || !a.mask[ps]) ? 1 : 0;
    }
    long long f = wgt;
    for (int o = 1; o < 64; o <<= 1) {
      const long long u = __shfl_up(f, o, 64);
      if (lane >= o) f += u;
    }
    const unsigned long long above = __ballot(f > dk);
    const int l = above ? __ffsll((long long)above) - 1 : 0;
    const long long dw = __shfl(wgt, l, 64);
    if (lane == d) {
      pick = dg * INIT_GROUP + l;
      wpx = dw;
    }
  }
  if (!mine) return;
  const float *jit = roi ? jit_roi + 2 * (size_t)i : jit_out + 2 * (size_t)(i - a.n_roi);
  const float sc = clamp_scale(roi ? 0.5 * sqrt((double)Wt / ((double)a.n_roi * (double)wpx))
                                   : 0.5 * sqrt((double)O / (double)a.n_out));
  const int py = pick / a.W, px = pick - py * a.W;
  xy[2 * i] = f32_add(f32_add((float)px, 0.5f), jit[0]);
  xy[2 * i + 1] = f32_add(f32_add((float)py, 0.5f), jit[1]);
  chol[3 * i] = sc;
  chol[3 * i + 1] = 0.f;
  chol[3 * i + 2] = sc;
#pragma unroll
  for (int ch = 0; ch < 3; ++ch)
    rgb[3 * i + ch] = (float)((double)a.T[ch * (size_t)HW + pick] * a.kappa);
  if (picked) picked[i] = pick;
}

}  // namespace

}  // namespace gs2d

using namespace gs2d;

extern "C" size_t gs2d_init_workspace_bytes(int32_t W, int32_t H) {
  InitLayout L;
  return init_layout(W, H, &L) ? L.total : 0;
}

extern "C" int gs2d_init_plain(int32_t W, int32_t H, const float *target, const uint8_t *roi_mask,
                               int32_t n_roi, const int64_t *pick_roi, const float *jit_roi,
                               int32_t n_out, const int64_t *pick_out, const float *jit_out,
                               float *xy, float *chol, float *rgb, int32_t *picked, void *ws,
                               size_t ws_bytes, void *stream) {
  try {
    InitLayout L;
    if (!init_layout(W, H, &L)) return GS2D_EINVAL;
    if (n_roi < 0 || n_out < 0 || n_roi + n_out < 1 || n_roi + (long long)n_out > 65536)
      return GS2D_EINVAL;
    if (!target || !roi_mask || !xy || !chol || !rgb || !ws) return GS2D_EINVAL;
    if ((n_roi > 0 && (!pick_roi || !jit_roi)) || (n_out > 0 && (!pick_out || !jit_out)))
      return GS2D_EINVAL;
    if (reinterpret_cast<uintptr_t>(ws) & 255) return GS2D_EINVAL;
    if (ws_bytes < L.total) return GS2D_ENOSPACE;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    const size_t HW = (size_t)W * H;
    const double kappa = 1.0 / (2.0 * M_PI * 0.25 * (1.0 - std::exp(-4.5)));
    hipLaunchKernelGGL(k_init_groups, dim3(L.n_chunks), dim3(INIT_LEVELS), 0, st, W, H, L.n_groups,
                       L.chunk_groups, target, roi_mask, at<long long>(ws, L.gqm),
                       at<long long>(ws, L.gqa), at<int>(ws, L.gr), at<long long>(ws, L.part));
    const DrawArgs a{W,
                     H,
                     n_roi,
                     n_out,
                     L.n_groups,
                     L.chunk_groups,
                     L.n_chunks,
                     target,
                     roi_mask,
                     at<const long long>(ws, L.gqm),
                     at<const long long>(ws, L.gqa),
                     at<const long long>(ws, L.part),
                     at<const int>(ws, L.gr),
                     kappa};
    constexpr int per_block = INIT_WAVES * INIT_DRAWS;
    hipLaunchKernelGGL(k_init_draw, dim3((n_roi + n_out + per_block - 1) / per_block),
                       dim3(INIT_BLOCK), 0, st, a, pick_roi, jit_roi, pick_out, jit_out, xy, chol,
                       rgb, picked);
    return hipGetLastError() == hipSuccess ? GS2D_OK : GS2D_EHIP;
  } catch (...) {
    return GS2D_EHIP;
  }
}
