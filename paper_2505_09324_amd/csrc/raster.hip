// Tile rasteriser for Eq. 2 (accumulated summation, Sec. 3.1) and its
// backward pass.
//
// SPLIT workgroups per TILE x TILE screen tile.  Each wavefront owns a sub-block
// 8 pixels wide and 8*PPL pixels tall: lane (lx, ly) = (lane & 7, lane >> 3)
// handles the PPL vertically adjacent pixels (x0 + lx, y0 + ly*PPL + k),
// which share d_x, u1 = d_x / l1 and u1^2.  The tile's Gaussian list is
// staged through LDS in chunks; while staging, each Gaussian's 3-sigma box
// and its cutoff ellipse's cut with each row of sub-blocks select the
// sub-blocks it can reach, and each wavefront compacts the chunk into its own
// list.
//
// Per (pixel, Gaussian), with d = (x+1/2, y+1/2) - mu and u = L^-1 d:
//   u1 = d1 / l1;  u2 = (d2 - l2 u1) / l3;  q = u1^2 + u2^2
//   w = exp(-q/2) if q <= 9 else 0;  C += c' w
// Backward, with g = dL/dC at the pixel, s = (g . c') w, v = L^-T u:
//   dL/dmu += s v;  dL/dl1 += s v1 u1;  dL/dl2 += s v2 u1;  dL/dl3 += s v2 u2;
//   dL/dc' += g w.
// The backward takes 16 Gaussians of a list at a time, each lane summing one
// over its row's pixels; those left over go one by one, their eight per-lane
// sums reduced across the wavefront by a transposing butterfly (each exchange
// halves the values a lane carries).  The sums are added into an LDS accumulator
// shared by the workgroup's wavefronts and flushed with one global atomic per
// (workgroup, Gaussian, parameter).
#include "raster_tile.h"

namespace gs2d {

// ----------------------------------------------------------------- forward --
template <int TILE, int PPL, int SPLIT, int LS>
__global__ void __launch_bounds__((Cfg<TILE, PPL, SPLIT, LS>::NT)) GS2D_RASTER_OCCUPANCY
k_render_fwd(FrameArgs f, const float *__restrict__ target, float *__restrict__ img,
             float *__restrict__ dl_dimg, float *__restrict__ loss_part, float grad_scale,
             int n_tiles) {
  using C = Cfg<TILE, PPL, SPLIT, LS>;
  __shared__ Smem<C> S;
  __shared__ float xch[C::XCH];
  int part;
  const int tile = tile_of_block<SPLIT>(&part);
  if (SPLIT > 1 && tile >= n_tiles) return;
  const int tx = tile % f.TX, ty = tile / f.TX;
  const int beg = f.tile_start[tile], end = f.tile_start[tile + 1];
  int px, py0;
  pixel_of_thread<C, TILE, PPL>(tx, ty, &px, &py0, part);
  const float pxc = (float)px + 0.5f, pyc0 = (float)py0 + 0.5f;
  const unsigned inside = inside_mask<PPL>(f, px, py0);
  float acc[PPL][3] = {};
  for (int c = beg; c < end; c += C::CH) {
    const int cnt = min(C::CH, end - c);
    if (c != beg) __syncthreads();
    stage_chunk<C, TILE>(S, f.keys, c, cnt, tx, ty, f.W, f.H, f.geom, f.rgb, nullptr, part);
    __syncthreads();
    int kb, ke;
    list_run<C>(compact_chunk<C>(S, cnt), &kb, &ke);
    fwd_chunk<C, PPL, false>(S, kb, ke, pxc, pyc0, inside, acc);
  }
  exchange_sums<C, PPL>(xch, acc);
  const int w = threadIdx.x >> 6;
  if (w >= C::NB) return;  // the first wavefront of a sub-block writes it
  float l = 0.f;
  const size_t HW = (size_t)f.W * f.H;
#pragma unroll
  for (int r = 0; r < PPL; ++r) {
    if (!((inside >> r) & 1u)) continue;
    const size_t p = (size_t)(py0 + r) * f.W + px;
    if (img) {
      img[p] = acc[r][0];
      img[HW + p] = acc[r][1];
      img[2 * HW + p] = acc[r][2];
    }
    if (target) {
      const float r0 = acc[r][0] - target[p], r1 = acc[r][1] - target[HW + p],
                  r2 = acc[r][2] - target[2 * HW + p];
      l += r0 * r0 + r1 * r1 + r2 * r2;
      if (dl_dimg) {
        dl_dimg[p] = r0 * grad_scale;
        dl_dimg[HW + p] = r1 * grad_scale;
        dl_dimg[2 * HW + p] = r2 * grad_scale;
      }
    }
  }
  if (loss_part) wave_loss(l, loss_part + tile * C::NWT + part * C::NB + w);
}

// ---------------------------------------------------------------- backward --
template <int TILE, int PPL, int SPLIT, int LS>
__global__ void __launch_bounds__((Cfg<TILE, PPL, SPLIT, LS>::NT)) GS2D_RASTER_OCCUPANCY
k_render_bwd(FrameArgs f, const float *__restrict__ dl_dimg, float *__restrict__ g_xy,
             float *__restrict__ g_chol, float *__restrict__ g_rgb, int n_tiles) {
  using C = Cfg<TILE, PPL, SPLIT, LS>;
  __shared__ Smem<C> S;
  __shared__ float acc[C::CH * 8];
  int part;
  const int tile = tile_of_block<SPLIT>(&part);
  if (SPLIT > 1 && tile >= n_tiles) return;
  const int tx = tile % f.TX, ty = tile / f.TX;
  const int beg = f.tile_start[tile], end = f.tile_start[tile + 1];
  if (beg >= end) return;
  int px, py0;
  pixel_of_thread<C, TILE, PPL>(tx, ty, &px, &py0, part);
  const float pxc = (float)px + 0.5f, pyc0 = (float)py0 + 0.5f;
  const unsigned inside = inside_mask<PPL>(f, px, py0);
  float g[PPL][3];
  const size_t HW = (size_t)f.W * f.H;
#pragma unroll
  for (int r = 0; r < PPL; ++r) {
    g[r][0] = g[r][1] = g[r][2] = 0.f;
    if ((inside >> r) & 1u) {
      const size_t p = (size_t)(py0 + r) * f.W + px;
      g[r][0] = dl_dimg[p];
      g[r][1] = dl_dimg[HW + p];
      g[r][2] = dl_dimg[2 * HW + p];
    }
  }
  for (int c = beg; c < end; c += C::CH) {
    const int cnt = min(C::CH, end - c);
    if (c != beg) __syncthreads();
    stage_chunk<C, TILE>(S, f.keys, c, cnt, tx, ty, f.W, f.H, f.geom, f.rgb, nullptr, part);
    for (int i = threadIdx.x; i < cnt * 8; i += C::NT) acc[i] = 0.f;
    __syncthreads();
    int kb, ke;
    list_run<C>(compact_chunk<C>(S, cnt), &kb, &ke);
    bwd_chunk<C, PPL, false>(S, acc, kb, ke, pxc, pyc0, g);
    __syncthreads();
    flush_grads<C, true>(S, acc, cnt, g_xy, g_chol, g_rgb);
  }
}

// ------------------------------------------- fused forward + loss + backward --
template <int TILE, int PPL, int SPLIT, int LS, bool BATCH = true>
__global__ void __launch_bounds__((Cfg<TILE, PPL, SPLIT, LS>::NT)) GS2D_RASTER_OCCUPANCY
k_render_fused(FrameArgs f, const float *__restrict__ target, float *__restrict__ loss_part,
               float grad_scale, float *__restrict__ g_xy, float *__restrict__ g_chol,
               float *__restrict__ g_rgb, int n_tiles) {
  using C = Cfg<TILE, PPL, SPLIT, LS>;
  __shared__ Smem<C> S;
  __shared__ float acc[C::CH * 8];
  __shared__ float xch[C::XCH];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (f.lazy_misc && f.lazy_misc[MISC_STALE]) {
      const bool ok = !(f.lazy_misc[MISC_STICKY] & (int)STATUS_STALLED);
      f.lazy_misc[MISC_LISTS_LO] = ok ? (int)f.sig_lo : 0;
      f.lazy_misc[MISC_LISTS_HI] = ok ? (int)f.sig_hi : 0;
      f.lazy_misc[MISC_STALE] = 0;
    }
    if (f.tick) *f.tick += 1;
  }
  int part;
  const int tile = tile_of_block<SPLIT>(&part);
  if (SPLIT > 1 && tile >= n_tiles) return;
  fused_tile<C, TILE, PPL, true, true, BATCH>(S, acc, xch, f, tile, target,
                                              loss_part + tile * C::NWT, grad_scale, g_xy, g_chol,
                                              g_rgb, part);
}

// ------------------------------------------------- in-cutoff pair counting --
// Number of (pixel, Gaussian) pairs with q <= 9 inside the frame: the terms
// Eq. 2 actually sums (the algorithmic work of one render).
template <int TILE>
__global__ void __launch_bounds__((Cfg<TILE, 1>::NT))
k_count_pairs(FrameArgs f, unsigned long long *__restrict__ out) {
  using C = Cfg<TILE, 1>;
  __shared__ Smem<C> S;
  const int tile = blockIdx.x;
  const int tx = tile % f.TX, ty = tile / f.TX;
  const int beg = f.tile_start[tile], end = f.tile_start[tile + 1];
  int px, py;
  pixel_of_thread<C, TILE, 1>(tx, ty, &px, &py);
  const float pxc = (float)px + 0.5f, pyc = (float)py + 0.5f;
  const bool inside = px < f.W && py < f.H;
  const int w = threadIdx.x >> 6;
  unsigned int n = 0;
  for (int c = beg; c < end; c += C::CH) {
    const int cnt = min(C::CH, end - c);
    __syncthreads();
    stage_chunk<C, TILE>(S, f.keys, c, cnt, tx, ty, f.W, f.H, f.geom, nullptr);
    __syncthreads();
    const int len = compact_chunk<C>(S, cnt);
    __syncthreads();
    for (int k = 0; k < len; ++k) {
      const int j = S.list[w][k];
      const float4 A = S.A[j], B = S.B[j];
      const float u1 = (pxc - A.x) * A.z;
      const float u2 = pair_base(A, u1, pyc - A.y) * B.x;
      n += (inside && pair_q<1>(u1, u1 * u1, u2) <= CUTOFF_QS) ? 1u : 0u;
    }
  }
  for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o, 64);
  if ((threadIdx.x & 63) == 0 && n) atomicAdd(out, (unsigned long long)n);
}

// ------------------------------------------------------------- loss reduce --
__global__ void __launch_bounds__(1024)
k_loss_reduce(const float *__restrict__ part, int n, float scale, float *__restrict__ out) {
  __shared__ double red[16];
  double s = 0.0;
  s = thread_sum_parts(part, n);
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < 16; ++w) t += red[w];
    *out = (float)(t * (double)scale);
  }
}

// ------------------------------------------------------------------ launch --
static FrameArgs frame_args(const Layout &L, void *ws, const float *rgb) {
  FrameArgs f;
  f.W = L.W;
  f.H = L.H;
  f.TX = L.TX;
  f.geom = at<const float4>(ws, L.geom);
  f.keys = at<const uint32_t>(ws, L.keys_sorted());
  f.tile_start = at<const int>(ws, L.tile_start);
  f.rgb = rgb;
  f.active = nullptr;
  f.lazy_misc = nullptr;
  f.sig_lo = f.sig_hi = 0;
  f.tick = nullptr;
  return f;
}

static float grad_scale(const Layout &L) { return (float)(2.0 / (3.0 * L.W * (double)L.H)); }

// KERNEL<TT, PP, SPLIT, LS> for the layout's variant.
#define GS2D_LAUNCH_LS(KERNEL, TT, PP, SP, LS, ...)                             \
  hipLaunchKernelGGL((KERNEL<TT, PP, SP, LS>), dim3(split_grid(L.n_tiles, SP)), \
                     dim3(Cfg<TT, PP, SP, LS>::NT), 0, st, __VA_ARGS__, L.n_tiles)
#define GS2D_LAUNCH(KERNEL, TT, PP, SP, SPS, ...)                        \
  if (!done && L.T == TT && L.ppl == PP) {                               \
    const int share = raster_share(L.loss_parts);                        \
    if (share == 4) GS2D_LAUNCH_LS(KERNEL, TT, PP, SPS, 4, __VA_ARGS__); \
    else if (share == 2) GS2D_LAUNCH_LS(KERNEL, TT, PP, SPS, 2, __VA_ARGS__); \
    else GS2D_LAUNCH_LS(KERNEL, TT, PP, SP, 1, __VA_ARGS__);             \
    done = true;                                                         \
  }

hipError_t launch_render_fwd(const Layout &L, void *ws, const float *rgb, const float *target,
                             float *img, float *dl_dimg, hipStream_t st) {
  FrameArgs f = frame_args(L, ws, rgb);
  float *lp = target ? at<float>(ws, L.loss_part) : nullptr;
  bool done = false;
#define CALL(TT, PP, SP, SPS) \
  GS2D_LAUNCH(k_render_fwd, TT, PP, SP, SPS, f, target, img, dl_dimg, lp, grad_scale(L))
  GS2D_VARIANTS(CALL)
#undef CALL
  return done ? hipGetLastError() : hipErrorInvalidValue;
}

hipError_t launch_render_bwd(const Layout &L, void *ws, const float *rgb, const float *dl_dimg,
                             float *g_xy, float *g_chol, float *g_rgb, hipStream_t st) {
  FrameArgs f = frame_args(L, ws, rgb);
  bool done = false;
#define CALL(TT, PP, SP, SPS) \
  GS2D_LAUNCH(k_render_bwd, TT, PP, SP, SPS, f, dl_dimg, g_xy, g_chol, g_rgb)
  GS2D_VARIANTS(CALL)
#undef CALL
  return done ? hipGetLastError() : hipErrorInvalidValue;
}

hipError_t launch_render_fused(const Layout &L, void *ws, const float *rgb, const float *target,
                               float *g_xy, float *g_chol, float *g_rgb, hipStream_t st,
                               const uint8_t *active, bool lazy, int32_t *tick,
                               bool fixed_sums) {
  FrameArgs f = frame_args(L, ws, rgb);
  f.active = active;
  if (lazy) {
    f.lazy_misc = at<int>(ws, L.misc);
    f.sig_lo = L.sig_lo;
    f.sig_hi = L.sig_hi;
  }
  f.tick = tick;
  float *lp = at<float>(ws, L.loss_part);
  bool done = false;
  // Quantisation-aware fits.  A quantiser turns the last bit of a parameter near
  // a rounding boundary into a whole step of its code, and the gradients of its
  // neighbours follow, so a sum formed in another order moves single parameters
  // by 1e-3: these fits keep one form of every sum whatever the frame's size and
  // the lists' lengths.  1280x720 / 15,000, 20 iterations: 925 us, with the
  // parts, shares and batches of the other fits 787.
#define CALL_FIXED(TT, PP, SP, SPS)                                                            \
  if (!done && L.T == TT && L.ppl == PP) {                                                     \
    hipLaunchKernelGGL((k_render_fused<TT, PP, 1, 1, false>), dim3(L.n_tiles),                 \
                       dim3(Cfg<TT, PP>::NT), 0, st, f, target, lp, grad_scale(L), g_xy, g_chol, \
                       g_rgb, L.n_tiles);                                                      \
    done = true;                                                                               \
  }
  if (fixed_sums) {
    GS2D_VARIANTS(CALL_FIXED)
    return done ? hipGetLastError() : hipErrorInvalidValue;
  }
#undef CALL_FIXED
#define CALL(TT, PP, SP, SPS)                                                        \
  GS2D_LAUNCH(k_render_fused, TT, PP, SP, SPS, f, target, lp, grad_scale(L), g_xy, g_chol, \
              g_rgb)
  GS2D_VARIANTS(CALL)
#undef CALL
  return done ? hipGetLastError() : hipErrorInvalidValue;
}

hipError_t launch_count_pairs(const Layout &L, void *ws, unsigned long long *out, hipStream_t st) {
  FrameArgs f = frame_args(L, ws, nullptr);
  hipError_t e = launch_fill_zero_u32(reinterpret_cast<uint32_t *>(out), 2, st);
  if (e != hipSuccess) return e;
  switch (L.T) {
    case 8: hipLaunchKernelGGL(k_count_pairs<8>, dim3(L.n_tiles), dim3(64), 0, st, f, out); break;
    case 16: hipLaunchKernelGGL(k_count_pairs<16>, dim3(L.n_tiles), dim3(256), 0, st, f, out); break;
    case 32: hipLaunchKernelGGL(k_count_pairs<32>, dim3(L.n_tiles), dim3(1024), 0, st, f, out); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_loss_reduce(const Layout &L, void *ws, float *loss, hipStream_t st) {
  hipLaunchKernelGGL(k_loss_reduce, dim3(1), dim3(1024), 0, st, at<const float>(ws, L.loss_part),
                     L.loss_parts, (float)(1.0 / (3.0 * L.W * (double)L.H)), loss);
  return hipGetLastError();
}

}  // namespace gs2d
