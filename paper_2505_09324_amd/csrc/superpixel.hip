// Superpixel initialisation of the ROI Gaussians (Sec. 3.2.A, Fig. 2):
// K-means clustering of the ROI pixels in (x, y, colour) from K seed pixels,
// then one Gaussian per segment from the segment's centre, covariance and
// mean colour.
//
// Clustering (SLIC-style, one grid of cells of side S):
//   S = max(1, rint(sqrt(R / K))) (R ROI pixels, FP64, ties to even),
//   w = (m / S)^2 in FP32; pixel p joins the centre k minimising
//   D = ((dr^2 + dg^2) + db^2) + w (dx^2 + dy^2)  (FP32, this order, no
//   contraction; d = pixel - centre, pixel position = its centre) among the
//   centres whose cell floor(c / S) lies within one cell of the pixel's
//   cell x // S, ties to the lowest k.  Centres are exact means: positions
//   sum / n + 1/2 and colours sum / (n 65536) in FP64 from int64 sums of the
//   pixel indices and of the colours in 1/65536 units; an empty segment keeps
//   its centre.  After the last round each non-empty segment gives
//     mu = mean + 1/2,  L = chol(cov + I/12),
//     c' = colour sum / (2 pi l1 l3 (1 - e^-4.5))
//   (FP64, the order written in seg_gaussian, rounded to FP32 once), so the
//   Gaussian's rendered mass under the q <= 9 cutoff is the segment's colour
//   total; empty segments keep the caller's Gaussian.
//
// Kernels per round: k_sp_assign, whose blocks each take one 32 x 8 tile of
// pixels, collect the candidate centres of the tile's cells in LDS, label
// their pixels and add the segments' moments, first in LDS and then with one
// 64-bit integer atomic per (tile, segment, moment); and k_sp_update, which
// turns the moments into the new centres and chains each into its cell for
// the next round.  Integer sums do not depend on the atomics' order, so the
// result is deterministic.  S, the cell grid and w are computed on the
// device: the call never synchronises.
#include <climits>
#include <cmath>

#include "gs2d_internal.h"

namespace gs2d {
namespace {

constexpr int SP_BLOCK = 256;
constexpr int SP_MAX_K = 65536;
constexpr int SP_MAX_ITERS = 100;
constexpr double SP_COLOUR = 65536.0;
constexpr double SP_SCALE_2PI = 65536.0 * 2.0 * 3.14159265358979323846;
constexpr double SP_MASS = 0.98889100346175773;  // 1 - exp(-4.5)

// meta: tiles with an ROI pixel, roi_all, S, ncx, ncy, w (float bits)
enum { M_TILES = 0, M_ALL, M_S, M_NCX, M_NCY, M_W, M_N };

// Pixel tile of one assignment block: 32 pixels wide, so that a row of the
// frame is read in whole 128-byte lines, and 8 or 16 high, with one or two
// pixels of a column per thread (PX).
constexpr int SP_TW = 32;
template <int PX>
constexpr int SP_TH = 8 * PX;
static_assert(SP_TW * SP_TH<1> == SP_BLOCK, "one pixel per thread");
constexpr int SP_CAP = 256;        // candidate centres of a tile held in LDS
constexpr int SP_SEGS = 1024;       // most segments the tiles are counted in
constexpr int SP_SEG_MIN = 16;      // fewest tiles of a segment: four per wavefront

// A cell's chain head is (round + 1) << 17 | centre: a head left by another
// round reads as an empty cell, so the heads are cleared once per call and
// not once per round.
constexpr int SP_TAG = 17;
static_assert(SP_MAX_K <= 1 << SP_TAG && ((SP_MAX_ITERS + 1LL) << SP_TAG) < (1LL << 31), "tag");

// One centre as the assignment reads it: position, colour and the next centre
// of its cell (-1: none), so that one step along a chain is one 32-byte load.
struct alignas(16) SpCentre {
  float x, y, r, g;
  float b;
  int next, pad[2];
};

struct SpLayout {
  size_t cen, sums, sums2, rec, heads, seg, seg_tiles, tiles, meta, total;
  int px, tx, ty, n_tiles, seg_len, n_segs;  // px: pixels per thread (tile height 8 px)
};

bool sp_layout(int W, int H, int K, SpLayout *L) {
  if (W < 1 || H < 1 || K < 1 || K > SP_MAX_K) return false;
  const long long HW = (long long)W * H;
  if (HW > (1LL << 28)) return false;
  size_t o = 0;
  auto take = [&o](size_t b) {
    const size_t a = o;
    o = (o + b + 255) & ~(size_t)255;
    return a;
  };
  // Two pixels per thread share the candidates' reads but lengthen the chain
  // of one block.  An assignment takes 9 us at 640 x 360 with one pixel and 12
  // with two; at 1920 x 1080 a quarter of the frame as ROI (2163 tiles of one
  // pixel per thread) no longer fits the 2048 resident blocks: 18.5 and 16.9.
  L->tx = (W + SP_TW - 1) / SP_TW;
  L->px = (long long)L->tx * ((H + SP_TH<1> - 1) / SP_TH<1>) > 4 * 2048 * 7 / 8 ? 2 : 1;
  const int th = SP_TH<1> * L->px;
  L->ty = (H + th - 1) / th;
  L->n_tiles = L->tx * L->ty;
  L->seg_len = std::max(SP_SEG_MIN, (L->n_tiles + SP_SEGS - 1) / SP_SEGS);
  L->n_segs = (L->n_tiles + L->seg_len - 1) / L->seg_len;
  L->cen = take((size_t)2 * 5 * K * 4);        // two centre sets, SoA x y r g b
  L->sums = take((size_t)8 * K * 8);           // n, Sx, Sy, Sr, Sg, Sb, -, - per centre
  L->sums2 = take((size_t)4 * K * 8);          // Sxx, Sxy, Syy, - (last round)
  L->rec = take((size_t)K * sizeof(SpCentre)); // the centres of the next assignment
  L->heads = take((size_t)HW * 4);             // first centre of every cell, tagged
  L->seg = take((size_t)L->n_segs * 8);        // per segment: ROI pixels, ROI tiles
  L->seg_tiles = take((size_t)L->n_tiles * 4); // the ROI tiles of every segment
  L->tiles = take((size_t)L->n_tiles * 4);     // all ROI tiles
  L->meta = take(M_N * 4);
  L->total = o;
  return true;
}

__device__ inline long long colour_code(float v) { return (long long)rint((double)v * SP_COLOUR); }

// The start of a call.  The first n_segs blocks each count one segment of
// seg_len tiles: its ROI pixels and the list of its tiles that hold one (a
// wavefront per tile, four pixels of a row per lane); k_sp_seed joins the
// segments, so that no counter is shared (one atomic per block on one word
// measured 15 us at 1920 x 1080).  Every block clears a share of the moments
// and the cell heads and places a share of the seeds.
__global__ void __launch_bounds__(SP_BLOCK)
k_sp_begin(int W, int H, int K, int px, int tx, int n_tiles, int seg_len, int n_segs,
           const float *__restrict__ T, const uint8_t *__restrict__ mask,
           const int32_t *__restrict__ seeds, float *__restrict__ cen,
           unsigned long long *__restrict__ sums, unsigned long long *__restrict__ sums2,
           int *__restrict__ heads, int2 *__restrict__ seg, int *__restrict__ seg_tiles) {
  __shared__ int n_found, n_roi;
  const size_t HW = (size_t)W * H;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if ((int)blockIdx.x < n_segs) {
    if (threadIdx.x == 0) n_found = n_roi = 0;
    __syncthreads();
    const int t0 = blockIdx.x * seg_len, t1 = min(n_tiles, t0 + seg_len);
    int roi = 0;
    for (int tb = t0 + 4 * wid; tb < t1; tb += 4 * (SP_BLOCK / 64)) {
      int c[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {  // four tiles' loads in flight
        const int t = tb + j;
        const int x = (t % tx) * SP_TW + (lane & 7) * 4, y0 = (t / tx) * SP_TH<1> * px;
        c[j] = 0;
        for (int y = y0 + (lane >> 3); t < t1 && y < min(H, y0 + SP_TH<1> * px); y += SP_TH<1>) {
          const uint8_t *row = mask + (size_t)y * W;
#pragma unroll
          for (int i = 0; i < 4; ++i) c[j] += x + i < W && row[x + i] != 0;
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (__ballot(c[j] > 0) && lane == 0) seg_tiles[t0 + atomicAdd(&n_found, 1)] = tb + j;
        roi += c[j];
      }
    }
    for (int o = 32; o > 0; o >>= 1) roi += __shfl_xor(roi, o, 64);
    if (lane == 0 && roi) atomicAdd(&n_roi, roi);
    __syncthreads();
    if (threadIdx.x == 0) seg[blockIdx.x] = make_int2(n_roi, n_found);
  }
  const size_t i0 = blockIdx.x * (size_t)SP_BLOCK + threadIdx.x;
  const size_t nt = (size_t)gridDim.x * SP_BLOCK;
  for (size_t i = i0; i < HW; i += nt) heads[i] = 0;
  for (size_t i = i0; i < (size_t)8 * K; i += nt) sums[i] = 0;
  for (size_t i = i0; i < (size_t)4 * K; i += nt) sums2[i] = 0;
  for (size_t k = i0; k < (size_t)K; k += nt) {
    const int p = min(max(seeds[k], 0), (int)(HW - 1));
    cen[k] = (float)(p % W) + 0.5f;
    cen[K + k] = (float)(p / W) + 0.5f;
#pragma unroll
    for (int c = 0; c < 3; ++c)
      cen[(2 + c) * K + k] = (float)((double)colour_code(T[c * HW + p]) / SP_COLOUR);
  }
}

// Centre k into its cell's chain for round `round`.
__device__ inline void sp_chain(int k, float x, float y, float r, float g, float b, int S, int ncx,
                                int ncy, int round, int *__restrict__ heads,
                                SpCentre *__restrict__ rec) {
  const float fS = (float)S;
  // centres are means of pixel centres, so these lie inside the grid; the
  // clamp only keeps the index in range
  const int cx = min(max((int)floorf(__fdiv_rn(x, fS)), 0), ncx - 1);
  const int cy = min(max((int)floorf(__fdiv_rn(y, fS)), 0), ncy - 1);
  const int old = atomicExch(&heads[(size_t)cy * ncx + cx], ((round + 1) << SP_TAG) | k);
  const int next = (old >> SP_TAG) == round + 1 ? old & ((1 << SP_TAG) - 1) : -1;
  float4 *q = reinterpret_cast<float4 *>(rec + k);
  q[0] = make_float4(x, y, r, g);
  q[1] = make_float4(b, __int_as_float(next), 0.f, 0.f);
}

// Every block adds up the segments (at most SP_SEGS / SP_BLOCK per thread):
// the ROI count gives S, the cell grid and w, which block 0 records for the
// later kernels; a share of the segments' tile lists goes to its place in the
// whole list, and the seeds are chained into their cells.
__global__ void __launch_bounds__(SP_BLOCK)
k_sp_seed(int W, int H, int K, float m, int seg_len, int n_segs, const int2 *__restrict__ seg,
          const int *__restrict__ seg_tiles, int *__restrict__ tiles,
          const float *__restrict__ cen, int *__restrict__ meta, int *__restrict__ heads,
          SpCentre *__restrict__ rec) {
  constexpr int PER = SP_SEGS / SP_BLOCK;
  __shared__ int before[SP_SEGS + 1];  // tiles of the earlier segments
  __shared__ int red[2][SP_BLOCK / 64];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  int cnt[PER], c = 0, roi = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int i = tid * PER + j;
    const int2 v = i < n_segs ? seg[i] : make_int2(0, 0);
    roi += v.x;
    c += cnt[j] = v.y;
  }
  int x = c;
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(x, o, 64);
    if (lane >= o) x += u;
  }
  for (int o = 32; o > 0; o >>= 1) roi += __shfl_xor(roi, o, 64);
  if (lane == 63) red[0][wid] = x, red[1][wid] = roi;
  __syncthreads();
  int run = x - c, total = 0;
  long long R = 0;
  for (int w = 0; w < SP_BLOCK / 64; ++w) {
    if (w < wid) run += red[0][w];
    total += red[0][w];
    R += red[1][w];
  }
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    before[tid * PER + j] = run;
    run += cnt[j];
  }
  if (tid == SP_BLOCK - 1) before[SP_SEGS] = run;
  __syncthreads();
  for (int i = blockIdx.x * (SP_BLOCK / 64) + wid; i < n_segs; i += gridDim.x * (SP_BLOCK / 64))
    for (int j = lane; j < before[i + 1] - before[i]; j += 64)
      tiles[before[i] + j] = seg_tiles[i * seg_len + j];
  const int all = R == 0;
  if (all) R = (long long)W * H;
  const int S = max(1, (int)rint(sqrt((double)R / (double)K)));
  const int ncx = (W + S - 1) / S, ncy = (H + S - 1) / S;
  if (blockIdx.x == 0 && tid == 0) {
    const float r = __fdiv_rn(m, (float)S);
    meta[M_TILES] = total;
    meta[M_ALL] = all;
    meta[M_S] = S;
    meta[M_NCX] = ncx;
    meta[M_NCY] = ncy;
    meta[M_W] = __float_as_int(f32_mul(r, r));
  }
  const int k = blockIdx.x * SP_BLOCK + tid;
  if (k < K)
    sp_chain(k, cen[k], cen[K + k], cen[2 * K + k], cen[3 * K + k], cen[4 * K + k], S, ncx, ncy, 0,
             heads, rec);
}

// A pixel and its nearest candidate so far: least D, ties to the lowest
// centre index.
struct SpPixel {
  float py, r, g, b;
  float D;
  int k, slot;
};

__device__ inline void sp_try(SpPixel &q, bool ok, float dx2, float w, float cy, float cr,
                              float cg, float cb, int k, int slot) {
  const float dr = f32_sub(q.r, cr), dg = f32_sub(q.g, cg), db = f32_sub(q.b, cb);
  const float dy = f32_sub(q.py, cy);
  const float dcol = f32_add(f32_add(f32_mul(dr, dr), f32_mul(dg, dg)), f32_mul(db, db));
  const float dpos = f32_add(dx2, f32_mul(dy, dy));
  const float D = f32_add(dcol, f32_mul(w, dpos));
  if (ok && (D < q.D || (D == q.D && k < q.k))) {
    q.D = D;
    q.k = k;
    q.slot = slot;
  }
}

// Labels of one round and the segments' moments.  Grid-stride over the tiles
// that hold an ROI pixel (all tiles for an empty mask, and when the labels
// of the whole frame are asked for, which only the last round writes).  A
// tile's window is the cells of its pixels and one more on every side, row
// by row, so that the three cells of a row around a pixel are one run of the
// LDS pool.  LDS accumulators: {n | Slx << 16 | Sly << 32}, the three colour
// sums, and in the last round {Slxx | Slxy << 20 | Slyy << 40}, with lx, ly
// the pixel's place in the tile (a tile's sums fit these fields).  Where the
// window holds more than SP_CAP centres (many seeds on few pixels) the
// pixels walk the chains in memory and add to the moments there directly.
// Bound by the vector unit and by latency: at 1920 x 1080 with 21,000
// segments (S = 5) a pixel scores about ten candidates, and a block spends 3
// us on reaching them (meta and tile, cell heads, centres: three dependent
// loads) and as long on scoring.
template <int PX, bool LAST>
__global__ void __launch_bounds__(SP_BLOCK)
k_sp_assign(int W, int H, int tx, int n_tiles, int round, const float *__restrict__ T,
            const uint8_t *__restrict__ mask, const int *__restrict__ meta,
            const int *__restrict__ tiles, const int *__restrict__ heads,
            const SpCentre *__restrict__ rec, unsigned long long *__restrict__ sums,
            unsigned long long *__restrict__ sums2,
            int32_t *__restrict__ labels) {
  constexpr int TH = SP_TH<PX>;
  constexpr int CELLS = (SP_TW + 2) * (TH + 2);  // cells of the window at S = 1
  __shared__ float4 pool[SP_CAP];   // x, y, r, g
  __shared__ float2 pool2[SP_CAP];  // b, centre index
  __shared__ unsigned long long acc[LAST ? 5 : 4][SP_CAP];
  __shared__ int start[CELLS + 1];
  __shared__ int red[SP_BLOCK / 64];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const size_t HW = (size_t)W * H;
  int listed = (int)blockIdx.x < n_tiles ? tiles[blockIdx.x] : 0;  // read beside meta
  const int S = meta[M_S], ncx = meta[M_NCX], ncy = meta[M_NCY], all = meta[M_ALL];
  const float w = __int_as_float(meta[M_W]);
  const bool every = all || (LAST && labels);
  const int n = every ? n_tiles : meta[M_TILES];
  const int tag = round + 1, kmask = (1 << SP_TAG) - 1;
  for (int i = blockIdx.x; i < n; i += gridDim.x) {
    const int t = every ? i : listed;
    if (i + (int)gridDim.x < n_tiles) listed = tiles[i + gridDim.x];
    const int X0 = (t % tx) * SP_TW, Y0 = (t / tx) * TH;
    const int lx = tid & (SP_TW - 1), x = X0 + lx, ly0 = PX * (tid / SP_TW), y0 = Y0 + ly0;
    SpPixel px[PX];
    bool roi[PX], any = false;
#pragma unroll
    for (int j = 0; j < PX; ++j) {
      const bool inside = x < W && y0 + j < H;
      const size_t p = inside ? (size_t)(y0 + j) * W + x : 0;
      roi[j] = inside && (all || mask[p]);
      any |= roi[j];
      px[j] = {(float)(y0 + j) + 0.5f, T[p], T[HW + p], T[2 * HW + p], INFINITY, INT_MAX, -1};
    }
    // the window of cells
    const int cx0 = max(X0 / S - 1, 0), cx1 = min((min(X0 + SP_TW, W) - 1) / S + 1, ncx - 1);
    const int cy0 = max(Y0 / S - 1, 0), cy1 = min((min(Y0 + TH, H) - 1) / S + 1, ncy - 1);
    const int cw = cx1 - cx0 + 1, cells = cw * (cy1 - cy0 + 1);
    __syncthreads();  // the previous tile's LDS is free
    int total = 0;
    for (int c0 = 0; c0 < cells; c0 += SP_BLOCK) {
      const int c = c0 + tid;
      int first = -1, cnt = 0;
      if (c < cells) {
        const int h = heads[(size_t)(cy0 + c / cw) * ncx + cx0 + c % cw];
        first = (h >> SP_TAG) == tag ? h & kmask : -1;
      }
      // the cell's first two centres stay in registers (nearly all cells have
      // no more), the others are read again when the pool is filled
      float4 a0, b0, a1, b1;
      int k1 = -1, k2 = -1;
      if (first >= 0) {
        const float4 *q = reinterpret_cast<const float4 *>(rec + first);
        a0 = q[0];
        b0 = q[1];
        cnt = 1;
        k1 = __float_as_int(b0.y);
        if (k1 >= 0) {
          q = reinterpret_cast<const float4 *>(rec + k1);
          a1 = q[0];
          b1 = q[1];
          cnt = 2;
          k2 = __float_as_int(b1.y);
          for (int k = k2; k >= 0; k = rec[k].next) ++cnt;
        }
      }
      int v = cnt;
      for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(v, o, 64);
        if (lane >= o) v += u;
      }
      if (lane == 63) red[wid] = v;
      __syncthreads();
      int at = total + v - cnt;
      for (int q = 0; q < SP_BLOCK / 64; ++q) {
        if (q < wid) at += red[q];
        total += red[q];
      }
      if (c < cells) start[c] = at;
      auto put = [&](int k, const float4 &a, float cb) {
        if (at < SP_CAP) {
          pool[at] = a;
          pool2[at] = make_float2(cb, __int_as_float(k));
        }
        ++at;
      };
      if (cnt > 0) put(first, a0, b0.x);
      if (cnt > 1) put(k1, a1, b1.x);
      for (int k = k2; k >= 0 && at < SP_CAP;) {
        const float4 *q = reinterpret_cast<const float4 *>(rec + k);
        const float4 a = q[0], b = q[1];
        put(k, a, b.x);
        k = __float_as_int(b.y);
      }
      __syncthreads();
    }
    if (tid == 0) start[cells] = total;
    const bool pooled = total <= SP_CAP;
    if (pooled)
      for (int j = tid; j < total; j += SP_BLOCK) {
#pragma unroll
        for (int a = 0; a < (LAST ? 5 : 4); ++a) acc[a][j] = 0;
      }
    __syncthreads();
    if (any) {
      const float pxc = (float)x + 0.5f;
      // the candidate rows; two pixels may lie in adjacent rows of cells
      const int gx = x / S, ga = y0 / S, gb = (y0 + PX - 1) / S;
      const int ca = max(gx - 1, 0) - cx0, cb = min(gx + 1, ncx - 1) - cx0;
      const int cy_last = min(gb + 1, ncy - 1);
      int cy = max(ga - 1, 0);
      auto score = [&](int row, const float4 &a, const float2 &b, int slot) {
        const float dx = f32_sub(pxc, a.x), dx2 = f32_mul(dx, dx);
#pragma unroll
        for (int j = 0; j < PX; ++j)
          sp_try(px[j], PX == 1 || (roi[j] && (j == 0 ? row <= ga + 1 : row >= gb - 1)), dx2, w,
                 a.y, a.z, a.w, b.x, __float_as_int(b.y), slot);
      };
      for (; cy <= cy_last; ++cy) {
        if (pooled) {
          const int row = (cy - cy0) * cw, e = start[row + cb + 1];
          for (int j = start[row + ca]; j < e; ++j) score(cy, pool[j], pool2[j], j);
        } else {
          for (int cx = ca; cx <= cb; ++cx) {
            const int h = heads[(size_t)cy * ncx + cx0 + cx];
            for (int k = (h >> SP_TAG) == tag ? h & kmask : -1; k >= 0;) {
              const float4 *q = reinterpret_cast<const float4 *>(rec + k);
              const float4 a = q[0], b = q[1];
              score(cy, a, make_float2(b.x, __int_as_float(k)), -1);
              k = __float_as_int(b.y);
            }
          }
        }
      }
    }
#pragma unroll 1
    for (int j = 0; j < PX; ++j) {
      const SpPixel q = j == 0 ? px[0] : px[PX - 1];
      const int ly = ly0 + j, y = Y0 + ly;
      const bool hit = q.k != INT_MAX;
      if (LAST && labels && x < W && y < H) labels[(size_t)y * W + x] = hit ? q.k : -1;
      if (!hit) continue;
      const unsigned long long c0 = (unsigned long long)colour_code(q.r),
                               c1 = (unsigned long long)colour_code(q.g),
                               c2 = (unsigned long long)colour_code(q.b);
      if (pooled) {
        const int sl = q.slot;
        atomicAdd(&acc[0][sl], 1ull | (unsigned long long)lx << 16 | (unsigned long long)ly << 32);
        atomicAdd(&acc[1][sl], c0);
        atomicAdd(&acc[2][sl], c1);
        atomicAdd(&acc[3][sl], c2);
        if constexpr (LAST)
          atomicAdd(&acc[4][sl], (unsigned long long)(lx * lx) |
                                     (unsigned long long)(lx * ly) << 20 |
                                     (unsigned long long)(ly * ly) << 40);
      } else {
        unsigned long long *s = sums + 8 * (size_t)q.k;
        const unsigned long long ux = (unsigned long long)x, uy = (unsigned long long)y;
        atomicAdd(s, 1ull);
        atomicAdd(s + 1, ux);
        atomicAdd(s + 2, uy);
        atomicAdd(s + 3, c0);
        atomicAdd(s + 4, c1);
        atomicAdd(s + 5, c2);
        if constexpr (LAST) {
          atomicAdd(sums2 + 4 * (size_t)q.k, ux * ux);
          atomicAdd(sums2 + 4 * (size_t)q.k + 1, ux * uy);
          atomicAdd(sums2 + 4 * (size_t)q.k + 2, uy * uy);
        }
      }
    }
    if (!pooled) continue;  // uniform over the block
    __syncthreads();
    // eight adjacent lanes per segment: its atomics share two 32-byte blocks
    for (int e = tid; e < 8 * total; e += SP_BLOCK) {
      const int j = e >> 3, c = e & 7;
      const unsigned long long a = acc[0][j], cnt = a & 0xFFFF;
      if (cnt == 0 || c > 5) continue;
      const unsigned long long v = c == 0   ? cnt
                                   : c == 1 ? cnt * X0 + (a >> 16 & 0xFFFF)
                                   : c == 2 ? cnt * Y0 + (a >> 32)
                                            : acc[c - 2][j];
      atomicAdd(sums + 8 * (size_t)__float_as_int(pool2[j].y) + c, v);
    }
    if constexpr (LAST)
      for (int e = tid; e < 4 * total; e += SP_BLOCK) {
        const int j = e >> 2, c = e & 3;
        const unsigned long long a = acc[0][j], cnt = a & 0xFFFF;
        if (cnt == 0 || c > 2) continue;
        const unsigned long long b = acc[4][j], ux = X0, uy = Y0;
        const unsigned long long sx = a >> 16 & 0xFFFF, sy = a >> 32;
        const unsigned long long v =
            c == 0   ? cnt * ux * ux + 2 * ux * sx + (b & 0xFFFFF)
            : c == 1 ? cnt * ux * uy + ux * sy + uy * sx + (b >> 20 & 0xFFFFF)
                     : cnt * uy * uy + 2 * uy * sy + (b >> 40);
        atomicAdd(sums2 + 4 * (size_t)__float_as_int(pool2[j].y) + c, v);
      }
  }
}

// Segment Gaussian from exact moments s = n, Sx, Sy, Sxx, Sxy, Syy, Sr, Sg, Sb.
__device__ void seg_gaussian(const long long *s, float *xy, float *chol, float *rgb) {
#pragma clang fp contract(off)
  const double n = (double)s[0];
  const double ex = (double)s[1] / n, ey = (double)s[2] / n;
  const double vxx = ((double)s[3] / n - ex * ex) + 1.0 / 12.0;
  const double vxy = (double)s[4] / n - ex * ey;
  const double vyy = ((double)s[5] / n - ey * ey) + 1.0 / 12.0;
  const double l1 = sqrt(vxx);
  const double l2 = vxy / l1;
  const double l3 = sqrt(vyy - l2 * l2);
  const double den = ((SP_SCALE_2PI * l1) * l3) * SP_MASS;
  xy[0] = (float)(ex + 0.5);
  xy[1] = (float)(ey + 0.5);
  chol[0] = (float)l1;
  chol[1] = (float)l2;
  chol[2] = (float)l3;
#pragma unroll
  for (int c = 0; c < 3; ++c) rgb[c] = (float)((double)s[6 + c] / den);
}

__device__ void seg_centre(const long long *s, int K, int k, float *dst) {
#pragma clang fp contract(off)
  const double n = (double)s[0];
  dst[k] = (float)((double)s[1] / n + 0.5);
  dst[K + k] = (float)((double)s[2] / n + 0.5);
#pragma unroll
  for (int c = 0; c < 3; ++c) dst[(2 + c) * K + k] = (float)((double)s[6 + c] / (n * SP_COLOUR));
}

// The new centre of every segment from its moments, which are cleared for
// the next round; it is chained into its cell for that round or, after the
// last one, gives the segment's Gaussian and (if asked for) the centres
// before and after.  64-thread blocks: the work is a chain of a few loads,
// so it is spread over as many compute units as there are.
constexpr int SP_UPDATE = 64;

template <bool LAST>
__global__ void __launch_bounds__(SP_UPDATE)
k_sp_update(int K, int round, const int *__restrict__ meta, unsigned long long *__restrict__ sums,
            const unsigned long long *__restrict__ sums2, const float *__restrict__ src,
            float *__restrict__ dst, int *__restrict__ heads, SpCentre *__restrict__ rec,
            float *__restrict__ centres, float *__restrict__ xy, float *__restrict__ chol,
            float *__restrict__ rgb) {
  const int k = blockIdx.x * SP_UPDATE + threadIdx.x;
  if (k >= K) return;
  unsigned long long *m = sums + 8 * (size_t)k;
  long long s[9] = {(long long)m[0], (long long)m[1], (long long)m[2], 0, 0, 0,
                    (long long)m[3], (long long)m[4], (long long)m[5]};
  if (s[0] == 0) {
#pragma unroll
    for (int a = 0; a < 5; ++a) dst[a * K + k] = src[a * K + k];
  } else {
    seg_centre(s, K, k, dst);
  }
  if constexpr (LAST) {
    if (centres) {
#pragma unroll
      for (int a = 0; a < 5; ++a) {
        centres[a * K + k] = src[a * K + k];
        centres[(5 + a) * K + k] = dst[a * K + k];
      }
    }
    if (s[0] == 0) return;
#pragma unroll
    for (int a = 0; a < 3; ++a) s[3 + a] = (long long)sums2[4 * (size_t)k + a];
    seg_gaussian(s, xy + 2 * k, chol + 3 * k, rgb + 3 * k);
  } else {
#pragma unroll
    for (int a = 0; a < 6; ++a) m[a] = 0;
    sp_chain(k, dst[k], dst[K + k], dst[2 * K + k], dst[3 * K + k], dst[4 * K + k], meta[M_S],
             meta[M_NCX], meta[M_NCY], round + 1, heads, rec);
  }
}

unsigned grid_for(size_t n) { return (unsigned)std::min<size_t>((n + SP_BLOCK - 1) / SP_BLOCK, 8192); }

}  // namespace
}  // namespace gs2d

using namespace gs2d;

extern "C" size_t gs2d_superpixel_workspace_bytes(int32_t W, int32_t H, int32_t K) {
  SpLayout L;
  return sp_layout(W, H, K, &L) ? L.total : 0;
}

extern "C" int gs2d_init_superpixel(int32_t W, int32_t H, const float *target,
                                    const uint8_t *roi_mask, int32_t K, const int32_t *seeds,
                                    int32_t iters, float compactness, float *xy, float *chol,
                                    float *rgb, int32_t *labels, float *centres, void *ws,
                                    size_t ws_bytes, void *stream) {
  try {
    SpLayout L;
    if (!sp_layout(W, H, K, &L)) return GS2D_EINVAL;
    if (iters < 1 || iters > SP_MAX_ITERS || !(compactness > 0.f) || !std::isfinite(compactness))
      return GS2D_EINVAL;
    if (!target || !roi_mask || !seeds || !xy || !chol || !rgb || !ws) return GS2D_EINVAL;
    if (reinterpret_cast<uintptr_t>(ws) & 255) return GS2D_EINVAL;
    if (ws_bytes < L.total) return GS2D_ENOSPACE;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    const size_t HW = (size_t)W * H;
    float *cen = at<float>(ws, L.cen);
    auto *sums = at<unsigned long long>(ws, L.sums), *sums2 = at<unsigned long long>(ws, L.sums2);
    auto *rec = at<SpCentre>(ws, L.rec);
    auto *seg = at<int2>(ws, L.seg);
    int *heads = at<int>(ws, L.heads), *seg_tiles = at<int>(ws, L.seg_tiles);
    int *tiles = at<int>(ws, L.tiles), *meta = at<int>(ws, L.meta);
    const dim3 block(SP_BLOCK), gu((unsigned)((K + SP_UPDATE - 1) / SP_UPDATE));
    const unsigned gb = std::max(std::min(grid_for(std::max(HW, (size_t)8 * K)), 2048u),
                                 (unsigned)L.n_segs);
    hipLaunchKernelGGL(k_sp_begin, dim3(gb), block, 0, st, W, H, K, L.px, L.tx, L.n_tiles,
                       L.seg_len, L.n_segs, target, roi_mask, seeds, cen, sums, sums2, heads, seg, seg_tiles);
    hipLaunchKernelGGL(k_sp_seed, dim3((K + SP_BLOCK - 1) / SP_BLOCK), block, 0, st, W, H, K,
                       compactness, L.seg_len, L.n_segs, seg, seg_tiles, tiles, cen, meta, heads,
                       rec);
    // at most one tile per block up to 4096 tiles (a block without a tile
    // leaves at once), then by grid stride
    const dim3 ga((unsigned)std::min(L.n_tiles, 4096));
    for (int it = 0; it < iters; ++it) {
      float *src = cen + (size_t)(it & 1) * 5 * K, *dst = cen + (size_t)((it + 1) & 1) * 5 * K;
      const bool last = it == iters - 1;
      const auto assign = L.px == 1 ? (last ? k_sp_assign<1, true> : k_sp_assign<1, false>)
                                    : (last ? k_sp_assign<2, true> : k_sp_assign<2, false>);
      hipLaunchKernelGGL(assign, ga, block, 0, st, W, H, L.tx, L.n_tiles, it, target, roi_mask,
                         meta, tiles, heads, rec, sums, sums2, labels);
      hipLaunchKernelGGL(last ? k_sp_update<true> : k_sp_update<false>, gu, dim3(SP_UPDATE), 0, st,
                         K, it, meta, sums, sums2, src, dst, heads, rec, centres, xy, chol, rgb);
    }
    return hipGetLastError() == hipSuccess ? GS2D_OK : GS2D_EHIP;
  } catch (...) {
    return GS2D_EHIP;
  }
}
