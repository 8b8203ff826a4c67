// Device-side building blocks of the tile rasteriser for Eq. 2 and its
// backward pass, shared by the one-frame kernels (raster.hip) and the
// persistent batched kernel (batch.hip).  See raster.hip for the scheme.
#pragma once

#include "gs2d_internal.h"

namespace gs2d {

// exp(-q/2) = exp2(-q h) with h = log2(e)/2.  Staging multiplies 1/l1 and
// 1/l3 by sqrt(h) and divides l2 by it, so the per-pixel quantities are
// u' = sqrt(h) u and q' = h q: the exponent needs no multiply and the cutoff
// q <= 9 becomes q' <= 9 h.  Gradients summed in these units are rescaled
// by 1/h (mean) and 1/h^1.5 (Cholesky vector) when flushed.
constexpr float EXP_SCALE = 0.84932180028801904f;     // sqrt(log2(e)/2)
constexpr float CUTOFF_QS = 6.4921276840003355f;      // 9 log2(e)/2
constexpr float INV_H = 1.3862943611198906f;          // 2 / log2(e)
constexpr float INV_H15 = 1.6322368749392462f;        // (2 / log2(e))^1.5

// Raster kernels are compiled for 8 wavefronts per SIMD (at most 64 VGPRs):
// with 256-thread workgroups that is 8 workgroups per CU, the wave-slot limit,
// which the latency of staging and the barriers between a tile's phases need.
#define GS2D_RASTER_OCCUPANCY __attribute__((amdgpu_waves_per_eu(8, 8)))

// SPLIT workgroups share a tile, each taking NB consecutive sub-blocks of it
// (whole rows of sub-blocks, or part of one row); LS wavefronts share a
// sub-block, each taking one of LS runs of its Gaussian list and exchanging
// the forward sums through LDS.  Wavefront w: sub-block w % NB, run w / NB.
template <int TILE, int PPL, int SPLIT = 1, int LS = 1, int CHUNK = 0>
struct Cfg {
  static constexpr int SBH = 8 * PPL;      // sub-block height (px)
  static constexpr int SBX = TILE / 8;     // sub-blocks per tile row
  static constexpr int SBY = TILE / SBH;   // sub-block rows per tile
  static constexpr int NWT = SBX * SBY;    // sub-blocks per tile
  static constexpr int NB = NWT / SPLIT;   // sub-blocks per workgroup
  static constexpr int NW = NB * LS;       // wavefronts per workgroup
  static constexpr int NT = NW * 64;       // threads per workgroup
  // Gaussians staged per LDS chunk: fewer where a workgroup has only one or
  // two sub-blocks, so that the LDS of 32 wavefronts' workgroups fits one
  // compute unit (256 everywhere left 8 x 8 tiles 2 and 16 x 16 tiles with 2
  // pixels per lane 4 of 8 wavefronts per SIMD).  CHUNK: another choice.
  static constexpr int CH = CHUNK ? CHUNK : NWT == 1 ? 64 : NWT == 2 ? 128 : 256;
  // floats the wavefronts of a sub-block exchange
  static constexpr int XCH = LS > 1 ? NW * 64 * PPL * 3 : 1;
  static_assert(SBY >= 1 && NWT <= 16, "unsupported tile / pixels-per-lane");
  static_assert(NB * SPLIT == NWT && (NB % SBX == 0 || SBX % NB == 0), "unsupported split");
  static_assert(NT <= 1024, "workgroup too large");
};

// (tile, pixels per lane) variants that are compiled, with SPLIT where the
// frame's sub-blocks fill the device and where they do not (LS > 1).
//
// SPLIT: a workgroup of 4 wavefronts.  A tile's workgroup lives until its
// slowest wavefront is done, so smaller ones leave a shorter tail at the end
// of a launch and fewer idle wavefronts before each barrier, at the price of
// staging the tile's list once per part.  Fits of 20 iterations at 1920x1080 /
// 30,000, us: 32/2 (8 sub-blocks) whole 1144, halves 1107, quarters 1191; 32/1
// (16) whole 1277, halves 1223, quarters 1197; halves of 16/1 2301 against 1971,
// of 16/2 2136 against 1854, of 32/4 no gain.
#define GS2D_VARIANTS(X) \
  X(8, 1, 1, 1) X(16, 1, 1, 1) X(16, 2, 1, 1) X(32, 1, 4, 4) X(32, 2, 2, 4) X(32, 4, 1, 2)

// LS: the device holds 8192 wavefronts.  A frame with at most a quarter as
// many sub-blocks is bound by the serial pass over each one's list, so four
// wavefronts share it; somewhat below a half, two.  us per iteration at
// 480x270 / 1200 (32/2: 1080 sub-blocks) alone 22.4, four 19.2; 640x360 / 1000
// (1920) 20.5, 19.1; 800x450 / 4500 (3000) alone 27.4, two 25.6, four 28.5;
// 640x360 with 16/1 (3680) 21.9, 20.9, 24.6; 960x540 / 7000 (4080) 28.4, 30.0,
// 32.0; at 1280x720 (7360) two take 38.5 against 34.3.  The separate forward and
// backward follow the same lines: 480x270 / 1200 alone 4.8 and 8.9 us, four 4.4
// and 8.5; 800x450 / 4500 6.7 and 12.2, two 6.6 and 13.1; 640x360 with 16/1 4.7
// and 10.0, two 5.1 and 9.7; 960x540 / 7000 7.1 and 12.6, two 7.8 and 17.2.
inline int raster_share(long long sub_blocks) {
  return sub_blocks <= 2048 ? 4 : sub_blocks <= 3840 ? 2 : 1;
}

// The workgroup's tile (or work item) and its part of it: the parts run on one
// XCD (workgroup b runs on XCD b % 8).  A grid of split_grid workgroups covers
// every part; those past the last tile leave at once.
template <int SPLIT>
__device__ inline int tile_of_block(int *part) {
  const int b = (int)blockIdx.x;
  *part = SPLIT == 1 ? 0 : (b >> 3) % SPLIT;
  return SPLIT == 1 ? b : b / (8 * SPLIT) * 8 + (b & 7);
}
inline unsigned split_grid(unsigned n_tiles, unsigned split) {
  return split == 1 ? n_tiles : (n_tiles + 7) / 8 * 8 * split;
}

template <class C>
struct Smem {
  float4 A[C::CH];           // mx, my, 1/l1, l2
  float4 B[C::CH];           // 1/l3, c'0, c'1, c'2
  uint16_t mask[C::CH];      // bit w: box meets sub-block w (at most 16)
  int id[C::CH];
  uint16_t list[C::NW][C::CH];
  uint8_t act[C::CH];        // the Gaussian is optimised (FrameArgs::active)
};

// This wavefront's run [beg, end) of a list of len entries.
template <class C>
__device__ inline void list_run(int len, int *beg, int *end) {
  if constexpr (C::NW == C::NB) {
    *beg = 0;
    *end = len;
  } else {
    constexpr int LS = C::NW / C::NB;
    const int r = (int)(threadIdx.x >> 6) / C::NB;
    *beg = len * r / LS;
    *end = len * (r + 1) / LS;
  }
}

struct FrameArgs {
  int W, H, TX;
  const float4 *geom;
  const uint32_t *keys;
  const int *tile_start;
  const float *rgb;
  // nullable [N]: the fused backward skips Gaussians with active[n] == 0
  // (they are not optimised, Sec. 3.2.C); the forward renders them all
  const uint8_t *active;
  // nullable, lazy binning: the workspace's misc array.  The binning
  // kernels that read misc[MISC_STALE] have finished when the fused raster
  // runs; if the flag is set (this iteration rebuilt the lists) the raster
  // stamps the lists with (sig_lo, sig_hi), or clears the stamp if a
  // rebuild's wait ran out, then clears the flag.
  int *lazy_misc;
  uint32_t sig_lo, sig_hi;
  // nullable: the fused raster adds 1 to *tick (the optimiser's step)
  int *tick;
};

// The ellipse q' <= qmax (staged units: u1 = dx a, u2 = dy r3s - c u1 with c =
// l2s r3s), cut by the strip of rows d0 <= dy <= d1: true unless it misses the
// strip, and then the least and largest u1 of the cut.  sq = sqrt(qmax).  The
// rightmost point is (sq, l2s sq); where that lies outside the strip, the cut
// ends on the strip's nearer edge e = dy r3s, at a root of (1 + c^2) u1^2 - 2
// c e u1 + e^2 = qmax.  A NaN anywhere comes out as a NaN range.  The cut is
// convex, so it meets the sub-blocks of the strip whose columns its range
// meets: 57 vector instructions per row of sub-blocks, where a test per
// sub-block took 42 each (1920x1080 / 30,000, 20 iterations, with the loss sum
// in DPP adds: 1154 -> 1133 us; 4 pixels per lane 1422 -> 1367 us).
__device__ inline bool ellipse_in_strip(float l2s, float r3s, float d0, float d1, float qmax,
                                        float sq, float *lo, float *hi) {
  const float c = l2s * r3s, k = 1.f + c * c, ik = __builtin_amdgcn_rcpf(k), t = l2s * sq;
  const float er = (t < d0 ? d0 : d1) * r3s, el = (-t < d0 ? d0 : d1) * r3s;
  const float sr = qmax * k - er * er, sl = qmax * k - el * el;
  const bool in_r = t >= d0 && t <= d1, in_l = -t >= d0 && -t <= d1;
  *hi = in_r ? sq : (c * er + __builtin_amdgcn_sqrtf(sr)) * ik;
  *lo = in_l ? -sq : (c * el - __builtin_amdgcn_sqrtf(sl)) * ik;
  return !((!in_r && sr < 0.f) || (!in_l && sl < 0.f));
}

// Stage keys[beg, beg+cnt) into LDS with their sub-block masks: bit w is set
// when the Gaussian's 3-sigma box meets sub-block w and, with EXACT, its
// cutoff ellipse also comes within a rounding margin of one of the
// sub-block's in-frame pixel centres (on fitted frames about one box-met
// sub-block in six fails the ellipse test).  The margin, 0.01 (1 + |l2 /
// l3|) in staged q units, bounds the rounding of both this test and the
// per-pixel evaluation (each about 1e-5 (1 + |l2 / l3|)), so no sub-block
// with a pixel the raster counts inside the cutoff is dropped.  Exact masks
// leave few Gaussians without a pixel in the cutoff, so their users skip
// the per-Gaussian hit checks; the persistent batched kernel, whose
// register budget the test's live values overrun, keeps box masks.
template <class C, int TILE, bool EXACT = true>
__device__ inline void stage_chunk(Smem<C> &S, const uint32_t *__restrict__ keys, int beg, int cnt,
                                   int tx, int ty, int W, int H, const float4 *__restrict__ geom,
                                   const float *__restrict__ rgb,
                                   const uint8_t *__restrict__ active = nullptr, int part = 0) {
  // the workgroup's sub-blocks: rows [sy0, sy1], columns [sx0, sx1] of the tile's
  constexpr int ROWS = C::NB >= C::SBX ? C::NB / C::SBX : 1;
  const int sb0 = part * C::NB, sy0 = sb0 / C::SBX, sy1 = sy0 + ROWS - 1;
  const int sx0 = sb0 % C::SBX, sx1 = C::NB >= C::SBX ? C::SBX - 1 : sx0 + C::NB - 1;
  constexpr float inv_w = 0.125f, inv_h = 1.0f / (float)C::SBH;
  const float xlast = (float)W - 0.5f, ylast = (float)H - 0.5f;  // last pixel centres
  for (int j = threadIdx.x; j < cnt; j += C::NT) {
    const int id = (int)(keys[beg + j] & 0xFFFFu);
    const float4 g0 = geom[2 * id], g1 = geom[2 * id + 1];
    float c0 = 0.f, c1 = 0.f, c2 = 0.f;
    if (rgb) {  // pair counting stages geometry only
      c0 = rgb[3 * id];
      c1 = rgb[3 * id + 1];
      c2 = rgb[3 * id + 2];
    }
    const float a = g0.z * EXP_SCALE, l2s = g0.w * (1.0f / EXP_SCALE), r3s = g1.x * EXP_SCALE;
    S.A[j] = make_float4(g0.x, g0.y, a, l2s);
    S.B[j] = make_float4(r3s, c0, c1, c2);
    S.id[j] = id;
    if (active) S.act[j] = active[id];
    const float xlo = __fsub_rn(g0.x, g1.y), xhi = __fadd_rn(g0.x, g1.y);
    const float ylo = __fsub_rn(g0.y, g1.z), yhi = __fadd_rn(g0.y, g1.z);
    // sub-block columns/rows met by the box, tile-local
    const float bx0f = floorf(xlo * inv_w) - (float)(tx * C::SBX);
    const float bx1f = floorf(xhi * inv_w) - (float)(tx * C::SBX);
    const float by0f = floorf(ylo * inv_h) - (float)(ty * C::SBY);
    const float by1f = floorf(yhi * inv_h) - (float)(ty * C::SBY);
    const int bx0 = (int)fmaxf(bx0f, (float)sx0), bx1 = (int)fminf(bx1f, (float)sx1);
    const int by0 = (int)fmaxf(by0f, (float)sy0), by1 = (int)fminf(by1f, (float)sy1);
    const float qmax = CUTOFF_QS + 0.01f * (1.0f + fabsf(l2s * r3s));
    uint32_t m = 0;
    if constexpr (EXACT) {
      const float sq = __builtin_amdgcn_sqrtf(qmax), ia = __builtin_amdgcn_rcpf(a);
      // the centre and the last pixel column, from the tile's first
      const float first = (float)(tx * TILE) + 0.5f, left = g0.x - first, xl = xlast - first;
      for (int by = by0; by <= by1; ++by) {
        const float Y0 = (float)(ty * TILE + by * C::SBH) + 0.5f;
        const float Y1 = fminf(Y0 + (float)(C::SBH - 1), ylast);
        float u0, u1;
        if (Y0 > Y1 || !ellipse_in_strip(l2s, r3s, Y0 - g0.y, Y1 - g0.y, qmax, sq, &u0, &u1))
          continue;
        // columns from the first whose last pixel is not left of the cut, to
        // the last whose first is not right of it; the box's after a NaN
        const bool cut = u0 <= u1;
        const float x0 = left + fminf(u0 * ia, u1 * ia), x1 = left + fmaxf(u0 * ia, u1 * ia);
        const int c0 = cut ? (int)fmaxf(ceilf((x0 - 7.f) * inv_w), (float)bx0) : bx0;
        const int c1 = cut ? (int)fminf(floorf(fminf(x1, xl) * inv_w), (float)bx1) : bx1;
        if (c0 <= c1 && !(x0 > xl)) m |= ((2u << (c1 - c0)) - 1u) << (by * C::SBX + c0 - sb0);
      }
    } else {
      for (int by = by0; by <= by1; ++by)
        for (int bx = bx0; bx <= bx1; ++bx) m |= 1u << (by * C::SBX + bx - sb0);
    }
    S.mask[j] = (uint16_t)m;
  }
}

// Each wavefront builds its list of staged Gaussians; returns its length.
template <class C>
__device__ inline int compact_chunk(Smem<C> &S, int cnt) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, sb = w % C::NB;
  const unsigned long long lt = lanemask_lt();
  int len = 0;
  for (int j0 = 0; j0 < cnt; j0 += 64) {
    const int j = j0 + lane;
    const bool hit = (j < cnt) && ((S.mask[j] >> sb) & 1u);
    const unsigned long long bal = __ballot(hit);
    if (hit) S.list[w][len + __popcll(bal & lt)] = (uint16_t)j;
    len += __popcll(bal);
  }
  return len;
}

// ---- wavefront reduction of 8 values ----
// Sum of 8 per-lane values over the wavefront; lane L returns the total of
// value ((L >> 3) & 7).  Each exchange halves the number of values a lane
// carries:
//   - across the two 32-lane halves, v_permlane32_swap of (value i, value
//     i+4) leaves value i of both halves in the low half and value i+4 of
//     both halves in the high half; one add finishes the pair;
//   - across 16-lane rows, v_permlane16_swap, the same way;
//   - across 8 lanes inside a row and then within each 8-lane group, DPP
//     (row_ror:8, row_half_mirror, quad_perm) folded into the adds.
template <int CTRL>
__device__ inline float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}

constexpr int DPP_ROW_ROR8 = 0x128;
constexpr int DPP_ROW_HALF_MIRROR = 0x141;
constexpr int DPP_QUAD_XOR2 = 0x4E;  // quad_perm [2,3,0,1]
constexpr int DPP_QUAD_XOR1 = 0xB1;  // quad_perm [1,0,3,2]

__device__ inline float reduce8_transpose(const float (&a)[8]) {
  const int lane = threadIdx.x & 63;
  float b[4], c[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a[i]), __float_as_uint(a[i + 4]),
                                              false, false);
    b[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(b[i]), __float_as_uint(b[i + 2]),
                                              false, false);
    c[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  const bool hi = lane & 8;
  float d = (hi ? c[1] : c[0]) + dpp<DPP_ROW_ROR8>(hi ? c[0] : c[1]);
  d += dpp<DPP_ROW_HALF_MIRROR>(d);
  d += dpp<DPP_QUAD_XOR2>(d);
  d += dpp<DPP_QUAD_XOR1>(d);
  return d;
}

// Drop the Gaussians whose staged active flag is 0 from this wavefront's
// list (in place, order kept); returns the new length.
template <class C>
__device__ inline int keep_active(Smem<C> &S, int len) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const unsigned long long lt = lanemask_lt();
  int kept = 0;
  for (int k0 = 0; k0 < len; k0 += 64) {
    const int j = (k0 + lane < len) ? S.list[w][k0 + lane] : 0;
    const bool keep = (k0 + lane < len) && S.act[j];
    const unsigned long long bal = __ballot(keep);
    if (keep) S.list[w][kept + __popcll(bal & lt)] = (uint16_t)j;
    kept += __popcll(bal);
  }
  return kept;
}

// Pixel column and first row of this thread.
template <class C, int TILE, int PPL>
__device__ inline void pixel_of_thread(int tx, int ty, int *px, int *py0, int part = 0) {
  const int w = part * C::NB + (int)(threadIdx.x >> 6) % C::NB, lane = threadIdx.x & 63;
  *px = tx * TILE + (w % C::SBX) * 8 + (lane & 7);
  *py0 = ty * TILE + (w / C::SBX) * C::SBH + (lane >> 3) * PPL;
}

// q' of a (pixel, Gaussian) pair, each operation and its rounding written out
// and nothing left to the compiler's contraction: in every pass and route with
// the same pixels per lane the cutoff holds for the same pixels.  A lane's
// first row starts from base = dy - l2 u1; the rows below add 1/l3 to u2.  One
// pixel per lane and several round the last step differently (they share
// u1^2), so two such variants may differ on a pixel whose q' is within a few
// ulp of the cutoff.
__device__ __forceinline__ float pair_base(const float4 &A, float u1, float dy) {
  return __builtin_fmaf(-A.w, u1, dy);
}
__device__ __forceinline__ float pair_next_row(int r, float base, float u2, float inv_l3) {
  return r == 0 ? __builtin_fmaf(base, inv_l3, inv_l3) : u2 + inv_l3;
}
template <int PPL>
__device__ __forceinline__ float pair_q(float u1, float u1s, float u2) {
  return PPL == 1 ? __builtin_fmaf(u1, u1, u2 * u2) : __builtin_fmaf(u2, u2, u1s);
}

// Forward accumulation over entries [beg, end) of this wavefront's list of a
// staged, compacted chunk.  With KEEP_HITS (the whole list: beg = 0) the
// wavefront's list is compacted in place to the Gaussians that have at least
// one in-frame pixel with q <= 9 in this sub-block (the only ones the
// backward pass needs); returns the new length (else `end`).
template <class C, int PPL, bool KEEP_HITS>
__device__ inline int fwd_chunk(Smem<C> &S, int beg, int end, float pxc, float pyc0,
                                unsigned inside, float (&acc)[PPL][3]) {
  const int w = threadIdx.x >> 6;
  int kept = 0;
  for (int k = beg; k < end; ++k) {
    const int j = S.list[w][k];
    const float4 A = S.A[j], B = S.B[j];
    const float u1 = (pxc - A.x) * A.z;
    const float u1s = u1 * u1;
    const float base = pair_base(A, u1, pyc0 - A.y);
    bool any = false;
    float u2 = base * B.x;
#pragma unroll
    for (int r = 0; r < PPL; u2 = pair_next_row(r, base, u2, B.x), ++r) {
      const float q = pair_q<PPL>(u1, u1s, u2);
      const float e = __builtin_amdgcn_exp2f(-q);
      const bool in_cut = q <= CUTOFF_QS;
      const float wgt = in_cut ? e : 0.f;
      acc[r][0] += wgt * B.y;
      acc[r][1] += wgt * B.z;
      acc[r][2] += wgt * B.w;
      any |= in_cut && ((inside >> r) & 1u);
    }
    if (KEEP_HITS) {
      if (__ballot(any)) {
        if ((threadIdx.x & 63) == 0) S.list[w][kept] = (uint16_t)j;  // kept <= k
        ++kept;
      }
    }
  }
  return KEEP_HITS ? kept : end;
}

// The sums of the LS wavefronts that share a sub-block, added in the order of
// their runs: every one of them then holds the sub-block's pixels.
template <class C, int PPL>
__device__ inline void exchange_sums(float *xch, float (&acc)[PPL][3]) {
  if constexpr (C::NW > C::NB) {
    constexpr int LS = C::NW / C::NB, V = PPL * 3;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < V; ++i) xch[(w * V + i) * 64 + lane] = acc[i / 3][i % 3];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < V; ++i) {
      float s = 0.f;
#pragma unroll
      for (int r = 0; r < LS; ++r) s += xch[((r * C::NB + w % C::NB) * V + i) * 64 + lane];
      acc[i / 3][i % 3] = s;
    }
  }
}

// dL/dC of lane N of this lane's row of 16 (g, as DPP operands): its product
// with the colour B.yzw, and its share `wgt` added to the sums c.  s_nop: a
// register that a DPP operand reads must be two states old.
template <int N>
__device__ __forceinline__ float row_pixel(const float (&g)[3], const float4 &B, float wgt,
                                           float *c) {
  float d;
  asm("s_nop 1\n"
      "v_mul_f32_dpp %0, %4, %7 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f32_dpp %0, %5, %8 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f32_dpp %0, %6, %9 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f32_dpp %1, %4, %10 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f32_dpp %2, %5, %10 row_newbcast:%11 row_mask:0xf bank_mask:0xf\n"
      "v_fmac_f32_dpp %3, %6, %10 row_newbcast:%11 row_mask:0xf bank_mask:0xf"
      : "=&v"(d), "+v"(c[0]), "+v"(c[1]), "+v"(c[2])
      : "v"(g[0]), "v"(g[1]), "v"(g[2]), "v"(B.y), "v"(B.z), "v"(B.w), "v"(wgt), "n"(N));
  return d;
}

// bwd_batch's state over the pixel columns: v[0..4] as bwd_chunk's vals before
// the factors 1/l1 (0, 2) and 1/l3 (4), v[5..7] the colours.
struct BatchSums {
  float v[8];
  bool any;
};
template <int PPL, bool CHECK_HITS, int N>
__device__ __forceinline__ void batch_pixels(BatchSums &T, float &t0, float &t2, const float4 &B,
                                             float cut, float u1, float u1s, float base,
                                             const float (&g)[PPL][3]) {
  float u2 = base * B.x;
#pragma unroll
  for (int r = 0; r < PPL; u2 = pair_next_row(r, base, u2, B.x), ++r) {
    const float q = pair_q<PPL>(u1, u1s, u2);
    const float e = __builtin_amdgcn_exp2f(-q);
    const bool in_cut = q <= cut;
    const float wgt = in_cut ? e : 0.f;
    if (CHECK_HITS) T.any |= in_cut;
    const float sn = row_pixel<N>(g[r], B, wgt, T.v + 5) * wgt;
    const float s2 = sn * u2;
    t0 += sn;
    t2 += s2;
    T.v[4] += s2 * u2;
  }
}
template <int PPL, bool CHECK_HITS, int COL>
__device__ __forceinline__ void batch_column(BatchSums &T, const float4 &A, const float4 &B,
                                             float cut, float x0, const float (&yb)[2],
                                             const float (&g)[PPL][3]) {
  const float u1 = ((x0 + (float)COL) - A.x) * A.z;
  const float u1s = u1 * u1;
  float t0 = 0.f, t2 = 0.f;
  batch_pixels<PPL, CHECK_HITS, COL>(T, t0, t2, B, cut, u1, u1s, pair_base(A, u1, yb[0]),
                                     g);
  batch_pixels<PPL, CHECK_HITS, COL + 8>(T, t0, t2, B, cut, u1, u1s, pair_base(A, u1, yb[1]), g);
  t2 *= B.x;
  const float s1 = u1 * t0 - A.w * t2;
  T.v[0] += s1;
  T.v[1] += t2;
  T.v[2] += s1 * u1;
  T.v[3] += t2 * u1;
  if constexpr (COL < 7) batch_column<PPL, CHECK_HITS, COL + 1>(T, A, B, cut, x0, yb, g);
}

// Backward of up to 16 Gaussians at once, entries [k0, min(k0 + 16, end)): lane
// L takes Gaussian L & 15 over the pixels of its row of 16 lanes, whose dL/dC
// reach it as DPP operands, and sums in registers.  The raster is bound by
// vector instructions (about 85 % of the issue slots at 1920 x 1080).  One
// Gaussian at a time, 18 of its 67 for 128 pixels reduce 8 sums over 64 lanes
// and 12 more set it up; here 16 Gaussians share 12 for the reduction over 4
// rows, a pixel column's terms are formed once for its pixels, and no LDS is
// read for dL/dC (with lanes fetching it by ds_bpermute, 8 Gaussians at a time,
// the LDS became the bound and nothing was gained).  1920x1080 / 30,000, 20
// iterations 1296 -> 1146 us, 12 mixed frames, 10 iterations 2858 -> 2468 us.
template <class C, int PPL, bool CHECK_HITS>
__device__ __forceinline__ void bwd_batch(const Smem<C> &S, float *acc, int k0, int end, float pxc,
                                          float pyc0, const float (&g)[PPL][3]) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int k = k0 + (lane & 15);
  const bool live = k < end;
  const int j = S.list[w][min(k, end - 1)];
  const float4 A = S.A[j], B = S.B[j];
  const float x0 = pxc - (float)(lane & 7);
  const float y0 = pyc0 - (float)(((lane >> 3) & 1) * PPL);  // the row's first pixel row
  const float yb[2] = {y0 - A.y, (y0 + (float)PPL) - A.y};
  BatchSums T = {};
  batch_column<PPL, CHECK_HITS, 0>(T, A, B, live ? CUTOFF_QS : -1.f, x0, yb, g);
  T.v[0] *= A.z;
  T.v[2] *= A.z;
  T.v[4] *= B.x;
  // the four rows' sums: each exchange halves the values a lane carries
  float b[4], c[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(T.v[i]), __float_as_uint(T.v[i + 4]),
                                              false, false);
    b[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(b[i]), __float_as_uint(b[i + 2]),
                                              false, false);
    c[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  }
  bool add = live;
  if (CHECK_HITS) {
    const unsigned long long m = __ballot(T.any);
    add = add && (((m | m >> 16 | m >> 32 | m >> 48) >> (lane & 15)) & 1);
  }
  if (add) {
    float *dst = acc + j * 8 + (lane >> 5) * 4 + ((lane >> 4) & 1) * 2;
    atomicAdd(dst, c[0]);
    atomicAdd(dst + 1, c[1]);
  }
}

// Gaussians from which a batch is faster than one at a time: 16 take about 645
// vector instructions at 2 pixels per lane, one by itself 67 (us per 20
// iterations at 1920x1080 / 30,000, from 8: 1146, from 10: 1151, full batches
// only: 1200, never: 1296).  Where four wavefronts share a list they split it
// finer than that (640x360 / 1000, 50 iterations: 962 without, 989 with); two
// gain.
constexpr int BATCH_MIN = 8;

// Backward over entries [beg, end) of this wavefront's list of a staged,
// compacted chunk; adds into acc[CH][8] in LDS.
// CHECK_HITS skips (uniformly per wavefront) Gaussians with no pixel inside
// the cutoff, for lists that were not already reduced to such Gaussians.
// BATCH false: one Gaussian at a time whatever the list's length.
template <class C, int PPL, bool CHECK_HITS, bool BATCH = true>
__device__ inline void bwd_chunk(const Smem<C> &S, float *acc, int beg, int end, float pxc,
                                 float pyc0, const float (&g)[PPL][3]) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int k = beg;
  if constexpr (BATCH && C::NW <= 2 * C::NB)
    for (; end - k >= BATCH_MIN; k += 16)
      bwd_batch<C, PPL, CHECK_HITS>(S, acc, k, end, pxc, pyc0, g);
  for (; k < end; ++k) {
    const int j = S.list[w][k];
    const float4 A = S.A[j], B = S.B[j];
    const float u1 = (pxc - A.x) * A.z;
    const float u1s = u1 * u1;
    const float base = pair_base(A, u1, pyc0 - A.y);
    float u2[PPL], q[PPL];
    bool any = false;
#pragma unroll
    for (int r = 0; r < PPL; ++r) {
      u2[r] = r == 0 ? base * B.x : pair_next_row(r - 1, base, u2[r - 1], B.x);
      q[r] = pair_q<PPL>(u1, u1s, u2[r]);
      any |= q[r] <= CUTOFF_QS;
    }
    if (CHECK_HITS && !__ballot(any)) continue;  // wavefront-uniform skip
    float s0 = 0.f, s2 = 0.f, s3 = 0.f, c0 = 0.f, c1 = 0.f, c2 = 0.f;
#pragma unroll
    for (int r = 0; r < PPL; ++r) {
      const float e = __builtin_amdgcn_exp2f(-q[r]);
      const float wgt = (q[r] <= CUTOFF_QS) ? e : 0.f;
      const float sn = (g[r][0] * B.y + g[r][1] * B.z + g[r][2] * B.w) * wgt;
      const float v2 = u2[r] * B.x;
      const float t2 = sn * v2;
      s0 += sn;
      s2 += t2;
      s3 += t2 * u2[r];
      c0 += g[r][0] * wgt;
      c1 += g[r][1] * wgt;
      c2 += g[r][2] * wgt;
    }
    // v1 = (u1 - l2 v2) / l1 with u1 common to the lane's pixels, so
    // sum s v1 = (u1 sum s - l2 sum s v2) / l1; likewise dL/dl1 = sum s v1 u1
    // and dL/dl2 = sum s v2 u1 take the lane's u1 once.  In the staged units
    // (u' = sqrt(h) u, v2' = h v2) these sums come out as h dL/dmu and
    // h^1.5 dL/dl; flush_grads rescales them.
    const float s1 = (u1 * s0 - A.w * s2) * A.z;
    const float vals[8] = {s1, s2, s1 * u1, s2 * u1, s3, c0, c1, c2};
    const float red = reduce8_transpose(vals);
    if ((lane & 7) == 0) atomicAdd(&acc[j * 8 + (lane >> 3)], red);
  }
}

// Flush the LDS accumulators of a chunk to the global gradients: thread t
// adds parameter t % 8 of the chunk's Gaussians t / 8, t / 8 + NT / 8, ...,
// so the eight parameters of a Gaussian leave from adjacent lanes of one
// instruction and every wavefront of the tile takes a share.  PIN forms the
// lane's pointer, stride and scale at the flush rather than letting the
// compiler hoist them out of a caller's chunk loop, where they would hold
// registers through the passes (which of the two spills less depends on the
// caller).
template <class C, bool PIN = false>
__device__ inline void flush_grads(const Smem<C> &S, const float *acc, int cnt,
                                   float *__restrict__ g_xy, float *__restrict__ g_chol,
                                   float *__restrict__ g_rgb) {
  static_assert(C::NT % 8 == 0, "a thread keeps one parameter");
  int k = threadIdx.x & 7;
  if constexpr (PIN) asm volatile("" : "+v"(k));
  float *base;
  int stride;
  float scale;
  if (k < 2) {
    base = g_xy + k;
    stride = 2;
    scale = INV_H;
  } else if (k < 5) {
    base = g_chol + (k - 2);
    stride = 3;
    scale = INV_H15;
  } else {
    base = g_rgb + (k - 5);
    stride = 3;
    scale = 1.f;
  }
  for (int e = threadIdx.x; e < cnt * 8; e += C::NT) {
    const float v = acc[e];
    if (v != 0.f) atomicAdd(base + stride * S.id[e >> 3], v * scale);
  }
}

// Wavefront sum of one float per lane; lane 0 writes it to *slot.  Loss
// partials are kept per sub-block (tile t, sub-block b at t * NWT + b), so a
// wavefront never waits for the rest of its tile to record its loss.
__device__ inline void wave_loss(float v, float *__restrict__ slot) {
  v += dpp<DPP_QUAD_XOR1>(v);
  v += dpp<DPP_QUAD_XOR2>(v);
  v += dpp<DPP_ROW_HALF_MIRROR>(v);
  v += dpp<DPP_ROW_ROR8>(v);
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  if ((threadIdx.x & 63) == 0) *slot = __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// base[i] with a 32-bit byte offset beside a uniform base (a frame has at most
// 65536 tiles, so its planes stay below 2^28 bytes; Gaussians below 2^16).
__device__ __forceinline__ float at_index(const float *base, uint32_t i) {
  return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(base) + 4u * i);
}

// Bit r set: pixel row r of this lane lies inside the frame.
template <int PPL>
__device__ inline unsigned inside_mask(const FrameArgs &f, int px, int py0) {
  unsigned m = 0;
#pragma unroll
  for (int r = 0; r < PPL; ++r) m |= (px < f.W && py0 + r < f.H) ? (1u << r) : 0u;
  return m;
}


// ------------------------------------------- fused forward + loss + backward --
// Eq. 2 is an order-free sum and every Gaussian reaching a pixel is in that
// pixel's tile list, so a tile can finish its forward pass, form
// dL/dC = 2 (C - target) / (3HW) in registers and run its backward pass
// without dL/dC ever reaching memory.  One call processes one tile with the
// whole workgroup; each wavefront's sum of squared residuals goes to
// loss_slots[w].
//
// A list that fits one LDS chunk (the common case) is staged once; after
// one barrier every wavefront compacts it to its sub-block, runs its
// forward pass (with box masks also keeping only the Gaussians that reach
// its pixels), its residuals and its backward pass on its own, and a second
// barrier precedes the flush
// of the tile's gradient accumulators.  Longer lists are staged chunk by
// chunk, twice.
template <int TILE, int PPL>
__device__ inline void residuals(const float (&a)[PPL][3], const float (&tg)[PPL][3],
                                 unsigned inside, float grad_scale, float (&g)[PPL][3], float *l) {
  float s = 0.f;
#pragma unroll
  for (int r = 0; r < PPL; ++r) {
    g[r][0] = g[r][1] = g[r][2] = 0.f;
    if ((inside >> r) & 1u) {
      const float r0 = a[r][0] - tg[r][0], r1 = a[r][1] - tg[r][1], r2 = a[r][2] - tg[r][2];
      s += r0 * r0 + r1 * r1 + r2 * r2;
      g[r][0] = r0 * grad_scale;
      g[r][1] = r1 * grad_scale;
      g[r][2] = r2 * grad_scale;
    }
  }
  *l = s;
}

// ONE: the caller runs one tile per workgroup (no LDS of an earlier tile to
// wait for before staging).  loss_slots: the tile's, one per sub-block.
template <class C, int TILE, int PPL, bool EXACT = true, bool ONE = false, bool BATCH = true>
__device__ inline void fused_tile(Smem<C> &S, float *acc, float *xch, const FrameArgs &f, int tile,
                                  const float *__restrict__ target,
                                  float *__restrict__ loss_slots, float grad_scale,
                                  float *__restrict__ g_xy, float *__restrict__ g_chol,
                                  float *__restrict__ g_rgb, int part = 0) {
  static_assert(EXACT || C::NW == C::NB, "shared sub-blocks need exact masks");
  const int w = threadIdx.x >> 6;
  const int tx = tile % f.TX, ty = tile / f.TX;
  const int beg = f.tile_start[tile], end = f.tile_start[tile + 1];
  int px, py0;
  pixel_of_thread<C, TILE, PPL>(tx, ty, &px, &py0, part);
  const float pxc = (float)px + 0.5f, pyc0 = (float)py0 + 0.5f;
  const unsigned inside = inside_mask<PPL>(f, px, py0);
  // the target pixels are loaded first, their latency hidden by the staging
  const size_t HW = (size_t)f.W * f.H;
  float tg[PPL][3];
#pragma unroll
  for (int r = 0; r < PPL; ++r) {
    const uint32_t p = ((inside >> r) & 1u) ? (uint32_t)((py0 + r) * f.W + px) : 0;
    tg[r][0] = at_index(target, p);
    tg[r][1] = at_index(target + HW, p);
    tg[r][2] = at_index(target + 2 * HW, p);
  }
  float a[PPL][3] = {};
  float g[PPL][3];
  float l;
  int kb, ke;
  const bool once = end - beg <= C::CH;  // the whole list fits one chunk
  int len = 0;
  for (int c = beg; c < end; c += C::CH) {
    const int cnt = min(C::CH, end - c);
    if (!ONE || c != beg) __syncthreads();  // LDS of a previous tile or chunk is free
    stage_chunk<C, TILE, EXACT>(S, f.keys, c, cnt, tx, ty, f.W, f.H, f.geom, f.rgb, f.active,
                                part);
    if (once)
      for (int i = threadIdx.x; i < cnt * 8; i += C::NT) acc[i] = 0.f;
    __syncthreads();
    len = compact_chunk<C>(S, cnt);
    list_run<C>(len, &kb, &ke);
    const int kept = fwd_chunk<C, PPL, !EXACT>(S, kb, ke, pxc, pyc0, inside, a);
    if constexpr (!EXACT) len = kept;
  }
  exchange_sums<C, PPL>(xch, a);
  residuals<TILE, PPL>(a, tg, inside, grad_scale, g, &l);
  if (w < C::NB) wave_loss(l, loss_slots + part * C::NB + w);
  for (int c = beg; c < end; c += C::CH) {
    const int cnt = min(C::CH, end - c);
    if (!once) {
      __syncthreads();
      stage_chunk<C, TILE, EXACT>(S, f.keys, c, cnt, tx, ty, f.W, f.H, f.geom, f.rgb, f.active,
                                  part);
      for (int i = threadIdx.x; i < cnt * 8; i += C::NT) acc[i] = 0.f;
      __syncthreads();
      len = compact_chunk<C>(S, cnt);
    }
    if (f.active) len = keep_active<C>(S, len);
    list_run<C>(len, &kb, &ke);
    bwd_chunk<C, PPL, !EXACT, BATCH>(S, acc, kb, ke, pxc, pyc0, g);
    __syncthreads();
    flush_grads<C, ONE>(S, acc, cnt, g_xy, g_chol, g_rgb);
  }
}

}  // namespace gs2d
