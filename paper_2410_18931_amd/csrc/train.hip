// The training step around the renderer (Sec. 5, implementation details):
// the rendering loss of 3D Gaussian Splatting -- an l1 term plus a D-SSIM
// term weighted lambda = 0.2 -- with its gradient with respect to the
// rendered image, and the Adam update of the parameters.
//
//   L_v = (1 - lambda) mean|x - y| + lambda (1 - mean SSIM(x, y)),  L = mean_v L_v
//
// SSIM per colour channel (Wang et al. 2004): local statistics under an
// 11 x 11 Gaussian window (sigma 1.5) with zero padding, C1 = 0.01^2,
// C2 = 0.03^2.  The map depends on x through u = G*x, Sxx = G*x^2 and
// Sxy = G*(x y); the gradient of its mean is therefore
//   dmean/dx = (G*dS/du + 2 x G*dS/dSxx + y G*dS/dSxy) / P
// (the window is symmetric, so its adjoint is the same zero-padded filter).
//
// Two passes, the separable filter applied along rows, then columns:
//   pass1: the five windowed statistics -> map, the three derivative maps (to
//          the workspace) and each workgroup's (or wave's) share of the loss;
//   pass2: the three derivative maps filtered again -> dL/dx.
// The shares are summed in FP64 in a fixed order (loss_finalize).
//
// Small images are cut into 16 x 16 pixel tiles, one workgroup per tile and
// channel, staged with a 5-pixel halo in LDS (loss_pass1, loss_pass2): many
// short workgroups, but every row is filtered 1.6 times and the filtered rows
// pass through LDS again.  Large ones are cut into strips 64 pixels wide and
// 34 rows high, one wave per channel and one column per lane, which walk down
// the strip (loss_strip_pass1, loss_strip_pass2): a row with its halo is staged
// in LDS and filtered along the row once (1.3 times with the halo rows), and
// the last eleven filtered rows stay in registers for the filter along the
// column.  Fused multiply-adds are most of what either issues; a strip's rows
// are a serial chain of about 0.6 us each, so it needs enough pixels to give
// every SIMD some waves.  Both passes with the loss's sum, us, tiles and strips:
// 17 x 9 and 65 x 33 14 / 49, 640 x 360 34 / 54, three views of 400 x 300
// 43 / 55, 960 x 540 60 / 54, 1280 x 720 90 / 69, sixteen views of 400 x 300
// 171 / 102, 1920 x 1080 209 / 108, four of them 719 / 400.  Each launch of up to
// 16 views takes the form that suits its views (loss_in_strips).
#include <cmath>
#include <type_traits>
#include <mutex>

#include "adam.h"
#include "plan.h"
#include "wsr_internal.h"

// Workspace of the allocation-free loss entry point: the derivative maps and
// per-tile shares of wsr_loss, in a device array of fixed size.  Every device
// the library runs on holds its own copy until the process ends.  In host
// code this name stands for a host-side shadow, not a device address: host
// code uses only the address hipGetSymbolAddress returns for the current
// device (loss_static_workspace).
static __device__ __align__(256) unsigned char scratch[WSR_LOSS_STATIC_BYTES];

namespace wsr {
namespace {

constexpr int kLT = kLossTile;        // output tile edge
constexpr int kHalo = 5;              // window radius
constexpr int kLE = kLT + 2 * kHalo;  // staged edge (26)
constexpr int kTaps = 2 * kHalo + 1;
constexpr int kStrip = kStripCols;    // output columns of a strip, one a lane; its kStripRows output rows take 44
                                      // staged ones, four rounds of eleven (23 rows: 130 us at 1920 x 1080 instead
                                      // of 108, 45 rows: 116)
static_assert(kStrip == kWave, "a strip's columns are a wave's lanes");
constexpr int kStaged = kStrip + 2 * kHalo;
constexpr int kStripThreads = 3 * kWave;  // one wave per channel
constexpr int kAhead = 3;             // rows loaded ahead (2: 116 us at 1920 x 1080, 3: 108, 4: 118, 5: 129)
constexpr int kLossViewsPerLaunch = 16;
constexpr float kC1 = 0.01f * 0.01f;
constexpr float kC2 = 0.03f * 0.03f;

// Views of one launch, passed by value: sizes, first pixel of each view in
// the concatenated images, first tile (16 x 16, or a strip) of each view and
// the loss scale 1 / (P_v V) of each view.
struct LossViews {
  int32_t nv;
  int32_t tile0;  // first tile of this launch (global index)
  int32_t width[kLossViewsPerLaunch];
  int32_t height[kLossViewsPerLaunch];
  int32_t tiles_x[kLossViewsPerLaunch];
  int32_t tile_base[kLossViewsPerLaunch + 1];  // local to the launch
  int64_t pix_base[kLossViewsPerLaunch];
  float scale[kLossViewsPerLaunch];
  float gauss[11];  // normalised window taps
};

struct LossArgs {
  const float* img;
  const float* target;
  float* dmaps;           // [3][channel][pixel] derivative maps (tiles)
  float2* dmap2;          // the same for strips: [channel][pixel] dS/du and dS/dSxx
  float* dmap1;           // and [channel][pixel] dS/dSxy
  double* part;           // [tile * 3 + channel] loss shares
  float* dL;
  int64_t total_pixels;
  float lambda;
};

struct TileWhere {
  int v, tx0, ty0;
};

__device__ __forceinline__ TileWhere loss_tile(const LossViews& lv, int t) {
  int v = 0;
  while (v + 1 < lv.nv && lv.tile_base[v + 1] <= t) ++v;
  const int local = t - lv.tile_base[v];
  return {v, (local % lv.tiles_x[v]) * kLT, (local / lv.tiles_x[v]) * kLT};
}

// Stage the (26 x 26) region of the tile in M sources -- channel `ch` of the
// interleaved [pix][3] images (stride 3) or planar maps (stride 1) -- with
// zeros outside the view, interleaved in LDS (source q in component q of a
// float2 or float4), so that a filter tap reads all of them at once.  Every
// load of the thread is issued before the first LDS store, so a workgroup
// pays one memory round trip for all M.
constexpr int kStageIters = (kLE * kLE + 255) / 256;

template <int M>
using StageVec = typename std::conditional<M == 2, float2, float4>::type;

template <int M>
__device__ __forceinline__ void stage(StageVec<M> (*dst)[kLE + 1], const float* const src[M], int stride, int ch,
                                      const LossViews& lv, const TileWhere& w) {
  static_assert(M == 2 || M == 3, "two or three interleaved sources");
  const int width = lv.width[w.v], height = lv.height[w.v];
  const int64_t base = lv.pix_base[w.v];
  float val[M][kStageIters];
#pragma unroll
  for (int it = 0; it < kStageIters; ++it) {
    const int k = threadIdx.x + 256 * it;
    const int r = k / kLE, cc = k % kLE;
    const int py = w.ty0 - kHalo + r, px = w.tx0 - kHalo + cc;
    const bool in = k < kLE * kLE && px >= 0 && py >= 0 && px < width && py < height;
    // outside the view the load reads the view's first pixel and is discarded
    const int64_t pix = base + (in ? static_cast<int64_t>(py) * width + px : 0);
#pragma unroll
    for (int q = 0; q < M; ++q) {
      const float x = src[q][pix * stride + ch];
      val[q][it] = in ? x : 0.f;
    }
  }
#pragma unroll
  for (int it = 0; it < kStageIters; ++it) {
    const int k = threadIdx.x + 256 * it;
    if (k < kLE * kLE) {
      if constexpr (M == 2)
        dst[k / kLE][k % kLE] = make_float2(val[0][it], val[1][it]);
      else
        dst[k / kLE][k % kLE] = make_float4(val[0][it], val[1][it], val[2][it], 0.f);
    }
  }
}

__device__ __forceinline__ double block_sum_256(double x, double* sh) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, kWave);
  if ((threadIdx.x & (kWave - 1)) == 0) sh[threadIdx.x / kWave] = x;
  __syncthreads();
  const double t = sh[0] + sh[1] + sh[2] + sh[3];
  __syncthreads();
  return t;
}

// The map at a pixel and its derivatives, from the windowed statistics.  Every
// fused operation is written out and none is left to the compiler, so that tiles
// and strips give the same bits.
struct SsimTerm {
  float s, d_u, d_sxx, d_sxy;
};
__device__ __forceinline__ SsimTerm ssim_term(float u, float v, float sxx, float syy, float sxy) {
#pragma clang fp contract(off)
  const float u2 = u + u, v2 = v + v;
  const float a1 = fmaf(v, u2, kC1);
  const float a2 = fmaf(2.f, fmaf(-v, u, sxy), kC2);
  const float b1 = fmaf(v, v, u * u) + kC1;
  const float b2 = (fmaf(-v, v, syy) + fmaf(-u, u, sxx)) + kC2;
  const float ib = 1.f / (b1 * b2);
  SsimTerm t;
  t.s = a1 * a2 * ib;
  t.d_u = fmaf(fmaf(v2, a2, -(v2 * a1)), ib, (u2 / b1 - u2 / b2) * -t.s);
  t.d_sxx = -t.s / b2;
  t.d_sxy = (a1 + a1) * ib;
  return t;
}

// An entry's part of L_v V P_v: (1 - lambda)|x - y| + lambda (1 - S).
__device__ __forceinline__ double loss_share(float x, float y, float s, float lambda) {
  return (1.0 - lambda) * fabs(static_cast<double>(x) - y) + lambda * (1.0 - static_cast<double>(s));
}

// dL/dx of an entry from the filtered derivative maps f (see ssim_term).
__device__ __forceinline__ float loss_grad(float x, float y, float f0, float f1, float f2, float lambda, float scale) {
#pragma clang fp contract(off)
  const float sgn = x > y ? 1.f : (x < y ? -1.f : 0.f);
  const float dmean = fmaf(y, f2, fmaf(x + x, f1, f0));
  return scale * fmaf(1.f - lambda, sgn, -(lambda * dmean));
}

__global__ __launch_bounds__(256) void loss_pass1(LossArgs a, LossViews lv) {
  __shared__ float2 s_xy[kLE][kLE + 1];   // (x, y)
  __shared__ float4 s_h4[kLE][kLT + 1];   // row-filtered x, y, x^2, y^2
  __shared__ float s_h1[kLE][kLT + 1];    // row-filtered x y
  __shared__ double s_red[4];
  const int t = blockIdx.x, ch = blockIdx.y;
  const TileWhere w = loss_tile(lv, t);
  {
    const float* const src[2] = {a.img, a.target};
    stage<2>(s_xy, src, 3, ch, lv, w);
  }
  __syncthreads();
  // row pass of the separable filter: the 26 rows, the 16 output columns
  for (int k = threadIdx.x; k < kLE * kLT; k += 256) {
    const int r = k / kLT, c = k % kLT;
    float hx = 0.f, hy = 0.f, hxx = 0.f, hyy = 0.f, hxy = 0.f;
#pragma unroll
    for (int b = 0; b < 11; ++b) {
      const float gb = lv.gauss[b];
      const float2 xy = s_xy[r][c + b];
      const float x = xy.x, y = xy.y;
      hx = fmaf(gb, x, hx);
      hy = fmaf(gb, y, hy);
      hxx = fmaf(gb, x * x, hxx);
      hyy = fmaf(gb, y * y, hyy);
      hxy = fmaf(gb, x * y, hxy);
    }
    s_h4[r][c] = make_float4(hx, hy, hxx, hyy);
    s_h1[r][c] = hxy;
  }
  __syncthreads();
  const int i = threadIdx.x / kLT, j = threadIdx.x % kLT;
  const int px = w.tx0 + j, py = w.ty0 + i;
  double share = 0.0;
  if (px < lv.width[w.v] && py < lv.height[w.v]) {
    // column pass
    float u = 0.f, v = 0.f, sxx = 0.f, syy = 0.f, sxy = 0.f;
#pragma unroll
    for (int q = 0; q < 11; ++q) {
      const float gq = lv.gauss[q];
      const float4 h = s_h4[i + q][j];
      const float h1 = s_h1[i + q][j];
      u = fmaf(gq, h.x, u);
      v = fmaf(gq, h.y, v);
      sxx = fmaf(gq, h.z, sxx);
      syy = fmaf(gq, h.w, syy);
      sxy = fmaf(gq, h1, sxy);
    }
    const SsimTerm m = ssim_term(u, v, sxx, syy, sxy);
    const int64_t pix = lv.pix_base[w.v] + static_cast<int64_t>(py) * lv.width[w.v] + px;
    const int64_t P = a.total_pixels;
    a.dmaps[(0 * 3 + ch) * P + pix] = m.d_u;
    a.dmaps[(1 * 3 + ch) * P + pix] = m.d_sxx;
    a.dmaps[(2 * 3 + ch) * P + pix] = m.d_sxy;
    const float x = s_xy[i + kHalo][j + kHalo].x, y = s_xy[i + kHalo][j + kHalo].y;
    share = loss_share(x, y, m.s, a.lambda);
  }
  share = block_sum_256(share, s_red);
  if (threadIdx.x == 0) a.part[static_cast<int64_t>(lv.tile0 + t) * 3 + ch] = share * lv.scale[w.v];
}

__global__ __launch_bounds__(256) void loss_pass2(LossArgs a, LossViews lv) {
  __shared__ float4 s_m[kLE][kLE + 1];   // the three derivative maps (fourth component unused)
  __shared__ float4 s_h[kLE][kLT + 1];   // the same, row-filtered
  const int t = blockIdx.x, ch = blockIdx.y;
  const TileWhere w = loss_tile(lv, t);
  const int i = threadIdx.x / kLT, j = threadIdx.x % kLT;
  const int64_t P = a.total_pixels;
  {
    const float* const src[3] = {a.dmaps + (0 * 3 + ch) * P, a.dmaps + (1 * 3 + ch) * P, a.dmaps + (2 * 3 + ch) * P};
    stage<3>(s_m, src, 1, 0, lv, w);
  }
  __syncthreads();
  for (int k = threadIdx.x; k < kLE * kLT; k += 256) {
    const int r = k / kLT, c = k % kLT;
    float h0 = 0.f, h1 = 0.f, h2 = 0.f;
#pragma unroll
    for (int b = 0; b < 11; ++b) {
      const float gb = lv.gauss[b];
      const float4 m = s_m[r][c + b];
      h0 = fmaf(gb, m.x, h0);
      h1 = fmaf(gb, m.y, h1);
      h2 = fmaf(gb, m.z, h2);
    }
    s_h[r][c] = make_float4(h0, h1, h2, 0.f);
  }
  __syncthreads();
  float f[3] = {0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < 11; ++q) {
    const float gq = lv.gauss[q];
    const float4 h = s_h[i + q][j];
    f[0] = fmaf(gq, h.x, f[0]);
    f[1] = fmaf(gq, h.y, f[1]);
    f[2] = fmaf(gq, h.z, f[2]);
  }
  const int px = w.tx0 + j, py = w.ty0 + i;
  if (px >= lv.width[w.v] || py >= lv.height[w.v]) return;
  const int64_t pix = lv.pix_base[w.v] + static_cast<int64_t>(py) * lv.width[w.v] + px;
  const float x = a.img[3 * pix + ch], y = a.target[3 * pix + ch];
  a.dL[3 * pix + ch] = loss_grad(x, y, f[0], f[1], f[2], a.lambda, lv.scale[w.v]);
}

// Where a strip lies, and the lane's part of a staged row: its own pixel at
// the strip's left edge - 5 + lane and, for the first ten lanes, the one 64
// further on.  A pixel outside the view reads a pixel of it and counts as zero.
struct Strip {
  int v, x0, y0;
  int width, height;
  int64_t pix_base;
  int c0, c1;        // columns read
  bool in0, in1;
};

__device__ __forceinline__ Strip loss_strip(const LossViews& lv, int t, int lane) {
  Strip w;
  w.v = 0;
  while (w.v + 1 < lv.nv && lv.tile_base[w.v + 1] <= t) ++w.v;
  const int local = t - lv.tile_base[w.v];
  w.x0 = local % lv.tiles_x[w.v] * kStrip;
  w.y0 = local / lv.tiles_x[w.v] * kStripRows;
  w.width = lv.width[w.v];
  w.height = lv.height[w.v];
  w.pix_base = lv.pix_base[w.v];
  const int a = w.x0 - kHalo + lane, b = a + kWave;
  w.in0 = a >= 0 && a < w.width;
  w.in1 = lane < 2 * kHalo && b < w.width;
  w.c0 = min(max(a, 0), w.width - 1);
  w.c1 = min(b, w.width - 1);
  return w;
}

// The taps in vector registers (an operand from a scalar register halves the
// rate of a fused multiply-add), six values since the window is symmetric.
struct Taps {
  float g[kHalo + 1];
  __device__ __forceinline__ float operator[](int k) const { return g[k <= kHalo ? k : 2 * kHalo - k]; }
};
__device__ __forceinline__ Taps load_taps(const LossViews& lv) {
  Taps t;
#pragma unroll
  for (int k = 0; k <= kHalo; ++k) {
    t.g[k] = lv.gauss[k];
    asm("" : "+v"(t.g[k]));
  }
  return t;
}

// LDS writes of this wave before, LDS reads of this wave after.
__device__ __forceinline__ void row_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__global__ __launch_bounds__(kStripThreads, 4) void loss_strip_pass1(LossArgs a, LossViews lv) {
  __shared__ float2 s_xy[3][kStaged + 6];
  const int lane = threadIdx.x % kWave, ch = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const Strip w = loss_strip(lv, blockIdx.x, lane);
  const Taps g = load_taps(lv);
  float2* row = s_xy[ch];
  const int y1 = min(w.y0 + kStripRows, w.height);  // end of the output rows
  const bool out_col = w.x0 + lane < w.width;

  // staged rows: the k-th is image row y0 - 5 + k
  struct Loaded {
    float x0, y0, x1, y1;
  } ahead[kTaps];
  auto load = [&](int k) {
    const int py = min(max(w.y0 - kHalo + k, 0), w.height - 1);
    const int64_t at = 3 * (w.pix_base + static_cast<int64_t>(py) * w.width) + ch;
    const float *img = a.img + at, *tgt = a.target + at;
    return Loaded{img[3 * w.c0], tgt[3 * w.c0], img[3 * w.c1], tgt[3 * w.c1]};
  };
#pragma unroll
  for (int k = 0; k < kAhead; ++k) ahead[k] = load(k);

  float hx[kTaps], hy[kTaps], hxx[kTaps], hyy[kTaps], hxy[kTaps], cx[kTaps], cy[kTaps];
  double share = 0.0;
  for (int k0 = 0; w.y0 + k0 - 2 * kHalo < y1; k0 += kTaps) {
#pragma unroll
    for (int k = 0; k < kTaps; ++k) {
      const Loaded l = ahead[k];
      ahead[(k + kAhead) % kTaps] = load(k0 + k + kAhead);
      const int py = w.y0 - kHalo + k0 + k;
      const bool in = py >= 0 && py < w.height;
      row_fence();
      row[lane] = w.in0 && in ? make_float2(l.x0, l.y0) : make_float2(0.f, 0.f);
      if (lane < 2 * kHalo) row[kWave + lane] = w.in1 && in ? make_float2(l.x1, l.y1) : make_float2(0.f, 0.f);
      row_fence();
      float sx = 0.f, sy = 0.f, sxx = 0.f, syy = 0.f, sxy = 0.f;
#pragma unroll
      for (int b = 0; b < kTaps; ++b) {
        const float2 xy = row[lane + b];
        const float x = xy.x, y = xy.y;
        sx = fmaf(g[b], x, sx);
        sy = fmaf(g[b], y, sy);
        sxx = fmaf(g[b], x * x, sxx);
        syy = fmaf(g[b], y * y, syy);
        sxy = fmaf(g[b], x * y, sxy);
        if (b == kHalo) {
          cx[k] = x;
          cy[k] = y;
        }
      }
      hx[k] = sx;
      hy[k] = sy;
      hxx[k] = sxx;
      hyy[k] = syy;
      hxy[k] = sxy;
      const int oy = w.y0 + k0 + k - 2 * kHalo;  // the output row whose window ends here
      if (oy < w.y0 || oy >= y1) continue;
      // along the column, the oldest row first
      float u = 0.f, v = 0.f;
      sxx = syy = sxy = 0.f;
#pragma unroll
      for (int q = 0; q < kTaps; ++q) {
        const int r = (k + 1 + q) % kTaps;
        u = fmaf(g[q], hx[r], u);
        v = fmaf(g[q], hy[r], v);
        sxx = fmaf(g[q], hxx[r], sxx);
        syy = fmaf(g[q], hyy[r], syy);
        sxy = fmaf(g[q], hxy[r], sxy);
      }
      const SsimTerm m = ssim_term(u, v, sxx, syy, sxy);
      if (out_col) {
        const int64_t at = ch * a.total_pixels + w.pix_base + static_cast<int64_t>(oy) * w.width + w.x0;
        (a.dmap2 + at)[lane] = make_float2(m.d_u, m.d_sxx);
        (a.dmap1 + at)[lane] = m.d_sxy;
        const float x = cx[(k + 1 + kHalo) % kTaps], y = cy[(k + 1 + kHalo) % kTaps];
        share += loss_share(x, y, m.s, a.lambda);
      }
    }
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) share += __shfl_xor(share, d, kWave);
  if (lane == 0) a.part[static_cast<int64_t>(lv.tile0 + static_cast<int>(blockIdx.x)) * 3 + ch] = share * lv.scale[w.v];
}

// The gradient's rows go through LDS so that the three waves' channels are
// stored interleaved, whole rows at a time.
__global__ __launch_bounds__(kStripThreads, 4) void loss_strip_pass2(LossArgs a, LossViews lv) {
  __shared__ float2 s_m2[3][kStaged + 6];
  __shared__ float s_m1[3][kStaged + 6];
  __shared__ float s_out[kTaps][3 * kStrip];
  const int lane = threadIdx.x % kWave, ch = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const Strip w = loss_strip(lv, blockIdx.x, lane);
  const Taps g = load_taps(lv);
  float2* row2 = s_m2[ch];
  float* row1 = s_m1[ch];
  const int y1 = min(w.y0 + kStripRows, w.height);
  const int64_t plane = ch * a.total_pixels + w.pix_base;
  const int cols = min(kStrip, w.width - w.x0);
  const int oc = min(lane, cols - 1);  // output column read
  const float sc = lv.scale[w.v], lambda = a.lambda;

  struct Loaded {
    float2 m0, m1;
    float n0, n1, x, y;  // (x, y): the output pixel whose window ends with this row
  } ahead[kTaps];
  auto load = [&](int k) {
    const int py = min(max(w.y0 - kHalo + k, 0), w.height - 1);
    const int64_t at = plane + static_cast<int64_t>(py) * w.width;
    const float2* m2 = a.dmap2 + at;
    const float* m1 = a.dmap1 + at;
    const int oy = min(max(w.y0 + k - 2 * kHalo, 0), w.height - 1);
    const int64_t o = 3 * (w.pix_base + static_cast<int64_t>(oy) * w.width + w.x0) + ch;
    return Loaded{m2[w.c0], m2[w.c1], m1[w.c0], m1[w.c1], (a.img + o)[3 * oc], (a.target + o)[3 * oc]};
  };
#pragma unroll
  for (int k = 0; k < kAhead; ++k) ahead[k] = load(k);

  float h0[kTaps], h1[kTaps], h2[kTaps];
  for (int k0 = 0; w.y0 + k0 - 2 * kHalo < y1; k0 += kTaps) {
#pragma unroll
    for (int k = 0; k < kTaps; ++k) {
      const Loaded l = ahead[k];
      ahead[(k + kAhead) % kTaps] = load(k0 + k + kAhead);
      const int py = w.y0 - kHalo + k0 + k;
      const bool in = py >= 0 && py < w.height;
      row_fence();
      row2[lane] = w.in0 && in ? l.m0 : make_float2(0.f, 0.f);
      row1[lane] = w.in0 && in ? l.n0 : 0.f;
      if (lane < 2 * kHalo) {
        row2[kWave + lane] = w.in1 && in ? l.m1 : make_float2(0.f, 0.f);
        row1[kWave + lane] = w.in1 && in ? l.n1 : 0.f;
      }
      row_fence();
      float s0 = 0.f, s1 = 0.f, s2 = 0.f;
#pragma unroll
      for (int b = 0; b < kTaps; ++b) {
        const float2 m = row2[lane + b];
        s0 = fmaf(g[b], m.x, s0);
        s1 = fmaf(g[b], m.y, s1);
        s2 = fmaf(g[b], row1[lane + b], s2);
      }
      h0[k] = s0;
      h1[k] = s1;
      h2[k] = s2;
      const int oy = w.y0 + k0 + k - 2 * kHalo;
      if (oy < w.y0 || oy >= y1) continue;
      float f0 = 0.f, f1 = 0.f, f2 = 0.f;
#pragma unroll
      for (int q = 0; q < kTaps; ++q) {
        const int r = (k + 1 + q) % kTaps;
        f0 = fmaf(g[q], h0[r], f0);
        f1 = fmaf(g[q], h1[r], f1);
        f2 = fmaf(g[q], h2[r], f2);
      }
      s_out[k][3 * lane + ch] = loss_grad(l.x, l.y, f0, f1, f2, lambda, sc);
    }
    __syncthreads();
    const int t = static_cast<int>(threadIdx.x);
#pragma unroll
    for (int k = 0; k < kTaps; ++k) {
      const int oy = w.y0 + k0 + k - 2 * kHalo;
      if (oy < w.y0 || oy >= y1 || t >= 3 * cols) continue;
      (a.dL + 3 * (w.pix_base + static_cast<int64_t>(oy) * w.width + w.x0))[t] = s_out[k][t];
    }
    __syncthreads();
  }
}

// Sum of the tiles' shares in a fixed order: one block, strided partial sums,
// then a tree over the block.
__global__ __launch_bounds__(256) void loss_finalize(const double* part, int64_t n, float* loss) {
  __shared__ double s_red[4];
  double s = 0.0;
  // unrolled so that a thread's loads are in flight together (same order of additions)
#pragma unroll 8
  for (int64_t k = threadIdx.x; k < n; k += 256) s += part[k];
  s = block_sum_256(s, s_red);
  if (threadIdx.x == 0) *loss = static_cast<float>(s);
}

// Adam with bias correction; bc1 = 1 - beta1^t, bc2 = 1 - beta2^t.
__global__ __launch_bounds__(256) void adam_kernel(float* p, const float* g, float* m, float* v, int64_t n,
                                                   float lr, AdamStep as) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * 256;
  for (int64_t k = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; k < n; k += stride) {
    float mk = m[k], vk = v[k];
    p[k] = adam_update(p[k], g[k], mk, vk, lr, as);
    m[k] = mk;
    v[k] = vk;
  }
}

// Taps of the normalised 11-tap Gaussian window (sigma 1.5), in double then
// rounded once.
void gauss_taps(float* g) {
  double sum = 0.0, gd[11];
  for (int k = 0; k < 11; ++k) {
    const double d = k - 5;
    gd[k] = std::exp(-(d * d) / (2.0 * 1.5 * 1.5));
    sum += gd[k];
  }
  for (int k = 0; k < 11; ++k) g[k] = static_cast<float>(gd[k] / sum);
}

}  // namespace

// Tiles of all views, `w` by `h` pixels each.
int64_t loss_tiles(const wsr_camera* cams, int32_t nv, int w, int h) {
  int64_t t = 0;
  for (int v = 0; v < nv; ++v)
    t += static_cast<int64_t>((cams[v].width + w - 1) / w) * ((cams[v].height + h - 1) / h);
  return t;
}

int64_t loss_workspace_bytes(const wsr_camera* cams, int32_t nv) {
  int64_t pixels = 0;
  for (int v = 0; v < nv; ++v) pixels += static_cast<int64_t>(cams[v].width) * cams[v].height;
  const int64_t maps = (sizeof(float) * 9 * pixels + 255) / 256 * 256;
  return maps + static_cast<int64_t>(sizeof(double)) * 3 * loss_tiles(cams, nv, kLT, kLT);
}

hipError_t launch_loss(const wsr_camera* cams, int32_t nv, const float* img, const float* target, float lambda,
                       void* ws, float* loss, float* dL, hipStream_t st) {
  int64_t pixels = 0;
  for (int v = 0; v < nv; ++v) pixels += static_cast<int64_t>(cams[v].width) * cams[v].height;
  LossArgs a;
  a.img = img;
  a.target = target;
  a.dmaps = static_cast<float*>(ws);
  a.dmap2 = static_cast<float2*>(ws);
  a.dmap1 = static_cast<float*>(ws) + 6 * pixels;
  a.part = reinterpret_cast<double*>(static_cast<char*>(ws) + (sizeof(float) * 9 * pixels + 255) / 256 * 256);
  a.dL = dL;
  a.total_pixels = pixels;
  a.lambda = lambda;
  int64_t pix_base = 0;
  int32_t tile0 = 0;
  for (int v0 = 0; v0 < nv; v0 += kLossViewsPerLaunch) {
    LossViews lv = {};
    gauss_taps(lv.gauss);
    lv.nv = nv - v0 < kLossViewsPerLaunch ? nv - v0 : kLossViewsPerLaunch;
    lv.tile0 = tile0;
    const wsr_camera* c = cams + v0;
    int64_t here = 0;
    for (int k = 0; k < lv.nv; ++k) here += static_cast<int64_t>(c[k].width) * c[k].height;
    const bool strips = loss_in_strips(loss_tiles(c, lv.nv, kLT, kLT), loss_tiles(c, lv.nv, kStrip, kStripRows), here);
    const int tw = strips ? kStrip : kLT, th = strips ? kStripRows : kLT;
    int32_t tiles = 0;
    for (int k = 0; k < lv.nv; ++k) {
      lv.width[k] = c[k].width;
      lv.height[k] = c[k].height;
      lv.tiles_x[k] = (c[k].width + tw - 1) / tw;
      lv.tile_base[k] = tiles;
      lv.pix_base[k] = pix_base;
      lv.scale[k] = static_cast<float>(1.0 / (3.0 * c[k].width * c[k].height * nv));
      tiles += lv.tiles_x[k] * ((c[k].height + th - 1) / th);
      pix_base += static_cast<int64_t>(c[k].width) * c[k].height;
    }
    lv.tile_base[lv.nv] = tiles;
    tile0 += tiles;
    if (tiles == 0) continue;
    // both passes of these views before the next ones, whose maps may lie
    // otherwise in the same workspace
    const unsigned count = static_cast<unsigned>(tiles);
    if (strips) {
      loss_strip_pass1<<<count, kStripThreads, 0, st>>>(a, lv);
      loss_strip_pass2<<<count, kStripThreads, 0, st>>>(a, lv);
    } else {
      loss_pass1<<<dim3(count, 3), 256, 0, st>>>(a, lv);
      loss_pass2<<<dim3(count, 3), 256, 0, st>>>(a, lv);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  loss_finalize<<<1, 256, 0, st>>>(a.part, static_cast<int64_t>(tile0) * 3, loss);
  return hipGetLastError();
}

// Device address of `scratch` on the current device, looked up once per
// device (with that device current) and kept.
namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch[kMaxDevices] = {};
}  // namespace

hipError_t loss_static_workspace(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p || reinterpret_cast<uintptr_t>(p) % 256 != 0) return hipErrorInvalidValue;
    g_scratch[dev] = p;
  }
  *out = g_scratch[dev];
  return hipSuccess;
}

hipError_t launch_adam(float* p, const float* g, float* m, float* v, int64_t n, int32_t step, float lr, float b1,
                       float b2, float eps, hipStream_t st) {
  if (n == 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  adam_kernel<<<static_cast<unsigned>(blocks), 256, 0, st>>>(p, g, m, v, n, lr, make_adam_step(step, b1, b2, eps));
  return hipGetLastError();
}

}  // namespace wsr
