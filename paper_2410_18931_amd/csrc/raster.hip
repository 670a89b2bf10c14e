// Steps a7 and a8 of the WSR path: the per-pixel weighted sums of Sec. 4.2,
// Eq. 7, and their gradient.
//
//   forward:  N = c_B w_B + sum_i c_i a_i,  D = w_B + sum_i a_i,  C = N / D
//             a_i = amp_i exp(-q_i / 2) for q_i <= tau   (amp_i = u_i w(d_i))
//   backward: per pixel gbar = dL/dC / D and s = gbar . C; per pair
//             dL/da = gbar . c_i - s, then the chain to (mu, conic, c, amp).
//
// One workgroup per work item (at most kItemSplats splats of one tile's list); the
// items are dispatched longest first (the full ones, then the tiles' last
// items by decreasing length; see tile_scan_single), so that the launch ends
// on short items.
// Each wave owns an 8x8 pixel block of the tile.  Per batch the group stages
// splat records into LDS; each wave then keeps only the splats whose support
// reaches its own block (support box, then the exact minimum of q over the
// block; wave ballot + compaction into an LDS list).  In the forward every
// lane evaluates its pixel against that list with FP32 register
// accumulation; in the backward every lane takes one splat of the list and
// walks the block.  The sums are commutative, so the list order does not
// matter, and no per-pair data is stored between forward and backward: the
// backward recomputes every pair.
#include <algorithm>
#include <map>
#include <mutex>
#include <type_traits>
#include <utility>

#include "wsr_internal.h"

namespace wsr {
namespace {

// Every wave owns an 8x8 pixel block of the tile (one pixel per lane): tile 8
// is one wave, tile 16 four, tile 32 sixteen.  Up to 256 records are staged
// per batch.
//
// A splat is culled against sub-blocks: the 8 wide, 4 high halves of the 8x8
// blocks, which it must pay for 10 to 24 % fewer pixels than for whole blocks
// (1.45 -> 1.31 evaluated pixels per pixel in its support at 1 M Gaussians /
// 1080p, 1.71 -> 1.48 at 200 k / 720p, 3.0 -> 2.3 at 30 k / 400 x 300).
// Quarters (4 x 4) would save as much again, but a row of four pixels shares
// its row terms among too few.  Tile 32 keeps whole blocks: its 32 halves'
// culling masks would not fit the pair buffer.
template <int T>
struct TileGeom {
  static constexpr int kSub = 8;                       // wave block edge
  static constexpr int kWaves = (T / 8) * (T / 8);
  static constexpr int kHalves = T == 32 ? 1 : 2;      // sub-blocks of a wave block, one above the other
  static constexpr int kRows = 8 / kHalves;            // rows of a sub-block
  static constexpr int kSubs = kWaves * kHalves;       // sub-blocks of the tile: wave block b's are b kHalves ..
  static constexpr int kThreads = kWaves * kWave;
  static constexpr int kBatch = kThreads < 256 ? kThreads : 256;
  static_assert(kBatch <= 256, "the sorted composite's lists hold 8-bit record indices");
  // first pixel centre of a sub-block relative to the tile's centre (exact)
  static __device__ __forceinline__ float sub_x(int s) {
    return static_cast<float>((s / kHalves % (T / 8)) * 8 - T / 2) + 0.5f;
  }
  static __device__ __forceinline__ float sub_y(int s) {
    return static_cast<float>((s / kHalves / (T / 8)) * 8 + (s % kHalves) * kRows - T / 2) + 0.5f;
  }
};

// A record as staged in LDS for one tile (48 bytes; stage_and_cull builds it
// from the projected record):
//   r0 = (mx, my, A, B2)   centre relative to the tile's centre; conic
//                          (A, B2 = 2B, C) times log2(e) / 2
//   r1 = (c0, c1, c2, amp) colour (times amp in the forward)
//   r2 = (C, ext | cut, u, K)  support half-extents (two halves), or with
//                          the early-out the record's own cutoff times
//                          log2(e) / 2 and its support_k; u = the opacity,
//                          used by OIT only
// The tile-relative centre is (integer origin - tile centre) + fractional
// centre: the difference is exact, the sum rounds once (to within 2^-24 of
// its magnitude, which is at most the pixel's distance plus half the tile
// size).  Pixel centres relative to the tile centre are exact, so dx and dy
// round once more.  With the conic scaled, the form below is q log2(e) / 2, the
// falloff exp(-q / 2) is one hardware exp2 of its negation, and every cutoff
// it is compared with (tau, a record's own cutoff) carries the same factor.
struct StagedRec {
  float4 r0, r1, r2;
};
static_assert(sizeof(StagedRec) == 48, "staged record layout");

constexpr float kHalfLog2e = 0.72134752044448170f;  // log2(e) / 2
constexpr float kTwoLn2 = 1.38629436111989061f;     // its inverse

// The support predicate and the Gaussian falloff.  Forward and backward
// evaluate q with exactly this sequence of float operations (the backward
// hoists the row-constant products B2*dy and (C*dy)*dy, which does not change
// their values), so both take the same support decision for every pair.
// Different tile sizes round the tile-relative centre differently, so they
// can disagree on a pair within that rounding of the cutoff.
__device__ __forceinline__ float quad_form(float A, float B2dy, float Cdy2, float dx) {
  return fmaf(fmaf(A, dx, B2dy), dx, Cdy2);
}

// px, py: the pixel centre relative to the tile's centre
__device__ __forceinline__ float pair_q(const StagedRec& r, float px, float py) {
  const float dx = px - r.r0.x;
  const float dy = py - r.r0.y;
  return quad_form(r.r0.z, r.r0.w * dy, (r.r2.x * dy) * dy, dx);
}

// exp(-q/2) from the scaled form q log2(e) / 2
__device__ __forceinline__ float falloff(float qs) { return __builtin_amdgcn_exp2f(-qs); }

// Transcendentals of one row of eight pixels, back to back at raised wave
// priority.  A SIMD issues two plain FP32 operations of different waves at
// once (2.5 cycles per wave instruction with four or eight waves) but a
// transcendental alone (8.5 cycles); scattered among the waves' other work
// each one also breaks up pairs around it.  Issued as one burst that the other
// waves let pass, they leave those to pair up again.  A loop of the forward's
// operations per pixel took 44 cycles per wave with the exp2 in its natural
// place or in bursts of eight, and 30.6 in bursts at raised priority; the
// backward's 64.6 and 40.8.
template <typename F>
__device__ __forceinline__ void trans_burst(F&& f) {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_setprio(3);
  __builtin_amdgcn_sched_barrier(0);
  f();
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_setprio(0);
  __builtin_amdgcn_sched_barrier(0);
}

// The support predicate q <= cut as a factor in plain FP32 arithmetic, which
// pairs with other waves' work (a compare and select are half-rate operations
// with wait states between them): clamp(K - q 2^64) to [0, 1] with
// K = 2^64 next(cut), next the following float.  K - q 2^64 is rounded once,
// so it is <= 0 for q > cut (q >= next(cut)) and, an ulp of the cutoff being
// at least 2^-64 for cut >= 2^-41, >= 1 for q <= cut.  A smaller cutoff
// (tau = 0) keeps q = 0; one above 2^63 keeps every q, whose falloff is 0
// there.  A NaN clamps to 0.  cut < 0 passes no pixel.
constexpr float kSupportScale = 0x1p64f;
__device__ __forceinline__ float support_k(float cut) {
  return cut < 0.f ? -kSupportScale : fmaxf(__uint_as_float(__float_as_uint(cut) + 1u) * kSupportScale, 1.f);
}
__device__ __forceinline__ float in_support(float q, float K) {
  return __builtin_amdgcn_fmed3f(fmaf(q, -kSupportScale, K), 0.f, 1.f);
}

// x m with 0 m = x 0 = 0 whatever the other factor, NaN included.
__device__ __forceinline__ float mul_zero_wins(float x, float m) {
  float r;
  asm("v_mul_legacy_f32 %0, %1, %2" : "=v"(r) : "v"(x), "v"(m));
  return r;
}

// exp(-q/2) of a row's eight pixels where q <= cut (K = support_k(cut)), else
// 0, also where q is NaN.
__device__ __forceinline__ void falloff_row(const float (&q)[8], float K, float (&G)[8]) {
  float x[8];
  trans_burst([&] {
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = falloff(q[k]);
  });
#pragma unroll
  for (int k = 0; k < 8; ++k) G[k] = mul_zero_wins(x[k], in_support(q[k], K));
}

__device__ __forceinline__ float2 rec_extent(const StagedRec& r) {
  const uint32_t e = __float_as_uint(r.r2.y);
  const _Float16 ex = __builtin_bit_cast(_Float16, static_cast<uint16_t>(e & 0xffffu));
  const _Float16 ey = __builtin_bit_cast(_Float16, static_cast<uint16_t>(e >> 16));
  return make_float2(static_cast<float>(ex), static_cast<float>(ey));
}

// Does the splat's support reach the pixel centres spanning
// [bx, bx + 7] x [by, by + h] (relative to the tile's centre)?  First the
// (conservative) support box; then, unless the conic is badly conditioned, the
// exact minimum of q over the rectangle against tau with a margin far above
// the float error of q.  The minimum is at the centre, or on one of the (at
// most two) edges that face it: on the nearest vertical line at its clamped 1D
// minimiser, or on the nearest horizontal one.  Where the centre lies within
// the rectangle's columns the nearest vertical line passes through it and that
// point is one of the rectangle, no further below the minimum.  For
// needle-like splats (eigenvalue ratio above ~100) float q loses digits to
// cancellation, so the box decision is kept.
//
// With CUT (the opacity early-out) the record's fourth word is the splat's
// own cutoff instead of the half-extents, which are then derived from the
// conic: the extents of q <= cut are sqrt(cut C / det) and sqrt(cut A / det),
// with det = A C - B^2 formed by Kahan's algorithm (B^2 split exactly with an
// FMA) so that it stays accurate for needle-like conics.
struct SupportBox {
  float ex, ey;     // half-extents with their rounding slack
  float tau;        // cutoff with its margin (infinite where the box decides)
  float kx, ky;     // -B / A, -B / C
};

template <bool CUT>
__device__ __forceinline__ SupportBox support_box(const StagedRec& r, float tau_in) {
  SupportBox b;
  const float A = r.r0.z, B = 0.5f * r.r0.w, C = r.r2.x;
  float tau = tau_in;
  if (CUT) {
    tau = r.r2.y;
    const float bb = B * B;
    const float det = fmaf(A, C, -bb) - fmaf(B, B, -bb);
    const float s = det > 0.f ? tau * __builtin_amdgcn_rcpf(det) : __builtin_inff();
    b.ex = sqrtf(s * C) * 1.0001f;
    b.ey = sqrtf(s * A) * 1.0001f;
  } else {
    const float2 e = rec_extent(r);
    b.ex = e.x;
    b.ey = e.y;
  }
  b.ex += 1e-3f * fabsf(r.r0.x) + 1e-2f;
  b.ey += 1e-3f * fabsf(r.r0.y) + 1e-2f;
  const float tr = A + C, det = A * C - B * B;
  b.tau = tr * tr <= 102.f * det ? tau * 1.002f + 1e-3f : __builtin_inff();
  // hardware reciprocals (within 1 ulp): they only place the edge minimisers,
  // whose error changes q there by a second-order amount far inside the margin
  b.kx = -B * __builtin_amdgcn_rcpf(A);
  b.ky = -B * __builtin_amdgcn_rcpf(C);
  return b;
}

// (without branches: the comparisons of the box are shared by the sub-blocks
// of a column or row)
__device__ __forceinline__ bool rect_hits(const StagedRec& r, const SupportBox& b, float bx, float by, float h) {
  const float A = r.r0.z, B2 = r.r0.w, C = r.r2.x;
  // the rectangle relative to the centre, and its nearest column and row
  const float x0 = bx - r.r0.x, x1 = (bx + 7.f) - r.r0.x;
  const float y0 = by - r.r0.y, y1 = (by + h) - r.r0.y;
  const float cx = __builtin_amdgcn_fmed3f(0.f, x0, x1), cy = __builtin_amdgcn_fmed3f(0.f, y0, y1);
  const float dy = __builtin_amdgcn_fmed3f(b.ky * cx, y0, y1);
  const float qv = fmaf(fmaf(C, dy, B2 * cx), dy, (A * cx) * cx);
  const float dx = __builtin_amdgcn_fmed3f(b.kx * cy, x0, x1);
  const float qh = fmaf(fmaf(A, dx, B2 * cy), dx, (C * cy) * cy);
  return static_cast<bool>(static_cast<int>(fabsf(cx) <= b.ex) & static_cast<int>(fabsf(cy) <= b.ey) &
                           static_cast<int>(!(fminf(qv, qh) > b.tau)));
}

// The sub-blocks s0 .. s0 + N - 1 of the tile that the splat reaches, one bit
// each (bit s0 + i).
template <int T, int N, bool CUT>
__device__ __forceinline__ uint32_t sub_hits(const StagedRec& r, float tau, bool valid, int s0) {
  using G = TileGeom<T>;
  SupportBox box = support_box<CUT>(r, tau);
  if (!valid) box.ex = -1.f;
  uint32_t h = 0;
#pragma unroll
  for (int s = 0; s < N; ++s)
    h |= rect_hits(r, box, G::sub_x(s0 + s), G::sub_y(s0 + s), G::kRows - 1) ? 1u << s : 0u;
  return h << s0;
}

struct RasterArgs {
  const DevCamera* cams;
  const DevSplat* rec;
  const uint32_t* tile_start;  // start of every tile's id list
  const uint2* ent;       // list entries (Gaussian id, Gaussian-major slot)
  int64_t n;
  int64_t capacity;
  int32_t nv;
  float tau;              // support cutoff, times log2(e) / 2 like the staged conic
  int32_t unnormalised;   // write the raw sums (no background, no division)
  const float* globals;
  // forward outputs
  float* out_rgb;
  float* out_den;
  int32_t* out_count;
  // backward inputs / outputs
  const float* dL_drgb;
  const float* rgb;
  const float* den;
  float3* part;           // per-pair partial 2D gradients, 3 float3 per slot
  float* tilepart;
  // work items (see tile_scan_single); the split-tile partial sums of the
  // forward: item 0 of a split tile in the per-pixel accumulator, item k > 0
  // of the tile with first item i0 at slot i0 - tile + k - 1 of split4 (and
  // splitlog for Eq. 2's coverage), [split_slots][T * T]
  const uint32_t* items;
  const uint4* tile_order;     // the tiles' last items in dispatch order (see tile_scan_single)
  int64_t total_tiles;
  float* acc;
  float4* split4;
  float* splitlog;
  int64_t split_slots;
  // OIT (Eq. 2): per pixel (weighted average, coverage P) from the forward,
  // the split-tile accumulator of ln P and the per-pair partial dL/du
  float4* oit;
  float* acclog;
  float* du;
  // persistent launches: the counter the workgroups take work items from
  // (zeroed before the launch); null for one workgroup per work item
  uint32_t* queue;
  // culling masks: per list entry the sub-blocks of the tile its splat reaches
  // (one bit each, HitBits<T> per entry), or null for none;
  // flags->cull_masks says whether they hold the current lists' masks
  void* masks;
  DevFlags* flags;
};

// A persistent workgroup's next work item: the next unclaimed one, taken
// from the counter by thread 0 and shared through LDS.
__device__ __forceinline__ uint32_t claim_item(const RasterArgs& a, uint32_t* s_item) {
  __syncthreads();  // every thread has read the previous item
  if (threadIdx.x == 0) *s_item = atomicAdd(a.queue, 1u);
  __syncthreads();
  return *s_item;
}

__device__ __forceinline__ int find_view(const DevCamera* cams, int nv, int tile) {
  int v = 0;
  while (v + 1 < nv && cams[v + 1].tile_base <= tile) ++v;
  return v;
}

// Common set-up of one work item: its tile (view, tile coordinates), the
// sub-range [start, end) of the tile's id list it covers, and this lane's
// pixels.
template <int T>
struct TileCtx {
  int v, tx, ty;
  int64_t tile;
  int64_t n;
  uint32_t start, end;
  uint32_t list0;                 // first list position of the tile (capped at the capacity)
  uint32_t k, nk;                 // item index within the tile, items of the tile
  int wave, lane;
  int bx0, by0;                   // first pixel of this wave's block
  int px, py;                     // this lane's pixel
  int fx0, fy0;                   // frame origin of the staged centres: the tile's centre
};

// The sub-blocks of a tile, one bit each.
template <int T>
using HitBits = typename std::conditional<(TileGeom<T>::kSubs <= 8), uint8_t, uint16_t>::type;
static_assert(TileGeom<32>::kSubs <= 16, "sub-block bits");

template <int T>
__device__ __forceinline__ void tile_setup(const RasterArgs& a, uint32_t item, TileCtx<T>& c, const DevCamera*& cam) {
  using G = TileGeom<T>;
  // dispatch slot -> (tile, item within the tile), in the order the binning
  // laid out: first the full items, tile by tile, then the tiles' last items
  // in tile_order
  const uint32_t nfull = a.items[a.total_tiles] - static_cast<uint32_t>(a.total_tiles);
  uint32_t s0, e0;  // the tile's list, capped at the capacity
  if (item < nfull) {
    // largest tile t with items[t] - t <= item (nondecreasing in t)
    int64_t lo = 0, hi = a.total_tiles - 1;
    while (lo < hi) {
      const int64_t mid = (lo + hi + 1) >> 1;
      if (static_cast<int64_t>(a.items[mid]) - mid <= static_cast<int64_t>(item)) lo = mid; else hi = mid - 1;
    }
    c.tile = lo;
    c.k = item - (a.items[lo] - static_cast<uint32_t>(lo));
    c.nk = a.items[lo + 1] - a.items[lo];
    const uint64_t cap = static_cast<uint64_t>(a.capacity);
    s0 = static_cast<uint32_t>(min(static_cast<uint64_t>(a.tile_start[lo]), cap));
    e0 = static_cast<uint32_t>(min(static_cast<uint64_t>(a.tile_start[lo + 1]), cap));
    if (e0 < s0) e0 = s0;
  } else {
    const uint4 d = a.tile_order[item - nfull];
    c.tile = d.x;
    c.nk = d.w;
    c.k = d.w - 1;
    s0 = d.y;
    e0 = d.z;
  }
  const int tile = static_cast<int>(c.tile);
  c.v = find_view(a.cams, a.nv, tile);
  cam = &a.cams[c.v];
  const int local = tile - cam->tile_base;
  c.tx = local % cam->tiles_x;
  c.ty = local / cam->tiles_x;
  c.n = a.n;
  c.list0 = s0;
  const uint64_t ss = s0 + static_cast<uint64_t>(c.k) * kItemSplats;
  const uint64_t ee = ss + kItemSplats;
  c.start = static_cast<uint32_t>(ss < e0 ? ss : e0);
  c.end = static_cast<uint32_t>(ee < e0 ? ee : e0);
  c.wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  c.lane = threadIdx.x % kWave;
  c.bx0 = c.tx * T + (c.wave % (T / 8)) * G::kSub;
  c.by0 = c.ty * T + (c.wave / (T / 8)) * G::kSub;
  c.fx0 = c.tx * T + T / 2;
  c.fy0 = c.ty * T + T / 2;
  c.px = c.bx0 + (c.lane & 7);
  c.py = c.by0 + (c.lane >> 3);
}

// The staged form of a projected record, relative to the tile centre
// (tox, toy).
template <bool CUT, bool OIT, bool PREMUL>
__device__ __forceinline__ StagedRec make_staged(const DevSplat* d, float tox, float toy) {
  const SplatRec s = d->s;  // (fx, fy, A, B2) (C, ox, oy, amp) (c0, c1, c2, ext | cut)
  const float amp = s.r1.w;
  float c0 = s.r2.x, c1 = s.r2.y, c2 = s.r2.z;
  if (PREMUL) {
    c0 *= amp;
    c1 *= amp;
    c2 *= amp;
  }
  StagedRec r;
  r.r0 = make_float4((s.r1.y - tox) + s.r0.x, (s.r1.z - toy) + s.r0.y, s.r0.z * kHalfLog2e, s.r0.w * kHalfLog2e);
  r.r1 = make_float4(c0, c1, c2, amp);
  // OIT: the opacity u rides in the record's third word
  r.r2 = make_float4(s.r1.x * kHalfLog2e, CUT ? s.r2.w * kHalfLog2e : s.r2.w, OIT ? __uint_as_float(d->slot.w) : 0.f,
                     CUT ? support_k(s.r2.w * kHalfLog2e) : 0.f);
  return r;
}

// Barrier between LDS writes and reads of a workgroup.  __syncthreads would
// also wait for the outstanding global stores and loads.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// LDS writes of this wave before, LDS reads of this wave after.
__device__ __forceinline__ void lds_wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// For the sorted composite: stage one batch of records into LDS and list, in
// order, those whose support reaches this wave's block (as staged-record
// indices).  Returns the list length.
template <int T, int BATCH>
__device__ __forceinline__ int stage_and_cull(const RasterArgs& a, const TileCtx<T>& c, uint32_t b,
                                              StagedRec* s_rec, uint8_t* s_list) {
  using G = TileGeom<T>;
  const float tox = static_cast<float>(c.fx0), toy = static_cast<float>(c.fy0);
  __syncthreads();  // previous batch fully consumed
  for (int q = threadIdx.x; q < BATCH; q += G::kThreads) {
    const uint32_t j = b + q;
    if (j < c.end) s_rec[q] = make_staged<false, false, false>(a.rec + static_cast<int64_t>(c.v) * c.n + a.ent[j].x, tox, toy);
  }
  __syncthreads();
  const int cnt = static_cast<int>(min(static_cast<uint32_t>(BATCH), c.end - b));
  uint8_t* list = s_list + c.wave * BATCH;
  int m = 0;
  const float bx = static_cast<float>(c.bx0 - c.fx0) + 0.5f, by = static_cast<float>(c.by0 - c.fy0) + 0.5f;
  for (int k0 = 0; k0 < cnt; k0 += kWave) {
    const int k = k0 + c.lane;
    bool hit = false;
    if (k < cnt) {
      const StagedRec& r = s_rec[k];
      hit = rect_hits(r, support_box<false>(r, a.tau), bx, by, 7.f);
    }
    const uint64_t mask = __ballot(hit);
    if (hit) list[m + __popcll(mask & ((1ull << c.lane) - 1ull))] = static_cast<uint8_t>(k);
    m += __popcll(mask);
  }
  lds_wave_fence();
  return m;
}

// Eq. 7 for one pixel from its sums (or the raw sums in unnormalised mode).
__device__ __forceinline__ void write_pixel(const RasterArgs& a, int64_t pix, float nr, float ng, float nb,
                                            float dd) {
  if (a.unnormalised) {
    a.out_rgb[3 * pix] = nr;
    a.out_rgb[3 * pix + 1] = ng;
    a.out_rgb[3 * pix + 2] = nb;
    a.out_den[pix] = dd;
    return;
  }
  const float wbg = a.globals[2];
  const float bgr = a.globals[3], bgg = a.globals[4], bgb = a.globals[5];
  const float D = wbg + dd;
  const float Nr = fmaf(bgr, wbg, nr), Ng = fmaf(bgg, wbg, ng), Nb = fmaf(bgb, wbg, nb);
  float Cr = bgr, Cg = bgg, Cb = bgb;
  if (D != 0.f) {
    Cr = Nr / D;
    Cg = Ng / D;
    Cb = Nb / D;
  }
  a.out_rgb[3 * pix] = Cr;
  a.out_rgb[3 * pix + 1] = Cg;
  a.out_rgb[3 * pix + 2] = Cb;
  a.out_den[pix] = D;
}

// Eq. 2 for one pixel: C = P c_B + (1 - P) N / D (the average is 0 where
// D = 0); D goes to out_den and (N / D, P) to the workspace for the backward.
__device__ __forceinline__ void write_pixel_oit(const RasterArgs& a, int64_t pix, float nr, float ng, float nb,
                                                float dd, float P) {
  const float inv = dd != 0.f ? 1.f / dd : 0.f;
  const float ar = nr * inv, ag = ng * inv, ab = nb * inv;
  const float Q = 1.f - P;
  a.out_rgb[3 * pix] = fmaf(P, a.globals[3], Q * ar);
  a.out_rgb[3 * pix + 1] = fmaf(P, a.globals[4], Q * ag);
  a.out_rgb[3 * pix + 2] = fmaf(P, a.globals[5], Q * ab);
  a.out_den[pix] = dd;
  a.oit[pix] = make_float4(ar, ag, ab, P);
}

// The lanes of a forward wave: lane = (slot, row).  Row r of the 8x8 block is
// evaluated by the eight lanes that hold it, each against another splat of the
// row's sub-block list (slot s takes positions s, s + 8, ... of the lists of
// the item's batches taken together), eight pixels per lane.  Against one
// pixel per lane and one splat per step this shares a row's dy, B2 dy and
// C dy^2 among eight pixels (9.5 instead of 14.25 VALU operations per pixel
// and splat besides the exp2), one LDS read fetches eight records instead of
// one (5 instead of 40 B of LDS per lane and splat), and the two halves of the
// block walk lists of their own.
constexpr int kFwdSlots = 8;

// Sum over the slots (lane bits 3 to 5) of each row's eight columns, or their
// product: three exchange steps, each halving the columns a lane still holds,
// so that lane (slot, row) ends with column `slot` in v[0].
template <bool PRODUCT, typename V>
__device__ __forceinline__ V slots_combine(V (&v)[8], int lane) {
#pragma unroll
  for (int h = 4; h >= 1; h >>= 1) {
    const bool hi = (lane & (8 * h)) != 0;
#pragma unroll
    for (int i = 0; i < h; ++i) {
      const V lo_v = v[i], hi_v = v[i + h];
      const V keep = hi ? hi_v : lo_v, send = hi ? lo_v : hi_v;
      const V got = __shfl_xor(send, 8 * h, kWave);
      v[i] = PRODUCT ? keep * got : keep + got;
    }
  }
  return v[0];
}

// LDS of the forward.  Lists hold byte offsets into `rec`, which serve as LDS
// addresses directly; they are cleared once, so that an entry past the end of
// a list, read ahead but not used, is a valid offset too.  Behind the batch's
// records, `rec` holds up to eight records per sub-block carried over from the
// batch before: those of its last, incomplete group of eight.
template <int T, int S>
struct FwdShared {
  using G = TileGeom<T>;
  static constexpr int kGroups = S / kWave;              // groups of 64 records per batch
  static constexpr int kParts = G::kWaves / kGroups;     // waves that share a group's culling
  static constexpr int kList = S + 3 * kFwdSlots;        // entries of a list: carried, new, read ahead
  StagedRec rec[S + G::kSubs * kFwdSlots];
  uint16_t list[G::kSubs * kList];
  HitBits<T> hits[kParts][S];
};

// The forward of one work item (tile_setup's c), S records staged per batch.
// Thread k stages record k, requested while the previous batch is evaluated;
// each wave tests one group of 64 records against a share of the tile's
// sub-blocks, and the waves then list the records that reach their own.  A
// sub-block's groups of eight splats run on across the batches, so the order
// of every pixel's sums follows from the list alone, whatever the batch size.
template <int T, int S, bool COUNT, bool CUT, bool OIT>
__device__ __forceinline__ void raster_fwd_item(const RasterArgs& a, const TileCtx<T>& c, const DevCamera* cam,
                                                FwdShared<T, S>& sh) {
  using G = TileGeom<T>;
  using F = FwdShared<T, S>;
  constexpr int NT = G::kSubs / F::kParts;  // sub-blocks each wave tests
  constexpr bool kOwn = F::kParts == 1;     // a wave tests the records its threads stage
  static_assert(S <= G::kThreads && G::kWaves % F::kGroups == 0 && G::kSubs % F::kParts == 0, "culling shares");
  float nr[8], ng[8], nb[8], dd[8];
  float cov[8];  // OIT: prod (1 - alpha)
  int cntp[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    nr[k] = ng[k] = nb[k] = dd[k] = 0.f;
    cov[k] = 1.f;
    cntp[k] = 0;
  }
  const int slot = c.lane >> 3, row = c.lane & 7;
  const int half = row / G::kRows;
  // pixel centres relative to the tile's centre (exact): the row's y and the
  // block's columns
  const float pcy = static_cast<float>(c.by0 + row - c.fy0) + 0.5f;
  float xs[8];  // wave-uniform: kept in scalar registers
#pragma unroll
  for (int k = 0; k < 8; ++k)
    xs[k] = __uint_as_float(
        __builtin_amdgcn_readfirstlane(__float_as_uint(static_cast<float>(c.bx0 + k - c.fx0) + 0.5f)));
  const float none = support_k(-1.f), Kall = support_k(a.tau);

  const float tox = static_cast<float>(c.fx0), toy = static_cast<float>(c.fy0);
  const DevSplat* recs = a.rec + static_cast<int64_t>(c.v) * c.n;
  StagedRec mine = {};  // the record this thread stages next
  auto fetch = [&](uint32_t b) {
    const uint32_t j = b + threadIdx.x;
    if (threadIdx.x < S && j < c.end) mine = make_staged<CUT, OIT, true>(recs + a.ent[j].x, tox, toy);
  };
  fetch(c.start);

  // this lane's record of the present group: the geometry is replaced by the
  // next group's as soon as q is formed, the rest after the sums
  float4 r0, r1;
  float C, u = 0.f, Kown = 0.f;
  auto at_offset = [&](uint32_t off) -> const StagedRec& {
    return *reinterpret_cast<const StagedRec*>(reinterpret_cast<const char*>(sh.rec) + off);
  };
  auto load_geom = [&](uint32_t off) {
    r0 = at_offset(off).r0;
    C = at_offset(off).r2.x;
  };
  auto load_rest = [&](uint32_t off) {
    r1 = at_offset(off).r1;
    if (OIT) u = at_offset(off).r2.z;
    if (CUT) Kown = at_offset(off).r2.w;
  };
  // q of the row's pixels, then next_geom, then the sums; the staged colour
  // carries the amplitude
  auto evaluate = [&](bool use, auto&& next_geom) {
    const float K = use ? (CUT ? Kown : Kall) : none;
    const float dy = pcy - r0.y;
    const float B2dy = r0.w * dy, Cdy2 = (C * dy) * dy;
    float q[8], g[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) q[k] = quad_form(r0.z, B2dy, Cdy2, xs[k] - r0.x);
    next_geom();
    falloff_row(q, K, g);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      nr[k] = fmaf(g[k], r1.x, nr[k]);
      ng[k] = fmaf(g[k], r1.y, ng[k]);
      nb[k] = fmaf(g[k], r1.z, nb[k]);
      dd[k] = fmaf(g[k], r1.w, dd[k]);
      if (OIT) cov[k] *= 1.f - __builtin_amdgcn_fmed3f(u * g[k], 0.f, 1.f);
      if (COUNT) cntp[k] += static_cast<int>(in_support(q[k], K));
    }
  };
  // this wave's lists (of its sub-blocks), and this lane's
  uint16_t* const lists = sh.list + c.wave * G::kHalves * F::kList;
  const uint16_t* const list = lists + half * F::kList;
  // this lane's slot among its sub-block's carried records
  const int mysub = c.wave * G::kHalves + half;
  const uint32_t carry = static_cast<uint32_t>((S + mysub * kFwdSlots + slot) * sizeof(StagedRec));
  int held[G::kHalves] = {};  // carried records of each sub-block
  for (uint32_t b = c.start; b < c.end; b += S) {
    const int cnt = static_cast<int>(min(static_cast<uint32_t>(S), c.end - b));
    const int groups = (cnt + kWave - 1) / kWave;
    lds_barrier();  // previous batch fully consumed
    if (threadIdx.x < S) sh.rec[threadIdx.x] = mine;
    if (!kOwn) lds_barrier();
    {
      const int g = kOwn ? c.wave : c.wave % F::kGroups, part = kOwn ? 0 : c.wave / F::kGroups;
      const int k = g * kWave + c.lane;
      if (g < groups)
        sh.hits[part][k] =
            static_cast<HitBits<T>>(sub_hits<T, NT, CUT>(kOwn ? mine : sh.rec[k], a.tau, k < cnt, part * NT));
    }
    lds_barrier();
    if (a.masks && threadIdx.x < cnt) {
      uint32_t h = 0;
#pragma unroll
      for (int part = 0; part < F::kParts; ++part) h |= sh.hits[part][threadIdx.x];
      static_cast<HitBits<T>*>(a.masks)[b + threadIdx.x] = static_cast<HitBits<T>>(h);
    }
    fetch(b + S);
    int n[G::kHalves];  // records of each sub-block: carried and new
#pragma unroll
    for (int h = 0; h < G::kHalves; ++h) {
      n[h] = held[h];
      if (half == h && slot < held[h]) lists[h * F::kList + slot] = static_cast<uint16_t>(carry);
    }
#pragma unroll
    for (int g = 0; g < F::kGroups; ++g) {
      if (g >= groups) break;
      const uint32_t bits = sh.hits[c.wave * G::kHalves / NT][g * kWave + c.lane];
#pragma unroll
      for (int h = 0; h < G::kHalves; ++h) {
        const bool hit = (bits >> (c.wave * G::kHalves + h)) & 1u;
        const uint64_t w = __ballot(hit);
        if (hit)
          lists[h * F::kList + n[h] + __popcll(w & ((1ull << c.lane) - 1ull))] =
              static_cast<uint16_t>((g * kWave + c.lane) * sizeof(StagedRec));
        n[h] += __popcll(w);
      }
    }
    lds_wave_fence();
    int rounds = 0, mine_rounds = 0;  // groups of eight: the longer half's, this lane's
#pragma unroll
    for (int h = 0; h < G::kHalves; ++h) {
      rounds = max(rounds, n[h] / kFwdSlots);
      if (half == h) mine_rounds = n[h] / kFwdSlots;
    }
    const uint16_t* next = list + slot;
    uint32_t off = next[0];
    load_geom(off);
    load_rest(off);
    off = next[kFwdSlots];
    next += 2 * kFwdSlots;
    for (int i = 0; i < rounds; ++i) {
      evaluate(i < mine_rounds, [&] { load_geom(off); });
      load_rest(off);
      off = *next;
      next += kFwdSlots;
    }
    // the incomplete groups' records are carried over: row j of a sub-block's
    // first three copies the j-th third of its slot's record
#pragma unroll
    for (int h = 0; h < G::kHalves; ++h) {
      held[h] = n[h] % kFwdSlots;
      const int j = row % G::kRows;
      if (half == h && slot < held[h] && j < 3) {
        const uint32_t src = list[n[h] - held[h] + slot];
        const float4 x = reinterpret_cast<const float4*>(&at_offset(src))[j];
        reinterpret_cast<float4*>(const_cast<StagedRec*>(&at_offset(carry)))[j] = x;
      }
    }
    lds_wave_fence();
  }
  {
    bool use = false, any = false;
#pragma unroll
    for (int h = 0; h < G::kHalves; ++h) {
      any |= held[h] > 0;
      if (half == h) use = slot < held[h];
    }
    if (any) {
      load_geom(carry);
      load_rest(carry);
      evaluate(use, [] {});
    }
  }

  const float Nr = slots_combine<false>(nr, c.lane), Ng = slots_combine<false>(ng, c.lane);
  const float Nb = slots_combine<false>(nb, c.lane), Dd = slots_combine<false>(dd, c.lane);
  const float Cv = OIT ? slots_combine<true>(cov, c.lane) : 1.f;
  const int count = COUNT ? slots_combine<false>(cntp, c.lane) : 0;
  const int px = c.bx0 + slot, py = c.by0 + row;  // the pixel this lane ends with
  if (px >= cam->width || py >= cam->height) return;
  const int64_t pix = cam->pix_base + static_cast<int64_t>(py) * cam->width + px;
  if (COUNT) atomicAdd(a.out_count + pix, count);
  if (c.nk > 1) {
    // split tile: this item's partial sums, added in item order by
    // raster_fwd_finalize (the coverage products of the parts multiply, so
    // their logarithms add).  Item 0 stores into the per-pixel accumulator,
    // item k > 0 into its own slot of the split-tile partials.
    const float4 sums = make_float4(Nr, Ng, Nb, Dd);
    if (c.k == 0) {
      reinterpret_cast<float4*>(a.acc)[pix] = sums;
      if (OIT) a.acclog[pix] = __logf(Cv);
    } else {
      const int64_t e = static_cast<int64_t>(a.items[c.tile]) - c.tile + c.k - 1;
      if (e < a.split_slots) {
        const int64_t q = e * (T * T) + (py - c.ty * T) * T + (px - c.tx * T);
        a.split4[q] = sums;
        if (OIT) a.splitlog[q] = __logf(Cv);
      }
    }
    return;
  }
  if (OIT)
    write_pixel_oit(a, pix, Nr, Ng, Nb, Dd, Cv);
  else
    write_pixel(a, pix, Nr, Ng, Nb, Dd);
}

// Forward.  Lists hold LDS byte offsets of the staged records.  S records
// are staged per batch.  A workgroup renders the work item of dispatch slot
// blockIdx.x (the grid covers them all), or, PERSIST, claims slots from a
// counter until none is left.  Tile 16 asks for four waves per SIMD (at most
// 128 VGPRs): five spill, 412 instead of 386 us at 1 M Gaussians / 1080p.
template <int T, int S, bool COUNT, bool CUT, bool OIT, bool PERSIST>
__global__ __launch_bounds__(TileGeom<T>::kThreads, T == 16 ? 4 : 1) void raster_fwd_kernel(RasterArgs a) {
  __shared__ FwdShared<T, S> sh;
  __shared__ uint32_t s_item;
  for (int k = threadIdx.x; k < TileGeom<T>::kSubs * FwdShared<T, S>::kList; k += TileGeom<T>::kThreads) sh.list[k] = 0;
  for (int k = threadIdx.x; k < TileGeom<T>::kSubs * kFwdSlots; k += TileGeom<T>::kThreads) sh.rec[S + k] = StagedRec{};
  // every work item stores its waves' culling masks (when there is room):
  // valid for the backward once this launch has finished
  if (blockIdx.x == 0 && threadIdx.x == 0) a.flags->cull_masks = a.masks ? (kCullMasks | (CUT ? 2u : 0u)) : 0u;
  const uint32_t n_items = a.items[a.total_tiles];
  uint32_t item = PERSIST ? claim_item(a, &s_item) : blockIdx.x;
  while (item < n_items) {
    TileCtx<T> c;
    const DevCamera* cam;
    tile_setup<T>(a, item, c, cam);
    raster_fwd_item<T, S, COUNT, CUT, OIT>(a, c, cam, sh);
    if (!PERSIST) break;
    item = claim_item(a, &s_item);
  }
}

// Normalisation of the tiles whose list was split over several work items:
// the items' partial sums are added in item order (item 0's from the
// per-pixel accumulator, the others' from their slots), so the image does
// not depend on the order in which the items ran.
template <int T, bool OIT>
__global__ __launch_bounds__(256) void raster_fwd_finalize(RasterArgs a) {
  const int64_t t = blockIdx.x;
  const uint32_t i0 = a.items[t], nk = a.items[t + 1] - i0;
  if (nk <= 1) return;
  const int tile = static_cast<int>(t);
  const int v = find_view(a.cams, a.nv, tile);
  const DevCamera& cam = a.cams[v];
  const int local = tile - cam.tile_base;
  const int tx = local % cam.tiles_x, ty = local / cam.tiles_x;
  const int64_t e0 = static_cast<int64_t>(i0) - t;  // slot of the tile's item 1
  for (int q = threadIdx.x; q < T * T; q += 256) {
    const int px = tx * T + q % T, py = ty * T + q / T;
    if (px >= cam.width || py >= cam.height) continue;
    const int64_t pix = cam.pix_base + static_cast<int64_t>(py) * cam.width + px;
    float4 s = reinterpret_cast<const float4*>(a.acc)[pix];
    float lg = OIT ? a.acclog[pix] : 0.f;
    for (uint32_t k = 1; k < nk; ++k) {
      const int64_t e = e0 + k - 1;
      if (e >= a.split_slots) break;
      const float4 x = a.split4[e * (T * T) + q];
      s.x += x.x;
      s.y += x.y;
      s.z += x.z;
      s.w += x.w;
      if (OIT) lg += a.splitlog[e * (T * T) + q];
    }
    if (OIT)
      write_pixel_oit(a, pix, s.x, s.y, s.z, s.w, __expf(lg));
    else
      write_pixel(a, pix, s.x, s.y, s.z, s.w);
  }
}

// Per-pixel factors of a sub-block in LDS: its pixels', and one of padding, so
// that the same pixel of different sub-blocks lies in different banks.
template <int T>
constexpr int kPdStride = TileGeom<T>::kRows * 8 + 1;

__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, kWave);
  return x;
}

// Moments of a block.  A lane sums, per pixel of its splat's walk,
// e = G dL/da against the pixel centre's offset xc from the 8x8 block's centre
// (a compile-time constant per column: no per-pixel dx or dx^2 for the
// moments) and folds each row with dy = pixel y - splat y:
//   X1 = sum e xc, X2 = sum e xc^2, XY = sum e xc dy, My = sum e dy,
//   Myy = sum e dy^2, S = sum e.
// With dx = xc - m (m the splat centre's offset from the block centre) the
// moments about the splat centre follow once per block:
//   Mx = X1 - m S,  Mxx = X2 - 2 m X1 + m^2 S,  Mxy = XY - m My,
// whose rounding is bounded like that of summing e dx directly (|xc| + |m|
// bounds |dx| over the block).
struct BlockMoments {
  float X1 = 0.f, X2 = 0.f, XY = 0.f, My = 0.f, Myy = 0.f, S = 0.f;
};

__device__ __forceinline__ void fold_row(BlockMoments& M, float dy, float S0, float S1, float S2) {
  M.S += S0;
  M.X1 += S1;
  M.X2 += S2;
  M.My = fmaf(dy, S0, M.My);
  M.XY = fmaf(dy, S1, M.XY);
  M.Myy = fmaf(dy * dy, S0, M.Myy);
}

// One splat's gradient sums over its pixels of the tile: with G = exp(-q/2)
// and e = G dL/da, the moments of e about the splat's centre and sum G gbar.
//
// OIT (Eq. 2): plus the coverage term.  A layer's opacity alpha = u G
// (clamped to [0, 1], no gradient where clamped) gets
// dL/dalpha = -k / (1 - alpha) with k from pixel_factors, so per pixel
// dq = -G (amp dL/da + u dL/dalpha) / 2, the moments carry the amplitude, and
// there are two more sums, sum G dL/da and dL/du = sum G dL/dalpha.
template <bool OIT>
struct WalkSums {
  float Mx = 0.f, My = 0.f, Mxx = 0.f, Mxy = 0.f, Myy = 0.f, S = 0.f;
  float g_r = 0.f, g_g = 0.f, g_b = 0.f, g_amp = 0.f, g_u = 0.f;

  __device__ __forceinline__ void add_block(const BlockMoments& B, float m) {
    Mx += fmaf(-m, B.S, B.X1);
    Mxx += fmaf(m, fmaf(m, B.S, -2.f * B.X1), B.X2);
    Mxy += fmaf(-m, B.My, B.XY);
    My += B.My;
    Myy += B.Myy;
    S += B.S;
  }

  // the sums of the lanes d apart, added
  __device__ __forceinline__ void add_lanes(int d) {
    float* const v[] = {&Mx, &My, &Mxx, &Mxy, &Myy, &S, &g_r, &g_g, &g_b, &g_amp, &g_u};
#pragma unroll
    for (int k = 0; k < (OIT ? 11 : 9); ++k) *v[k] += __shfl_xor(*v[k], d, kWave);
  }
};

// One row of eight pixels of the walk.  dx: the row's pixel centres minus the
// splat's, dy likewise; pd, pk: the row's per-pixel factors in LDS.  Columns
// j and 7 - j lie at -xc and +xc from the block centre, so their e enter the
// moments as a sum and a difference: 6 instead of 8 operations per pair.
template <bool OIT>
__device__ __forceinline__ void walk_row(WalkSums<OIT>& W, BlockMoments& B, const StagedRec& r, const float (&dx)[8], float dy,
                                         float K, const float4* pd_row, const float* pk_row) {
  const float A = r.r0.z, B2 = r.r0.w, Cc = r.r2.x;
  const float cr = r.r1.x, cg = r.r1.y, cb = r.r1.z, amp = r.r1.w;
  const float B2dy = B2 * dy, Cdy2 = (Cc * dy) * dy;
  float4 pds[8];  // requested before the arithmetic below, which covers their latency
#pragma unroll
  for (int k = 0; k < 8; ++k) pds[k] = pd_row[k];
  float q[8], G[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) q[k] = quad_form(A, B2dy, Cdy2, dx[k]);
  falloff_row(q, K, G);
  float rc[8];  // OIT: 1 / (1 - alpha)
  if constexpr (OIT) {
    const float u = r.r2.z;
    float om[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) om[k] = fmaf(-u, G[k], 1.f);
    // hardware reciprocal (within 1 ulp) instead of an IEEE division
    trans_burst([&] {
#pragma unroll
      for (int k = 0; k < 8; ++k) rc[k] = __builtin_amdgcn_rcpf(om[k]);
    });
  }
  float S0 = 0.f, S1 = 0.f, S2 = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float xc = 3.5f - static_cast<float>(j);
    float f[2];  // the factor of G in e, at columns j and 7 - j
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = h ? 7 - j : j;
      const float4 pd = pds[k];
      const float dLda = fmaf(pd.x, cr, fmaf(pd.y, cg, fmaf(pd.z, cb, -pd.w)));
      W.g_r = fmaf(G[k], pd.x, W.g_r);
      W.g_g = fmaf(G[k], pd.y, W.g_g);
      W.g_b = fmaf(G[k], pd.z, W.g_b);
      if constexpr (OIT) {
        const float u = r.r2.z;
        const float al = u * G[k];
        const float dLdal = (al > 0.f && al < 1.f) ? -pk_row[k] * rc[k] : 0.f;
        W.g_amp = fmaf(G[k], dLda, W.g_amp);
        W.g_u = fmaf(G[k], dLdal, W.g_u);
        f[h] = fmaf(amp, dLda, u * dLdal);
      } else {
        f[h] = dLda;
      }
    }
    const float eb = G[7 - j] * f[1];
    const float sum = fmaf(G[j], f[0], eb), dif = fmaf(-G[j], f[0], eb);
    S0 += sum;
    S1 = fmaf(dif, xc, S1);
    S2 = fmaf(sum, xc * xc, S2);
  }
  fold_row(B, dy, S0, S1, S2);
}

// The walk's sums as the pair's partial 2D gradient at its Gaussian-major
// slot, with plain stores: the dq factors of the mean and conic gradients
// (dq = -a e / 2 per pixel, with a = amp G; the staged conic is scaled by
// log2(e) / 2, undone here), dL/dc = amp sum G gbar and dL/damp = sum G dL/da.
// The amplitude multiplies the moments once (OIT: they carry it).
template <bool OIT>
__device__ __forceinline__ void walk_store(const RasterArgs& a, uint32_t slot, const WalkSums<OIT>& W,
                                           const StagedRec& r) {
  if (slot >= a.capacity) return;
  const float amp = r.r1.w, A = r.r0.z, B2 = r.r0.w, Cc = r.r2.x;
  const float ampm = OIT ? 1.f : amp, ampc = ampm * kTwoLn2;
  float3* dst = a.part + 3 * static_cast<int64_t>(slot);
  dst[0] = make_float3(ampc * (A * W.Mx + 0.5f * B2 * W.My), ampc * (0.5f * B2 * W.Mx + Cc * W.My),
                       -0.5f * ampm * W.Mxx);
  dst[1] = make_float3(-ampm * W.Mxy, -0.5f * ampm * W.Myy, amp * W.g_r);
  dst[2] = make_float3(amp * W.g_g, amp * W.g_b, OIT ? W.g_amp : W.S);
  if (OIT) a.du[slot] = W.g_u;
}

// The backward's per-pixel factors for pixel (px, py) of view `cam`:
// gbar = dL/dC / D and s = gbar . C (zero outside the image), and the pixel's
// share of the background gradients dL/dc_B (rgb) and dL/dw_B.
//
// OIT (Eq. 2, C = P c_B + (1 - P) N / D): gbar = dL/dC (1 - P) / D and
// s = gbar . (N / D), so that dL/da = gbar . c - s as for Eq. 7, and the
// coverage factor k = P dL/dC . (c_B - N / D), so that a layer's opacity
// alpha gets dL/dalpha = -k / (1 - alpha); dL/dc_B = P dL/dC, dL/dw_B = 0.
template <bool OIT>
__device__ __forceinline__ void pixel_factors(const RasterArgs& a, const DevCamera& cam, int px, int py,
                                              float4* pd_o, float* kcov_o, float* bacc) {
  const float wbg = a.globals[2];
  const float bgr = a.globals[3], bgg = a.globals[4], bgb = a.globals[5];
  float4 pd = make_float4(0.f, 0.f, 0.f, 0.f);
  float kcov = 0.f;
  bacc[0] = bacc[1] = bacc[2] = bacc[3] = 0.f;
  if (px < cam.width && py < cam.height) {
    const int64_t pix = cam.pix_base + static_cast<int64_t>(py) * cam.width + px;
    const float D = a.den[pix];
    const float g0 = a.dL_drgb[3 * pix], g1 = a.dL_drgb[3 * pix + 1], g2 = a.dL_drgb[3 * pix + 2];
    if (OIT) {
      const float4 o = a.oit[pix];  // (N / D, P)
      const float P = o.w;
      const float f = D != 0.f ? (1.f - P) / D : 0.f;
      pd.x = g0 * f;
      pd.y = g1 * f;
      pd.z = g2 * f;
      pd.w = pd.x * o.x + pd.y * o.y + pd.z * o.z;
      kcov = P * (g0 * (bgr - o.x) + g1 * (bgg - o.y) + g2 * (bgb - o.z));
      bacc[0] = g0 * P;
      bacc[1] = g1 * P;
      bacc[2] = g2 * P;
    } else if (D != 0.f) {
      const float iD = 1.f / D;
      pd.x = g0 * iD;
      pd.y = g1 * iD;
      pd.z = g2 * iD;
      pd.w = pd.x * a.rgb[3 * pix] + pd.y * a.rgb[3 * pix + 1] + pd.z * a.rgb[3 * pix + 2];
      bacc[0] = wbg * pd.x;
      bacc[1] = wbg * pd.y;
      bacc[2] = wbg * pd.z;
      bacc[3] = pd.x * bgr + pd.y * bgg + pd.z * bgb - pd.w;
    } else {
      // C is the background colour where the denominator vanishes
      bacc[0] = g0;
      bacc[1] = g1;
      bacc[2] = g2;
    }
  }
  *pd_o = pd;
  *kcov_o = kcov;
}

// A backward workgroup has four waves whatever the tile size, and the compiler
// is asked for four resident waves per SIMD, as many as the SIMD needs to issue
// two FP32 operations at once throughout (at most 128 VGPRs).
constexpr int kBwdWaves = 4;
constexpr int kBwdThreads = kBwdWaves * kWave;
// Backward of one work item.  Every lane takes one splat of the item and walks
// the sub-blocks of the tile that its support reaches, so a splat's
// gradient sums stay in its lane's registers from the first pixel to the
// store: no merging between waves, and no barrier, once the walk has begun.
// The lanes of a wave walk the sub-blocks of their own splats (a lane's j-th
// is its splat's j-th); for them to finish together the item's splats are
// first sorted by the number of sub-blocks they reach (a counting sort in LDS),
// the most first.  Splats that reach none get zeros.  The records of a
// wave's next splats are requested before it walks the present ones.
//
// The previous form (waves owning blocks, lanes owning splats of the wave's
// culled list, the waves' sums merged through LDS in lockstep rounds) spent
// 47 % of its wave time waiting at the rounds' barriers, at the staging's and
// on LDS.
//
// The last splats, fewer than the workgroup has lanes, are shared by W = 1, 2,
// 4 or 8 lanes each, which split the rows of every sub-block (and, where it
// has fewer rows than W, the sub-blocks); the lanes' sums are added with
// shuffles.  A splat's sums
// depend on its place in the sort through W alone, and the sort is stable, so
// they do not vary from run to run.
template <int T>
struct BwdShared {
  // the item's splats, most sub-blocks first: Gaussian id; index in the item,
  // and in the upper half the sub-blocks it reaches (one bit each)
  uint2 order[kItemSplats];
  uint32_t count[TileGeom<T>::kSubs + 1][kBwdWaves];  // per number of sub-blocks and wave
};

// Wave w sorts the w-th share of the item, whole groups of 64 splats.  All
// global loads of the sort are issued by bwd_sort_begin, so that they and the
// pixel factors' cost one memory round trip.
template <int T>
struct BwdShare {
  static constexpr int kGroups = kItemSplats / kBwdThreads;
  int w0, w1;              // the share, relative to the item
  uint32_t id[kGroups];    // of each group's entry: the Gaussian
  uint32_t hits[kGroups];  // and the sub-blocks it reaches
};

template <int T, bool CUT, bool OIT>
__device__ __forceinline__ void bwd_sort_begin(const RasterArgs& a, const TileCtx<T>& c, BwdShare<T>& q,
                                               const HitBits<T>* masks_in) {
  using G = TileGeom<T>;
  const int len = static_cast<int>(c.end - c.start);
  const int per = ((len + kBwdWaves - 1) / kBwdWaves + kWave - 1) & ~(kWave - 1);
  q.w0 = min(c.wave * per, len);
  q.w1 = min(q.w0 + per, len);
#pragma unroll
  for (int g = 0; g < BwdShare<T>::kGroups; ++g) {
    const int e = q.w0 + g * kWave + c.lane;
    q.id[g] = e < q.w1 ? a.ent[c.start + e].x : 0u;
    q.hits[g] = masks_in && e < q.w1 ? masks_in[c.start + e] : 0u;
  }
  if (!masks_in) {
#pragma unroll
    for (int g = 0; g < BwdShare<T>::kGroups; ++g) {
      const int e = q.w0 + g * kWave + c.lane;
      if (e < q.w1)
        q.hits[g] = sub_hits<T, G::kSubs, CUT>(
            make_staged<CUT, OIT, false>(a.rec + static_cast<int64_t>(c.v) * c.n + q.id[g],
                                         static_cast<float>(c.fx0), static_cast<float>(c.fy0)),
            a.tau, true, 0);
    }
  }
}

template <int T>
__device__ __forceinline__ int bwd_sort(const TileCtx<T>& c, BwdShare<T>& q, BwdShared<T>& sh) {
  using G = TileGeom<T>;
  constexpr int NB = G::kSubs;
  constexpr int NG = BwdShare<T>::kGroups;
  uint32_t at[NB + 1];  // per number of sub-blocks: this wave's splats, then the place of its next one
#pragma unroll
  for (int k = 0; k <= NB; ++k) at[k] = 0;
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    if (q.w0 + g * kWave >= q.w1) break;
    const int n = q.w0 + g * kWave + c.lane < q.w1 ? __popc(q.hits[g]) : -1;
#pragma unroll
    for (int k = 0; k <= NB; ++k) at[k] += static_cast<uint32_t>(__popcll(__ballot(n == k)));
  }
  if (c.lane == 0) {
#pragma unroll
    for (int k = 0; k <= NB; ++k) sh.count[k][c.wave] = at[k];
  }
  lds_barrier();
  int total = 0, reaching = 0;
#pragma unroll
  for (int k = NB; k >= 0; --k) {
    if (k == 0) reaching = total;
#pragma unroll
    for (int w = 0; w < kBwdWaves; ++w) {
      if (w == c.wave) at[k] = static_cast<uint32_t>(total);
      total += static_cast<int>(sh.count[k][w]);
    }
  }
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    if (q.w0 + g * kWave >= q.w1) break;
    const int e = q.w0 + g * kWave + c.lane;
    const uint32_t h = q.hits[g];
    const int n = e < q.w1 ? __popc(h) : -1;
    uint32_t place = 0;
#pragma unroll
    for (int k = 0; k <= NB; ++k) {
      const uint64_t same = __ballot(n == k);
      if (n == k) place = at[k] + static_cast<uint32_t>(__popcll(same & ((1ull << c.lane) - 1ull)));
      at[k] += static_cast<uint32_t>(__popcll(same));
    }
    if (n >= 0) sh.order[place] = make_uint2(q.id[g], static_cast<uint32_t>(e) | (h << 16));
  }
  lds_barrier();
  return reaching;
}

// Walk the splats of a wave, W lanes each.  order: index in the item, and in
// the upper half the sub-blocks the splat reaches (0: no splat).
template <int T, bool CUT, bool OIT, int W>
__device__ __forceinline__ void bwd_walk(const RasterArgs& a, const TileCtx<T>& c, const float4* s_pd,
                                         const float* s_pk, const StagedRec& r, uint32_t order) {
  using G = TileGeom<T>;
  constexpr int S = kWave / W;                       // splats per wave
  constexpr int WR = W < G::kRows ? W : G::kRows;    // lanes that share a sub-block's rows
  constexpr int R = G::kRows / WR;                   // rows per lane
  const int g = c.lane / S;
  uint32_t h = order >> 16;
  const bool valid = h != 0;
  if (W > WR) h &= g / WR == 0 ? 0x5555u : 0xaaaau;  // two lanes share the sub-blocks
  const uint32_t slot = a.ent[c.start + (order & 0xffffu)].y;  // needed at the end only
  const float Kv = CUT ? r.r2.w : support_k(a.tau);
  WalkSums<OIT> sums;
  while (__any(h != 0)) {
    const float K = h != 0 ? Kv : support_k(-1.f);
    const int b = h != 0 ? __ffs(static_cast<int>(h)) - 1 : 0;
    h &= h - 1u;
    // the first pixel centre relative to the tile's centre (exact, so that dx
    // and dy match the forward's)
    const float ex0 = G::sub_x(b);
    float yrow = G::sub_y(b) + static_cast<float>(g % WR * R);
    float dx[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) dx[k] = (ex0 + static_cast<float>(k)) - r.r0.x;
    const int at = b * kPdStride<T> + g % WR * R * 8;
    const float4* pd = s_pd + at;
    const float* pk = OIT ? s_pk + at : nullptr;
    BlockMoments B;
#pragma unroll 1
    for (int row = 0; row < R; ++row, yrow += 1.f)
      walk_row<OIT>(sums, B, r, dx, yrow - r.r0.y, K, pd + row * 8, OIT ? pk + row * 8 : nullptr);
    sums.add_block(B, r.r0.x - (ex0 + 3.5f));
  }
#pragma unroll
  for (int d = S; d < kWave; d <<= 1) sums.add_lanes(d);
  if (g == 0 && valid) walk_store<OIT>(a, slot, sums, r);
}

template <int T, bool CUT, bool OIT, bool PERSIST>
__global__ __launch_bounds__(kBwdThreads, 4) void raster_bwd_kernel(
    RasterArgs a) {
  using G = TileGeom<T>;
  __shared__ BwdShared<T> sh;
  __shared__ float4 s_pd[G::kSubs * kPdStride<T>];            // per-pixel factors, sub-block by sub-block
  __shared__ float s_pk[OIT ? G::kSubs * kPdStride<T> : 1];   // OIT: per-pixel coverage factors
  __shared__ float s_bg[kBwdWaves][4];
  __shared__ uint32_t s_item;
  // the forward's culling masks, if it stored them for these lists with the
  // same early-out setting
  const HitBits<T>* masks_in = (a.masks && a.flags->cull_masks == (kCullMasks | (CUT ? 2u : 0u)))
                                   ? static_cast<const HitBits<T>*>(a.masks) : nullptr;
  const uint32_t n_items = a.items[a.total_tiles];
  uint32_t item = PERSIST ? claim_item(a, &s_item) : blockIdx.x;
  while (item < n_items) {
    TileCtx<T> c;
    const DevCamera* cam;
    tile_setup<T>(a, item, c, cam);
    BwdShare<T> share;
    bwd_sort_begin<T, CUT, OIT>(a, c, share, masks_in);
    // every thread's pixel factors into LDS; the tile's first work item also
    // stores the tile's background-gradient partial sums
    {
      float back[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int p = threadIdx.x; p < T * T; p += kBwdThreads) {
        const int sub = p / (G::kRows * 8), at = p % (G::kRows * 8);  // pixel `at` of a sub-block
        float4 pd;
        float kcov, bacc[4];
        pixel_factors<OIT>(a, *cam, c.tx * T + sub / G::kHalves % (T / 8) * 8 + (at & 7),
                           c.ty * T + sub / G::kHalves / (T / 8) * 8 + sub % G::kHalves * G::kRows + (at >> 3), &pd,
                           &kcov, bacc);
        s_pd[sub * kPdStride<T> + at] = pd;
        if (OIT) s_pk[sub * kPdStride<T> + at] = kcov;
#pragma unroll
        for (int j = 0; j < 4; ++j) back[j] += bacc[j];
      }
      if (c.k == 0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float sj = wave_sum(back[j]);
          if (c.lane == 0) s_bg[c.wave][j] = sj;
        }
      }
    }
    const int n = bwd_sort<T>(c, share, sh);
    if (c.k == 0 && threadIdx.x < 4) {
      float sj = 0.f;
#pragma unroll
      for (int w = 0; w < kBwdWaves; ++w) sj += s_bg[w][threadIdx.x];
      a.tilepart[c.tile * 4 + threadIdx.x] = sj;
    }
    // rounds of one lane per splat that keep every wave busy, then the rest
    // with W lanes per splat
    const int rounds = n / kBwdThreads, rest = n % kBwdThreads;
    const int wsh = rest * 8 <= kBwdThreads ? 3 : rest * 4 <= kBwdThreads ? 2 : rest * 2 <= kBwdThreads ? 1 : 0;
    const DevSplat* recs = a.rec + static_cast<int64_t>(c.v) * c.n;
    const float tox = static_cast<float>(c.fx0), toy = static_cast<float>(c.fy0);
    // this lane's splat of a round (its record, and item index and blocks; no
    // blocks past the end)
    auto fetch = [&](int round, uint32_t& order, StagedRec& r) {
      const int first = round < rounds ? round * kBwdThreads + c.wave * kWave
                                       : rounds * kBwdThreads + c.wave * (kWave >> wsh);
      const int j = first + (round < rounds ? c.lane : c.lane & ((kWave >> wsh) - 1));
      const uint2 o = sh.order[min(j, n - 1)];
      order = j < n ? o.y : o.y & 0xffffu;
      r = make_staged<CUT, OIT, false>(recs + o.x, tox, toy);
    };
    if (n > 0) {
      uint32_t o;
      StagedRec r;
      fetch(0, o, r);
      for (int round = 0; round < rounds; ++round) {
        uint32_t on;
        StagedRec rn;
        fetch(round + 1, on, rn);
        bwd_walk<T, CUT, OIT, 1>(a, c, s_pd, s_pk, r, o);
        o = on;
        r = rn;
      }
      if (wsh == 3)
        bwd_walk<T, CUT, OIT, 8>(a, c, s_pd, s_pk, r, o);
      else if (wsh == 2)
        bwd_walk<T, CUT, OIT, 4>(a, c, s_pd, s_pk, r, o);
      else if (wsh == 1)
        bwd_walk<T, CUT, OIT, 2>(a, c, s_pd, s_pk, r, o);
      else
        bwd_walk<T, CUT, OIT, 1>(a, c, s_pd, s_pk, r, o);
    }
    // the splats that reach no pixel of the tile: zeros
    for (int j = n + threadIdx.x; j < static_cast<int>(c.end - c.start); j += kBwdThreads) {
      const uint32_t slot = a.ent[c.start + (sh.order[j].y & 0xffffu)].y;
      if (slot < a.capacity) {
        float3* dst = a.part + 3 * static_cast<int64_t>(slot);
        dst[0] = dst[1] = dst[2] = make_float3(0.f, 0.f, 0.f);
        if (OIT) a.du[slot] = 0.f;
      }
    }
    if (!PERSIST) break;
    item = claim_item(a, &s_item);  // (its first barrier: the shared arrays are free again)
  }
}

// ---- Sorted alpha blending (Eq. 6): the baseline the method removes the
// sort from.  The splats are those of the weighted sum (projected with the
// DIR weight, so a record's amplitude is the opacity u), ordered per tile by
// camera depth and composited front to back.

// The per-tile sort.  A list is spread over equal steps of its depth range,
// about as many buckets as entries (counted and placed with LDS atomics), and
// every entry then finds its place by counting, in its bucket alone, the keys
// below its own.  A key is (depth bits, list position), so the order is strict
// and does not depend on how the atomics fell; binning leaves every list in
// increasing id order, so ties in depth stay in id order.  Entries are held in
// registers from before the first barrier until they are stored at their new
// positions.  Lists with many equal or crowded depths, where the comparisons
// (the sum of the squared bucket sizes) would pass kSortCrowd per entry, are
// sorted by a bitonic network over the keys instead.
//
// Most lists are short: sort_short_kernel gives each a small workgroup, several
// to a CU, and leaves the longer ones to two kernels with more shared memory.
// More buckets pay where the shared memory allows them: depths come in clumps,
// and the comparisons are most of the work (lists of 2,049 to 8,192 entries
// with 2,048, 4,096 and 8,192 buckets: 84, 67 and 63 us; up to 2,048 entries
// with 2,048 and 1,024, which lets two more workgroups share a CU: 65 and
// 62 us).  All lists of 1 M Gaussians at 1080p: 596 us with bitonic networks
// throughout (66 barriers for 2,048 entries), 133 us now, of which the dense
// depths take 11 and save 31.
constexpr int kSortSmall = kItemSplats;
constexpr int kSortMid = 8192;
constexpr uint32_t kSortCrowd = 64;

// The tiles whose lists are longer than kSortSmall, as sort_short_kernel comes
// across them: up to kSortMid entries from the front of `tiles`, longer ones
// from its back.  head = (number, number claimed) of the former, then of the
// latter.
struct SortQueue {
  uint32_t* head;
  uint32_t* tiles;  // [room]
  uint32_t room;    // all tiles
};

// Shared memory of one sort: CAP keys, NB buckets, TH threads.
template <int CAP, int NB, int TH>
struct SortShared {
  uint64_t keys[CAP];
  uint32_t hist[NB];  // bucket sizes, then (first place << 16 | size)
  uint32_t lo, hi, work, wave[TH / kWave];
};

template <int TH>
__device__ __forceinline__ void sort_sync() {
  if constexpr (TH == kWave) lds_wave_fence(); else lds_barrier();
}

// Sorts keys[0, npow) in place (npow a power of two), between barriers.
template <int TH>
__device__ __forceinline__ void bitonic_keys(uint64_t* keys, int npow, int tid) {
  for (int size = 2; size <= npow; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int i = tid; i < (npow >> 1); i += TH) {
        const int a = (i / stride) * 2 * stride + (i % stride);
        const int b = a + stride;
        const bool up = (a & size) == 0;
        const uint64_t x = keys[a], y = keys[b];
        if ((x > y) == up) {
          keys[a] = y;
          keys[b] = x;
        }
      }
      sort_sync<TH>();
    }
  }
}

template <int CAP, int NB, int TH>
__device__ __forceinline__ void sort_list(SortShared<CAP, NB, TH>& sh, const uint32_t* depths, uint2* ent, int len) {
  constexpr int R = CAP / TH;  // list positions per thread
  const int tid = static_cast<int>(threadIdx.x) % TH, lane = tid % kWave;
  int npow = 64;
  while (npow < len) npow <<= 1;
  const int nb = min(npow, NB);
  uint2 e[R];
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (r * TH < len) e[r] = ent[min(tid + r * TH, len - 1)];
  for (int k = tid; k < nb; k += TH) sh.hist[k] = 0u;
  if (TH > kWave && tid == 0) {
    sh.lo = ~0u;
    sh.hi = 0u;
    sh.work = 0u;
  }
  uint32_t depth[R], lo = ~0u, hi = 0u;
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (r * TH < len) depth[r] = depths[e[r].x];
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (r * TH < len) {
      lo = min(lo, depth[r]);
      hi = max(hi, depth[r]);
    }
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    lo = min(lo, static_cast<uint32_t>(__shfl_xor(lo, d, kWave)));
    hi = max(hi, static_cast<uint32_t>(__shfl_xor(hi, d, kWave)));
  }
  sort_sync<TH>();
  if (TH > kWave) {
    if (lane == 0) {
      atomicMin(&sh.lo, lo);
      atomicMax(&sh.hi, hi);
    }
    sort_sync<TH>();
    lo = sh.lo;
    hi = sh.hi;
  }
  const uint32_t span = hi - lo;
  // bucket of a depth: (depth - lo) nb / (span + 1), a little less
  const float step = 0.999f * 4294967296.f * static_cast<float>(nb) / (static_cast<float>(span) + 1.f);
  const uint32_t mult = span < static_cast<uint32_t>(nb) ? 0u : static_cast<uint32_t>(step);
  uint32_t place[R];  // (bucket << 16 | arrival in it)
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (tid + r * TH < len) {
      const uint32_t d = depth[r] - lo, b = mult ? __umulhi(d, mult) : d;
      place[r] = b << 16 | atomicAdd(&sh.hist[b], 1u);
    }
  sort_sync<TH>();
  uint32_t work = 0u;  // comparisons
  {
    constexpr int P = (NB + TH - 1) / TH;
    uint32_t c[P], sum = 0u;
    const int per = (nb + TH - 1) / TH, k0 = tid * per;
#pragma unroll
    for (int k = 0; k < P; ++k) {
      c[k] = k < per && k0 + k < nb ? sh.hist[k0 + k] : 0u;
      sum += c[k];
      work += c[k] * c[k];
    }
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) work += __shfl_xor(work, d, kWave);
    uint32_t first = sum;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const uint32_t o = __shfl_up(first, d, kWave);
      if (lane >= d) first += o;
    }
    if (TH > kWave) {
      if (lane == kWave - 1) {
        sh.wave[tid / kWave] = first;
        atomicAdd(&sh.work, work);
      }
      lds_barrier();
#pragma unroll
      for (int k = 0; k < TH / kWave; ++k) first += k < tid / kWave ? sh.wave[k] : 0u;
      work = sh.work;
    }
    first -= sum;
#pragma unroll
    for (int k = 0; k < P; ++k)
      if (k < per && k0 + k < nb) {
        sh.hist[k0 + k] = first << 16 | c[k];
        first += c[k];
      }
  }
  sort_sync<TH>();
  auto key_of = [&](int r) { return static_cast<uint64_t>(depth[r]) << 32 | static_cast<uint32_t>(tid + r * TH); };
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (tid + r * TH < len) {
      const uint32_t h = sh.hist[place[r] >> 16];
      sh.keys[(h >> 16) + (place[r] & 0xffffu)] = key_of(r);
      place[r] = h;
    }
  if (work <= kSortCrowd * static_cast<uint32_t>(len)) {
    sort_sync<TH>();
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (tid + r * TH < len) {
        const uint64_t key = key_of(r);
        const uint32_t k0 = place[r] >> 16, k1 = k0 + (place[r] & 0xffffu);
        uint32_t pos = k0;
        for (uint32_t k = k0; k < k1; k += 2) {
          const uint64_t x = sh.keys[k], y = sh.keys[min(k + 1, k1 - 1)];
          pos += (x < key ? 1u : 0u) + ((y < key && k + 1 < k1) ? 1u : 0u);
        }
        place[r] = pos;
      }
    // through LDS, so that the list is stored in order
    sort_sync<TH>();
    uint2* sorted = reinterpret_cast<uint2*>(sh.keys);
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (tid + r * TH < len) sorted[place[r]] = e[r];
    sort_sync<TH>();
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (tid + r * TH < len) ent[tid + r * TH] = sorted[tid + r * TH];
  } else {
    for (int k = len + tid; k < npow; k += TH) sh.keys[k] = ~0ull;  // sorts last
    sort_sync<TH>();
    bitonic_keys<TH>(sh.keys, npow, tid);
    // the position in a key leads back to its entry
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (tid + r * TH < len) e[r] = ent[static_cast<uint32_t>(sh.keys[tid + r * TH])];
    if (TH > kWave) __syncthreads();  // every old entry has been read
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (tid + r * TH < len) ent[tid + r * TH] = e[r];
  }
}

// The lists of up to kSortSmall entries, i.e. the tiles of one work item, one
// workgroup each, longest first; the others' tiles go to the queue.
constexpr int kSortThreads = 256;
__global__ __launch_bounds__(kSortThreads, 8) void sort_short_kernel(const DevCamera* cams, int32_t nv,
                                                                     const uint32_t* depths, int64_t n,
                                                                     const uint4* tile_order, uint2* ent,
                                                                     SortQueue queue, DevFlags* flags) {
  __shared__ SortShared<kSortSmall, 1024, kSortThreads> sh;
  // entries move: culling masks stored for the old positions no longer apply
  if (blockIdx.x == 0 && threadIdx.x == 0) flags->cull_masks = 0u;
  const uint4 d = tile_order[blockIdx.x];  // (tile, list first, list end, work items)
  const uint32_t len = d.z - d.y;
  if (len > static_cast<uint32_t>(kSortSmall)) {
    if (threadIdx.x == 0) {
      if (len > static_cast<uint32_t>(kSortMax)) flags->sort_overflow = 1u;
      else if (len > static_cast<uint32_t>(kSortMid)) queue.tiles[queue.room - 1u - atomicAdd(&queue.head[2], 1u)] = d.x;
      else queue.tiles[atomicAdd(&queue.head[0], 1u)] = d.x;
    }
  } else if (len > 1u) {
    const int v = find_view(cams, nv, static_cast<int>(d.x));
    sort_list(sh, depths + static_cast<int64_t>(v) * n, ent + d.y, static_cast<int>(len));
  }
}

// The longer lists, claimed from the queue by workgroups that stay until it is
// empty.
template <int CAP>
__global__ __launch_bounds__(1024, 4) void sort_long_kernel(
    const DevCamera* cams, int32_t nv, const uint32_t* depths, int64_t n, const uint32_t* tile_start,
    int64_t capacity, uint2* ent, SortQueue queue) {
  __shared__ SortShared<CAP, CAP == kSortMid ? kSortMid : 4096, 1024> sh;
  __shared__ uint32_t s_next;
  uint32_t* head = queue.head + (CAP == kSortMid ? 0 : 2);
  const uint32_t count = head[0];
  while (true) {
    if (threadIdx.x == 0) s_next = atomicAdd(&head[1], 1u);
    __syncthreads();
    const uint32_t k = s_next;
    if (k >= count) return;
    const uint32_t t = queue.tiles[CAP == kSortMid ? k : queue.room - 1u - k];
    const uint64_t cap = static_cast<uint64_t>(capacity);
    const uint32_t s = tile_start[t];
    const int len = static_cast<int>(min(static_cast<uint64_t>(tile_start[t + 1]), cap) - s);
    const int v = find_view(cams, nv, static_cast<int>(t));
    sort_list(sh, depths + static_cast<int64_t>(v) * n, ent + s, len);
    __syncthreads();  // the shared arrays are free again
  }
}

// The records' depths as a dense array: the sort's gathers then stay in the
// caches, 4 bytes instead of a 64-byte record each.  Also empties the queue.
__global__ __launch_bounds__(256) void sort_depths_kernel(const DevSplat* rec, uint32_t* depths, int64_t slots,
                                                          uint32_t* head) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i < 4) head[i] = 0u;
  if (i < slots) depths[i] = rec[i].slot.w;
}

// One workgroup per tile (no splitting: the composition is sequential), the
// same staging and per-wave culling as the weighted sum (the culled list
// keeps the depth order); per pixel alpha = min(alpha_max, u G), layers
// below alpha_min skipped, C += c alpha T and T *= 1 - alpha, a pixel stops
// once T < t_min and the tile once all its pixels have stopped.
template <int T>
__global__ __launch_bounds__(TileGeom<T>::kThreads) void raster_sorted_kernel(RasterArgs a, float alpha_max,
                                                                              float alpha_min, float t_min,
                                                                              float* out_T) {
  using G = TileGeom<T>;
  __shared__ StagedRec s_rec[G::kBatch];
  __shared__ __align__(16) uint8_t s_list[G::kWaves * G::kBatch];
  TileCtx<T> c;
  const int tile = static_cast<int>(blockIdx.x);
  c.v = find_view(a.cams, a.nv, tile);
  const DevCamera* cam = &a.cams[c.v];
  const int local = tile - cam->tile_base;
  c.tile = tile;
  c.tx = local % cam->tiles_x;
  c.ty = local / cam->tiles_x;
  c.n = a.n;
  const uint64_t cap = static_cast<uint64_t>(a.capacity);
  uint64_t s = a.tile_start[tile], e = a.tile_start[tile + 1];
  s = s < cap ? s : cap;
  e = e < cap ? e : cap;
  if (e < s) e = s;
  c.start = static_cast<uint32_t>(s);
  c.end = static_cast<uint32_t>(e);
  c.k = 0;
  c.nk = 1;
  c.wave = threadIdx.x / kWave;
  c.lane = threadIdx.x % kWave;
  c.bx0 = c.tx * T + (c.wave % (T / 8)) * G::kSub;
  c.by0 = c.ty * T + (c.wave / (T / 8)) * G::kSub;
  c.fx0 = c.tx * T + T / 2;
  c.fy0 = c.ty * T + T / 2;
  c.px = c.bx0 + (c.lane & 7);
  c.py = c.by0 + (c.lane >> 3);
  const bool inside = c.px < cam->width && c.py < cam->height;
  bool live = inside;
  float cr = 0.f, cg = 0.f, cb = 0.f, Tr = 1.f;
  const float pcx = static_cast<float>(c.px - c.fx0) + 0.5f;  // relative to the tile's centre
  const float pcy = static_cast<float>(c.py - c.fy0) + 0.5f;
  const float tau = a.tau;
  for (uint32_t b = c.start; b < c.end; b += G::kBatch) {
    const int m = stage_and_cull<T, G::kBatch>(a, c, b, s_rec, s_list);
    const uint8_t* list = s_list + c.wave * G::kBatch;
    for (int i = 0; i < m && live; ++i) {
      const StagedRec r = s_rec[list[i]];
      const float q = pair_q(r, pcx, pcy);
      const float al = fminf(alpha_max, r.r1.w * falloff(q));
      if (q <= tau && al >= alpha_min) {
        const float w = al * Tr;
        cr = fmaf(w, r.r1.x, cr);
        cg = fmaf(w, r.r1.y, cg);
        cb = fmaf(w, r.r1.z, cb);
        Tr *= 1.f - al;
        if (Tr < t_min) live = false;
      }
    }
    if (!__syncthreads_or(live ? 1 : 0)) break;
  }
  if (!inside) return;
  const int64_t pix = cam->pix_base + static_cast<int64_t>(c.py) * cam->width + c.px;
  a.out_rgb[3 * pix] = fmaf(Tr, a.globals[3], cr);
  a.out_rgb[3 * pix + 1] = fmaf(Tr, a.globals[4], cg);
  a.out_rgb[3 * pix + 2] = fmaf(Tr, a.globals[5], cb);
  out_T[pix] = Tr;
}

RasterArgs make_args(const Layout& L, void* ws, const void* pairs, int64_t capacity,
                     const wsr_params* P, const float* globals) {
  RasterArgs a = {};
  const PairView pv = pair_view(pairs, capacity);
  a.cams = at<DevCamera>(ws, L.off_cams);
  a.rec = at<DevSplat>(ws, L.off_rec);
  a.tile_start = at<uint32_t>(ws, L.off_tstart);
  a.ent = pv.ent;
  a.part = pv.part;
  a.n = L.n;
  a.capacity = capacity;
  a.nv = L.nv;
  a.tau = P->tau * kHalfLog2e;  // in the scale of the staged conic
  a.unnormalised = (P->flags & WSR_FLAG_UNNORMALISED) ? 1 : 0;
  a.globals = globals;
  a.items = at<uint32_t>(ws, L.off_items);
  a.tile_order = at<uint4>(ws, L.off_torder);
  a.total_tiles = L.total_tiles;
  a.acc = at<float>(ws, L.off_acc);
  // The forward's split-tile slots live in the pair buffer's partial-gradient
  // region, which the raster backward fills only later.  A tile of l pairs
  // has ceil(l / kItemSplats) - 1 items beyond its first, so at most
  // (capacity - 1) / kItemSplats slots exist; their T^2 x 20 bytes each fit
  // in the region's 36 bytes per pair for every tile size (T <= 32).
  a.split_slots = capacity > 0 ? (capacity - 1) / kItemSplats : 0;
  a.split4 = reinterpret_cast<float4*>(pv.part);
  a.splitlog = reinterpret_cast<float*>(a.split4 + a.split_slots * L.tile * L.tile);
  a.oit = at<float4>(ws, L.off_oit);
  a.acclog = at<float>(ws, L.off_acclog);
  a.du = pv.du;
  a.flags = at<DevFlags>(ws, L.off_flags);
  a.masks = capacity > 0 ? pv.masks : nullptr;
  return a;
}

// Workgroups of `kernel` (with `threads` threads) the current device holds
// at once: its compute units times the workgroups one of them can host.
// Looked up once per kernel and device; 0 if the runtime cannot tell.
int64_t resident_workgroups(const void* kernel, int threads) {
  static std::mutex mu;
  static std::map<std::pair<const void*, int>, int64_t> known;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  std::lock_guard<std::mutex> lock(mu);
  const auto key = std::make_pair(kernel, dev);
  const auto it = known.find(key);
  if (it != known.end()) return it->second;
  int per_cu = 0, cus = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  const int64_t r = static_cast<int64_t>(per_cu) * cus;
  known[key] = r;
  return r;
}

// Launch a raster kernel over the work items: one workgroup per item (the
// grid covers the upper bound of the item count; workgroups beyond the
// actual count exit at once), or, with a queue, the persistent kernel on as
// many workgroups as the device holds at once, claiming items from the
// queue (cleared here first) until none is left.
hipError_t launch_items(void (*grid_kernel)(RasterArgs), void (*persistent_kernel)(RasterArgs), RasterArgs a,
                        int64_t max_items, uint32_t* queue, int threads, hipStream_t st) {
  if (queue) {
    const int64_t r = resident_workgroups(reinterpret_cast<const void*>(persistent_kernel), threads);
    if (r > 0 && r < max_items) {
      a.queue = queue;
      const hipError_t e = launch_fill_zero(queue, sizeof(uint32_t), st);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL(persistent_kernel, dim3(static_cast<unsigned>(r)), dim3(threads), 0, st, a);
      return hipGetLastError();
    }
  }
  a.queue = nullptr;
  hipLaunchKernelGGL(grid_kernel, dim3(static_cast<unsigned>(max_items)), dim3(threads), 0, st, a);
  return hipGetLastError();
}

template <int T, int S, bool COUNT, bool CUT, bool OIT>
hipError_t fwd_k(const RasterArgs& a, int64_t grid, uint32_t* queue, hipStream_t st) {
  return launch_items(raster_fwd_kernel<T, S, COUNT, CUT, OIT, false>, raster_fwd_kernel<T, S, COUNT, CUT, OIT, true>,
                      a, grid, queue, TileGeom<T>::kThreads, st);
}

template <int T, int S>
hipError_t fwd_ts(const RasterArgs& a, int64_t grid, bool count, bool cut, bool oit, uint32_t* queue,
                  hipStream_t st) {
  if (oit) return count ? fwd_k<T, S, true, false, true>(a, grid, queue, st) : fwd_k<T, S, false, false, true>(a, grid, queue, st);
  if (cut) return count ? fwd_k<T, S, true, true, false>(a, grid, queue, st) : fwd_k<T, S, false, true, false>(a, grid, queue, st);
  return count ? fwd_k<T, S, true, false, false>(a, grid, queue, st) : fwd_k<T, S, false, false, false>(a, grid, queue, st);
}

template <int T, bool CUT, bool OIT>
hipError_t bwd_k(const RasterArgs& a, int64_t grid, uint32_t* queue, hipStream_t st) {
  return launch_items(raster_bwd_kernel<T, CUT, OIT, false>, raster_bwd_kernel<T, CUT, OIT, true>, a, grid, queue,
                      kBwdThreads, st);
}

template <int T>
hipError_t bwd_t(const RasterArgs& a, int64_t grid, bool cut, bool oit, uint32_t* queue, hipStream_t st) {
  if (oit) return bwd_k<T, false, true>(a, grid, queue, st);
  if (cut) return bwd_k<T, true, false>(a, grid, queue, st);
  return bwd_k<T, false, false>(a, grid, queue, st);
}

// Records the forward stages per batch: tile 8 (one wave, 64 threads) stages 64; tiles
// 16 and 32 take 64 (tile 16 only), 128 or 256 (the default).
template <int T>
hipError_t fwd_t(const RasterArgs& a, int64_t grid, int64_t tiles, int batch, bool count, bool cut, bool oit,
                 uint32_t* queue, hipStream_t st) {
  hipError_t e;
  if constexpr (T == 8) {
    e = fwd_ts<8, 64>(a, grid, count, cut, oit, queue, st);
  } else {
    if (batch == 128)
      e = fwd_ts<T, 128>(a, grid, count, cut, oit, queue, st);
    else if (T == 16 && batch == 64)
      e = fwd_ts<16, 64>(a, grid, count, cut, oit, queue, st);
    else
      e = fwd_ts<T, 256>(a, grid, count, cut, oit, queue, st);
  }
  if (e != hipSuccess) return e;
  if (oit)
    raster_fwd_finalize<T, true><<<dim3(static_cast<unsigned>(tiles)), 256, 0, st>>>(a);
  else
    raster_fwd_finalize<T, false><<<dim3(static_cast<unsigned>(tiles)), 256, 0, st>>>(a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_raster_fwd(const Layout& L, void* ws, const void* pairs, int64_t capacity,
                             const wsr_params* P, const float* globals, float* out_rgb,
                             float* out_den, int32_t* out_count, hipStream_t st) {
  if (L.total_tiles == 0) return hipSuccess;
  RasterArgs a = make_args(L, ws, pairs, capacity, P, globals);
  a.out_rgb = out_rgb;
  a.out_den = out_den;
  a.out_count = out_count;
  const bool cnt = out_count != nullptr;
  if (cnt) {
    const hipError_t e = launch_fill_zero(out_count, sizeof(int32_t) * L.total_pixels, st);
    if (e != hipSuccess) return e;
  }
  const int64_t grid = max_raster_items(L, capacity);
  const bool oit = (P->flags & WSR_FLAG_OIT) != 0;
  uint32_t* queue = (P->flags & WSR_FLAG_PERSISTENT) ? at<uint32_t>(ws, L.off_queue) : nullptr;
  const bool cut = P->alpha_cut > 0.f;
  switch (L.tile) {
    case 8: return fwd_t<8>(a, grid, L.total_tiles, P->batch, cnt, cut, oit, queue, st);
    case 32: return fwd_t<32>(a, grid, L.total_tiles, P->batch, cnt, cut, oit, queue, st);
    default: return fwd_t<16>(a, grid, L.total_tiles, P->batch, cnt, cut, oit, queue, st);
  }
}

hipError_t launch_raster_bwd(const Layout& L, void* ws, void* pairs, int64_t capacity,
                             const wsr_params* P, const float* globals, const float* dL_drgb,
                             const float* rgb, const float* den, hipStream_t st) {
  if (L.total_tiles == 0) return hipSuccess;
  RasterArgs a = make_args(L, ws, pairs, capacity, P, globals);
  a.dL_drgb = dL_drgb;
  a.rgb = rgb;
  a.den = den;
  a.tilepart = at<float>(ws, L.off_tilepart);
  const int64_t grid = max_raster_items(L, capacity);
  const bool oit = (P->flags & WSR_FLAG_OIT) != 0;
  uint32_t* queue = (P->flags & WSR_FLAG_PERSISTENT) ? at<uint32_t>(ws, L.off_queue) + 1 : nullptr;
  const bool cut = P->alpha_cut > 0.f;
  switch (L.tile) {
    case 8: return bwd_t<8>(a, grid, cut, oit, queue, st);
    case 32: return bwd_t<32>(a, grid, cut, oit, queue, st);
    default: return bwd_t<16>(a, grid, cut, oit, queue, st);
  }
}

}  // namespace wsr

namespace wsr {

hipError_t launch_sort_tiles(const Layout& L, void* ws, void* pairs, int64_t capacity, hipStream_t st) {
  if (L.total_tiles == 0) return hipSuccess;
  const PairView pv = pair_view(pairs, capacity);
  const DevCamera* cams = at<DevCamera>(ws, L.off_cams);
  const uint32_t* tstart = at<uint32_t>(ws, L.off_tstart);
  DevFlags* flags = at<DevFlags>(ws, L.off_flags);
  // the 2D dL/du array and the count matrix are scratch outside the projection
  // backward and the binning
  uint32_t* depths = at<uint32_t>(ws, L.off_du2d);
  SortQueue queue;
  queue.head = at<uint32_t>(ws, L.off_sortq);
  queue.tiles = at<uint32_t>(ws, L.off_hist);
  queue.room = static_cast<uint32_t>(L.total_tiles);
  const int64_t slots = L.n * L.nv;
  sort_depths_kernel<<<static_cast<unsigned>(slots / 256 + 1), 256, 0, st>>>(at<DevSplat>(ws, L.off_rec), depths,
                                                                             slots, queue.head);
  sort_short_kernel<<<static_cast<unsigned>(L.total_tiles), kSortThreads, 0, st>>>(
      cams, L.nv, depths, L.n, at<uint4>(ws, L.off_torder), pv.ent, queue, flags);
  // as many workgroups as run at once, and no more than there can be lists
  if (capacity > kSortSmall)
    sort_long_kernel<kSortMid><<<static_cast<unsigned>(std::min<int64_t>({512, L.total_tiles, capacity / kSortSmall})),
                                 1024, 0, st>>>(cams, L.nv, depths, L.n, tstart, capacity, pv.ent, queue);
  if (capacity > kSortMid)
    sort_long_kernel<kSortMax><<<static_cast<unsigned>(std::min<int64_t>({256, L.total_tiles, capacity / kSortMid})),
                                 1024, 0, st>>>(cams, L.nv, depths, L.n, tstart, capacity, pv.ent, queue);
  return hipGetLastError();
}

hipError_t launch_raster_sorted(const Layout& L, void* ws, const void* pairs, int64_t capacity,
                                const wsr_params* P, const float* globals, float alpha_max, float alpha_min,
                                float t_min, float* out_rgb, float* out_T, hipStream_t st) {
  if (L.total_tiles == 0) return hipSuccess;
  RasterArgs a = make_args(L, ws, pairs, capacity, P, globals);
  a.masks = nullptr;  // the sorted lists are culled on their own
  a.out_rgb = out_rgb;
  const dim3 grid(static_cast<unsigned>(L.total_tiles));
  switch (L.tile) {
    case 8:
      raster_sorted_kernel<8><<<grid, TileGeom<8>::kThreads, 0, st>>>(a, alpha_max, alpha_min, t_min, out_T);
      break;
    case 32:
      raster_sorted_kernel<32><<<grid, TileGeom<32>::kThreads, 0, st>>>(a, alpha_max, alpha_min, t_min, out_T);
      break;
    default:
      raster_sorted_kernel<16><<<grid, TileGeom<16>::kThreads, 0, st>>>(a, alpha_max, alpha_min, t_min, out_T);
  }
  return hipGetLastError();
}

}  // namespace wsr
