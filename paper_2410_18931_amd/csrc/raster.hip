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
template <int T>
struct TileGeom {
  static constexpr int kSub = 8;                       // wave block edge
  static constexpr int kWaves = (T / 8) * (T / 8);
  static constexpr int kThreads = kWaves * kWave;
  static constexpr int kBatch = kThreads < 256 ? kThreads : 256;
  static_assert(kBatch <= 256, "the backward's lists hold 8-bit record indices");
};

// A record as staged in LDS for one tile (48 bytes; stage_and_cull builds it
// from the projected record):
//   r0 = (mx, my, A, B2)   centre relative to the tile's centre; conic
//                          (A, B2 = 2B, C) times log2(e) / 2
//   r1 = (C, amp, c0, c1)  colour (times amp in the forward)
//   r2 = (c2, ext | cut, u, K)  support half-extents (two halves), or with
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
  return quad_form(r.r0.z, r.r0.w * dy, (r.r1.x * dy) * dy, dx);
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

// Does the splat's support reach the wave block whose pixel centres span
// [bx, bx + sub1] x [by, by + sub1] (relative to the tile's centre)?  First
// the (conservative) support box; then, unless the conic is badly
// conditioned, the exact minimum of q over
// the block (the unconstrained minimum is the centre; otherwise the minimum
// lies on an edge, at the clamped 1D minimiser of that edge) against tau with
// a margin far above the float error of q.  For needle-like splats
// (eigenvalue ratio above ~100) float q loses digits to cancellation, so the
// box decision is kept.
//
// With CUT (the opacity early-out) the record's fourth word is the splat's
// own cutoff instead of the half-extents, which are then derived from the
// conic: the extents of q <= cut are sqrt(cut C / det) and sqrt(cut A / det),
// with det = A C - B^2 formed by Kahan's algorithm (B^2 split exactly with an
// FMA) so that it stays accurate for needle-like conics.
template <bool CUT>
__device__ __forceinline__ bool block_hits(const StagedRec& r, float bx, float by, float sub1, float tau_in) {
  float2 e;
  float tau = tau_in;
  if (CUT) {
    tau = r.r2.y;
    const float A = r.r0.z, B = 0.5f * r.r0.w, C = r.r1.x;
    const float bb = B * B;
    const float det = fmaf(A, C, -bb) - fmaf(B, B, -bb);
    const float s = det > 0.f ? tau * __builtin_amdgcn_rcpf(det) : __builtin_inff();
    e = make_float2(sqrtf(s * C) * 1.0001f, sqrtf(s * A) * 1.0001f);
  } else {
    e = rec_extent(r);
  }
  const float mx = r.r0.x, my = r.r0.y;
  const float sx = 1e-3f * fabsf(mx) + 1e-2f, sy = 1e-3f * fabsf(my) + 1e-2f;  // rounding slack
  if (!((mx + e.x + sx >= bx) && (mx - e.x - sx <= bx + sub1) && (my + e.y + sy >= by) &&
        (my - e.y - sy <= by + sub1)))
    return false;
  const float A = r.r0.z, B = 0.5f * r.r0.w, C = r.r1.x;
  const float tr = A + C, det = A * C - B * B;
  if (!(tr * tr <= 102.f * det)) return true;
  // block corners relative to the centre
  const float x0 = bx - mx, x1 = (bx + sub1) - mx;
  const float y0 = by - my, y1 = (by + sub1) - my;
  if (x0 <= 0.f && x1 >= 0.f && y0 <= 0.f && y1 >= 0.f) return true;
  // hardware reciprocals (within 1 ulp): they only place the edge minimisers,
  // whose error changes q there by a second-order amount far inside the margin
  const float iA = __builtin_amdgcn_rcpf(A), iC = __builtin_amdgcn_rcpf(C);
  float qmin = 3.0e38f;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const float dy = k ? y1 : y0;
    const float dx = fminf(fmaxf(-B * dy * iA, x0), x1);
    qmin = fminf(qmin, A * dx * dx + 2.f * B * dx * dy + C * dy * dy);
    const float ex2 = k ? x1 : x0;
    const float ey2 = fminf(fmaxf(-B * ex2 * iC, y0), y1);
    qmin = fminf(qmin, A * ex2 * ex2 + 2.f * B * ex2 * ey2 + C * ey2 * ey2);
  }
  return qmin <= tau * 1.002f + 1e-3f;
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
  // culling masks (see cull_mask_word), or null where the pair buffer has no
  // room for them; flags->cull_masks says whether they hold the current
  // lists' masks
  uint64_t* masks;
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

// The culling masks: wave w's 64-bit ballot for the 64-entry group g of tile
// t's list (entries list0 + 64 g ...) is word (list0 / 64 + t + g) W + w, W the
// waves of a tile.  A tile of l entries has ceil(l / 64) groups and the next
// tile's first group is at least floor((list0 + l) / 64) + t + 1, so the
// tiles' words never overlap; all of them lie below
// (ceil(capacity / 64) + tiles + 2) W.
template <int T>
__device__ __forceinline__ int64_t cull_mask_word(const TileCtx<T>& c, uint32_t pos, int wave) {
  constexpr int W = TileGeom<T>::kWaves;
  const int64_t g = static_cast<int64_t>(c.list0 >> 6) + c.tile + ((pos - c.list0) >> 6);
  return g * W + wave;
}

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
  r.r1 = make_float4(s.r1.x * kHalfLog2e, amp, c0, c1);
  // OIT: the opacity u rides in the record's third word
  r.r2 = make_float4(c2, CUT ? s.r2.w * kHalfLog2e : s.r2.w, OIT ? __uint_as_float(d->slot.w) : 0.f,
                     CUT ? support_k(s.r2.w * kHalfLog2e) : 0.f);
  return r;
}

// Stage one batch of records into LDS (as StagedRec) and build this wave's
// culled list.  Returns the list length.  With PREMUL (the forward) the
// staged colour is premultiplied by the amplitude, so a pair adds G (amp c)
// and G amp.  The list holds staged-record indices (uint8_t) or, as uint16_t,
// their byte offsets in s_rec, which the forward uses as LDS addresses
// directly.  mask_out (may be null) receives the wave's culling masks.
template <int T, int BATCH, bool CUT, bool OIT, bool PREMUL, typename LT>
__device__ __forceinline__ int stage_and_cull(const RasterArgs& a, const TileCtx<T>& c, uint32_t b,
                                              StagedRec* s_rec, LT* s_list, uint64_t* mask_out = nullptr) {
  using G = TileGeom<T>;
  const float tox = static_cast<float>(c.fx0), toy = static_cast<float>(c.fy0);
  __syncthreads();  // previous batch fully consumed
  for (int q = threadIdx.x; q < BATCH; q += G::kThreads) {
    const uint32_t j = b + q;
    if (j < c.end) {
      const DevSplat* d = a.rec + static_cast<int64_t>(c.v) * c.n + a.ent[j].x;
      s_rec[q] = make_staged<CUT, OIT, PREMUL>(d, tox, toy);
    }
  }
  __syncthreads();
  const int cnt = static_cast<int>(min(static_cast<uint32_t>(BATCH), c.end - b));
  LT* list = s_list + c.wave * BATCH;
  int m = 0;
  const float bx = static_cast<float>(c.bx0 - c.fx0) + 0.5f, by = static_cast<float>(c.by0 - c.fy0) + 0.5f;
  for (int k0 = 0; k0 < cnt; k0 += kWave) {
    const int k = k0 + c.lane;
    const bool hit = k < cnt && block_hits<CUT>(s_rec[k], bx, by, static_cast<float>(G::kSub - 1), a.tau);
    const uint64_t mask = __ballot(hit);
    if (mask_out && c.lane == 0) mask_out[cull_mask_word(c, b + k0, c.wave)] = mask;
    const int pos = m + __popcll(mask & ((1ull << c.lane) - 1ull));
    if (hit) list[pos] = static_cast<LT>(sizeof(LT) == 1 ? k : k * static_cast<int>(sizeof(StagedRec)));
    m += __popcll(mask);
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
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

__device__ __forceinline__ const StagedRec& rec_at(const StagedRec* base, uint32_t off) {
  return *reinterpret_cast<const StagedRec*>(reinterpret_cast<const char*>(base) + off);
}

// The lanes of a forward wave: lane = (slot, row).  Row r of the 8x8 block is
// evaluated by the eight lanes that hold it, each against another splat of the
// list (slot s takes positions s, s + 8, ... of the wave's lists taken
// together), eight pixels per lane.  Against one pixel per lane and one splat
// per step this shares a row's dy, B2 dy and C dy^2 among eight pixels (9.5
// instead of 14.25 VALU operations per pixel and splat besides the exp2), and
// one LDS read fetches eight records instead of one (the forward read 40 B of
// LDS per lane and splat, now 5).
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

// The forward of one work item (tile_setup's c), S records staged per batch.
// The groups of eight splats run on across the batches (a lane keeps the
// record of an incomplete group), so the order of every pixel's sums follows
// from the list alone, whatever the batch size.
template <int T, int S, bool COUNT, bool CUT, bool OIT>
__device__ __forceinline__ void raster_fwd_item(const RasterArgs& a, const TileCtx<T>& c, const DevCamera* cam,
                                                StagedRec* s_rec, uint16_t* s_list) {
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
  // pixel centres relative to the tile's centre (exact): the row's y and the
  // block's first column
  const float pcy = static_cast<float>(c.by0 + row - c.fy0) + 0.5f;
  float xs[8];  // wave-uniform: kept in scalar registers
#pragma unroll
  for (int k = 0; k < 8; ++k)
    xs[k] = __uint_as_float(
        __builtin_amdgcn_readfirstlane(__float_as_uint(static_cast<float>(c.bx0 + k - c.fx0) + 0.5f)));
  // the staged colour carries the amplitude
  auto accumulate = [&](const StagedRec& r, float K) {
    const float dy = pcy - r.r0.y;
    const float B2dy = r.r0.w * dy, Cdy2 = (r.r1.x * dy) * dy;
    float q[8], G[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) q[k] = quad_form(r.r0.z, B2dy, Cdy2, xs[k] - r.r0.x);
    falloff_row(q, K, G);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      nr[k] = fmaf(G[k], r.r1.z, nr[k]);
      ng[k] = fmaf(G[k], r.r1.w, ng[k]);
      nb[k] = fmaf(G[k], r.r2.x, nb[k]);
      dd[k] = fmaf(G[k], r.r1.y, dd[k]);
      if (OIT) cov[k] *= 1.f - __builtin_amdgcn_fmed3f(r.r2.z * G[k], 0.f, 1.f);
      if (COUNT) cntp[k] += static_cast<int>(in_support(q[k], K));
    }
  };
  const float K = support_k(a.tau);
  StagedRec rec = {};  // this lane's record of the next group (a slot that never held one adds G = 0 times 0)
  int held = 0;        // slots whose record waits in `rec` for the group to fill
  for (uint32_t b = c.start; b < c.end; b += S) {
    const int m = stage_and_cull<T, S, CUT, OIT, true, uint16_t>(a, c, b, s_rec, s_list, a.masks);
    const uint16_t* list = s_list + c.wave * S;
    int k = slot - held;  // list position of this lane's next record
    if (k >= 0 && k < m) rec = rec_at(s_rec, list[k]);
    held += m;
    // the next group's records are requested before this one's arithmetic
    // (past the end of the list, where no slot is held, any record will do);
    // two groups per turn, so that no record is copied between registers
    while (held >= 2 * kFwdSlots) {
      const StagedRec next = rec_at(s_rec, list[min(k + kFwdSlots, m - 1)]);
      accumulate(rec, CUT ? rec.r2.w : K);
      k += 2 * kFwdSlots;
      rec = rec_at(s_rec, list[min(k, m - 1)]);
      accumulate(next, CUT ? next.r2.w : K);
      held -= 2 * kFwdSlots;
    }
    if (held >= kFwdSlots) {
      const StagedRec next = rec_at(s_rec, list[min(k + kFwdSlots, m - 1)]);
      accumulate(rec, CUT ? rec.r2.w : K);
      rec = next;
      held -= kFwdSlots;
    }
  }
  if (held > 0) accumulate(rec, slot < held ? (CUT ? rec.r2.w : K) : support_k(-1.f));

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
// counter until none is left.
// Resident waves per SIMD asked of the compiler at tile 16: as many as fit
// without spilled registers.
template <int T, bool OIT>
constexpr int fwd_min_blocks() {
  return T == 16 ? (OIT ? 4 : 5) : 1;
}

template <int T, int S, bool COUNT, bool CUT, bool OIT, bool PERSIST>
__global__ __launch_bounds__(TileGeom<T>::kThreads, (fwd_min_blocks<T, OIT>())) void raster_fwd_kernel(RasterArgs a) {
  using G = TileGeom<T>;
  __shared__ StagedRec s_rec[S];
  __shared__ __align__(16) uint16_t s_list[G::kWaves * S];
  __shared__ uint32_t s_item;
  // every work item stores its waves' culling masks (when there is room):
  // valid for the backward once this launch has finished
  if (blockIdx.x == 0 && threadIdx.x == 0) a.flags->cull_masks = a.masks ? (kCullMasks | (CUT ? 2u : 0u)) : 0u;
  const uint32_t n_items = a.items[a.total_tiles];
  uint32_t item = PERSIST ? claim_item(a, &s_item) : blockIdx.x;
  while (item < n_items) {
    TileCtx<T> c;
    const DevCamera* cam;
    tile_setup<T>(a, item, c, cam);
    raster_fwd_item<T, S, COUNT, CUT, OIT>(a, c, cam, s_rec, s_list);
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

// Per-pixel factors of an 8x8 block in LDS: 64 of them, and one of padding, so
// that the same pixel of different blocks lies in different banks.
constexpr int kPdStride = kWave + 1;

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
  const float A = r.r0.z, B2 = r.r0.w, Cc = r.r1.x;
  const float amp = r.r1.y, cr = r.r1.z, cg = r.r1.w, cb = r.r2.x;
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
  const float amp = r.r1.y, A = r.r0.z, B2 = r.r0.w, Cc = r.r1.x;
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

// Resident waves per SIMD asked of the compiler at tile 16: four, as many as
// the SIMD needs to issue two FP32 operations at once throughout (at most 128
// VGPRs).
template <int T, bool OIT>
constexpr int bwd_min_blocks() {
  return T == 16 ? 4 : 1;
}

// Barrier between LDS writes and reads of a workgroup.  __syncthreads would
// also wait for the outstanding global stores.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Backward of one work item.  Every lane takes one splat of the item and walks
// the 8x8 pixel blocks of the tile that its support reaches, so a splat's
// gradient sums stay in its lane's registers from the first pixel to the
// store: no merging between waves, and no barrier, once the walk has begun.
// The lanes of a wave walk the blocks of their own splats (a lane's j-th block
// is its splat's j-th); for them to finish together the item's splats are
// first sorted by the number of blocks they reach (a counting sort in LDS),
// the most first.  Splats that reach no block get zeros.  The records of a
// wave's next splats are requested before it walks the present ones.
//
// The previous form (waves owning blocks, lanes owning splats of the wave's
// culled list, the waves' sums merged through LDS in lockstep rounds) spent
// 47 % of its wave time waiting at the rounds' barriers, at the staging's and
// on LDS.
//
// The last splats, fewer than the workgroup has lanes, share their blocks
// among W = 1, 2, 4 or 8 lanes: lane group g walks rows [g 8/W, (g+1) 8/W) of
// every block and the groups' sums are added with shuffles.  A splat's sums
// depend on its place in the sort through W alone, and the sort is stable, so
// they do not vary from run to run.
template <int T>
struct BwdShared {
  static constexpr int kBlocks = TileGeom<T>::kWaves;
  // the item's splats, most blocks first: Gaussian id; index in the item, and
  // in the upper half the blocks it reaches (one bit per block)
  uint2 order[kItemSplats];
  uint32_t count[kBlocks + 1][TileGeom<T>::kWaves];  // per number of blocks and wave
};

// Wave w sorts the w-th share of the item, whole groups of 64 splats: at most
// 32 / NB groups, whose NB 64-bit ballots fit the wave's lanes (lane g NB + b
// holds group g's ballot for block b).  All global loads of the sort are
// issued by bwd_sort_begin, so that they and the pixel factors' cost one
// memory round trip.
template <int T>
struct BwdShare {
  static constexpr int kGroups = kItemSplats / (kWave * TileGeom<T>::kWaves);
  int w0, w1;            // the share, relative to the item
  uint32_t id[kGroups];  // Gaussian of each group's entry
  uint64_t word;         // the forward's ballots
};

template <int T>
__device__ __forceinline__ void bwd_sort_begin(const RasterArgs& a, const TileCtx<T>& c, BwdShare<T>& q,
                                               const uint64_t* masks_in) {
  using G = TileGeom<T>;
  const int len = static_cast<int>(c.end - c.start);
  const int per = ((len + G::kWaves - 1) / G::kWaves + kWave - 1) & ~(kWave - 1);
  q.w0 = min(c.wave * per, len);
  q.w1 = min(q.w0 + per, len);
  const int groups = (q.w1 - q.w0 + kWave - 1) / kWave;
  q.word = 0;
  if (masks_in && c.lane < groups * G::kWaves) q.word = masks_in[cull_mask_word(c, c.start + q.w0, 0) + c.lane];
#pragma unroll
  for (int g = 0; g < BwdShare<T>::kGroups; ++g) {
    const int e = q.w0 + g * kWave + c.lane;
    q.id[g] = e < q.w1 ? a.ent[c.start + e].x : 0u;
  }
}

template <int T, bool CUT, bool OIT>
__device__ __forceinline__ int bwd_sort(const RasterArgs& a, const TileCtx<T>& c, BwdShare<T>& q, BwdShared<T>& sh,
                                        bool have_masks) {
  using G = TileGeom<T>;
  constexpr int NB = BwdShared<T>::kBlocks;
  constexpr int NG = BwdShare<T>::kGroups;
  static_assert(NG * NB <= kWave, "a wave's ballots fit its lanes");
  if (!have_masks) {
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const int e = q.w0 + g * kWave + c.lane;
      StagedRec r = {};
      if (e < q.w1)
        r = make_staged<CUT, OIT, false>(a.rec + static_cast<int64_t>(c.v) * c.n + q.id[g],
                                         static_cast<float>(c.fx0), static_cast<float>(c.fy0));
#pragma unroll 1
      for (int b = 0; b < NB; ++b) {
        const float bx = static_cast<float>((b % (T / 8)) * 8 - T / 2) + 0.5f;
        const float by = static_cast<float>((b / (T / 8)) * 8 - T / 2) + 0.5f;
        const uint64_t m = __ballot(e < q.w1 && block_hits<CUT>(r, bx, by, static_cast<float>(G::kSub - 1), a.tau));
        if (c.lane == g * NB + b) q.word = m;
      }
    }
  }
  // the blocks reached by this lane's splat of group g
  auto hits = [&](int g) {
    uint32_t h = 0;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(q.word), g * NB + b);
      const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(q.word >> 32), g * NB + b);
      const uint64_t m = (static_cast<uint64_t>(hi) << 32) | lo;
      h |= static_cast<uint32_t>((m >> c.lane) & 1ull) << b;
    }
    return h;
  };
  uint32_t at[NB + 1];  // per number of blocks: this wave's splats, then the place of its next one
#pragma unroll
  for (int k = 0; k <= NB; ++k) at[k] = 0;
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    if (q.w0 + g * kWave >= q.w1) break;
    const int n = q.w0 + g * kWave + c.lane < q.w1 ? __popc(hits(g)) : -1;
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
    for (int w = 0; w < G::kWaves; ++w) {
      if (w == c.wave) at[k] = static_cast<uint32_t>(total);
      total += static_cast<int>(sh.count[k][w]);
    }
  }
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    if (q.w0 + g * kWave >= q.w1) break;
    const int e = q.w0 + g * kWave + c.lane;
    const uint32_t h = hits(g);
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
// the upper half the blocks of the tile the splat reaches (0: no splat).
template <int T, bool CUT, bool OIT, int W>
__device__ __forceinline__ void bwd_walk(const RasterArgs& a, const TileCtx<T>& c, const float4* s_pd,
                                         const float* s_pk, const StagedRec& r, uint32_t order) {
  constexpr int S = kWave / W;  // splats per group
  constexpr int R = 8 / W;      // rows per lane group
  const int g = c.lane / S;
  uint32_t h = order >> 16;
  const bool valid = h != 0;
  const uint32_t slot = a.ent[c.start + (order & 0xffffu)].y;  // needed at the end only
  const float Kv = CUT ? r.r2.w : support_k(a.tau);
  WalkSums<OIT> sums;
  while (__any(h != 0)) {
    const float K = h != 0 ? Kv : support_k(-1.f);
    const int b = h != 0 ? __ffs(static_cast<int>(h)) - 1 : 0;
    h &= h - 1;
    // the block's first pixel centre relative to the tile's centre (exact, so
    // that dx and dy match the forward's)
    const float ex0 = static_cast<float>((b % (T / 8)) * 8 - T / 2) + 0.5f;
    float yrow = static_cast<float>((b / (T / 8)) * 8 - T / 2 + g * R) + 0.5f;
    float dx[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) dx[k] = (ex0 + static_cast<float>(k)) - r.r0.x;
    const float4* pd = s_pd + b * kPdStride + g * R * 8;
    const float* pk = OIT ? s_pk + b * kPdStride + g * R * 8 : nullptr;
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
__global__ __launch_bounds__(TileGeom<T>::kThreads, (bwd_min_blocks<T, OIT>())) void raster_bwd_kernel(
    RasterArgs a) {
  using G = TileGeom<T>;
  __shared__ BwdShared<T> sh;
  __shared__ float4 s_pd[G::kWaves * kPdStride];              // per-pixel factors, block by block
  __shared__ float s_pk[OIT ? G::kWaves * kPdStride : 1];     // OIT: per-pixel coverage factors
  __shared__ float s_bg[G::kWaves][4];
  __shared__ uint32_t s_item;
  // the forward's culling masks, if it stored them for these lists with the
  // same early-out setting
  const uint64_t* masks_in =
      (a.masks && a.flags->cull_masks == (kCullMasks | (CUT ? 2u : 0u))) ? a.masks : nullptr;
  const uint32_t n_items = a.items[a.total_tiles];
  uint32_t item = PERSIST ? claim_item(a, &s_item) : blockIdx.x;
  while (item < n_items) {
    TileCtx<T> c;
    const DevCamera* cam;
    tile_setup<T>(a, item, c, cam);
    BwdShare<T> share;
    bwd_sort_begin<T>(a, c, share, masks_in);
    // every thread's pixel factors into LDS; the tile's first work item also
    // stores the tile's background-gradient partial sums
    {
      float4 pd;
      float kcov, bacc[4];
      pixel_factors<OIT>(a, *cam, c.px, c.py, &pd, &kcov, bacc);
      s_pd[c.wave * kPdStride + c.lane] = pd;
      if (OIT) s_pk[c.wave * kPdStride + c.lane] = kcov;
      if (c.k == 0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float sj = wave_sum(bacc[j]);
          if (c.lane == 0) s_bg[c.wave][j] = sj;
        }
      }
    }
    const int n = bwd_sort<T, CUT, OIT>(a, c, share, sh, masks_in != nullptr);
    if (c.k == 0 && threadIdx.x < 4) {
      float sj = 0.f;
#pragma unroll
      for (int w = 0; w < G::kWaves; ++w) sj += s_bg[w][threadIdx.x];
      a.tilepart[c.tile * 4 + threadIdx.x] = sj;
    }
    // rounds of one lane per splat that keep every wave busy, then the rest
    // with W lanes per splat
    const int rounds = n / G::kThreads, rest = n % G::kThreads;
    const int wsh = rest * 8 <= G::kThreads ? 3 : rest * 4 <= G::kThreads ? 2 : rest * 2 <= G::kThreads ? 1 : 0;
    const DevSplat* recs = a.rec + static_cast<int64_t>(c.v) * c.n;
    const float tox = static_cast<float>(c.fx0), toy = static_cast<float>(c.fy0);
    // this lane's splat of a round (its record, and item index and blocks; no
    // blocks past the end)
    auto fetch = [&](int round, uint32_t& order, StagedRec& r) {
      const int first = round < rounds ? round * G::kThreads + c.wave * kWave
                                       : rounds * G::kThreads + c.wave * (kWave >> wsh);
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
    for (int j = n + threadIdx.x; j < static_cast<int>(c.end - c.start); j += G::kThreads) {
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

// One workgroup per tile: the tile's list, keyed by (depth bits, list
// position), is sorted in LDS by a bitonic network over the next power of two
// (padding keys sort last), and the entries (id and Gaussian-major slot) are
// then moved to their sorted positions: every thread first reads the entries
// its positions receive, then, after a barrier, writes them.  Binning leaves
// every list in increasing id order, so ties in depth stay in id order.  An
// instance holds CAP keys and sorts the lists of length lo < l <= CAP; the
// largest instance raises a flag for lists longer than kSortMax, which stay
// unsorted.  Three instances (16, 64 and 128 KB of LDS): most lists are
// short, and the smaller instances let more workgroups share a CU.
constexpr int kSortSmall = 2048;
constexpr int kSortMid = 8192;

template <int CAP>
__global__ __launch_bounds__(1024) void sort_tiles_kernel(const DevCamera* cams, int32_t nv, const DevSplat* rec,
                                                          int64_t n, const uint32_t* tile_start, uint2* ent,
                                                          int64_t capacity, int lo, DevFlags* flags) {
  constexpr int R = CAP / 1024;  // list positions per thread
  __shared__ uint64_t keys[CAP];
  const int tile = static_cast<int>(blockIdx.x);
  // entries move: culling masks stored for the old positions no longer apply
  if (CAP == kSortSmall && tile == 0 && threadIdx.x == 0) flags->cull_masks = 0u;
  const uint64_t cap = static_cast<uint64_t>(capacity);
  uint64_t s = tile_start[tile], e = tile_start[tile + 1];
  s = s < cap ? s : cap;
  e = e < cap ? e : cap;
  if (e <= s + 1 || e - s <= static_cast<uint64_t>(lo)) return;
  if (e - s > static_cast<uint64_t>(CAP)) {
    if (CAP == kSortMax && threadIdx.x == 0) flags->sort_overflow = 1u;
    return;
  }
  const int len = static_cast<int>(e - s);
  const int v = find_view(cams, nv, tile);
  int npow = 2;
  while (npow < len) npow <<= 1;
  for (int k = threadIdx.x; k < npow; k += 1024) {
    uint64_t key = ~0ull;
    if (k < len) {
      const uint32_t id = ent[s + k].x;
      const uint32_t depth = rec[static_cast<int64_t>(v) * n + id].slot.w;
      key = (static_cast<uint64_t>(depth) << 32) | static_cast<uint32_t>(k);
    }
    keys[k] = key;
  }
  __syncthreads();
  for (int size = 2; size <= npow; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int i = threadIdx.x; i < (npow >> 1); i += 1024) {
        const int a = (i / stride) * 2 * stride + (i % stride);
        const int b = a + stride;
        const bool up = (a & size) == 0;
        const uint64_t x = keys[a], y = keys[b];
        if ((x > y) == up) {
          keys[a] = y;
          keys[b] = x;
        }
      }
      __syncthreads();
    }
  }
  uint2 moved[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int k = threadIdx.x + r * 1024;
    if (k < len) moved[r] = ent[s + static_cast<uint32_t>(keys[k])];
  }
  __syncthreads();  // every old entry has been read
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int k = threadIdx.x + r * 1024;
    if (k < len) ent[s + k] = moved[r];
  }
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
    const int m = stage_and_cull<T, G::kBatch, false, false, false, uint8_t>(a, c, b, s_rec, s_list);
    const uint8_t* list = s_list + c.wave * G::kBatch;
    for (int i = 0; i < m && live; ++i) {
      const StagedRec r = s_rec[list[i]];
      const float q = pair_q(r, pcx, pcy);
      const float al = fminf(alpha_max, r.r1.y * falloff(q));
      if (q <= tau && al >= alpha_min) {
        const float w = al * Tr;
        cr = fmaf(w, r.r1.z, cr);
        cg = fmaf(w, r.r1.w, cg);
        cb = fmaf(w, r.r2.x, cb);
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
  // The culling masks have 4 bytes per pair of the pair buffer; a capacity
  // too small for the per-tile rounding of the groups leaves them off.
  {
    const int64_t waves = static_cast<int64_t>(L.tile / 8) * (L.tile / 8);
    const int64_t words = (((capacity + 63) >> 6) + L.total_tiles + 2) * waves;
    a.masks = capacity > 0 && 8 * words <= 4 * capacity ? pv.masks : nullptr;
  }
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
                      TileGeom<T>::kThreads, st);
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
  const dim3 grid(static_cast<unsigned>(L.total_tiles));
  // the three instances sort disjoint sets of tiles
  const DevCamera* cams = at<DevCamera>(ws, L.off_cams);
  const DevSplat* rec = at<DevSplat>(ws, L.off_rec);
  const uint32_t* tstart = at<uint32_t>(ws, L.off_tstart);
  DevFlags* flags = at<DevFlags>(ws, L.off_flags);
  sort_tiles_kernel<kSortSmall><<<grid, 1024, 0, st>>>(cams, L.nv, rec, L.n, tstart, pv.ent, capacity, 0, flags);
  sort_tiles_kernel<kSortMid><<<grid, 1024, 0, st>>>(cams, L.nv, rec, L.n, tstart, pv.ent, capacity, kSortSmall, flags);
  sort_tiles_kernel<kSortMax><<<grid, 1024, 0, st>>>(cams, L.nv, rec, L.n, tstart, pv.ent, capacity, kSortMid, flags);
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
