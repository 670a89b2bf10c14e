// Step a6 of the WSR path: per-tile lists of Gaussian ids with no depth key.
// Eq. 7 is a commutative sum (Sec. 4.2), so only membership matters; this is
// the step that replaces the per-tile depth sort of 3DGS (Sec. 4.1).
//
// A counting sort by tile, with no global atomics:
//   1. bin_pass<count>: block (b, z, v) takes Gaussians [b*chunk, ...) of
//      view v and counts their (tile, Gaussian) pairs in the tile rows of
//      band z, as prefix sums of the rectangles' corners in LDS, written
//      contiguously as row b of the block-major count matrix M[v][b][tile].
//   2. column_scan_wide: each tile's column of M becomes exclusive prefixes
//      over the blocks, and the tile's total; tile_scan_single scans the
//      totals into the start of every tile's list (tile_start).
//   3. bin_pass<scatter>: the same blocks re-expand their pairs and place
//      each pair's entry (Gaussian id, Gaussian-major slot, see below) at
//      tile_start[t] + M[v][b][t] + the pair's stable rank in the block.
// A wave expands its Gaussians 64 at a time: a wave-wide scan of their pair
// counts, then 64 pairs per step, one per lane, so one huge splat does not
// serialise on one thread.  The scatter is stable: every tile's list holds its
// Gaussian ids in increasing order, whatever the timing of the run.  Eq. 7
// does not need an order, but the float sums of the raster stages follow the
// list order, so a fixed order makes the whole path reproducible bit for bit.
//
// The same step also lays out the backward's per-pair scratch: every
// (view, Gaussian) gets a contiguous range of "Gaussian-major" slots, one per
// tile of its rectangle in row-major order.  Its first slot, goff, is the
// exclusive scan of the rectangle sizes in (view, Gaussian) order, formed by
// the same passes: the counting pass's first band also sums each block's
// rectangle sizes, scan_parts (in tile_scan_single's second workgroup) scans
// those block sums, and the scatter pass's first band writes goff.  The raster
// work items that split long tile lists come from tile_scan_single.
#include "plan.h"
#include "wsr_internal.h"

namespace wsr {
namespace {

constexpr int kBinWaves = kBinThreads / kWave;

// Inclusive sum over the lanes of a wave, in registers (DPP row shifts, then
// the row totals broadcast on).
__device__ __forceinline__ uint32_t wave_scan(uint32_t x) {
  x += __builtin_amdgcn_update_dpp(0u, x, 0x111, 0xf, 0xf, false);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0u, x, 0x112, 0xf, 0xf, false);  // row_shr:2
  x += __builtin_amdgcn_update_dpp(0u, x, 0x114, 0xf, 0xf, false);  // row_shr:4
  x += __builtin_amdgcn_update_dpp(0u, x, 0x118, 0xf, 0xf, false);  // row_shr:8
  x += __builtin_amdgcn_update_dpp(0u, x, 0x142, 0xa, 0xf, false);  // row_bcast:15 to rows 1, 3
  x += __builtin_amdgcn_update_dpp(0u, x, 0x143, 0xc, 0xf, false);  // row_bcast:31 to rows 2, 3
  return x;
}

// LDS writes of this wave before, LDS reads of this wave after.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

struct BinArgs {
  const DevCamera* cams;
  const uint2* rect;
  uint32_t* hist;              // block-major count matrix, then its column prefixes
  const uint32_t* tile_start;  // start of every tile's list (scatter pass)
  uint2* ent;                  // list entries (id, Gaussian-major slot)
  int64_t n;
  int64_t capacity;
  int32_t nblk;                // blocks per view
  int32_t chunk;               // Gaussians per block, a multiple of kBinThreads
  uint32_t* parts;             // per (view, block): sum of the rectangle sizes, then its exclusive scan
  uint32_t* goff;              // Gaussian-major first slot of every (view, Gaussian)
};

// One Gaussian's tile rectangle, whole and cut to a band of tile rows.
struct BinRect {
  uint32_t x0, w, y0, count;  // cut to the band: columns [x0, x0 + w), first row, tiles
  uint32_t full;              // tiles of the whole rectangle
  uint32_t first;             // row-major index of tile (0, 0) in it: y0 w + x0 of the whole, negated
};

__device__ __forceinline__ BinRect bin_rect(uint2 r, int ry0, int ry1) {
  BinRect b;
  const uint32_t x1 = r.x >> 16, y0 = r.y & 0xffffu, y1 = r.y >> 16;
  b.x0 = r.x & 0xffffu;
  b.w = x1 > b.x0 ? x1 - b.x0 : 0u;
  const int yl = max(static_cast<int>(y0), ry0), yh = min(static_cast<int>(y1), ry1);
  b.y0 = static_cast<uint32_t>(yl);
  b.count = yh > yl ? b.w * static_cast<uint32_t>(yh - yl) : 0u;
  b.full = y1 > y0 ? b.w * (y1 - y0) : 0u;
  b.first = 0u - (y0 * b.w + b.x0);
  return b;
}

// The pairs of a wave's 64 Gaussians (one rectangle per lane), in
// Gaussian-major order (a Gaussian's tiles row-major), 64 per step:
// f(valid, owner lane, tx, ty, w).  A pair's owner is the last Gaussian whose
// first pair is not behind it: the owners that begin in the step mark their
// place in `mark` (64 words of LDS of this wave's own).
template <typename F>
__device__ __forceinline__ void expand_pairs(const BinRect& r, uint32_t* mark, int lane, F&& f) {
  const uint32_t inc = wave_scan(r.count), off = inc - r.count;
  const uint32_t total = __builtin_amdgcn_readlane(inc, kWave - 1);
  const uint32_t span = r.x0 | (r.w << 16);
  int last = 0;  // owner of the previous step's last pair
  for (uint32_t p0 = 0; p0 < total; p0 += kWave) {
    mark[lane] = kWave;
    wave_lds_fence();
    if (r.count > 0 && off >= p0 && off - p0 < kWave) mark[off - p0] = lane;
    wave_lds_fence();
    const int here = static_cast<int>(mark[lane]);
    const uint64_t begun = __ballot(here < kWave) & ((2ull << lane) - 1ull);
    const int from = __shfl(here, begun ? 63 - __clzll(begun) : 0, kWave);
    const int owner = begun ? from : last;
    last = __builtin_amdgcn_readlane(owner, kWave - 1);
    const uint32_t p = p0 + lane;
    const bool valid = p < total;
    const uint32_t local = p - __shfl(off, owner, kWave);
    const uint32_t sp = __shfl(span, owner, kWave), y0 = __shfl(r.y0, owner, kWave);
    const uint32_t w = max(sp >> 16, 1u);
    // local / w: at most 4,096 rows, so the float quotient is within one of it
    int q = static_cast<int>(static_cast<float>(local) * __builtin_amdgcn_rcpf(static_cast<float>(w)));
    int rem = static_cast<int>(local) - q * static_cast<int>(w);
    if (rem < 0) {
      --q;
      rem += static_cast<int>(w);
    } else if (rem >= static_cast<int>(w)) {
      ++q;
      rem -= static_cast<int>(w);
    }
    f(valid, owner, (sp & 0xffffu) + static_cast<uint32_t>(rem), y0 + static_cast<uint32_t>(q), w);
  }
}

// Rectangles into a band's difference array d (rows x tiles_x, one word per
// tile): four corners each, whose two-dimensional prefix sums are the number of
// rectangles over every tile.  `one` is the unit to add (1, or 1 << 16 for a
// count kept in the upper half of the words; the sums are linear, so the
// halves do not mix in the end).
__device__ __forceinline__ void add_corners(uint32_t* d, const BinRect& r, int ry0, int ry1, int tiles_x, uint32_t one) {
  if (r.count == 0) return;
  const int top = (static_cast<int>(r.y0) - ry0) * tiles_x;
  const int bottom = top + static_cast<int>(r.count / r.w) * tiles_x;  // first row below
  const bool below = bottom < (ry1 - ry0) * tiles_x;
  const int left = static_cast<int>(r.x0), right = static_cast<int>(r.x0 + r.w);
  atomicAdd(&d[top + left], one);
  if (right < tiles_x) atomicAdd(&d[top + right], 0u - one);
  if (below) {
    atomicAdd(&d[bottom + left], 0u - one);
    if (right < tiles_x) atomicAdd(&d[bottom + right], one);
  }
}

// The prefix sums of NW difference arrays (contiguous, `tiles` words each), in
// place, by the whole workgroup: down the columns, then along the rows.
template <int NW>
__device__ __forceinline__ void prefix_counts(uint32_t* d, int tiles, int tiles_x, int wv, int lane) {
  const int rows = tiles / tiles_x;
  __syncthreads();
  for (int c = threadIdx.x; c < NW * tiles_x; c += kBinThreads) {
    uint32_t* col = d + c / tiles_x * tiles + c % tiles_x;
    uint32_t run = 0;
    for (int r = 0; r < rows; ++r) {
      run += col[r * tiles_x];
      col[r * tiles_x] = run;
    }
  }
  __syncthreads();
  for (int k = wv; k < NW * rows; k += kBinWaves) {
    uint32_t* row = d + k / rows * tiles + k % rows * tiles_x;
    uint32_t carry = 0;
    for (int x0 = 0; x0 < tiles_x; x0 += kWave) {
      const int x = x0 + lane;
      const uint32_t inc = wave_scan(x < tiles_x ? row[x] : 0u);
      if (x < tiles_x) row[x] = carry + inc;
      carry += __builtin_amdgcn_readlane(inc, kWave - 1);
    }
  }
  __syncthreads();
}

// Counting and scattering pass.  Every wave takes a quarter of the block's
// Gaussians.  Counting needs no pairs: a rectangle adds its four corners to a
// difference array in LDS, whose prefix sums are the counts.  The scatter
// counts each wave's pairs per tile in the same way, which gives each wave
// cursors of its own (16 bits per wave and tile, behind the block's 32-bit
// base), and then expands and places the pairs with no barrier between the
// waves.  (Before, every pair was expanded to be counted, its Gaussian found by
// binary search in LDS, and the waves took turns at one cursor per tile, four
// barriers per 256 pairs: at 1 M Gaussians / 1080p counting 43 instead of
// 18 us, scattering 130 us as before, at 200 k / 720p 21 and 45 instead of 7 and
// 23 us.)
//
// FEW: bands of at most kFewTiles tiles (see plan.h).
template <bool SCATTER, bool FEW>
__global__ __launch_bounds__(kBinThreads) void bin_pass(BinArgs a) {
  extern __shared__ uint32_t lds[];
  __shared__ uint32_t s_full[kBinWaves];

  // Workgroups go round the eight XCDs in turn.  Each XCD takes a contiguous
  // eighth of a view's blocks, band by band, so that the parts of a tile's list
  // that lie side by side are written through one L2 (the stage at 1 M
  // Gaussians / 1080p 175 -> 166 us, 16 views 1,398 -> 1,273 us; with a part of
  // the bands per XCD instead, whose loads differ, 203 and 1,475 us).
  const int b = blockIdx.x % 8 * (gridDim.x / 8) + blockIdx.x / 8, z = blockIdx.y, v = blockIdx.z;
  if (b >= a.nblk) return;
  const DevCamera& cam = a.cams[v];
  const int tiles_x = cam.tiles_x;
  const int tiles_v = cam.tiles_x * cam.tiles_y;
  const int rows = cam.band_rows, ry0 = z * rows;
  if (ry0 >= cam.tiles_y) return;
  const int ry1 = min(ry0 + rows, cam.tiles_y);
  const int chunk_tiles = (ry1 - ry0) * tiles_x;
  const int t0 = ry0 * tiles_x;  // first tile (view-local) of the band
  uint32_t* row = a.hist + cam.hist_base + static_cast<int64_t>(b) * tiles_v + t0;
  const int lane = threadIdx.x & (kWave - 1), wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);

  // count: one word per tile; scatter: two words of two counts each, then
  // cursors, and the block's base per tile
  constexpr int NW = SCATTER ? 2 : 1;
  uint32_t* counts = lds;
  uint32_t* base = lds + NW * chunk_tiles;
  for (int t = threadIdx.x; t < NW * chunk_tiles; t += kBinThreads) counts[t] = 0u;
  if (SCATTER)
    for (int t = threadIdx.x; t < chunk_tiles; t += kBinThreads) base[t] = a.tile_start[cam.tile_base + t0 + t] + row[t];
  __syncthreads();

  const int64_t g0 = static_cast<int64_t>(b) * a.chunk + static_cast<int64_t>(wv) * (a.chunk / kBinWaves);
  const int64_t g1 = min(g0 + a.chunk / kBinWaves, a.n);
  const uint2* rect = a.rect + static_cast<int64_t>(v) * a.n;
  const int64_t part = static_cast<int64_t>(v) * a.nblk + b;

  uint32_t full = 0;
  for (int64_t i = g0 + lane; i < g1; i += kWave) {
    const BinRect r = bin_rect(rect[i], ry0, ry1);
    full += r.full;
    add_corners(counts + (SCATTER ? (wv >> 1) * chunk_tiles : 0), r, ry0, ry1, tiles_x,
                SCATTER ? 1u << (16 * (wv & 1)) : 1u);
  }
  // (view, block) rectangle sums, for the Gaussian-major slots
  const uint32_t fsum = wave_scan(full);
  if (lane == kWave - 1) s_full[wv] = fsum;
  prefix_counts<NW>(counts, chunk_tiles, tiles_x, wv, lane);
  if constexpr (!SCATTER) {
    for (int t = threadIdx.x; t < chunk_tiles; t += kBinThreads) row[t] = counts[t];
    if (z == 0 && threadIdx.x == 0) a.parts[part] = s_full[0] + s_full[1] + s_full[2] + s_full[3];
  } else {
    __shared__ uint32_t s_mark[kBinWaves][kWave];
    __shared__ uint8_t s_tag[FEW ? 1 : kBinWaves][kTags];
    uint32_t* mark = s_mark[wv];
    uint8_t* tag = s_tag[FEW ? 0 : wv];
    const uint32_t pitch = cam.tag_pitch;
    // counts of waves 0 to 3 -> their first places
    for (int t = threadIdx.x; t < chunk_tiles; t += kBinThreads) {
      const uint32_t c0 = counts[t] & 0xffffu, c1 = counts[t] >> 16, c2 = counts[chunk_tiles + t] & 0xffffu;
      counts[t] = c0 << 16;
      counts[chunk_tiles + t] = (c0 + c1) | ((c0 + c1 + c2) << 16);
    }
    __syncthreads();
    uint32_t gcarry = a.parts[part];  // running Gaussian-major offset
    for (int w = 0; w < wv; ++w) gcarry += s_full[w];
    uint16_t* cursor = reinterpret_cast<uint16_t*>(counts + (wv >> 1) * chunk_tiles) + (wv & 1);  // tile t's: [2 t]
    auto load = [&](int64_t i) { return i < g1 ? rect[i] : make_uint2(0u, 0u); };
    uint2 next = load(g0 + lane);
    for (int64_t g = g0; g < g1; g += kWave) {
      const BinRect r = bin_rect(next, ry0, ry1);
      next = load(g + kWave + lane);
      const uint32_t finc = wave_scan(r.full);
      const uint32_t goff = gcarry + finc - r.full;
      gcarry += __builtin_amdgcn_readlane(finc, kWave - 1);
      if (z == 0 && g + lane < g1) a.goff[static_cast<int64_t>(v) * a.n + g + lane] = goff;
      const uint32_t gadj = goff + r.first;  // slot of tile (tx, ty): this + ty w + tx
      expand_pairs(r, mark, lane, [&](bool valid, int owner, uint32_t tx, uint32_t ty, uint32_t w) {
        // (24-bit products, at the full rate)
        const uint32_t tr = ty - ry0;
        const uint32_t t = valid ? __umul24(tr, tiles_x) + tx : 0u;
        const uint32_t slot = __shfl(gadj, owner, kWave) + __umul24(ty, w) + tx;
        // Stable rank among the step's pairs of the same tile, where lower
        // lanes hold earlier pairs.
        uint32_t at = 0, rank = 0;
        bool last = true;
        if constexpr (FEW) {
          uint64_t same = __ballot(valid);
#pragma unroll
          for (int k = 0; k < kFewBits; ++k) {
            const uint64_t ones = __ballot((t >> k) & 1u);
            same &= (t >> k) & 1u ? ones : ~ones;
          }
          rank = static_cast<uint32_t>(__popcll(same & ((1ull << lane) - 1ull)));
          last = (same >> lane) == 1ull;
          if (valid) at = base[t] + cursor[2 * t];
          wave_lds_fence();
        } else {
          // Every lane leaves its number at its tile's tag; those that find
          // another there share the tag, as a rule the tile, and their groups
          // are formed one by one.
          const uint32_t own = (__umul24(tr, pitch) + tx) % kTags;
          if (valid) tag[own] = static_cast<uint8_t>(lane);
          wave_lds_fence();
          if (valid) at = base[t] + cursor[2 * t];
          uint64_t left = __ballot(valid && tag[own] != lane);
          while (left) {
            const uint32_t tl = __builtin_amdgcn_readlane(t, __ffsll(static_cast<long long>(left)) - 1);
            const uint64_t same = __ballot(valid && t == tl);
            if (t == tl) {
              rank = static_cast<uint32_t>(__popcll(same & ((1ull << lane) - 1ull)));
              last = (same >> lane) == 1ull;
            }
            left &= ~same;
          }
        }
        if (valid) {
          const uint32_t pos = at + rank;
          if (pos < a.capacity) a.ent[pos] = make_uint2(static_cast<uint32_t>(g) + owner, slot);
          // the highest lane of its group moves the wave's cursor past the group
          if (last) cursor[2 * t] = static_cast<uint16_t>(at + rank + 1u - base[t]);
        }
        wave_lds_fence();
      });
    }
  }
}

// Column prefixes of the count matrix, 16 waves per 64 tiles: lane = tile (coalesced
// rows of the block-major matrix), wave w takes the w-th sixteenth of the
// blocks.  Pass 1 sums each wave's share, the waves' bases follow from LDS,
// pass 2 rewrites the share as exclusive prefixes.  Sixteen times the loads
// in flight of one thread per tile.
constexpr int kColWaves = 16;
__global__ __launch_bounds__(kColWaves * kWave) void column_scan_wide(const DevCamera* cams, int32_t nv,
                                                                      int32_t nblk, int64_t total_tiles,
                                                                      uint32_t* hist, uint32_t* tile_start) {
  __shared__ uint32_t s_sum[kColWaves][kWave];
  const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
  const int64_t t = static_cast<int64_t>(blockIdx.x) * kWave + lane;
  const bool ok = t < total_tiles;
  uint32_t* col = hist;
  int64_t tiles_v = 0;
  if (ok) {
    int v = 0;
    while (v + 1 < nv && cams[v + 1].tile_base <= t) ++v;
    const DevCamera& cam = cams[v];
    tiles_v = static_cast<int64_t>(cam.tiles_x) * cam.tiles_y;
    col = hist + cam.hist_base + (t - cam.tile_base);
  }
  const int b0 = static_cast<int>(static_cast<int64_t>(nblk) * wv / kColWaves);
  const int b1 = static_cast<int>(static_cast<int64_t>(nblk) * (wv + 1) / kColWaves);
  uint32_t sum = 0;
  if (ok)
    for (int b = b0; b < b1; ++b) sum += col[b * tiles_v];
  s_sum[wv][lane] = sum;
  __syncthreads();
  uint32_t run = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kColWaves; ++w) {
    const uint32_t x = s_sum[w][lane];
    if (w < wv) run += x;
    total += x;
  }
  if (ok) {
    for (int b = b0; b < b1; ++b) {
      const uint32_t c = col[b * tiles_v];
      col[b * tiles_v] = run;
      run += c;
    }
    if (wv == 0) tile_start[t] = total;
  }
  if (wv == 0 && t == total_tiles) tile_start[t] = 0u;
}

// Exclusive scan over a 1024-thread block of one value per thread; *total
// receives the block sum.  `sh` needs 16 words.
__device__ inline uint32_t block_scan_1024(uint32_t v, uint32_t* sh, uint32_t* total) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = threadIdx.x / kWave;
  uint32_t inc = v;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const uint32_t o = __shfl_up(inc, d, kWave);
    if (lane >= d) inc += o;
  }
  if (lane == kWave - 1) sh[wv] = inc;
  __syncthreads();
  uint32_t base = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const uint32_t x = sh[k];
    if (k < wv) base += x;
    tot += x;
  }
  __syncthreads();
  *total = tot;
  return base + inc - v;
}

// One workgroup, after the column prefixes: the exclusive scan of the tile
// totals in place (tile_start; 64-bit running total, so a pair count beyond
// 32 bits is detected), the overflow flags, the raster work items --
// max(1, ceil(list length / kItemSplats)) per tile -- with their exclusive
// scan (items[total_tiles] = number of items), and their dispatch order.
// One pass over the tiles forms the starts, the item counts and the order
// histogram; a second places the tiles in the order.
constexpr int kTileScanThreads = 1024;
constexpr int kTileScanPer = 8;
constexpr int kOrderBuckets = kItemSplats / 32 + 1;

// A tile's list length with both ends capped at the pair capacity.
__device__ __forceinline__ uint64_t capped_len(uint64_t a, uint64_t e, uint64_t cap) {
  a = a < cap ? a : cap;
  e = e < cap ? e : cap;
  return e > a ? e - a : 0;
}

// Bucket of a tile in the dispatch order, from its (capped) list length:
// longest last work item first.
__device__ __forceinline__ int order_bucket(uint64_t l) {
  const uint64_t last = l == 0 ? 0 : l - ((l - 1) / kItemSplats) * kItemSplats;  // in [1, kItemSplats]
  return kOrderBuckets - 1 - static_cast<int>(last / 32);
}

// Exclusive scan (in place) of the per-(view, block) rectangle sums, in
// (view, block) order, i.e. (view, Gaussian) order; the grand total goes to
// *total (goff's closing entry).
__device__ __forceinline__ void scan_parts(uint32_t* parts, int64_t nparts, uint32_t* total, uint32_t* sh) {
  const int lane = threadIdx.x & (kWave - 1);
  const int wv = threadIdx.x / kWave;
  uint64_t carry = 0;
  for (int64_t c0 = 0; c0 < nparts; c0 += 1024) {
    const int64_t j = c0 + threadIdx.x;
    const uint32_t v = j < nparts ? parts[j] : 0u;
    uint32_t inc = v;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const uint32_t o = __shfl_up(inc, d, kWave);
      if (lane >= d) inc += o;
    }
    if (lane == kWave - 1) sh[wv] = inc;
    __syncthreads();
    uint64_t before = 0, tot = 0;
    for (int k = 0; k < 16; ++k) {
      if (k < wv) before += sh[k];
      tot += sh[k];
    }
    if (j < nparts) parts[j] = static_cast<uint32_t>(carry + before + inc - v);
    carry += tot;
    __syncthreads();
  }
  if (threadIdx.x == 0) *total = static_cast<uint32_t>(carry);
}

// Dispatch order of the work items.  Items that hold a full kItemSplats
// splats run first (in tile order: dispatch slot i < F, F the number of such
// items, is tile t's full item i - (items[t] - t)); then every tile's last
// item, longest first: tile_order holds (tile, its list's first and end
// position, its number of items), what a raster workgroup needs to begin, by
// the length of that item, counting-sorted in buckets of 32 splats.  Heavy items start early,
// so the launch ends on short ones instead of waiting for a late heavy one.
// Only the order of execution changes (within a bucket it varies from run
// to run): every item writes the same outputs.
//
// The second workgroup runs scan_parts, which needs a launch of its own no more
// than it needs this kernel's results (the stage with 4,096, 90 k and 200 k
// (view, Gaussian) slots: 20.5, 29.1 and 46.0 us with two launches, 18.0, 26.4
// and 43.5 with one).
__global__ __launch_bounds__(kTileScanThreads) void tile_scan_single(uint32_t* tile_start, int64_t total_tiles,
                                                                     uint32_t* items, uint4* tile_order,
                                                                     DevFlags* flags, int64_t capacity,
                                                                     uint32_t* parts, int64_t nparts,
                                                                     uint32_t* total) {
  __shared__ uint32_t sh[16];
  __shared__ uint32_t bucket[kOrderBuckets];
  if (blockIdx.x == 1) {
    scan_parts(parts, nparts, total, sh);
    return;
  }
  for (int k = threadIdx.x; k < kOrderBuckets; k += kTileScanThreads) bucket[k] = 0u;
  const int64_t len = total_tiles + 1;
  const uint64_t cap = static_cast<uint64_t>(capacity);
  constexpr int64_t kChunk = static_cast<int64_t>(kTileScanThreads) * kTileScanPer;
  uint64_t carry = 0;
  uint32_t icarry = 0;
  for (int64_t c0 = 0; c0 < len; c0 += kChunk) {
    const int64_t base = c0 + static_cast<int64_t>(threadIdx.x) * kTileScanPer;
    uint32_t vals[kTileScanPer];
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kTileScanPer; ++k) {
      vals[k] = base + k < len ? tile_start[base + k] : 0u;
      s += vals[k];
    }
    uint32_t tot;
    uint64_t run = carry + block_scan_1024(s, sh, &tot);  // (its first barrier also orders the bucket clear)
    uint32_t icnt[kTileScanPer];
    uint32_t is = 0;
#pragma unroll
    for (int k = 0; k < kTileScanPer; ++k) {
      const int64_t t = base + k;
      if (t < len) tile_start[t] = static_cast<uint32_t>(run);
      icnt[k] = 0u;
      if (t < total_tiles) {
        // from the 32-bit starts as stored, which the placement pass reads
        const uint64_t l = capped_len(static_cast<uint32_t>(run), static_cast<uint32_t>(run + vals[k]), cap);
        icnt[k] = static_cast<uint32_t>(l == 0 ? 1 : (l + kItemSplats - 1) / kItemSplats);
        atomicAdd(&bucket[order_bucket(l)], 1u);
      }
      is += icnt[k];
      run += vals[k];
    }
    carry += tot;
    uint32_t itot;
    uint32_t irun = icarry + block_scan_1024(is, sh, &itot);
#pragma unroll
    for (int k = 0; k < kTileScanPer; ++k) {
      if (base + k < len) items[base + k] = irun;
      irun += icnt[k];
    }
    icarry += itot;
  }
  if (threadIdx.x == 0) {
    flags->total_pairs = carry;
    flags->wrapped = carry > 0xffffffffull ? 1u : 0u;
    flags->overflow = (carry > static_cast<uint64_t>(capacity) || carry > 0xffffffffull) ? 1u : 0u;
    flags->sort_overflow = 0u;
    flags->cull_masks = 0u;  // new lists: no culling masks yet
    uint32_t r = 0;
    for (int k = 0; k < kOrderBuckets; ++k) {
      const uint32_t c = bucket[k];
      bucket[k] = r;
      r += c;
    }
  }
  __syncthreads();  // the starts of every tile and the bucket offsets are in place
  for (int64_t t = threadIdx.x; t < total_tiles; t += kTileScanThreads) {
    const uint64_t a = tile_start[t], l = capped_len(a, tile_start[t + 1], cap);
    const uint64_t a0 = a < cap ? a : cap;
    tile_order[atomicAdd(&bucket[order_bucket(l)], 1u)] =
        make_uint4(static_cast<uint32_t>(t), static_cast<uint32_t>(a0), static_cast<uint32_t>(a0 + l),
                   static_cast<uint32_t>(l == 0 ? 1 : (l + kItemSplats - 1) / kItemSplats));
  }
}

}  // namespace

hipError_t launch_bin(const Layout& L, void* ws, void* pairs, int64_t capacity, hipStream_t st) {
  DevFlags* flags = at<DevFlags>(ws, L.off_flags);
  uint32_t* hist = at<uint32_t>(ws, L.off_hist);
  uint32_t* parts = at<uint32_t>(ws, L.off_scan);
  uint32_t* goff = at<uint32_t>(ws, L.off_goff);
  uint32_t* tstart = at<uint32_t>(ws, L.off_tstart);
  uint32_t* items = at<uint32_t>(ws, L.off_items);
  const PairView pv = pair_view(pairs, capacity);

  BinArgs a;
  a.cams = at<DevCamera>(ws, L.off_cams);
  a.rect = at<uint2>(ws, L.off_rect);
  a.hist = hist;
  a.tile_start = tstart;
  a.ent = pv.ent;
  a.n = L.n;
  a.capacity = capacity;
  a.nblk = L.nblk;
  a.parts = parts;
  a.goff = goff;
  a.chunk = L.bin_chunk;
  const size_t lds = static_cast<size_t>(L.band_tiles) * sizeof(uint32_t);
  const GridShape gs = bin_grid(L.nblk, L.bands, L.nv);
  const dim3 grid(gs.x, gs.y, gs.z);

  hipError_t e;
  bin_pass<false, false><<<grid, kBinThreads, lds, st>>>(a);
  column_scan_wide<<<static_cast<unsigned>((L.total_tiles + 1 + kWave - 1) / kWave), kColWaves * kWave, 0, st>>>(
      a.cams, L.nv, L.nblk, L.total_tiles, hist, tstart);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // one workgroup: tile starts, overflow flags and raster work items; a second
  // one: Gaussian-major offsets of the blocks (the counting pass summed each
  // block's rectangle sizes); the scatter pass writes goff
  tile_scan_single<<<2, kTileScanThreads, 0, st>>>(tstart, L.total_tiles, items, at<uint4>(ws, L.off_torder), flags,
                                                   capacity, parts, static_cast<int64_t>(L.nv) * L.nblk,
                                                   goff + L.n * L.nv);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (L.band_tiles <= kFewTiles)
    bin_pass<true, true><<<grid, kBinThreads, 3 * lds, st>>>(a);
  else
    bin_pass<true, false><<<grid, kBinThreads, 3 * lds, st>>>(a);
  return hipGetLastError();
}

}  // namespace wsr
