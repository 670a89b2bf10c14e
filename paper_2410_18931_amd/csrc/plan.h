// Launch shapes that follow from the caller's sizes alone.  Plain C++, so that
// the rules can be checked over their whole range without a GPU.
#pragma once
#include <algorithm>
#include <cstdint>

namespace wsr {

// Workgroups of a launch.  In each dimension workgroups times threads stay
// below 2^32, more than which the runtime refuses.
struct GridShape {
  uint32_t x, y, z;
};

// Gaussians per binning block: the fewest, 256 to 2,048, with at most kBinBlocks
// blocks a view and a count matrix (blocks x tiles) of at most kBinSmall
// entries.  With few Gaussians or tiles a block's serial expansion is the whole
// pass and wants to be short (4,096 Gaussians at 128 x 128: 43 us of binning
// passes in blocks of 2,048, 10 us in blocks of 256); with many the matrix's
// traffic grows with the blocks (1 M Gaussians at 1080p: the stage takes 175 us
// in blocks of 2,048, 206 us in blocks of 1,024, 177 us in blocks of 4,096).
// 200 k Gaussians at 1280 x 720 and 300 k at 1001 x 747 take 49 and 55 us with
// the line here, 54 and 56 us with it at half and 53 and 67 us at twice as many
// entries.  A column of the matrix is a serial chain over the blocks, which a
// small image has nothing to hide behind: the stage for 500 k Gaussians at
// 128 x 128 takes 50, 52 and 67 us with at most 256, 512 and 1,024 blocks
// (101 without a limit, 63 in blocks of 2,048 throughout), for 300 k in twelve
// views of 200 x 133 166, 177 and 211 us.  With one view, blocks of 2,048 leave
// the chip idle, and up to kBinBlocksFull blocks of 1,024 are better (300 k at
// 1001 x 747, 293 blocks: 53.2 us and 55.4 in blocks of 2,048).
//
// Where a view's part of the matrix has more than kBinLarge entries even so, what
// a block does for every tile (its counts, their prefix sums, its row of the
// matrix) is most of the stage, and blocks of 4,096 halve it: 1 M Gaussians at
// 3840 x 2160 and tiles 16 and 8 386 -> 340 and 1,466 -> 1,117 us (372 and 1,907
// before rectangles were counted by their corners), at 7680 x 4320 and tile 16
// 1,470 -> 1,113 us.
constexpr int32_t kBinChunkMin = 256, kBinChunkMax = 2048, kBinChunkLarge = 4096;
constexpr int64_t kBinSmall = 1 << 20, kBinLarge = 12 << 20, kBinBlocks = 256, kBinBlocksFull = 320;

inline int64_t bin_blocks(int64_t n, int64_t chunk) { return n > 0 ? (n + chunk - 1) / chunk : 1; }

// tiles: of all views; largest: of the view that has most
inline int32_t bin_chunk(int64_t n, int64_t views, int64_t tiles, int64_t largest) {
  int32_t chunk = kBinChunkMin;
  auto most = [&] { return views == 1 && 2 * chunk == kBinChunkMax ? kBinBlocksFull : kBinBlocks; };
  while (chunk < kBinChunkMax && (bin_blocks(n, chunk) > most() || bin_blocks(n, chunk) * tiles > kBinSmall))
    chunk *= 2;
  if (chunk == kBinChunkMax && bin_blocks(n, chunk) * largest > kBinLarge) chunk = kBinChunkLarge;
  return chunk;
}

// Entries to hold the count matrix of every Gaussian count up to n: a workspace
// never holds fewer Gaussians than it was sized for.
inline int64_t bin_matrix_room(int64_t n, int64_t tiles, int64_t largest) {
  const int64_t small = std::min(bin_blocks(n, kBinChunkMin) * tiles, kBinSmall);
  const int64_t most = std::min(bin_blocks(n, kBinChunkMax), kBinLarge / largest);
  return std::max({small, most * tiles, bin_blocks(n, kBinChunkLarge) * tiles});
}

// Binning passes: x the blocks of a view, rounded up to whole eighths (one for
// each XCD), y the bands, z the views.  Workgroups start with x fastest, so
// eight neighbours go to the eight XCDs.
constexpr int kBinThreads = 256;
inline GridShape bin_grid(int64_t nblk, int64_t bands, int64_t nv) {
  return {static_cast<uint32_t>((nblk + 7) / 8 * 8), static_cast<uint32_t>(bands), static_cast<uint32_t>(nv)};
}

// Tile rows of a band of a view: at most kTileChunk tiles, which share the
// scatter's LDS at 12 bytes each (57 KB), and at least kBinBands bands for the
// tallest view: each block then expands only the pairs of its band, and the more
// blocks keep more of the chip busy (the stage at 1 M Gaussians / 1080p,
// 200 k / 720p, 300 k / 1001 x 747 and 16 views: 166, 48, 52 and 1,273 us with
// 4 bands, 161, 46, 52 and 1,267 us with 6, 161, 47, 58 and 1,264 us with 8,
// 165, 52, 62 and 1,352 us with 12).  The first limit is each view's own: a wide
// view beside a tall one must not cut the tall one into bands of one row.
constexpr int32_t kTileChunk = 4864, kBinBands = 6;
constexpr int32_t bin_rows(int32_t tiles_x, int32_t max_tiles_y) {
  const int32_t fit = kTileChunk / tiles_x, even = (max_tiles_y + kBinBands - 1) / kBinBands;
  return fit < 1 ? 1 : fit < even ? fit : even;
}

// In bands of at most kFewTiles tiles many of a scatter step's 64 pairs share a
// tile, and the lanes of each tile are found bit by bit of its number, in
// kFewBits ballots, instead of tile by tile (300 k Gaussians in twelve views of
// 200 x 133, bands of 26 tiles: the stage 171 us tile by tile, 158 bit by bit;
// 100 k in 64 views of 128 x 128, 16 tiles: 322 and 292; with 33 to 64 tiles both
// are level).
constexpr int32_t kFewBits = 5, kFewTiles = 1 << kFewBits;

// Tag of a band's tile, by which the lanes of a scatter step that place pairs in
// one tile find each other.  Tiles may share a tag, but every shared one is a
// step of its own, so the tags of the pairs that one splat has in a step, up to
// 64 tiles of its rectangle row by row, are kept apart: the k-th row after one
// lies k pitches further on, modulo the number of tags, and as both are in the
// step only if a row has fewer than 64 / (k - 1) tiles, as many tags between them
// are enough.  The pitch is the view's width where that holds, which spreads a
// band's tiles best, and else the next larger one where it does.  Among the widths
// where it does not hold are the powers of two (1 M Gaussians, the stage at
// 2048 x 1024 and tile 8, 4096 x 2160 and tiles 16 and 8, 8192 x 4320 and tile 8:
// 443, 481, 2,472 and 10,451 us with tags by width, 328, 353, 1,147 and 4,784 now).
// A pitch of 67 throughout costs 149 instead of 142 us at 1080p, where a band's 12
// rows of 120 tiles then share 857 tags.
constexpr uint32_t kTags = 1024;
constexpr uint32_t bin_tag(uint32_t row, uint32_t col, uint32_t pitch) { return (row * pitch + col) % kTags; }

inline int32_t bin_tag_pitch(int32_t tiles_x) {
  auto apart = [&](int32_t pitch) {
    for (int32_t k = 1; k < 64; ++k) {
      const int32_t far = k * pitch % static_cast<int32_t>(kTags);
      const int32_t gap = std::min(far, static_cast<int32_t>(kTags) - far);
      if (gap < std::min(tiles_x, k == 1 ? 64 : 63 / (k - 1))) return false;
    }
    return true;
  };
  int32_t pitch = tiles_x;
  while (!apart(pitch)) ++pitch;
  return pitch;
}

// Pair sums: three lanes for each of `slots` (view, Gaussian)s, in rows of at
// most 2^22 workgroups.
constexpr int kSumPerWave = 64 / 3;  // Gaussians of a wave
constexpr int kSumWaves = 4;
inline GridShape sum_grid(int64_t slots) {
  constexpr int64_t kPerBlock = kSumWaves * kSumPerWave, kRow = int64_t{1} << 22;
  const int64_t blocks = (slots + kPerBlock - 1) / kPerBlock;
  const int64_t rows = (blocks + kRow - 1) / kRow;
  return {static_cast<uint32_t>(blocks < kRow ? blocks : kRow), static_cast<uint32_t>(rows), 1u};
}

// The loss of a launch's views in strips instead of tiles (see train.hip).  The
// strips' time hardly depends on their number while every compute unit has at
// most one, and then steps up; the tiles' grows with theirs.  Both passes, us,
// tiles and strips: 640 x 705 (1,800 tiles, 210 strips) 48 / 53, four views of
// 400 x 300 (1,900, 252) 51 / 53, 705 x 700 (1,980, 252) 61 / 53, 960 x 540
// (2,040, 240) 58 / 53, 97 x 4700 (2,058, 278) 54 / 61, 800 x 720 (2,250, 286)
// 59 / 61, 97 x 5700 (2,499, 336) 64 / 61, 1280 x 720 (3,600, 440) 84 / 64.
// Views that fill their strips badly stay with tiles: lanes would idle, and the
// workspace has room for the shares of the tiles.
constexpr int32_t kLossTile = 16, kStripCols = 64, kStripRows = 34;
constexpr int64_t kStripTiles = 1950, kStripTilesMore = 2300, kStripUnits = 256;
constexpr bool loss_in_strips(int64_t tiles, int64_t strips, int64_t pixels) {
  return tiles >= (strips <= kStripUnits ? kStripTiles : kStripTilesMore) &&
         2 * kStripCols * kStripRows * strips <= 3 * pixels;
}

}  // namespace wsr
