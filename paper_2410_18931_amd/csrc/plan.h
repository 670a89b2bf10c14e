// Launch shapes that follow from the caller's sizes alone.  Plain C++, so that
// the rules can be checked over their whole range without a GPU.
#pragma once
#include <cstdint>

namespace wsr {

// Workgroups of a launch.  In each dimension workgroups times threads stay
// below 2^32, more than which the runtime refuses.
struct GridShape {
  uint32_t x, y, z;
};

// Binning passes: x the blocks of a view, rounded up to whole eighths (one for
// each XCD), y the bands, z the views.  Workgroups start with x fastest, so
// eight neighbours go to the eight XCDs.
constexpr int kBinThreads = 256;
inline GridShape bin_grid(int64_t nblk, int64_t bands, int64_t nv) {
  return {static_cast<uint32_t>((nblk + 7) / 8 * 8), static_cast<uint32_t>(bands), static_cast<uint32_t>(nv)};
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

}  // namespace wsr
