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

}  // namespace wsr
