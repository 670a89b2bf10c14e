// Small page-locked buffers, one for each thread that reads status words.
//
// A thread takes a slot at its first read and gives it back when it ends.  The
// slots lie in one page that is allocated for the first of them and stays until
// the process ends: freeing it when a thread ends would be a call into the
// runtime that can wait for the device's work and break a stream capture of
// another thread.  While kSlots threads hold all of them, the others get none
// and copy to memory of their own.  Plain C++; the caller brings the allocation.
#pragma once
#include <cstddef>
#include <cstdint>
#include <mutex>

namespace wsr {

class StatusSlots {
 public:
  static constexpr int kSlots = 64;
  static constexpr size_t kSlotBytes = 64;

  // The process's slots; never destroyed, since threads may outlive static objects.
  static StatusSlots& process() {
    static StatusSlots* slots = new StatusSlots;
    return *slots;
  }

  // A slot, or null if there is none; alloc(bytes) returns the page or null.
  template <typename Alloc>
  void* take(Alloc&& alloc) {
    std::lock_guard<std::mutex> lock(mutex_);
    if (!page_) page_ = static_cast<char*>(alloc(kSlots * kSlotBytes));
    if (!page_ || free_ == 0) return nullptr;
    const int k = __builtin_ctzll(free_);
    free_ &= free_ - 1;
    return page_ + k * kSlotBytes;
  }

  void give(void* slot) {
    std::lock_guard<std::mutex> lock(mutex_);
    free_ |= 1ull << (static_cast<size_t>(static_cast<char*>(slot) - page_) / kSlotBytes);
  }

 private:
  std::mutex mutex_;
  char* page_ = nullptr;
  uint64_t free_ = ~0ull;  // one bit per slot
};

}  // namespace wsr
