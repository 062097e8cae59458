// Slots of host memory that polls of device words copy into.  A call takes one
// from before its copy until it has read the words, so that calls on other
// threads and streams of the device never write there meanwhile.  Host only.
#pragma once

#include <stdint.h>

#include <atomic>

namespace ens {

class PollSlots {
 public:
  static constexpr int kSlots = 64;   // polls in flight at once on a device
  static constexpr int kBytes = 128;  // a word for each of the 32 streams of the concurrent baseline

  // The lowest free slot, -1 when all are taken.
  int take() {
    uint64_t used = used_.load(std::memory_order_relaxed);
    while (~used) {
      const int i = __builtin_ctzll(~used);
      if (used_.compare_exchange_weak(used, used | (1ull << i), std::memory_order_acquire,
                                      std::memory_order_relaxed))
        return i;
    }
    return -1;
  }
  void give(int i) { used_.fetch_and(~(1ull << i), std::memory_order_release); }

 private:
  std::atomic<uint64_t> used_{0};
};

}  // namespace ens
