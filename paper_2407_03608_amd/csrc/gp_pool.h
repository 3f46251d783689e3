// Idle resources kept for reuse within the process, by device (host code).
#pragma once

#include <cstddef>
#include <mutex>
#include <utility>
#include <vector>

namespace gp {

// At most `most` idle ones in all; safe with several threads.  A resource is in
// the pool or with one caller, never both.
template <class R>
class IdlePool {
 public:
  explicit IdlePool(size_t most) : most_(most) {}
  // An idle resource of the device into *r; false: there is none.
  bool take(int device, R* r) {
    std::lock_guard<std::mutex> lk(mu_);
    for (size_t i = idle_.size(); i-- > 0;)
      if (idle_[i].first == device) {
        *r = idle_[i].second;
        idle_.erase(idle_.begin() + (std::ptrdiff_t)i);
        return true;
      }
    return false;
  }
  // Gives r back; false: the pool is full and r stays the caller's.
  bool put(int device, const R& r) {
    std::lock_guard<std::mutex> lk(mu_);
    if (idle_.size() >= most_) return false;
    idle_.emplace_back(device, r);
    return true;
  }

 private:
  const size_t most_;
  std::mutex mu_;
  std::vector<std::pair<int, R>> idle_;
};

}  // namespace gp
