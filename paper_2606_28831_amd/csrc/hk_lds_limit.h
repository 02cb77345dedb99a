// The dynamic-LDS limit of one kernel, raised as launches ask for more (host only).
#pragma once

#include <stddef.h>

#include <atomic>
#include <mutex>

namespace hk {

class LdsLimit {
 public:
  explicit LdsLimit(size_t granted) : granted_(granted) {}

  // set(bytes) when no earlier call granted as much.  The limit is set and recorded under one
  // lock: of two threads that raise it at once, the smaller one's set cannot come last.
  template <typename F>
  void raise(size_t bytes, F set) {
    if (bytes <= granted_.load(std::memory_order_acquire)) return;
    std::lock_guard<std::mutex> lk(mu_);
    if (bytes <= granted_.load(std::memory_order_relaxed)) return;
    set(bytes);
    granted_.store(bytes, std::memory_order_release);
  }

 private:
  std::mutex mu_;
  std::atomic<size_t> granted_;
};

}  // namespace hk
