// host_pool.h -- the pinned host buffers that host transfers borrow.
//
// A transfer needs its buffer from the first array staged until the stream has been
// waited for, that is for less than one call, so the objects of a process share a few:
// an object that is created finds one ready or has it allocated then, beside its init,
// and no call allocates while fewer threads than buffers transfer at once.  (A buffer
// per object, allocated by its first transfer, made that call 30 - 45 us longer than the
// single copy it replaced, and held 1 MiB for each object.)  With the last object the
// idle buffers are freed.
#pragma once

#include <cstddef>
#include <mutex>

namespace eco {

// Every function may be called from any thread; none throws.
class HostPool {
 public:
  static constexpr int kMost = 8;   // buffers at once, borrowed ones included
  HostPool(size_t bytes, void* (*get)(size_t), void (*put)(void*)) : bytes_(bytes), get_(get), put_(put) {}

  // An object is there (from its creation to its end): one buffer stands ready.
  void join() {
    std::lock_guard<std::mutex> g(lock_);
    ++objects_;
    if (n_idle_ == 0) grow();
  }
  // It is gone, and gives back what it had borrowed first.
  void leave() {
    std::lock_guard<std::mutex> g(lock_);
    if (--objects_ > 0) return;
    total_ -= n_idle_;
    while (n_idle_ > 0) put_(idle_[--n_idle_]);
  }
  // A buffer for one transfer, null if there is none.
  void* take() {
    std::lock_guard<std::mutex> g(lock_);
    if (n_idle_ == 0) grow();
    return n_idle_ > 0 ? idle_[--n_idle_] : nullptr;
  }
  // Back, with nothing on the GPU that may still use it.
  void give(void* p) {
    std::lock_guard<std::mutex> g(lock_);
    idle_[n_idle_++] = p;
  }

 private:
  void grow() {
    if (total_ == kMost) return;
    if (void* p = get_(bytes_)) {
      idle_[n_idle_++] = p;
      ++total_;
    }
  }
  const size_t bytes_;
  void* (*const get_)(size_t);
  void (*const put_)(void*);
  std::mutex lock_;
  void* idle_[kMost] = {};
  int n_idle_ = 0, total_ = 0;
  long objects_ = 0;
};

}  // namespace eco
