// The store of released device blocks: which block an allocation gets, which
// ones go when the store is full, and what happens when the device is.  No HIP
// calls here: getting and giving back memory are the caller's functions.
#pragma once
#include <stddef.h>

#include <mutex>

namespace famsa {

// Device blocks of kKeptLeast to kKeptBlock bytes are kept when they are
// released and handed to later allocations of about their size: getting and
// giving back such a block takes the driver 0.1 to 0.4 ms, more than many
// calls' work.  The store holds at most kKeptBytes in kKeptCount blocks, over
// all devices.
constexpr size_t kKeptBytes = 512u << 20, kKeptBlock = 256u << 20, kKeptLeast = 1u << 20;
constexpr size_t kKeptCount = 16;

struct KeptBlock {
  void* p;
  size_t bytes;
  int device;
};

class KeptStore {  // any thread; nothing here allocates host memory
 public:
  size_t held(int device) {
    std::lock_guard<std::mutex> lock(mu_);
    size_t n = 0;
    for (size_t i = 0; i < n_; ++i) n += b_[i].device == device ? b_[i].bytes : 0;
    return n;
  }
  // The smallest block that holds `bytes` and is at most an eighth larger (an
  // object's memory is reported and budgeted by its blocks' own sizes).
  bool take(int device, size_t bytes, KeptBlock* out) {
    std::lock_guard<std::mutex> lock(mu_);
    size_t best = n_;
    for (size_t i = 0; i < n_; ++i)
      if (b_[i].device == device && b_[i].bytes >= bytes && b_[i].bytes - bytes <= bytes / 8 &&
          (best == n_ || b_[i].bytes < b_[best].bytes))
        best = i;
    if (best == n_) return false;
    *out = b_[best];
    drop(best);
    return true;
  }
  // Keeps a block that no work uses any more, or frees it; the oldest blocks
  // go where the store would hold too much.
  template <class Free>
  void put(const KeptBlock& b, Free&& give_back) {
    if (b.bytes < kKeptLeast || b.bytes > kKeptBlock) return give_back(b);
    std::lock_guard<std::mutex> lock(mu_);
    b_[n_++] = b;
    size_t total = 0;
    for (size_t i = 0; i < n_; ++i) total += b_[i].bytes;
    while (total > kKeptBytes || n_ > kKeptCount) {
      const KeptBlock old = b_[0];
      total -= old.bytes;
      drop(0);
      give_back(old);
    }
  }
  // Frees every block of one device (every block: device < 0).
  template <class Free>
  void empty(int device, Free&& give_back) {
    std::lock_guard<std::mutex> lock(mu_);
    for (size_t i = n_; i-- > 0;)
      if (device < 0 || b_[i].device == device) {
        const KeptBlock old = b_[i];
        drop(i);
        give_back(old);
      }
  }
  // A block for `bytes`: a kept one (if `kept`), or get(bytes, &p); where the
  // device has no room for it (get returns no_room), once more after the
  // device's blocks are given back.
  template <class Get, class Free>
  int allocate(int device, size_t bytes, bool kept, int no_room, Get&& get, Free&& give_back, KeptBlock* out) {
    if (kept && bytes >= kKeptLeast && take(device, bytes, out)) return 0;
    *out = KeptBlock{nullptr, bytes, device};
    int e = get(bytes, &out->p);
    if (e == no_room && held(device)) {
      empty(device, give_back);
      e = get(bytes, &out->p);
    }
    return e;
  }

 private:
  void drop(size_t i) {
    for (--n_; i < n_; ++i) b_[i] = b_[i + 1];
  }
  std::mutex mu_;
  KeptBlock b_[kKeptCount + 1];  // oldest first
  size_t n_ = 0;
};

}  // namespace famsa
