// Device memory of one context under an optional byte budget, with the scratch of finished calls
// kept for the next call that borrows as much.  Bookkeeping only: Mem gets and puts the memory, so
// that a host-only test drives this code with a stub, under the sanitizers.
//
// Why keep any: a call's scratch otherwise costs more than its kernels (measured on one MI355X: the
// outputs of a 25-atom state 16.8 ms of which 2.0 ms kernels, a 12-atom Lindblad step with its 8.3
// GB Arnoldi space 260 ms of which 92 ms).
// What bounds it: kept blocks total at most keep_max bytes and kMaxKept blocks, oldest freed first.
// A block of kLarge bytes and more is kept only while half of the device is free, so that a program
// that fills the device finds everything there.  Registers, their workspaces and results are never
// kept.  All kept blocks are freed before the context's budget or a failed allocation refuses a
// request (its own kept blocks first, then through Mem::reclaim those of the process's other
// contexts on the device), and by trim().
#pragma once

#include <cstddef>
#include <mutex>
#include <vector>

namespace rsv {

// Mem: bool get(size_t, void**); void put(void*); void wait() (until nothing runs on the device);
// bool half_free() (half of the device's memory is free); void reclaim() (trims the other pools).
template <class Mem>
class ScratchPool {
 public:
  enum Status { kOk, kOverBudget, kNoMemory };
  static constexpr size_t kMaxKept = 32, kLarge = size_t(64) << 20;

  ScratchPool(size_t budget, size_t keep_max, Mem mem) : mem_(mem), budget_(budget), keep_max_(keep_max) {}
  ~ScratchPool() { trim(); }

  Status alloc(size_t bytes, void** p) { return take(bytes, bytes, false, p); }
  void release(void* p, size_t bytes) {
    if (!p) return;
    mem_.put(p);
    std::lock_guard<std::mutex> lk(mu_);
    in_use_ -= bytes;
  }

  // Memory for one call.  idle: the caller has waited for every kernel and copy that used the
  // block (a kept one may next be used on another stream).
  Status borrow(size_t bytes, void** p) { return take(bytes, block_size(bytes), true, p); }
  void give_back(void* p, size_t bytes, bool idle) {
    if (!p) return;
    if (!idle) mem_.wait();
    const size_t size = block_size(bytes);
    const bool keep = size <= keep_max_ && (size < kLarge || mem_.half_free());
    std::vector<void*> out;
    {
      std::lock_guard<std::mutex> lk(mu_);
      in_use_ -= bytes;
      if (keep) {
        kept_.push_back(Kept{p, size});
        kept_bytes_ += size;
      } else {
        out.push_back(p);
      }
      while (kept_bytes_ > keep_max_ || kept_.size() > kMaxKept) {
        out.push_back(kept_.front().p);
        kept_bytes_ -= kept_.front().size;
        kept_.erase(kept_.begin());
      }
    }
    for (void* q : out) mem_.put(q);
  }

  // Frees every kept block; returns their bytes.
  size_t trim() {
    std::vector<Kept> out;
    size_t bytes = 0;
    {
      std::lock_guard<std::mutex> lk(mu_);
      out.swap(kept_);
      bytes = kept_bytes_;
      kept_bytes_ = 0;
    }
    for (const Kept& k : out) mem_.put(k.p);
    return bytes;
  }
  size_t in_use() const {
    std::lock_guard<std::mutex> lk(mu_);
    return in_use_;
  }

 private:
  struct Kept {
    void* p;
    size_t size;
  };
  // Borrowed blocks are got, kept and matched by this size.
  static size_t block_size(size_t bytes) { return (bytes + 4095) / 4096 * 4096; }

  Status take(size_t bytes, size_t size, bool reuse, void** p) {
    *p = nullptr;
    bool squeeze = false;
    {
      std::lock_guard<std::mutex> lk(mu_);
      if (budget_ && (bytes > budget_ || in_use_ > budget_ - bytes)) return kOverBudget;
      in_use_ += bytes;
      for (size_t i = reuse ? kept_.size() : 0; i-- > 0;) {
        if (kept_[i].size != size) continue;
        *p = kept_[i].p;
        kept_bytes_ -= size;
        kept_.erase(kept_.begin() + i);
        return kOk;
      }
      squeeze = budget_ && in_use_ + kept_bytes_ > budget_;
    }
    if (squeeze) trim();  // the budget bounds what the context holds, kept blocks included
    if (mem_.get(size, p)) return kOk;
    trim();
    if (mem_.get(size, p)) return kOk;
    mem_.reclaim();
    if (mem_.get(size, p)) return kOk;
    *p = nullptr;
    std::lock_guard<std::mutex> lk(mu_);
    in_use_ -= bytes;
    return kNoMemory;
  }

  Mem mem_;
  const size_t budget_, keep_max_;
  size_t in_use_ = 0, kept_bytes_ = 0;
  std::vector<Kept> kept_;  // oldest first
  mutable std::mutex mu_;
};

}  // namespace rsv
