// Device memory of one context under an optional byte budget, with the scratch of finished calls
// kept for the next call that borrows as much.  Bookkeeping only: Mem gets and puts the memory, so
// that a host-only test drives this code with a stub, under the sanitizers.
//
// Why keep any: a call's scratch otherwise costs more than its kernels (measured on one MI355X: the
// outputs of a 25-atom state 16.8 ms of which 2.0 ms kernels, a 12-atom Lindblad step with its 8.3
// GB Arnoldi space 260 ms of which 92 ms).
// What bounds it: kept blocks total at most keep_max bytes and kMaxKept blocks, oldest freed first.
// A block of kLarge bytes and more is kept only while half of the device is free, so that a program
// that fills the device finds nearly everything there (asking takes about 20 us, 2 % of all outputs
// of a 25-atom state with their 512 MiB of scratch, hence not for smaller blocks).  Registers, their
// workspaces and results are never kept.  All kept blocks are freed before the context's budget or a
// failed allocation refuses a request (its own kept blocks first, then through Mem::reclaim those of
// the process's other contexts on the device), and by trim().
#pragma once

#include <cstddef>
#include <mutex>

namespace rsv {

// Mem: bool get(size_t, void**); void put(void*); void wait() (until nothing runs on the device);
// bool half_free() (half of the device's memory is free); void reclaim() (trims the other pools).
template <class Mem>
class ScratchPool {
 public:
  enum Status { kOk, kOverBudget, kNoMemory };
  static constexpr size_t kMaxKept = 32, kLarge = size_t(1) << 30;

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
    void* out[kMaxKept + 1];
    size_t n_out = 0;
    {
      std::lock_guard<std::mutex> lk(mu_);
      in_use_ -= bytes;
      if (keep) {
        while (n_kept_ == kMaxKept || kept_bytes_ + size > keep_max_) out[n_out++] = drop(0);
        kept_[n_kept_++] = Kept{p, size};
        kept_bytes_ += size;
      } else {
        out[n_out++] = p;
      }
    }
    for (size_t i = 0; i < n_out; ++i) mem_.put(out[i]);
  }

  // Frees every kept block; returns their bytes.
  size_t trim() {
    void* out[kMaxKept];
    size_t n_out = 0, bytes = 0;
    {
      std::lock_guard<std::mutex> lk(mu_);
      bytes = kept_bytes_;
      while (n_kept_ > 0) out[n_out++] = drop(n_kept_ - 1);
    }
    for (size_t i = 0; i < n_out; ++i) mem_.put(out[i]);
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
  // Takes kept block i out of the list (mu_ held).
  void* drop(size_t i) {
    void* p = kept_[i].p;
    kept_bytes_ -= kept_[i].size;
    for (--n_kept_; i < n_kept_; ++i) kept_[i] = kept_[i + 1];
    return p;
  }
  // Borrowed blocks are got, kept and matched by this size.
  static size_t block_size(size_t bytes) { return (bytes + 4095) / 4096 * 4096; }

  Status take(size_t bytes, size_t size, bool reuse, void** p) {
    *p = nullptr;
    bool squeeze = false;
    {
      std::lock_guard<std::mutex> lk(mu_);
      if (budget_ && (bytes > budget_ || in_use_ > budget_ - bytes)) return kOverBudget;
      in_use_ += bytes;
      for (size_t i = reuse ? n_kept_ : 0; i-- > 0;) {
        if (kept_[i].size != size) continue;
        *p = drop(i);
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
  size_t in_use_ = 0, kept_bytes_ = 0, n_kept_ = 0;
  Kept kept_[kMaxKept];  // oldest first
  mutable std::mutex mu_;
};

}  // namespace rsv
