// Device memory of a hierarchy.  A setup makes some 130 allocations and as many releases.  Each costs 1 us
// where the runtime holds a freed piece of that size, 10 to 40 us where it maps one again and about 250 us
// where the device's memory is new to the process (a third of the time of a 1.1M-row setup and its
// destruction).  The arrays a handle keeps therefore come from slabs that the handle owns, and the
// setup's temporary arrays are reused within that setup.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <vector>

namespace amgp {

// The handle's kept arrays: sub-allocated from slabs of 2 to 64 MB (each about as large as all
// before it together), arrays above a quarter of a slab on their own.  Released together.
class Arena {
 public:
  hipError_t alloc(void** p, size_t bytes) {
    const size_t need = (std::max<size_t>(bytes, 1) + 255) / 256 * 256;
    if (need > kMaxSlab / 4) {
      const hipError_t e = hipMalloc(p, need);
      if (e == hipSuccess) slabs_.push_back(Slab{static_cast<char*>(*p), need, need});
      return e;
    }
    for (Slab& s : slabs_)
      if (s.size - s.used >= need) return take(s, p, need);
    size_t size = std::max(need, std::min(kMaxSlab, std::max(kMinSlab, total_)));
    void* base = nullptr;
    hipError_t e = hipMalloc(&base, size);
    if (e != hipSuccess && size > need) {  // no room for a whole slab
      (void)hipGetLastError();
      size = need;
      e = hipMalloc(&base, size);
    }
    if (e != hipSuccess) return e;
    total_ += size;
    slabs_.push_back(Slab{static_cast<char*>(base), size, 0});
    return take(slabs_.back(), p, need);
  }
  bool owns(const void* p) const {
    for (const Slab& s : slabs_)
      if (p >= s.base && p < s.base + s.size) return true;
    return false;
  }
  void release() { rewind({}); }

  // How far the slabs are in use, and the return to that: later arrays are given back.
  std::vector<size_t> mark() const {
    std::vector<size_t> used;
    for (const Slab& s : slabs_) used.push_back(s.used);
    return used;
  }
  void rewind(const std::vector<size_t>& used) {
    while (slabs_.size() > used.size()) {
      hipFree(slabs_.back().base);
      slabs_.pop_back();
    }
    total_ = 0;
    for (size_t i = 0; i < slabs_.size(); ++i) {
      slabs_[i].used = used[i];
      if (slabs_[i].size <= kMaxSlab) total_ += slabs_[i].size;
    }
  }

 private:
  struct Slab {
    char* base;
    size_t size, used;
  };
  static constexpr size_t kMinSlab = size_t(2) << 20, kMaxSlab = size_t(64) << 20;
  static hipError_t take(Slab& s, void** p, size_t need) {
    *p = s.base + s.used;
    s.used += need;
    return hipSuccess;
  }
  std::vector<Slab> slabs_;
  size_t total_ = 0;
};

// For the duration of a setup (or a release) on this thread: kept arrays come from the handle's arena,
// released temporary arrays of up to 64 MB (512 MB in all) are kept for the setup's next ones of
// about their size.  All of a setup's work is on one stream, so an array is reused in the order of
// that stream.  Arrays still in use when the scope ends (the levels' CSR arrays) are the handle's.
class MemoryScope {
 public:
  explicit MemoryScope(Arena* arena) : arena_(arena), before_(current()) { current() = this; }
  ~MemoryScope() {
    for (Block& b : blocks_)
      if (!b.busy) hipFree(b.p);
    current() = before_;
  }
  MemoryScope(const MemoryScope&) = delete;
  MemoryScope& operator=(const MemoryScope&) = delete;

  static MemoryScope*& current() {
    static thread_local MemoryScope* scope = nullptr;
    return scope;
  }

  hipError_t keep(void** p, size_t bytes) {
    hipError_t e = arena_->alloc(p, bytes);
    if (e != hipSuccess && drop_idle()) e = arena_->alloc(p, bytes);
    return e;
  }

  hipError_t take(void** p, size_t bytes) {
    bytes = std::max<size_t>(bytes, 1);
    Block* best = nullptr;
    for (Block& b : blocks_)
      if (!b.busy && b.size >= bytes && b.size <= bytes + bytes / 4 + kSlack && (!best || b.size < best->size))
        best = &b;
    if (best) {
      best->busy = true;
      idle_ -= best->size;
      *p = best->p;
      return hipSuccess;
    }
    hipError_t e = hipMalloc(p, bytes);
    if (e != hipSuccess && drop_idle()) e = hipMalloc(p, bytes);
    if (e == hipSuccess) blocks_.push_back(Block{*p, bytes, true});
    return e;
  }

  // whether p is a block more than kSlack larger than the bytes that are in use of it
  bool outgrown(const void* p, size_t bytes) const {
    for (const Block& b : blocks_)
      if (b.p == p) return b.size > bytes + kSlack;
    return false;
  }

  void give(void* p) {
    if (!p || arena_->owns(p)) return;  // the arena's are released with the handle
    for (size_t i = 0; i < blocks_.size(); ++i) {
      Block& b = blocks_[i];
      if (b.p != p) continue;
      if (b.size <= kMaxBlock && idle_ + b.size <= kMaxIdle) {
        b.busy = false;
        idle_ += b.size;
        return;
      }
      blocks_.erase(blocks_.begin() + i);
      break;
    }
    hipFree(p);
  }

 private:
  struct Block {
    void* p;
    size_t size;
    bool busy;
  };
  static constexpr size_t kSlack = size_t(64) << 10, kMaxBlock = size_t(64) << 20, kMaxIdle = size_t(512) << 20;
  // After a refused request: give the idle arrays back; true when there were any, to try once more.
  bool drop_idle() {
    if (idle_ == 0) return false;
    (void)hipGetLastError();
    for (size_t i = blocks_.size(); i-- > 0;)
      if (!blocks_[i].busy) {
        hipFree(blocks_[i].p);
        blocks_.erase(blocks_.begin() + i);
      }
    idle_ = 0;
    return true;
  }
  Arena* arena_;
  MemoryScope* before_;
  std::vector<Block> blocks_;
  size_t idle_ = 0;
};

// An array the handle keeps; a temporary one; the release of either.
template <typename T>
hipError_t keep_malloc(T** p, size_t bytes) {
  MemoryScope* m = MemoryScope::current();
  return m ? m->keep(reinterpret_cast<void**>(p), bytes) : hipMalloc(reinterpret_cast<void**>(p), bytes);
}
template <typename T>
hipError_t temp_malloc(T** p, size_t bytes) {
  MemoryScope* m = MemoryScope::current();
  return m ? m->take(reinterpret_cast<void**>(p), bytes) : hipMalloc(reinterpret_cast<void**>(p), bytes);
}
inline void dev_free(void* p) {
  MemoryScope* m = MemoryScope::current();
  if (m)
    m->give(p);
  else
    hipFree(p);
}

// An array that outlives the setup, in a temporary one's block that is too large for it (by up to a
// quarter, see take): moved to memory of its own size, where there is room for it.
template <typename T>
hipError_t settle(hipStream_t s, T** p, size_t bytes) {
  MemoryScope* m = MemoryScope::current();
  if (!m || !m->outgrown(*p, bytes)) return hipSuccess;
  T* q = nullptr;
  if (keep_malloc(&q, bytes) != hipSuccess) {
    (void)hipGetLastError();
    return hipSuccess;
  }
  const hipError_t e = hipMemcpyAsync(q, *p, bytes, hipMemcpyDeviceToDevice, s);
  m->give(*p);
  *p = q;
  return e;
}

}  // namespace amgp
