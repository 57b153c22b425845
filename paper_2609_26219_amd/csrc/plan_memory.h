// Device memory of plans, and their upload.  Written over the few runtime calls it makes (Hip), so that it runs on a CPU
// against a simulated runtime.
#ifndef PKV_PLAN_MEMORY_H
#define PKV_PLAN_MEMORY_H

#include <stddef.h>
#include <stdint.h>

#include <cstddef>
#include <mutex>
#include <new>
#include <vector>

namespace pkv {

// Pieces cut from slabs: a resume's plan is 0.1-0.3 MB and lives for one
// restore, and an allocation of its own costs a hipMalloc and, when it is
// freed, a wait for everything the device still runs (hipFree).  Plans of more
// than a quarter slab, and plans that find no room for a slab, take an
// allocation of their own.
//
// A released piece is used again only after a device synchronisation that
// follows its release, so a plan that is freed while a launch still reads it
// stays readable, as with hipFree.  That synchronisation is made when no piece
// is left and the released ones add up to half a slab, so a plan that is kept
// holds back its own bytes and not its slab.  A slab but the newest is freed
// with its last plan, and all are when no plan of the device is left.
//
// No lock is held while memory is freed or copied, which may wait for the device.
template <typename Hip>
class PlanMemory {
 public:
  using Error = typename Hip::Error;
  static constexpr size_t kSlab = size_t(4) << 20;

  // On failure the runtime's last error is cleared: the status is the report.
  Error allocate(size_t bytes, void** out) {
    std::lock_guard<std::mutex> lock(mu_);
    Error e;
    try {
      e = place(bytes, out);
    } catch (const std::bad_alloc&) {
      e = Hip::kOutOfMemory;
    }
    if (e == Hip::kSuccess)
      ++plans_;
    else
      Hip::clear_error();
    return e;
  }

  void release(void* p) {
    void* gone = nullptr;     // an allocation of its own, or a slab without plans
    std::vector<Slab> slabs;  // every slab, with the last plan
    {
      std::lock_guard<std::mutex> lock(mu_);
      --plans_;
      size_t i = 0;
      while (i < slabs_.size() && !(p >= slabs_[i].base && p < slabs_[i].base + kSlab)) ++i;
      if (i == slabs_.size()) {
        gone = p;
      } else {
        Slab& s = slabs_[i];
        for (Piece& q : s.pieces)
          if (s.base + q.off == p) {
            q.state = State::kReleased;
            released_ += q.size;
          }
        if (--s.plans == 0 && i + 1 < slabs_.size()) {
          for (const Piece& q : s.pieces) released_ -= q.state == State::kReleased ? q.size : 0;
          gone = s.base;
          slabs_.erase(slabs_.begin() + std::ptrdiff_t(i));
        }
      }
      if (plans_ == 0) {
        slabs.swap(slabs_);
        released_ = 0;
      }
    }
    if (gone) Hip::free(gone);
    for (const Slab& s : slabs) Hip::free(s.base);
  }

  // Copy `bytes` of host memory to the device and wait for it, on a stream of
  // the library's own: the copy does not queue behind the restores that the
  // caller's streams still run.  A device reset ends that stream, so a copy
  // that fails is tried once more on a new one.
  Error upload(void* dst, const void* src, size_t bytes) {
    typename Hip::Stream tried = nullptr;
    Error e = Hip::kSuccess;
    for (int attempt = 0; attempt < 2; ++attempt) {
      typename Hip::Stream s = nullptr;
      {
        std::lock_guard<std::mutex> lock(stream_mu_);
        if (tried && stream_ == tried) stream_ = nullptr;
        if (!stream_ && (e = Hip::stream_create(&stream_)) != Hip::kSuccess) {
          stream_ = nullptr;
          break;
        }
        s = stream_;
      }
      e = Hip::copy(dst, src, bytes, s);
      if (e == Hip::kSuccess) e = Hip::stream_synchronize(s);
      if (e == Hip::kSuccess) return e;
      tried = s;
      Hip::clear_error();
    }
    Hip::clear_error();
    return e;
  }

 private:
  enum class State : uint32_t { kFree, kLive, kReleased };
  struct Piece {
    uint32_t off, size;
    State state;
  };
  struct Slab {
    char* base;
    int64_t plans;
    std::vector<Piece> pieces;  // ascending, the whole slab
  };

  Error place(size_t bytes, void** out) {
    if (bytes <= kSlab / 4) {
      const uint32_t size = uint32_t((bytes + 255) & ~size_t(255));
      if (cut(size, out)) return Hip::kSuccess;
      if (released_ >= kSlab / 2) {
        const Error e = reclaim();
        if (e != Hip::kSuccess) return e;
        if (cut(size, out)) return Hip::kSuccess;
      }
      slabs_.reserve(slabs_.size() + 1);
      Slab s{nullptr, 0, {Piece{0, uint32_t(kSlab), State::kFree}}};
      void* base = nullptr;
      if (Hip::malloc(&base, kSlab) == Hip::kSuccess) {
        s.base = static_cast<char*>(base);
        slabs_.push_back(std::move(s));
        return cut(size, out) ? Hip::kSuccess : Hip::kOutOfMemory;
      }
      Hip::clear_error();
      if (released_ > 0 && reclaim() == Hip::kSuccess && cut(size, out)) return Hip::kSuccess;
    }
    return Hip::malloc(out, bytes);
  }

  // The first free piece that `size` fits, newest slab first.
  bool cut(uint32_t size, void** out) {
    for (size_t i = slabs_.size(); i-- > 0;) {
      Slab& s = slabs_[i];
      for (size_t k = 0; k < s.pieces.size(); ++k) {
        if (s.pieces[k].state != State::kFree || s.pieces[k].size < size) continue;
        if (s.pieces[k].size > size) {
          const Piece rest{s.pieces[k].off + size, s.pieces[k].size - size, State::kFree};
          s.pieces.insert(s.pieces.begin() + std::ptrdiff_t(k + 1), rest);
        }
        s.pieces[k].size = size;
        s.pieces[k].state = State::kLive;
        ++s.plans;
        *out = s.base + s.pieces[k].off;
        return true;
      }
    }
    return false;
  }

  // Released pieces become free ones, neighbours as one.
  Error reclaim() {
    const Error e = Hip::device_synchronize();
    if (e != Hip::kSuccess) return e;
    for (Slab& s : slabs_) {
      size_t n = 0;
      for (Piece q : s.pieces) {
        if (q.state == State::kReleased) q.state = State::kFree;
        if (n > 0 && q.state == State::kFree && s.pieces[n - 1].state == State::kFree)
          s.pieces[n - 1].size += q.size;
        else
          s.pieces[n++] = q;
      }
      s.pieces.resize(n);
    }
    released_ = 0;
    return Hip::kSuccess;
  }

  std::mutex mu_;
  std::vector<Slab> slabs_;
  size_t released_ = 0;  // bytes released and not reclaimed
  int64_t plans_ = 0;    // plans that hold device memory
  std::mutex stream_mu_;
  typename Hip::Stream stream_ = nullptr;
};

}  // namespace pkv

#endif  // PKV_PLAN_MEMORY_H
