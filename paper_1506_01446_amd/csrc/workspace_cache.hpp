// Workspaces of the digit and rank sorts (host code, no HIP: the allocator is a
// parameter, so the policy is tested on the CPU).
//
// A sort on stream S takes S's buffer.  Work on one stream is ordered, so the
// next sort on S may write the buffer as soon as it runs; a buffer that is
// replaced is freed in stream order, behind the work that uses it.  A buffer
// is lent to one call at a time: another thread that enqueues on the same
// stream meanwhile gets a buffer of its own, since its launches may fall
// between this call's.
//
// What is kept is bounded: at most kKeepBytes a stream, kKeepTotal and
// kKeepSlots in all.  A new stream takes the place of the idle one that has
// not sorted for longest.  Anything beyond is allocated for the one call and
// freed in stream order behind it, and a stream whose calls have long needed
// an eighth of its buffer or less gives it back for a smaller one.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <mutex>

namespace bitonic {

// Alloc: `void* alloc(int dev, void* stream, size_t bytes)` (nullptr on
// failure) and `bool free(int dev, void* stream, void* ptr)`, stream-ordered;
// for eviction, `bool stamp(int dev, void* stream, int slot, uint32_t value)`
// (enqueues a write of value to the slot's word) and `uint32_t stamped(int
// slot)` (the word as it is now).  The cache itself allocates nothing and
// throws nothing (it runs under C entries).
template <class Alloc>
class WorkspaceCache {
 public:
  static constexpr size_t kMinBytes = size_t(1) << 20;
  static constexpr size_t kKeepBytes = size_t(256) << 20;
  static constexpr size_t kKeepTotal = size_t(2) << 30;
  static constexpr size_t kKeepSlots = 32;
  static constexpr size_t kParkSlots = 32;
  static constexpr int kShrinkCalls = 64;
  // Above either, calls are stamped (crowded()).  A stamp is a launch of one
  // thread, 2.5 us of the host's time, where allocating and freeing a workspace
  // per call takes 17.
  static constexpr size_t kQuietSlots = 16;
  static constexpr size_t kQuietBytes = size_t(1) << 30;

  explicit WorkspaceCache(Alloc a = Alloc{}) : alloc_(a) {}

  // A buffer of at least `bytes` for work on (dev, stream), nullptr if there
  // is none to be had.  keep == false: never a kept one (a stream handle that
  // names another stream in every thread).  only_kept: none that would be
  // allocated and freed for this call.  Every buffer is given back with
  // release() once the call's work is enqueued.
  void* acquire(int dev, void* stream, size_t bytes, bool keep = true, bool only_kept = false) {
    std::lock_guard<std::mutex> lock(mu_);
    for (Slot& s : parked_) {
      // a buffer whose free failed: its stream's work is still ordered
      if (!s.ptr || s.dev != dev || s.stream != stream || s.lent || !keep) continue;
      if (s.bytes >= bytes) {
        s.lent = true;
        return s.ptr;
      }
      if (alloc_.free(dev, stream, s.ptr)) s = Slot{};
    }
    if (keep && bytes <= kKeepBytes) {
      Slot* s = find(dev, stream);
      if (s && !s->lent) {
        s->small = bytes <= s->bytes / 8 ? s->small + 1 : 0;
        if (s->bytes >= bytes && s->small < kShrinkCalls) {
          s->lent = true;
          return s->ptr;
        }
        const size_t want = rounded(bytes);
        s->lent = true;  // not to be evicted for itself
        const bool room = make_room(dev, stream, kept_ - s->bytes, want);
        s->lent = false;
        if (room) {
          if (void* p = alloc_.alloc(dev, stream, want)) {
            give_back(*s);
            kept_ += want - s->bytes;
            *s = Slot{dev, stream, p, want, 0, true, 0, ++calls_};
            return p;
          }
          if (s->bytes >= bytes) {
            s->lent = true;
            return s->ptr;
          }
          return nullptr;
        }
      } else if (!s) {
        const size_t want = rounded(bytes);
        if (make_room(dev, stream, kept_, want, true)) {
          Slot* const f = free_slot();
          void* p = alloc_.alloc(dev, stream, want);
          if (!p) return nullptr;
          *f = Slot{dev, stream, p, want, 0, true, 0, ++calls_};
          kept_ += want;
          return p;
        }
      }
    }
    return only_kept ? nullptr : alloc_.alloc(dev, stream, bytes);
  }

  // After the work that uses p is enqueued on (dev, stream).
  void release(int dev, void* stream, void* p, size_t bytes) {
    std::lock_guard<std::mutex> lock(mu_);
    for (Slot& s : slots_)
      if (s.ptr == p) {
        s.lent = false;
        s.used = ++calls_;
        s.stamp = crowded() ? stamp(s) : 0;
        return;
      }
    for (Slot& s : parked_)
      if (s.ptr == p) {
        s.lent = false;
        return;
      }
    give_back(Slot{dev, stream, p, bytes});
  }

  // Gives back every buffer that is not lent.  wait(dev) waits until the
  // device is idle; buffers of a device for which it fails stay.  Then
  // after(allocator) runs, under the lock too.  False if anything stayed.
  template <class Wait, class After>
  bool give_back_all(Wait wait, After after) {
    std::lock_guard<std::mutex> lock(mu_);
    bool all = true;
    auto sweep = [&](Slot& s, size_t counted) {
      if (!s.ptr || s.lent) return;
      // idle now, so it may be freed on the null stream: its own may be gone
      if (wait(s.dev) && alloc_.free(s.dev, nullptr, s.ptr)) {
        kept_ -= counted;
        s = Slot{};
      } else {
        all = false;
      }
    };
    for (Slot& s : slots_) sweep(s, s.bytes);
    for (Slot& s : parked_) sweep(s, 0);
    return after(alloc_) && all;
  }

  size_t kept_bytes() const { return kept_; }
  size_t kept_slots() const { return used(slots_); }
  size_t parked() const { return used(parked_); }
  Alloc& allocator() { return alloc_; }

 private:
  struct Slot {
    int dev = 0;
    void* stream = nullptr;
    void* ptr = nullptr;  // nullptr: no buffer
    size_t bytes = 0;
    int small = 0;  // calls in a row that needed an eighth or less
    bool lent = false;
    // what the slot's word becomes when its last call's work is done; 0: that
    // call was not stamped
    uint32_t stamp = 0;
    uint64_t used = 0;  // order of the slots' last calls
  };
  static size_t rounded(size_t bytes) {
    size_t w = kMinBytes;
    while (w < bytes) w *= 2;
    return w;
  }
  template <size_t N>
  static size_t used(const Slot (&list)[N]) {
    size_t n = 0;
    for (const Slot& s : list) n += s.ptr != nullptr;
    return n;
  }
  Slot* find(int dev, const void* stream) {
    for (Slot& s : slots_)
      if (s.ptr && s.dev == dev && s.stream == stream) return &s;
    return nullptr;
  }
  Slot* free_slot() {
    for (Slot& s : slots_)
      if (!s.ptr) return &s;
    return nullptr;
  }
  // A stream may have been destroyed since its last sort, so nothing is asked
  // of the streams of other slots: once many buffers are kept, a call on a kept
  // one ends with a write to host memory, behind its work, and a slot whose
  // write has arrived is idle.  Few streams, as most programs have, never pay
  // for it; the slots they leave behind are at most kQuietSlots and kQuietBytes.
  bool crowded() const { return used(slots_) > kQuietSlots || kept_ > kQuietBytes; }
  uint32_t stamp(Slot& s) {
    if constexpr (requires { alloc_.stamp(0, nullptr, 0, 0u); }) {
      if (++last_stamp_ == 0) ++last_stamp_;
      if (alloc_.stamp(s.dev, s.stream, (int)(&s - slots_), last_stamp_)) return last_stamp_;
    }
    return 0;
  }
  bool idle(const Slot& s) {
    if constexpr (requires { alloc_.stamped(0); })
      return s.stamp != 0 && alloc_.stamped((int)(&s - slots_)) == s.stamp;
    return false;
  }
  // Whether `want` more bytes (and with `slot`, one more slot) fit beside
  // `others` kept ones, after giving back, the longest unused first, as many
  // idle buffers of the device as that takes.  They are freed on `stream`,
  // where the caller is about to work.
  bool make_room(int dev, void* stream, size_t others, size_t want, bool slot = false) {
    while (others + want > kKeepTotal || (slot && !free_slot())) {
      Slot* v = nullptr;
      for (Slot& s : slots_)
        if (s.ptr && s.dev == dev && !s.lent && idle(s) && (!v || s.used < v->used)) v = &s;
      if (!v) return false;
      const Slot gone = *v;
      *v = Slot{};
      kept_ -= gone.bytes;
      others -= gone.bytes;
      Slot freed = gone;
      freed.stream = stream;
      give_back(freed);
    }
    return true;
  }
  void give_back(Slot s) {
    s.lent = false;
    if (alloc_.free(s.dev, s.stream, s.ptr)) return;
    for (Slot& f : parked_)
      if (!f.ptr) {
        f = s;
        return;
      }
    // more refused frees than can be kept account of: the buffer stays
    // allocated
  }

  Alloc alloc_;
  std::mutex mu_;
  Slot slots_[kKeepSlots];
  Slot parked_[kParkSlots];
  size_t kept_ = 0;
  uint64_t calls_ = 0;
  uint32_t last_stamp_ = 0;
};

}  // namespace bitonic
