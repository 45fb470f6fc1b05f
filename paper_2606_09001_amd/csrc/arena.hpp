// Device memory handed out from a few slabs.  No HIP in here: Mem supplies
//   static char* take(size_t bytes, bool must)  null when out of memory, unless `must` (then it throws)
//   static void give(char* p)
// and the CPU tests run it over host memory.
#pragma once

#include <algorithm>
#include <cstddef>
#include <vector>

namespace amg {

// A setup makes over 200 buffers; each its own hipMalloc and synchronizing
// hipFree they took 19 of the 45 ms of a cold 100^3 setup and solve.  A
// hierarchy's buffers live in its own arena until it is destroyed or set up
// again; a setup's temporaries in a second one that is freed when the setup
// returns.  All work of a setup is on one stream, so memory given back is
// reused in order.
template <class Mem>
class ArenaOf {
 public:
  ArenaOf() = default;
  ArenaOf(const ArenaOf&) = delete;
  ArenaOf& operator=(const ArenaOf&) = delete;
  ~ArenaOf() {
    for (Slab& s : slabs_) Mem::give(s.p);
  }
  // 256-byte aligned: a hole that something given back has left, the end of a
  // slab, or a new slab: of what is expected and not held yet, then a quarter of
  // what is held (2 to 256 MB, or the request itself); where that cannot be had,
  // one of the request's size.
  void* get(size_t bytes) {
    bytes = round(bytes);
    for (Slab& s : slabs_) {
      for (size_t i = 0; i < s.holes.size(); ++i)
        if (s.holes[i].len >= bytes) {
          char* q = s.p + s.holes[i].at;
          s.holes[i].at += bytes;
          s.holes[i].len -= bytes;
          if (s.holes[i].len == 0) s.holes.erase(s.holes.begin() + i);
          return q;
        }
      if (s.cap - s.used >= bytes) {
        char* q = s.p + s.used;
        s.used += bytes;
        return q;
      }
    }
    const size_t h = held(), grow = expected_ > h ? expected_ - h : expected_ ? h / 4 : h;
    const size_t cap = std::max(bytes, std::min(std::max(grow, kMinSlab), kMaxSlab));
    slabs_.emplace_back();
    Slab& s = slabs_.back();
    try {
      s.p = cap > bytes ? Mem::take(cap, false) : nullptr;
      s.cap = s.p ? cap : bytes;
      if (!s.p) s.p = Mem::take(bytes, true);
    } catch (...) {
      slabs_.pop_back();
      throw;
    }
    s.used = bytes;
    return s.p;
  }
  // How much will be asked for in all.  From about 16 MB on a slab's allocation
  // and free take 0.2 to 0.5 ms whatever its size: doubling from 2 to the 134 MB
  // of a 300^2 hierarchy, and its setup's temporaries likewise, took 11 slabs and
  // 6.5 ms for a setup (with one allocation per buffer 5.0); two slabs of the sizes
  // expected 3.8.
  void expect(size_t bytes) { expected_ = round(bytes); }
  // Takes back what get(bytes) returned.
  void put(void* q, size_t bytes) noexcept {
    bytes = round(bytes);
    for (Slab& s : slabs_) {
      if ((char*)q < s.p || (char*)q >= s.p + s.used) continue;
      Hole h{(size_t)((char*)q - s.p), bytes};
      auto it = std::lower_bound(s.holes.begin(), s.holes.end(), h,
                                 [](const Hole& a, const Hole& b) { return a.at < b.at; });
      if (it != s.holes.end() && h.at + h.len == it->at) {  // joins the holes beside it
        h.len += it->len;
        it = s.holes.erase(it);
      }
      if (it != s.holes.begin() && (it - 1)->at + (it - 1)->len == h.at) {
        h.at = (it - 1)->at;
        h.len += (it - 1)->len;
        it = s.holes.erase(it - 1);
      }
      if (h.at + h.len == s.used) s.used = h.at;
      else try {
        s.holes.insert(it, h);
      } catch (...) {  // no host memory for the record: unused until the slab goes
      }
      return;
    }
  }
  // Everything is given back at once.
  void reset() {
    for (Slab& s : slabs_) {
      s.used = 0;
      s.holes.clear();
    }
  }
  // Frees the slabs that hold nothing.
  void trim() {
    for (size_t i = slabs_.size(); i-- > 0;)
      if (slabs_[i].used == 0) {
        Mem::give(slabs_[i].p);
        slabs_.erase(slabs_.begin() + i);
      }
  }
  size_t held() const {
    size_t h = 0;
    for (const Slab& s : slabs_) h += s.cap;
    return h;
  }

 private:
  static constexpr size_t kMinSlab = (size_t)2 << 20, kMaxSlab = (size_t)256 << 20;
  static size_t round(size_t bytes) { return (bytes + 255) & ~(size_t)255; }
  struct Hole {
    size_t at, len;
  };
  struct Slab {
    char* p = nullptr;
    size_t cap = 0, used = 0;
    std::vector<Hole> holes;  // given back below `used`, by address
  };
  std::vector<Slab> slabs_;
  size_t expected_ = 0;
};

}  // namespace amg
