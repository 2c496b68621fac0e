// Device scratch of a handle: grown on demand, with a smaller share taken where the device has no room.
#pragma once

#include <cstddef>
#include <cstdint>

namespace sf {

struct Scratch {
  void* ptr = nullptr;
  size_t bytes = 0;
};

// Makes room for `fixed` bytes and as many parts of `per` bytes as it can, at most `most`, and returns how many
// (0: not even one fits).  Asks for all of them first and for half as many after each refusal.  The present buffer
// is kept until a larger one is there if it holds at least one part, and serves if none is had.
// alloc(bytes) returns NULL where there is no room, release(ptr) gives a buffer back.
template <class Alloc, class Release>
int64_t scratch_parts(Scratch& s, size_t fixed, size_t per, int64_t most, Alloc alloc, Release release) {
  const int64_t held = s.bytes >= fixed + per ? (int64_t)((s.bytes - fixed) / per) : 0;
  if (held >= most) return most;
  if (held == 0 && s.ptr) {
    release(s.ptr);
    s = Scratch();
  }
  for (int64_t n = most; n > held; n /= 2) {
    void* p = alloc(fixed + (size_t)n * per);
    if (!p) continue;
    if (s.ptr) release(s.ptr);
    s.ptr = p;
    s.bytes = fixed + (size_t)n * per;
    return n;
  }
  return held;
}

}  // namespace sf
