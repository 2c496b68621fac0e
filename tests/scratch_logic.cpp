// Host check of the reverse mode's scratch growth: how many checkpoint segments it takes on a device with little
// room.  Built and run by tests/test_scratch.py; prints the number of failed checks.
#include "sf_scratch.h"

#include <cstdio>
#include <map>

int main() {
  int fails = 0, line = 0;
  auto chk = [&](bool c, const char* what) {
    ++line;
    if (!c) {
      std::printf("FAIL %d %s\n", line, what);
      ++fails;
    }
  };
  // a device of `room` bytes; addresses are serial numbers
  size_t room = 0, used = 0;
  std::map<void*, size_t> live;
  size_t serial = 0, asked = 0;
  auto alloc = [&](size_t bytes) -> void* {
    ++asked;
    if (used + bytes > room) return nullptr;
    used += bytes;
    void* p = reinterpret_cast<void*>(++serial);
    live[p] = bytes;
    return p;
  };
  auto release = [&](void* p) {
    used -= live.at(p);
    live.erase(p);
  };
  auto sound = [&](const sf::Scratch& s) { return live.size() <= 1 && (!s.ptr || live.at(s.ptr) == s.bytes); };
  {   // plenty of room: all segments, once
    sf::Scratch s;
    room = 1000;
    chk(sf::scratch_parts(s, 10, 20, 10, alloc, release) == 10 && s.bytes == 210 && sound(s), "all parts");
    const size_t before = asked;
    chk(sf::scratch_parts(s, 10, 20, 10, alloc, release) == 10 && asked == before, "nothing is asked for twice");
    chk(sf::scratch_parts(s, 30, 50, 3, alloc, release) == 3 && asked == before, "another shape in the same buffer");
    release(s.ptr);
  }
  {   // room for fewer: halves down to one, and none at all
    sf::Scratch s;
    room = 130;
    chk(sf::scratch_parts(s, 10, 20, 10, alloc, release) == 5 && sound(s), "half of the parts");
    release(s.ptr);
    s = sf::Scratch();
    room = 30;
    chk(sf::scratch_parts(s, 10, 20, 10, alloc, release) == 1 && sound(s), "one part");
    release(s.ptr);
    s = sf::Scratch();
    room = 29;
    chk(sf::scratch_parts(s, 10, 20, 10, alloc, release) == 0 && !s.ptr && s.bytes == 0, "none");
  }
  {   // a smaller working buffer survives a refusal and serves
    sf::Scratch s;
    room = 100;
    chk(sf::scratch_parts(s, 10, 20, 3, alloc, release) == 3 && sound(s), "three parts");
    void* p = s.ptr;
    chk(sf::scratch_parts(s, 10, 20, 10, alloc, release) == 3 && s.ptr == p && sound(s), "the present buffer serves");
    // too small for one part of another shape: it makes room first
    chk(sf::scratch_parts(s, 10, 85, 4, alloc, release) == 1 && sound(s) && used == 95, "the present buffer makes room");
    release(s.ptr);
  }
  {   // growth gives the old buffer back
    sf::Scratch s;
    room = 1000;
    chk(sf::scratch_parts(s, 0, 20, 1, alloc, release) == 1, "one part");
    chk(sf::scratch_parts(s, 0, 20, 8, alloc, release) == 8 && used == 160 && sound(s), "grown");
    chk(sf::scratch_parts(s, 0, 20, 9, alloc, release) == 9 && used == 180 && sound(s), "grown again");
    release(s.ptr);
  }
  std::printf("%d\n", fails);
  return fails != 0;
}
