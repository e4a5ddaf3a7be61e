// Arena::alloc_front and Arena::trim against Arena::alloc: a block taken from
// the front for more than is needed and then trimmed leaves the arena as an
// exact alloc would have, and a refused alloc_front leaves it as it was.
// Built and run by test_arena_front.py.
#include <cstdio>
#include <random>
#include <vector>

#include "../paper_1604_07515_amd/csrc/arena.h"

#define CHECK(c)                                                     \
  do {                                                               \
    if (!(c)) {                                                      \
      std::fprintf(stderr, "check failed line %d: %s\n", __LINE__, #c); \
      return 1;                                                      \
    }                                                                \
  } while (0)

int main() {
  char* base = reinterpret_cast<char*>(uintptr_t(1) << 40);  // never dereferenced
  plc::Arena A, B;
  A.reset(base, size_t(1) << 20);
  B.reset(base, size_t(1) << 20);
  std::mt19937_64 rng(3);
  std::vector<void*> live;
  int front = 0, refused = 0;
  for (int it = 0; it < 100000; it++) {
    if (live.empty() || rng() % 100 < (it / 500 % 2 ? 30u : 65u)) {
      const size_t want = rng() % 9000, room = want + (rng() % 3 ? rng() % 9000 : 0);
      void* a = A.alloc_front(room);
      if (a) {
        A.trim(a, want);
        front++;
      } else {
        a = A.alloc(want);
        refused++;
      }
      void* b = B.alloc(want);
      CHECK(a == b);
      if (a) live.push_back(a);
    } else {
      const size_t j = rng() % live.size();
      CHECK(A.release(live[j]) && B.release(live[j]));
      live.erase(live.begin() + (long)j);
    }
    CHECK(A.free_bytes() == B.free_bytes() && A.largest_free() == B.largest_free());
  }
  CHECK(front > 1000 && refused > 1000);
  std::puts("front ok");
  return 0;
}
