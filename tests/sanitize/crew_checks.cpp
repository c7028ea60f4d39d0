// The host threads that results are read back by (Crew, csrc/readback.h), CPU
// only: every piece is done once with any number of threads, and an allocation
// that fails at any point ends in fewer threads, not in std::terminate.  Exit
// status 0 = every check held.
#include <cstdio>
#include <cstdlib>
#include <new>

#include "readback.h"

static long g_countdown = -1;  // the allocation that fails, counted from the next one on (negative: none)
static std::atomic<long> g_live{0};
void *operator new(std::size_t n) {
  if (g_countdown >= 0 && g_countdown-- == 0) throw std::bad_alloc();
  void *p = std::malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  ++g_live;
  return p;
}
void operator delete(void *p) noexcept {
  if (p) --g_live;
  std::free(p);
}
void operator delete(void *p, std::size_t) noexcept { operator delete(p); }

#define CHECK(c)                                                      \
  do {                                                                \
    if (!(c)) {                                                       \
      std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #c); \
      return 1;                                                       \
    }                                                                 \
  } while (0)

static int jobs_are_done(int threads) {
  lda::Crew crew(threads);
  for (int turn = 0; turn < 3; ++turn) {
    std::atomic<int> hit[37] = {};
    crew.run(37, [&](size_t q) { ++hit[q]; });
    for (auto &h : hit) CHECK(h == 1);
  }
  return 0;
}

int main() {
  for (int threads : {0, 1, 2, 8})
    if (jobs_are_done(threads)) return 1;
  // every allocation of a crew of 8 in turn; the first that is never reached ends the loop
  for (long fail = 0; fail < 100; ++fail) {
    const long before = g_live;
    g_countdown = fail;
    const int r = jobs_are_done(8);
    const bool reached = g_countdown < 0;
    g_countdown = -1;
    CHECK(r == 0);
    CHECK(g_live == before);
    if (!reached) {
      std::printf("crew checks passed (%ld allocations)\n", fail);
      return 0;
    }
  }
  return 1;
}
