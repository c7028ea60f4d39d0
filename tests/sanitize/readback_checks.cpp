// Results read back through the pinned buffers (csrc/readback.h), CPU only:
// the HIP calls that it makes are replaced by host copies and by counts of
// what is alive.  Exit status 0 = every check held.
#include <cstdio>
#include <cstdlib>
#include <new>
#include <vector>

#include "readback.h"

static int g_events, g_fail_event = -1, g_pinned, g_pinned_room = 1 << 20;
static bool g_at_work, g_freed_at_work;  // queued kernels not waited for; memory given back meanwhile
static long g_countdown = -1;            // the host allocation that fails (negative: none)
void *operator new(std::size_t n) {
  if (g_countdown >= 0 && g_countdown-- == 0) throw std::bad_alloc();
  void *p = std::malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

extern "C" {
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(dst, src, n);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  g_at_work = false;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) {
  g_at_work = false;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
  if (g_fail_event >= 0 && g_fail_event-- == 0) return hipErrorOutOfMemory;
  ++g_events;
  *e = reinterpret_cast<hipEvent_t>(std::malloc(1));
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
  --g_events;
  std::free(e);
  return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
  if (g_pinned >= g_pinned_room) return hipErrorOutOfMemory;
  ++g_pinned;
  *p = std::malloc(n);
  return hipSuccess;
}
hipError_t hipHostFree(void *p) {
  --g_pinned;
  std::free(p);
  return hipSuccess;
}
hipError_t hipMalloc(void **, size_t) { return hipErrorOutOfMemory; }
hipError_t hipFree(void *) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
}
namespace lda {
thread_local std::string g_create_error;
void release_chunks(ChunkMode *) {}
}  // namespace lda

#define CHECK(c)                                                      \
  do {                                                                \
    if (!(c)) {                                                       \
      std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #c); \
      return 1;                                                       \
    }                                                                 \
  } while (0)

static void *dev_alloc(size_t n, void *) { return std::malloc(n); }
static void dev_free(void *p, void *) {
  g_freed_at_work = g_freed_at_work || g_at_work;
  std::free(p);
}

static void drop_stage(lda_handle &h) {
  for (int q = 0; q < 2; ++q) {
    if (h.stage[q]) (void)hipHostFree(h.stage[q]);
    if (h.stage_ev[q]) (void)hipEventDestroy(h.stage_ev[q]);
    h.stage[q] = nullptr;
    h.stage_ev[q] = nullptr;
  }
}

// n values arrive once each, in their places
static int arrive(lda_handle &h, int threads, size_t n) {
  std::vector<uint32_t> dev(n), got(n, 0xFFFFFFFFu);
  for (size_t q = 0; q < n; ++q) dev[q] = uint32_t(q * 2654435761u);
  lda::Crew crew(threads);
  CHECK(lda::read_back(&h, crew, static_cast<const uint32_t *>(dev.data()), n,
                       [&](const uint32_t *src, size_t first, size_t m) {
                         std::memcpy(got.data() + first, src, m * sizeof(uint32_t));
                       }) == LDA_OK);
  CHECK(got == dev);
  return 0;
}

int main() {
  const size_t small = lda::kReadSmall / 4, step = lda::kStageBytes / 4;
  for (int threads : {1, 4})
    for (size_t n : {size_t(0), size_t(1), small, small + 1, step, step + 1, 3 * step + 17}) {
      lda_handle h;
      if (arrive(h, threads, n)) return 1;
      if (arrive(h, threads, n)) return 1;  // the buffers are there already
      drop_stage(h);
      CHECK(g_events == 0 && g_pinned == 0);
    }
  // an event or a buffer that cannot be made leaves nothing behind, however often it is tried
  for (int fail = 0; fail < 2; ++fail) {
    lda_handle h;
    for (int call = 0; call < 3; ++call) {
      g_fail_event = fail;
      if (arrive(h, 2, small + 5)) return 1;
      CHECK(!h.stage[0] && g_events == 0 && g_pinned == 0);
    }
    g_fail_event = -1;
    g_pinned_room = fail;
    if (arrive(h, 2, small + 5)) return 1;
    CHECK(!h.stage[0] && g_events == 0 && g_pinned == 0);
    g_pinned_room = 1 << 20;
    drop_stage(h);
  }
  // host memory that runs out between a kernel's launch and the wait for its results: the device array that it
  // writes is given back to the caller's allocator only when the kernel is done
  for (long fail = 0; fail < 50; ++fail) {
    lda_handle h;
    h.dev_alloc = dev_alloc;
    h.dev_free = dev_free;
    bool threw = false;
    try {
      lda::Crew crew(1);
      lda::Scratch<uint32_t> a(&h);
      CHECK(a.get(1000) == LDA_OK);
      std::memset(a.ptr, 0, 4000);
      g_at_work = true;  // a launch
      g_countdown = fail;
      CHECK(lda::read_back(&h, crew, a, 1000, [](const uint32_t *, size_t, size_t) {}) == LDA_OK);
      g_countdown = -1;
    } catch (const std::bad_alloc &) {
      threw = true;
    }
    g_countdown = -1;
    CHECK(!g_freed_at_work && h.allocations.empty());
    if (!threw) {
      CHECK(fail > 0);  // at least one allocation failed
      break;
    }
  }
  std::printf("read-back checks passed\n");
  return 0;
}
