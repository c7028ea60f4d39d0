// Results to caller memory: device arrays stream through two pinned buffers of
// the handle, and a few host threads widen or split what has arrived into the
// caller's (pageable, often untouched) arrays while the next piece is copied.
#pragma once

#include <atomic>
#include <condition_variable>
#include <cstring>
#include <exception>
#include <functional>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "handle.h"

namespace lda {

// Host threads of one call; run() shares numbered pieces of a job among them
// and the calling thread and returns when all are done.
class Crew {
 public:
  explicit Crew(int threads) {
    try {
      th_.reserve(size_t(std::max(threads, 1)));  // no growth below: it could fail with threads running
      for (int q = 1; q < threads; ++q) th_.emplace_back([this] { loop(); });
    } catch (const std::exception &) {
      // no thread or no memory for one: the pieces are shared among those there are
    }
  }
  ~Crew() {
    {
      std::lock_guard<std::mutex> l(m_);
      stop_ = true;
    }
    go_.notify_all();
    for (std::thread &t : th_) t.join();
  }
  Crew(const Crew &) = delete;
  Crew &operator=(const Crew &) = delete;

  template <typename F>
  void run(size_t pieces, const F &job) {
    if (th_.empty() || pieces <= 1) {
      for (size_t i = 0; i < pieces; ++i) job(i);
      return;
    }
    {
      std::lock_guard<std::mutex> l(m_);
      job_ = std::cref(job);
      pieces_ = pieces;
      next_.store(0);
      busy_ = int(th_.size());
      ++turn_;
    }
    go_.notify_all();
    work();
    std::unique_lock<std::mutex> l(m_);
    done_.wait(l, [this] { return busy_ == 0; });
  }

 private:
  void work() {
    for (size_t i = next_.fetch_add(1); i < pieces_; i = next_.fetch_add(1)) job_(i);
  }
  void loop() {
    unsigned seen = 0;
    std::unique_lock<std::mutex> l(m_);
    for (;;) {
      go_.wait(l, [&] { return stop_ || turn_ != seen; });
      if (stop_) return;
      seen = turn_;
      l.unlock();
      work();
      l.lock();
      if (--busy_ == 0) done_.notify_one();
    }
  }
  std::vector<std::thread> th_;
  std::mutex m_;
  std::condition_variable go_, done_;
  std::function<void(size_t)> job_;
  std::atomic<size_t> next_{0};
  size_t pieces_ = 0;
  int busy_ = 0;
  unsigned turn_ = 0;
  bool stop_ = false;
};

// A device array of one call, given back when the call leaves by any path.
// Where the device or the caller's allocator has no room it is pinned host
// memory, which kernels reach over PCIe: an export needs no device memory to
// succeed, only to be fast.
template <typename T>
struct Scratch {
  lda_handle *h;
  T *ptr = nullptr;
  bool on_host = false;
  explicit Scratch(lda_handle *handle) : h(handle) {}
  ~Scratch() {
    // left by an exception (no host memory), kernels may still be at work on it
    if (ptr && std::uncaught_exceptions()) (void)hipStreamSynchronize(h->stream);
    if (on_host) (void)hipHostFree(ptr);
    else dfree(h, ptr);
  }
  Scratch(const Scratch &) = delete;
  Scratch &operator=(const Scratch &) = delete;

  lda_status get(size_t count) {
    const std::string err = h->err;
    const lda_status st = dalloc(h, &ptr, count);
    if (st != LDA_E_NOMEM) return st;
    (void)hipGetLastError();
    void *p = nullptr;
    if (hipHostMalloc(&p, std::max<size_t>(count, 1) * sizeof(T), hipHostMallocDefault) != hipSuccess) {
      (void)hipGetLastError();
      return st;
    }
    h->err = err;
    ptr = static_cast<T *>(p);
    on_host = true;
    return LDA_OK;
  }
  // The first n values from src, which the caller keeps until the stream is waited for.
  lda_status put(const T *src, size_t n) {
    if (on_host) {
      HIP_TRY(h, hipStreamSynchronize(h->stream));  // kernels before read what is overwritten
      std::memcpy(ptr, src, n * sizeof(T));
    } else {
      HIP_TRY(h, hipMemcpyAsync(ptr, src, n * sizeof(T), hipMemcpyHostToDevice, h->stream));
    }
    return LDA_OK;
  }
};

// Below this many bytes a result is copied at once and used by the calling
// thread (the threads' start costs more than they save).
constexpr size_t kReadSmall = size_t(1) << 20;
constexpr int kReadThreads = 8;
inline int read_threads(size_t bytes) {
  const unsigned hw = std::thread::hardware_concurrency();
  const size_t most = std::min<size_t>(kReadThreads, hw ? hw : 1);
  return int(std::min<size_t>(most, 1 + bytes / kReadSmall));
}

// use(src, first, count) for consecutive pieces of dev[0, n), which arrive in
// stream order after the work queued on the handle's stream; calls for
// different pieces may run at once, on several threads.
template <typename T, typename F>
lda_status read_back(lda_handle *h, Crew &crew, const T *dev, size_t n, const F &use) {
  const size_t bytes = n * sizeof(T);
  if (n == 0) return LDA_OK;
  if (bytes > kReadSmall && !h->stage[0]) {
    // all or none: without pinned memory the copies below go straight to host memory
    void *a = nullptr, *b = nullptr;
    hipEvent_t ea = nullptr, eb = nullptr;
    if (hipHostMalloc(&a, kStageBytes, hipHostMallocDefault) == hipSuccess &&
        hipHostMalloc(&b, kStageBytes, hipHostMallocDefault) == hipSuccess &&
        hipEventCreateWithFlags(&ea, hipEventDisableTiming) == hipSuccess &&
        hipEventCreateWithFlags(&eb, hipEventDisableTiming) == hipSuccess) {
      h->stage[0] = a;
      h->stage[1] = b;
      h->stage_ev[0] = ea;
      h->stage_ev[1] = eb;
    } else {
      (void)hipGetLastError();
      if (a) (void)hipHostFree(a);
      if (b) (void)hipHostFree(b);
      if (ea) (void)hipEventDestroy(ea);
      if (eb) (void)hipEventDestroy(eb);
    }
  }
  if (bytes <= kReadSmall || !h->stage[0]) {
    std::vector<T> tmp(std::min(n, kStageBytes / sizeof(T)));
    for (size_t i = 0; i < n; i += tmp.size()) {
      const size_t m = std::min(tmp.size(), n - i);
      HIP_TRY(h, hipMemcpyAsync(tmp.data(), dev + i, m * sizeof(T), hipMemcpyDeviceToHost, h->stream));
      HIP_TRY(h, hipStreamSynchronize(h->stream));
      use(tmp.data(), i, m);
    }
    return LDA_OK;
  }
  const size_t step = kStageBytes / sizeof(T), nst = (n + step - 1) / step;
  const size_t piece = (size_t(64) << 10) / sizeof(T);
  auto issue = [&](size_t i) -> lda_status {
    const size_t b = i * step, m = std::min(step, n - b);
    HIP_TRY(h, hipMemcpyAsync(h->stage[i & 1], dev + b, m * sizeof(T), hipMemcpyDeviceToHost, h->stream));
    HIP_TRY(h, hipEventRecord(h->stage_ev[i & 1], h->stream));
    return LDA_OK;
  };
  LDA_TRY(issue(0));
  for (size_t i = 0; i < nst; ++i) {
    if (i + 1 < nst) LDA_TRY(issue(i + 1));  // the other buffer's pieces were used below
    HIP_TRY(h, hipEventSynchronize(h->stage_ev[i & 1]));
    const size_t b = i * step, m = std::min(step, n - b);
    const T *src = static_cast<const T *>(h->stage[i & 1]);
    crew.run((m + piece - 1) / piece, [&](size_t q) {
      const size_t f = q * piece;
      use(src + f, b + f, std::min(piece, m - f));
    });
  }
  return LDA_OK;
}

template <typename T, typename F>
lda_status read_back(lda_handle *h, Crew &crew, const Scratch<T> &from, size_t n, const F &use) {
  if (!from.on_host) return read_back(h, crew, static_cast<const T *>(from.ptr), n, use);
  HIP_TRY(h, hipStreamSynchronize(h->stream));
  const T *src = from.ptr;
  const size_t piece = (size_t(64) << 10) / sizeof(T);
  crew.run((n + piece - 1) / piece, [&](size_t q) {
    const size_t f = q * piece;
    use(src + f, f, std::min(piece, n - f));
  });
  return LDA_OK;
}

// Caller arrays of one export.
lda_status read_z(lda_handle *h, Crew &crew, const uint16_t *z, size_t n, int32_t *out);
lda_status read_z(lda_handle *h, Crew &crew, const Scratch<uint16_t> &z, size_t n, int32_t *out);
// D rows of documents [0, M) of d (offsets d_cap) as CSR, appended at entry
// `at` of the topic and count arrays: off[q] = entry of document q's first
// (M + 1 written); returns the entries written in *entries.
lda_status export_d(lda_handle *h, Crew &crew, const DevState &d, int32_t M, int64_t at, int64_t *off, int32_t *topic,
                    int32_t *count, int64_t *entries);
// W in the caller's word ids as CSR.
lda_status export_w(lda_handle *h, Crew &crew, const DevState &d, const Params &p, int64_t *off, int32_t *topic,
                    int32_t *count);

}  // namespace lda
