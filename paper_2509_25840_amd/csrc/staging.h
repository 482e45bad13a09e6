// Copies between device memory and ordinary (pageable) host memory.
//
// hipMemcpyAsync moves a pageable buffer at 28 GB/s to the device and 10 GB/s
// from it (a new host array's first touch included), bound by one core that
// copies and takes the page faults; the link does 56 GB/s.  Here a few threads
// copy between the host buffer and a ring of pinned chunks, while this thread
// moves the chunks over the link.  In and out, before and after: 50 MB 1.8 and
// 5.0 -> 1.5 and 1.9 ms, 63 MB 2.2 and 6.2 -> 1.9 and 1.9 ms, 537 MB 18.3 and
// 50.7 -> 13.8 and 14.4 ms.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstring>
#include <exception>
#include <thread>
#include <vector>

namespace chfpe {

constexpr size_t kStageChunk = 2 << 20;
constexpr int kStageSlots = 12;
constexpr int kStageThreads = 8;
// Smaller copies are left to hipMemcpyAsync: 19 MB in take 0.56 ms there and 0.68
// here (starting the threads takes 0.1 ms), and 25 MB out 1.4 against 0.9, not
// enough for the 24 MiB that are pinned (1 ms, once) and for what the threads
// lose where others keep the CPUs busy (up to 4 ms, a time slice).
constexpr size_t kStageMin = 32 << 20;

// One object's ring of pinned chunks, allocated at its first large copy and
// freed with it; not for two threads at a time (as the context that owns it).
// Only the calling thread makes HIP calls.
class Staging {
 public:
  Staging() = default;
  Staging(const Staging &) = delete;
  Staging &operator=(const Staging &) = delete;
  ~Staging() {
    for (int i = 0; i < events_; ++i) (void)hipEventDestroy(moved_[i]);
    if (pinned_) (void)hipHostFree(pinned_);
  }

  // dst (device) = src (host), in stream order; src is free once the stream is
  // synchronized.
  hipError_t in(void *dst, const void *src, size_t bytes, hipStream_t st) {
    if (bytes < kStageMin || reached(src) || !ready())
      return hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, st);
    Ring r(bytes);
    // chunk k is filled once chunk k - slots has left (r.moved of them have)
    Threads copiers(r, [&](size_t k) {
      if (k >= kStageSlots) r.wait([&] { return r.moved.load(std::memory_order_acquire) + kStageSlots > k; });
      if (r.stop) return;
      std::memcpy(slot(k), static_cast<const char *>(src) + k * kStageChunk, r.size(k));
      r.copied[k % kStageSlots].store(k + 1, std::memory_order_release);
    });
    if (copiers.none()) return hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, st);
    constexpr size_t lag = kStageSlots / 2;  // chunks on the link
    hipError_t e = hipSuccess;
    for (size_t k = 0; k < r.n && e == hipSuccess; ++k) {
      r.wait([&] { return r.copied[k % kStageSlots].load(std::memory_order_acquire) == k + 1; });
      e = hipMemcpyAsync(static_cast<char *>(dst) + k * kStageChunk, slot(k), r.size(k), hipMemcpyHostToDevice, st);
      if (e == hipSuccess) e = hipEventRecord(moved_[k % kStageSlots], st);
      if (e == hipSuccess && k >= lag) {
        e = hipEventSynchronize(moved_[(k - lag) % kStageSlots]);
        r.moved.store(k - lag + 1, std::memory_order_release);
      }
    }
    r.stop = true;
    const hipError_t es = hipStreamSynchronize(st);
    return e == hipSuccess ? es : e;
  }

  // dst (host) = src (device), complete on return.
  hipError_t out(void *dst, const void *src, size_t bytes, hipStream_t st) {
    hipError_t e = hipSuccess;
    if (bytes >= kStageMin && !reached(dst) && ready()) {
      Ring r(bytes);
      // chunk k is copied once it has come (r.moved of them have)
      Threads copiers(r, [&](size_t k) {
        r.wait([&] { return r.moved.load(std::memory_order_acquire) > k; });
        if (r.stop) return;
        std::memcpy(static_cast<char *>(dst) + k * kStageChunk, slot(k), r.size(k));
        r.copied[k % kStageSlots].store(k + 1, std::memory_order_release);
      });
      if (!copiers.none()) {
        size_t issued = 0;
        for (size_t k = 0; k < r.n && e == hipSuccess; ++k) {
          while (e == hipSuccess && issued < r.n) {
            if (issued >= kStageSlots) {  // its slot's last chunk must be out
              auto &c = r.copied[issued % kStageSlots];
              const size_t last = issued - kStageSlots + 1;
              if (issued > k && c.load(std::memory_order_acquire) != last) break;
              r.wait([&] { return c.load(std::memory_order_acquire) == last; });
            }
            e = hipMemcpyAsync(slot(issued), static_cast<const char *>(src) + issued * kStageChunk, r.size(issued),
                               hipMemcpyDeviceToHost, st);
            if (e == hipSuccess) e = hipEventRecord(moved_[issued % kStageSlots], st);
            ++issued;
          }
          if (e == hipSuccess) e = hipEventSynchronize(moved_[k % kStageSlots]);
          if (e == hipSuccess) r.moved.store(k + 1, std::memory_order_release);
        }
        if (e != hipSuccess) {
          r.stop = true;
          (void)hipStreamSynchronize(st);
        }
        copiers.join();
        return e;
      }
    }
    e = hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, st);
    return e == hipSuccess ? hipStreamSynchronize(st) : e;
  }

 private:
  // One copy's chunks: moved counts those that have crossed the link, in order;
  // copied[slot] is one more than the last chunk that the host side is done
  // with there.  stop ends every wait.
  struct Ring {
    explicit Ring(size_t b) : bytes(b), n((b + kStageChunk - 1) / kStageChunk) {
      for (auto &c : copied) c.store(0, std::memory_order_relaxed);
    }
    size_t size(size_t k) const { return std::min(kStageChunk, bytes - k * kStageChunk); }
    template <typename F>
    void wait(F done) const {
      for (int spin = 0; !done() && !stop; ++spin)
        if (spin >= 64) std::this_thread::yield();
    }
    const size_t bytes, n;
    std::atomic<size_t> next{0}, moved{0};
    std::atomic<size_t> copied[kStageSlots];
    std::atomic<bool> stop{false};
  };

  // Threads that each take the next chunk until none is left.
  class Threads {
   public:
    template <typename F>
    Threads(Ring &r, F one) {
      const int want = std::min(kStageThreads, (int)std::thread::hardware_concurrency() - 1);
      try {
        t_.reserve(kStageThreads);
        for (int w = 0; w < want; ++w)
          t_.emplace_back([&r, one] {
            for (size_t k; !r.stop && (k = r.next.fetch_add(1)) < r.n;) one(k);
          });
      } catch (const std::exception &) {  // fewer threads, then
      }
    }
    ~Threads() { join(); }
    bool none() const { return t_.empty(); }
    void join() {
      for (std::thread &t : t_) t.join();
      t_.clear();
    }

   private:
    std::vector<std::thread> t_;
  };

  char *slot(size_t k) const { return pinned_ + k % kStageSlots * kStageChunk; }

  // Memory the link reaches by itself (pinned by the caller, managed): its
  // copies need no ring (84 MiB in and out 2.32 and 2.35 ms through it, 1.54 and
  // 1.60 directly).
  static bool reached(const void *p) {
    hipPointerAttribute_t a{};
    if (hipPointerGetAttributes(&a, p) == hipSuccess) return a.type != hipMemoryTypeUnregistered;
    (void)hipGetLastError();  // ordinary memory, as some releases answer
    return false;
  }

  bool ready() {
    if (pinned_ || failed_) return pinned_ != nullptr;
    void *p = nullptr;
    if (hipHostMalloc(&p, kStageSlots * kStageChunk, hipHostMallocDefault) == hipSuccess) {
      while (events_ < kStageSlots &&
             hipEventCreateWithFlags(&moved_[events_], hipEventDisableTiming) == hipSuccess)
        ++events_;
      if (events_ == kStageSlots) {
        pinned_ = static_cast<char *>(p);
        return true;
      }
      (void)hipHostFree(p);
    }
    failed_ = true;  // pageable copies from now on
    (void)hipGetLastError();
    return false;
  }

  char *pinned_ = nullptr;
  hipEvent_t moved_[kStageSlots] = {};
  int events_ = 0;
  bool failed_ = false;
};

}  // namespace chfpe
