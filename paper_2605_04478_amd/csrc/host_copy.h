// How the columns of a host batch get to the staging area, and the streams of the threads that help with large ones.
// Host code only: tests compile it against a HIP runtime of their own.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <mutex>
#include <thread>

namespace ccld {

struct HostCopy { void* dst; const void* src; uint64_t bytes; };

// Ordinary memory is made known to the device, copied and forgotten again by the runtime, column by column, and the calling
// thread waits for each; two more threads with a stream each keep the link busy meanwhile: a window of 1,024,000 records (42 MB)
// 1,620 -> 1,150 us (42 MB from pinned memory alone: 795).  The gain is 14% at 16 MB and nothing below 12.
constexpr uint64_t COPY_ALONE_BYTES = 32ull << 20;
constexpr int COPY_HELPERS = 2, COPY_DEVICES = 64;
// The streams are dear in a process that has none but the default one: 3 ms each to make and about 6 more with each one's first
// two large copies (42 MB: 1.7 ms alone, 14.4 with the streams made for it; 2 to 7 for the next two contexts where every context
// makes its own).  So a context's large batches are copied by the caller alone until they have come to as many bytes as make
// the streams worth their price, and whoever makes them makes them for the device: later contexts use them from their first
// batch on, and the last context of the device gives them back.
constexpr uint64_t COPY_EARN_BYTES = 1ull << 30;

struct CopyStreams {
  std::mutex lock;
  struct Device { hipStream_t stream[COPY_HELPERS]; uint32_t contexts; bool made, busy; } dev[COPY_DEVICES] = {};

  void join(int d) {
    std::lock_guard<std::mutex> hold(lock);
    ++dev[d].contexts;
  }
  void leave(int d) {
    std::lock_guard<std::mutex> hold(lock);
    Device& D = dev[d];
    if (--D.contexts || !D.made) return;
    for (hipStream_t s : D.stream) (void)hipStreamDestroy(s);
    D.made = false;
  }
  // One batch at a time uses them; a batch that meets another one is copied by its caller alone.  They belong to device d, whatever
  // device the calling thread has current.
  bool take(int d, bool make) {
    std::lock_guard<std::mutex> hold(lock);
    Device& D = dev[d];
    if (D.busy) return false;
    if (!D.made) {
      int current = d;
      if (!make || hipGetDevice(&current) != hipSuccess || (current != d && hipSetDevice(d) != hipSuccess)) {
        if (make) (void)hipGetLastError();
        return false;
      }
      int n = 0;
      while (n < COPY_HELPERS && hipStreamCreateWithFlags(&D.stream[n], hipStreamNonBlocking) == hipSuccess) ++n;
      D.made = n == COPY_HELPERS;
      if (!D.made) {
        (void)hipGetLastError();
        while (n) (void)hipStreamDestroy(D.stream[--n]);
      }
      if (current != d && hipSetDevice(current) != hipSuccess) (void)hipGetLastError();
    }
    return D.busy = D.made;
  }
  void give(int d) {
    std::lock_guard<std::mutex> hold(lock);
    dev[d].busy = false;
  }
};

// n columns of a batch, on their way in the order of stream st, which belongs to device d; earned: the bytes of large batches that the
// context's caller has copied alone.
inline hipError_t copy_from_host(CopyStreams& pool, int d, uint64_t& earned, hipStream_t st, const HostCopy* copies, int n) {
  uint64_t bytes = 0;
  for (int i = 0; i < n; ++i) bytes += copies[i].bytes;
  std::atomic<int> next{0};
  auto copy = [&](hipStream_t on) -> hipError_t {
    hipError_t e = hipSuccess;
    for (int i; e == hipSuccess && (i = next.fetch_add(1)) < n;)
      e = hipMemcpyAsync(copies[i].dst, copies[i].src, copies[i].bytes, hipMemcpyHostToDevice, on);
    return e;
  };
  if (bytes < COPY_ALONE_BYTES) return copy(st);
  const bool make = earned >= COPY_EARN_BYTES;
  if (!pool.take(d, make)) {
    earned = make ? 0 : earned + bytes;                    // streams that could not be made are not asked for in every batch
    return copy(st);
  }
  hipError_t e = hipStreamSynchronize(st);                 // what still uses the staging area
  if (e == hipSuccess) {
    hipError_t helped[COPY_HELPERS];
    std::thread helper[COPY_HELPERS];                      // what none of them takes, the calling thread copies
    for (int t = 0; t < COPY_HELPERS; ++t) {
      helped[t] = hipSuccess;
      try {
        helper[t] = std::thread([&, t] {
          if ((helped[t] = hipSetDevice(d)) != hipSuccess) return;
          helped[t] = copy(pool.dev[d].stream[t]);
          const hipError_t done = hipStreamSynchronize(pool.dev[d].stream[t]);
          if (helped[t] == hipSuccess) helped[t] = done;
        });
      } catch (...) {
        break;
      }
    }
    e = copy(st);
    for (int t = 0; t < COPY_HELPERS; ++t)
      if (helper[t].joinable()) { helper[t].join(); if (e == hipSuccess) e = helped[t]; }
  }
  pool.give(d);
  return e;
}

}  // namespace ccld
