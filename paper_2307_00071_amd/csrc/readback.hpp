// Small device results on the host: the status words and counters that a
// call returns, shared by the library's translation units.
//
// A copy of 4 bytes to ordinary host memory and a stream synchronisation
// measured 19.6 us on the MI355X beyond the call's own launches (pinned
// memory and a synchronisation 10.7 us); a kernel that stores the words to
// pinned memory, polled by the waiting thread, 6.0 us.  So the words go that
// way, each with the call's sequence number in one 8-byte store, and the
// thread polls for kPollLimit; a longer wait ends in a stream
// synchronisation.
//
// The pinned memory is one page of 16 slots, allocated once per process; a
// call holds one slot while it waits, and takes the copy when none is free,
// when the page cannot be allocated or may not be (the allocation-free fit),
// and while the stream is being captured (the copy then gives the error it
// always gave).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <atomic>
#include <chrono>
#include <mutex>

namespace gmm_host {

constexpr int kReadSlots = 16, kReadWords = 32;
constexpr std::chrono::microseconds kPollLimit{1000};

struct ReadPage {
  std::mutex mu;
  uint32_t missed = 0;                    // failed or skipped attempts
  uint64_t *host = nullptr, *dev = nullptr;
  std::atomic<uint32_t> busy{0};          // bit per slot
  uint32_t seq[kReadSlots] = {};          // written by the slot's holder only
};
inline ReadPage g_read;

// GMM_READ_TEST (tests of each way): copy - the copy always; page - an error
// where the page cannot be used; nopage - the page's allocation fails; refuse -
// a launch that the runtime refuses.
enum ReadTest { kReadAsIs, kReadCopy, kReadPageOnly, kReadNoPage, kReadRefuse };
inline ReadTest read_test() {
  const char *e = getenv("GMM_READ_TEST");
  if (!e) return kReadAsIs;
  const char *const names[] = {"", "copy", "page", "nopage", "refuse"};
  for (int i = 1; i < 5; ++i)
    if (strcmp(e, names[i]) == 0) return (ReadTest)i;
  return kReadAsIs;
}

// An attempt that fails is repeated at the 2nd, 4th, 8th, ... call after it.
// Another thread may be capturing a stream: in the relaxed mode the
// allocation is allowed then and leaves that capture alone.
inline bool read_page(bool may_alloc, ReadTest test) {
  std::lock_guard<std::mutex> lk(g_read.mu);
  if (g_read.host || !may_alloc) return g_read.host != nullptr;
  if ((g_read.missed & (g_read.missed - 1)) == 0) {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    void *h = nullptr, *d = nullptr;
    const size_t bytes = (size_t)kReadSlots * kReadWords * sizeof(uint64_t);
    if (test != kReadNoPage &&
        hipHostMalloc(&h, bytes, hipHostMallocPortable | hipHostMallocMapped) == hipSuccess) {
      if (hipHostGetDevicePointer(&d, h, 0) == hipSuccess && d) {
        memset(h, 0, bytes);
        g_read.dev = static_cast<uint64_t *>(d);
        g_read.host = static_cast<uint64_t *>(h);
      } else {
        (void)hipHostFree(h);
      }
    }
    if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
    if (!g_read.host) (void)hipGetLastError();
  }
  if (!g_read.host) ++g_read.missed;
  return g_read.host != nullptr;
}

namespace {
__global__ void publish_kernel(const uint32_t *__restrict__ src, int n, uint64_t *dst,
                               uint32_t seq) {
  const int i = threadIdx.x;
  if (i < n)
    __hip_atomic_store(dst + i, ((uint64_t)seq << 32) | src[i], __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}
}  // namespace

inline hipError_t read_words_copy(const uint32_t *src, int n, void *out, hipStream_t s) {
  hipError_t e = hipMemcpyAsync(out, src, (size_t)n * 4, hipMemcpyDeviceToHost, s);
  return e != hipSuccess ? e : hipStreamSynchronize(s);
}

// The n <= kReadWords 32-bit words at src (device memory) after everything
// queued on s; returns when they are in `out`.
inline hipError_t read_words(const void *src_, int n, void *out, hipStream_t s,
                             bool may_alloc = true) {
  const uint32_t *src = static_cast<const uint32_t *>(src_);
  const ReadTest test = read_test();
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &cap) != hipSuccess) {
    (void)hipGetLastError();
    cap = hipStreamCaptureStatusInvalidated;
  }
  if (n > kReadWords || cap != hipStreamCaptureStatusNone || test == kReadCopy ||
      !read_page(may_alloc, test))
    return test == kReadPageOnly ? hipErrorNotReady : read_words_copy(src, n, out, s);
  int slot = -1;
  for (uint32_t b = g_read.busy.load(); slot < 0;) {
    const uint32_t open = ~b & ((1u << kReadSlots) - 1u);
    if (!open) return read_words_copy(src, n, out, s);
    const uint32_t bit = open & (0u - open);
    if (g_read.busy.compare_exchange_weak(b, b | bit)) slot = __builtin_ctz(bit);
  }
  uint64_t *h = g_read.host + (size_t)slot * kReadWords;
  const uint32_t seq = ++g_read.seq[slot];
  uint64_t *dst = g_read.dev + (size_t)slot * kReadWords;
  void *args[] = {&src, &n, &dst, const_cast<uint32_t *>(&seq)};
  hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(&publish_kernel),
                                 dim3(test == kReadRefuse ? 0 : 1),
                                 dim3(64), args, 0, s);
  if (e != hipSuccess) {   // refused: nothing will store to the slot
    (void)hipGetLastError();
    g_read.busy.fetch_and(~(1u << slot));
    return read_words_copy(src, n, out, s);
  }
  auto arrived = [&] {
    for (int i = 0; i < n; ++i) {
      const uint64_t v = __atomic_load_n(h + i, __ATOMIC_ACQUIRE);
      if ((uint32_t)(v >> 32) != seq) return false;
      static_cast<uint32_t *>(out)[i] = (uint32_t)v;
    }
    return true;
  };
  bool ok = false;
  {
    const auto until = std::chrono::steady_clock::now() + kPollLimit;
    do {
      for (int k = 0; k < 64 && !(ok = arrived()); ++k) __builtin_ia32_pause();
    } while (!ok && std::chrono::steady_clock::now() < until);
    if (!ok) {
      e = hipStreamSynchronize(s);
      ok = arrived();
    }
  }
  // after a failure the kernel may still store: the slot stays taken
  if (ok || e == hipSuccess) g_read.busy.fetch_and(~(1u << slot));
  return ok ? hipSuccess : (e != hipSuccess ? e : hipErrorUnknown);
}

}  // namespace gmm_host
