// Runs one block of a HIP kernel on the CPU: every thread is a fiber that
// runs alone up to its next barrier or cross-lane operation.  The wave order
// of a step is chosen by the test, so an access that is not separated from
// another wave's by a barrier is seen in both orders.  A thread that waits
// at a block barrier while another thread of the block has returned ends the
// program: the barrier is not reached by the whole block.
#pragma once

#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <ucontext.h>

#include <functional>
#include <vector>

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __shared__ static
#define __launch_bounds__(...)

struct dim3 {
  unsigned x = 1, y = 1, z = 1;
};
struct double2 {
  double x, y;
};
inline double2 make_double2(double x, double y) { return {x, y}; }
using std::isfinite;

inline dim3 threadIdx, blockIdx, blockDim, gridDim;
inline uint32_t atomicOr(uint32_t *p, uint32_t v) {
  const uint32_t old = *p;
  *p |= v;
  return old;
}

namespace emulate {

constexpr int kWave = 64;
constexpr size_t kStack = 128 << 10;
enum State { kReady, kBlock, kLane, kDone };

struct Fiber {
  ucontext_t ctx;
  std::vector<char> stack;
  State state = kReady;
  double put = 0.0, got = 0.0;
  int mask = 0;   // partner of a lane exchange; -1: ballot
  uint64_t bits = 0;
};

inline std::vector<Fiber> fibers;
inline ucontext_t home;
inline int self = 0;
inline std::function<void()> body;

inline void entry() {
  body();
  fibers[self].state = kDone;
  swapcontext(&fibers[self].ctx, &home);
}

inline void wait(State s) {
  fibers[self].state = s;
  swapcontext(&fibers[self].ctx, &home);
}

// Every lane of a wave that has not returned waits: exchange and go on.
inline bool lanes_ready(int w0) {
  bool any = false;
  for (int i = w0; i < w0 + kWave; ++i) {
    if (fibers[i].state == kReady || fibers[i].state == kBlock) return false;
    any = any || fibers[i].state == kLane;
  }
  if (!any) return false;
  uint64_t bits = 0;
  for (int i = w0; i < w0 + kWave; ++i)
    if (fibers[i].state == kLane && fibers[i].put != 0.0) bits |= 1ull << (i - w0);
  for (int i = w0; i < w0 + kWave; ++i) {
    Fiber &f = fibers[i];
    if (f.state != kLane) continue;
    f.bits = bits;
    if (f.mask >= 0) f.got = fibers[w0 + ((i - w0) ^ f.mask)].put;
  }
  for (int i = w0; i < w0 + kWave; ++i)
    if (fibers[i].state == kLane) fibers[i].state = kReady;
  return true;
}

// One block of `threads` threads (whole waves); backwards: the last wave
// runs first in every step.
inline void run_block(int threads, bool backwards, std::function<void()> f) {
  body = std::move(f);
  blockDim.x = (unsigned)threads;
  fibers = std::vector<Fiber>((size_t)threads);
  for (Fiber &q : fibers) {
    q.stack.resize(kStack);
    getcontext(&q.ctx);
    q.ctx.uc_stack.ss_sp = q.stack.data();
    q.ctx.uc_stack.ss_size = kStack;
    q.ctx.uc_link = &home;
    makecontext(&q.ctx, entry, 0);
  }
  const int waves = threads / kWave;
  for (;;) {
    int blocked = 0, done = 0;
    for (int v = 0; v < waves; ++v) {
      const int w0 = kWave * (backwards ? waves - 1 - v : v);
      do {
        // (lanes from the last one down: lane 0, which often stores for the
        // wave, after the others have read, as in a wave in step)
        for (int i = w0 + kWave - 1; i >= w0; --i) {
          if (fibers[i].state != kReady) continue;
          self = i;
          threadIdx.x = (unsigned)i;
          swapcontext(&home, &fibers[i].ctx);
        }
      } while (lanes_ready(w0));
    }
    for (const Fiber &q : fibers) {
      blocked += q.state == kBlock;
      done += q.state == kDone;
    }
    if (done == threads) return;
    if (blocked != threads) {
      printf("barrier not reached by the whole block: %d wait, %d have returned, %d differ\n",
             blocked, done, threads - blocked - done);
      exit(1);
    }
    for (Fiber &q : fibers) q.state = kReady;
  }
}

}  // namespace emulate

inline void __syncthreads() { emulate::wait(emulate::kBlock); }
inline double __shfl_xor(double v, int mask, int) {
  emulate::Fiber &f = emulate::fibers[emulate::self];
  f.put = v;
  f.mask = mask;
  emulate::wait(emulate::kLane);
  return f.got;
}
inline uint64_t __ballot(int p) {
  emulate::Fiber &f = emulate::fibers[emulate::self];
  f.put = p ? 1.0 : 0.0;
  f.mask = -1;
  emulate::wait(emulate::kLane);
  return f.bits;
}
