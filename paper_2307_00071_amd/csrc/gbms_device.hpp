// Mean shift with a flat kernel over binned seeds (device code, included by
// gbms.hip): the estimate of the number of mixture components that precedes
// k-means++ seeding and EM (the paper, Sec. V "Gaussian Blurring Mean Shift"
// and the information-flow figure: bandwidth + point cloud -> K).
//
// Seeds are the centres b h of the occupied bins b = rint(x / h) (Comaniciu
// and Meer's binned estimator); a seed moves to the mean of the points within
// distance h of it until the move is at most 1e-3 h or the iteration cap is
// reached; its weight is the size of that last neighbourhood.  Modes are then
// merged: in the order (weight descending, coordinates descending, seed
// ascending) a mode still kept removes every later mode within h.
//
// GPU design:
//   * a uniform grid of cell side h, the cells being the bins themselves:
//     the points are sorted by the 64-bit packed bin key (stable LSD radix
//     sort, radix_device.hpp), the occupied cells are the runs of equal keys
//     (so the seeds come out in lexicographic bin order) and an open-
//     addressing hash table maps a key to its cell;
//   * one wave per seed: a ball of radius h around s overlaps at most four
//     cells per axis, and cell k goes to the slot given by k mod 4 on every
//     axis (4^D slots, lane = slot mod 64), so the cell that holds a point
//     reaches the same lane whatever s is: the neighbourhood sum is then a
//     function of the neighbourhood alone (each lane adds its cells' points
//     in sorted order, rounds in order, then a fixed DPP reduction: within
//     each 16-lane row, then the rows in order), and seeds
//     that reach the same neighbourhood get bitwise the same mean;
//   * the merge never sorts the modes: mode i is kept iff no kept mode that
//     precedes it lies within h, so it needs only the predecessors within h
//     (a second grid, over the modes).  Passes decide, in place, every mode
//     whose predecessors within h are all decided; each pass decides at
//     least the first undecided mode of the order, so the passes end.
// All arithmetic that decides a neighbourhood, a bin, a stop or a merge is
// FP64 with every product and sum rounded on its own (no contraction), in the
// order ((d0^2 + d1^2) + d2^2) + d3^2.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "radix_device.hpp"
#include "wave_f64.hpp"

#pragma clang fp contract(off)

namespace gbms_dev {

using namespace gmm_wave;

using gmm_dev::kSortChunk;
using gmm_dev::kSortItems;
using gmm_dev::kSortThreads;

constexpr int kMsThreads = 256;
constexpr int kMsWaves = kMsThreads / 64;   // seeds (or modes) per block
constexpr uint64_t kNoKey = ~0ull;          // empty hash slot; no real key has it
constexpr int kRoundBatch = 2;              // merge launches per host check

// device status bits
constexpr uint32_t kMsNonFinite = 1u;
constexpr uint32_t kMsRange = 2u;

__device__ inline void ms_set_status(uint32_t *st, uint32_t bit) { atomicOr(st, bit); }

// Bin keys: D fields of kBits[D] bits, the first coordinate most
// significant, each holding b + 2^(bits - 1) with |b| <= 2^(bits - 1) - 2,
// so that key order is the lexicographic order of the bins and no key is
// all ones.
template <int D> struct KeyBits;
template <> struct KeyBits<3> { static constexpr int v = 21; };
template <> struct KeyBits<4> { static constexpr int v = 16; };

template <int D>
__device__ __forceinline__ int64_t bin_limit() {
  return (int64_t(1) << (KeyBits<D>::v - 1)) - 2;
}

template <int D>
__device__ __forceinline__ bool pack_key(const int64_t *b, uint64_t *key) {
  constexpr int B = KeyBits<D>::v;
  const int64_t lim = bin_limit<D>();
  uint64_t k = 0;
#pragma unroll
  for (int j = 0; j < D; ++j) {
    if (b[j] < -lim || b[j] > lim) return false;
    k = (k << B) | (uint64_t)(b[j] + (int64_t(1) << (B - 1)));
  }
  *key = k;
  return true;
}

template <int D>
__device__ __forceinline__ void unpack_key(uint64_t key, int64_t *b) {
  constexpr int B = KeyBits<D>::v;
#pragma unroll
  for (int j = D - 1; j >= 0; --j) {
    b[j] = (int64_t)(key & ((uint64_t(1) << B) - 1)) - (int64_t(1) << (B - 1));
    key >>= B;
  }
}

// SplitMix64's output mix (Steele, Lea and Flood 2014) as the hash.
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z ^= z >> 30;
  z *= 0xbf58476d1ce4e5b9ull;
  z ^= z >> 27;
  z *= 0x94d049bb133111ebull;
  z ^= z >> 31;
  return z;
}

__device__ __forceinline__ int hash_find(const uint64_t *__restrict__ hk,
                                         const int *__restrict__ hv, uint64_t mask,
                                         uint64_t key) {
  uint64_t s = mix64(key) & mask;
  for (;;) {
    const uint64_t k = hk[s];
    if (k == key) return hv[s];
    if (k == kNoKey) return -1;
    s = (s + 1) & mask;
  }
}

// ((d0^2 + d1^2) + d2^2) (+ d3^2), each operation rounded on its own.
template <int D>
__device__ __forceinline__ double sq_norm(const double *d) {
  double q = d[0] * d[0] + d[1] * d[1];
#pragma unroll
  for (int j = 2; j < D; ++j) q = q + d[j] * d[j];
  return q;
}

// ------------------------------------------------------------ point keys
// Key of point i from b_j = rint(x_j / h) in FP64; vals[i] = i.
template <int D>
__global__ __launch_bounds__(kSortThreads) void ms_point_key_kernel(
    const float *__restrict__ pts, int64_t n, double h, unsigned *__restrict__ klo,
    unsigned *__restrict__ khi, unsigned *__restrict__ vals, uint32_t *__restrict__ status) {
  const int64_t i = (int64_t)blockIdx.x * kSortThreads + threadIdx.x;
  if (i >= n) return;
  int64_t b[D];
  bool fin = true;
#pragma unroll
  for (int j = 0; j < D; ++j) {
    const double x = (double)pts[i * D + j];
    fin = fin && isfinite(x);
    const double r = rint(x / h);
    b[j] = (fabs(r) < 4.0e18) ? (int64_t)r : 0;
  }
  uint64_t key = 0;
  if (!fin) {
    ms_set_status(status, kMsNonFinite);
  } else if (!pack_key<D>(b, &key)) {
    ms_set_status(status, kMsRange);
  }
  klo[i] = (unsigned)key;
  khi[i] = (unsigned)(key >> 32);
  vals[i] = (unsigned)i;
}

// out[i] = in[perm[i]] (32-bit words)
__global__ __launch_bounds__(kSortThreads) void ms_gather_u32_kernel(
    const unsigned *__restrict__ in, const unsigned *__restrict__ perm,
    const int *__restrict__ np, int64_t nmax, unsigned *__restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * kSortThreads + threadIdx.x;
  const int64_t n = np ? (int64_t)*np : nmax;
  if (i < n) out[i] = in[perm[i]];
}

// Sorted 64-bit keys and the points' sorted float4 copies.
template <int D>
__global__ __launch_bounds__(kSortThreads) void ms_sorted_kernel(
    const unsigned *__restrict__ klo, const unsigned *__restrict__ khi,
    const unsigned *__restrict__ perm, const float *__restrict__ pts, int64_t n,
    uint64_t *__restrict__ keys, float4 *__restrict__ ptsS) {
  const int64_t i = (int64_t)blockIdx.x * kSortThreads + threadIdx.x;
  if (i >= n) return;
  const unsigned p = perm[i];
  keys[i] = ((uint64_t)khi[p] << 32) | klo[p];
  const float *x = pts + (size_t)p * D;
  ptsS[i] = make_float4(x[0], x[1], x[2], D == 4 ? x[3] : 0.0f);
}

// ------------------------------------------------- flags and their scan
// Two flag kinds over n items: a new run of sorted keys (FLAG_CELL), or a
// kept mode (FLAG_KEPT).  Each block takes a chunk of kSortChunk items,
// thread t the kSortItems consecutive items from t kSortItems on.
enum { FLAG_CELL = 0, FLAG_KEPT = 1 };

template <int KIND>
__device__ __forceinline__ bool item_flag(const uint64_t *keys, const int *status, int64_t i) {
  if (KIND == FLAG_CELL) return i == 0 || keys[i] != keys[i - 1];
  return status[i] == 1;
}

template <int KIND>
__global__ __launch_bounds__(kSortThreads) void ms_flag_count_kernel(
    const uint64_t *__restrict__ keys, const int *__restrict__ status,
    const int *__restrict__ np, int64_t nmax, unsigned *__restrict__ bsum) {
  __shared__ unsigned wsum[kSortThreads / 64];
  const int64_t n = np ? (int64_t)*np : nmax;
  const int64_t base = (int64_t)blockIdx.x * kSortChunk + (int64_t)threadIdx.x * kSortItems;
  unsigned c = 0;
#pragma unroll
  for (int u = 0; u < kSortItems; ++u) {
    const int64_t i = base + u;
    if (i < n && item_flag<KIND>(keys, status, i)) ++c;
  }
  unsigned tot = 0;
  (void)gmm_dev::block_exclusive_scan256(c, wsum, &tot);
  if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// FLAG_CELL: start[cell] = first sorted index of the cell, ckey[cell] = its
// key.  FLAG_KEPT: the kept modes in seed order into (out_mode, out_w).
// boff = the exclusive scan of the block counts.
template <int KIND, int D>
__global__ __launch_bounds__(kSortThreads) void ms_flag_write_kernel(
    const uint64_t *__restrict__ keys, const int *__restrict__ status,
    const int *__restrict__ np, int64_t nmax, const unsigned *__restrict__ boff,
    int *__restrict__ start, uint64_t *__restrict__ ckey,
    const double *__restrict__ mode, const int *__restrict__ weight,
    double *__restrict__ out_mode, long long *__restrict__ out_w, int64_t out_cap) {
  __shared__ unsigned wsum[kSortThreads / 64];
  const int64_t n = np ? (int64_t)*np : nmax;
  const int64_t base = (int64_t)blockIdx.x * kSortChunk + (int64_t)threadIdx.x * kSortItems;
  unsigned c = 0;
  bool f[kSortItems];
#pragma unroll
  for (int u = 0; u < kSortItems; ++u) {
    const int64_t i = base + u;
    f[u] = i < n && item_flag<KIND>(keys, status, i);
    c += f[u] ? 1u : 0u;
  }
  unsigned tot = 0;
  unsigned pos = boff[blockIdx.x] + gmm_dev::block_exclusive_scan256(c, wsum, &tot);
#pragma unroll
  for (int u = 0; u < kSortItems; ++u) {
    if (!f[u]) continue;
    const int64_t i = base + u;
    if (KIND == FLAG_CELL) {
      start[pos] = (int)i;
      ckey[pos] = keys[i];
    } else if ((int64_t)pos < out_cap) {
#pragma unroll
      for (int j = 0; j < D; ++j) out_mode[(size_t)pos * D + j] = mode[(size_t)i * D + j];
      if (out_w) out_w[pos] = (long long)weight[i];
    }
    ++pos;
  }
}

// start[ncells] = n; the cell count to *count.
__global__ void ms_cells_end_kernel(const unsigned *__restrict__ dtot,
                                    const int *__restrict__ np, int64_t nmax,
                                    int *__restrict__ start, int *__restrict__ count) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const int nc = (int)dtot[0];
  start[nc] = np ? *np : (int)nmax;
  *count = nc;
}

// ---------------------------------------------------------------- hashing
__global__ __launch_bounds__(kSortThreads) void ms_hash_clear_kernel(
    uint64_t *__restrict__ hk, uint64_t cap) {
  const uint64_t i = (uint64_t)blockIdx.x * kSortThreads + threadIdx.x;
  if (i < cap) hk[i] = kNoKey;
}

// Cell c's key into the table.
__global__ __launch_bounds__(kSortThreads) void ms_hash_insert_kernel(
    const uint64_t *__restrict__ ckey, const int *__restrict__ ncp,
    uint64_t *__restrict__ hk, int *__restrict__ hv, uint64_t mask) {
  const int c = blockIdx.x * kSortThreads + threadIdx.x;
  if (c >= *ncp) return;
  const uint64_t key = ckey[c];
  if (key == kNoKey) return;
  uint64_t s = mix64(key) & mask;
  for (;;) {
    const unsigned long long prev =
        atomicCAS(reinterpret_cast<unsigned long long *>(hk + s),
                  (unsigned long long)kNoKey, (unsigned long long)key);
    if (prev == (unsigned long long)kNoKey) {
      hv[s] = c;
      return;
    }
    s = (s + 1) & mask;
  }
}

// ------------------------------------------------------- the grid query
// Cells whose bins can hold a point within h of s: per axis the bins from
// ceil(s/h - 1.5) to floor(s/h + 1.5), widened by 1e-7 (rounding of x / h
// and of the distance test); at most four per axis.  Slot u (4^D of them)
// stands for the cell whose bin is congruent to the base-4 digits of u on
// every axis; the slot is skipped when that bin is outside the range or its
// box is farther than h from s.  With a slack (below 1/2), the same for every
// point within slack h of s.
template <int D>
struct GridQuery {
  double t[D];
  int lo[D], nr[D];
  __device__ __forceinline__ void init(const double *s, double h, double slack = 0.0) {
#pragma unroll
    for (int j = 0; j < D; ++j) {
      t[j] = s[j] / h;
      lo[j] = (int)ceil(t[j] - 1.5 - slack - 1e-7);
      nr[j] = (int)floor(t[j] + 1.5 + slack + 1e-7) - lo[j] + 1;
    }
  }
  __device__ __forceinline__ bool slot_key(int u, uint64_t *key, double slack = 0.0) const {
    int64_t k[D];
    double g2 = 0.0;
    bool ok = true;
#pragma unroll
    for (int j = 0; j < D; ++j) {
      const int r = (u >> (2 * (D - 1 - j))) & 3;
      const int off = (r - lo[j]) & 3;
      k[j] = (int64_t)lo[j] + off;
      ok = ok && off < nr[j];
      const double g = fabs(t[j] - (double)k[j]) - 0.5;
      if (g > 0.0) g2 = g2 + g * g;
    }
    ok = ok && g2 <= (1.0 + slack) * (1.0 + slack) * (1.0 + 1e-6);
    return ok && pack_key<D>(k, key);
  }
};

// -------------------------------------------------------------- mean shift
// Cells with at most kMsSerial points are walked by the lane that owns their
// slot; larger cells by the whole wave (point p of a cell starting at b goes
// to lane (p - b) mod 64), one cell after another in slot order.  Every lane
// therefore sums its points in an order fixed by the cells alone: the mean
// of an iterate depends only on the set of points within h of it.
constexpr int kMsSerial = 16;
// At most this many seeds: a block per seed.  What decides is the longest
// chain and the size of a neighbourhood; the seeds' number stands for both.
// Calls, block per seed against wave per seed: 13,301 seeds of an image (4D)
// 1.57 and 3.63 ms; a few points a cell 15,529 0.61 and 0.62, 17,286 0.61 and
// 0.54, 24,966 0.81 and 0.68, 44,910 1.49 and 1.47.  (Images of more seeds
// would gain by the block too: 17,844 1.49 and 3.75, 29,796 1.65 and 2.45.)
constexpr int kMsBlockSeeds = 16384;

template <int D>
__device__ __forceinline__ void ms_take(const float4 &x, bool ok, const double *s, double h2,
                                        double *acc, int &in) {
  const double xv[4] = {(double)x.x, (double)x.y, (double)x.z, (double)x.w};
  double d[D];
#pragma unroll
  for (int j = 0; j < D; ++j) d[j] = xv[j] - s[j];
  if (ok && sq_norm<D>(d) <= h2) {
#pragma unroll
    for (int j = 0; j < D; ++j) acc[j] = acc[j] + xv[j];
    ++in;
  }
}

// One wave per seed (a cell, in sorted order = lexicographic bin order):
// mode, weight (the last neighbourhood's size; 0 = dropped) and the
// iteration count of the oracle's loop.
template <int D>
__global__ __launch_bounds__(kMsThreads) void ms_shift_kernel(
    const float4 *__restrict__ ptsS, const int *__restrict__ cstart,
    const uint64_t *__restrict__ ckey, const int *__restrict__ ncp,
    const uint64_t *__restrict__ hk, const int *__restrict__ hv, uint64_t mask,
    double h, int max_iter, double *__restrict__ mode, int *__restrict__ weight,
    int *__restrict__ iters, int *__restrict__ max_it, int thr) {
  const int lane = threadIdx.x & 63;
  const int c = blockIdx.x * kMsWaves + (threadIdx.x >> 6);
  const int ncells = *ncp;
  if (ncells <= thr) return;   // few seeds: ms_shift_block_kernel takes them
  if (c >= ncells) return;     // uniform per wave
  double s[D];
  {
    int64_t b[D];
    unpack_key<D>(ckey[c], b);
#pragma unroll
    for (int j = 0; j < D; ++j) s[j] = (double)b[j] * h;
  }
  const double h2 = h * h;
  const double stop = 1e-3 * h;
  int it = 0, cnt = 0;
  for (;;) {
    GridQuery<D> g;
    g.init(s, h);
    double acc[D];
#pragma unroll
    for (int j = 0; j < D; ++j) acc[j] = 0.0;
    int in = 0;
    for (int u0 = 0; u0 < (1 << (2 * D)); u0 += 64) {
      int b = 0, e = 0;
      uint64_t key;
      if (g.slot_key(u0 + lane, &key)) {
        const int id = hash_find(hk, hv, mask, key);
        if (id >= 0) {
          b = cstart[id];
          e = cstart[id + 1];
        }
      }
      const bool wide = e - b > kMsSerial;
      if (!wide) {
        for (int p0 = b; p0 < e; p0 += 4) {
          float4 x[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) x[k] = ptsS[min(p0 + k, e - 1)];
#pragma unroll
          for (int k = 0; k < 4; ++k) ms_take<D>(x[k], p0 + k < e, s, h2, acc, in);
        }
      }
      uint64_t big = __ballot(wide);
      while (big) {
        const int o = __builtin_ctzll(big);
        big &= big - 1;
        const int cb = __builtin_amdgcn_readlane(b, o);
        const int ce = __builtin_amdgcn_readlane(e, o);
        for (int p0 = cb + lane; p0 < ce; p0 += 256) {
          float4 x[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) x[k] = ptsS[min(p0 + 64 * k, ce - 1)];
#pragma unroll
          for (int k = 0; k < 4; ++k) ms_take<D>(x[k], p0 + 64 * k < ce, s, h2, acc, in);
        }
      }
    }
#pragma unroll
    for (int j = 0; j < D; ++j) acc[j] = wave_sum_f64(acc[j]);
    in = wave_sum_i32(in);
    if (in == 0) break;   // uniform: every lane holds the same sums
    cnt = in;
    double d[D];
#pragma unroll
    for (int j = 0; j < D; ++j) {
      const double v = acc[j] / (double)in;
      d[j] = v - s[j];
      s[j] = v;
    }
    if (sqrt(sq_norm<D>(d)) <= stop || it == max_iter) break;
    ++it;
  }
  if (lane == 0) {
#pragma unroll
    for (int j = 0; j < D; ++j) mode[(size_t)c * D + j] = s[j];
    weight[c] = cnt;
    iters[c] = it;
    atomicMax(max_it, it);
  }
}

// The same shift with a block of kMsSeedWaves waves on one seed, for calls
// with at most `thr` seeds (few seeds, large neighbourhoods: the time is the
// slowest seed's chain of iterations).  Thread t < 4^D holds slot t; a cell
// is cut into pieces of 64 points; piece p of the cell in slot t is wave
// (home(t) + p) mod kMsSeedWaves's, which takes its pieces in slot order; the
// wave sums are added in wave order.  Every lane's order is again fixed by
// the cells alone.
//
// The list of pieces is made for all positions within kMsSlack h of s and
// serves until s has left that range (a long chain moves by little more than
// the stop's 1e-3 h a step); the first kMsKeep pieces of a wave stay in
// registers meanwhile.  An iteration that keeps the list has one barrier and,
// up to kMsKeep pieces a wave, no loads.
// Measured on clouds with the seeds of images (76,800 points, 4D; 10,972
// seeds, 71,000 iterations, longest chain 268): the kernel 2.6 -> 1.4 ms
// against four waves a seed that look every cell up again and load every
// point in each iteration; 300,000 points, 3D (2,916 seeds, cap of 300
// reached): the call 3.8 -> 2.4 ms.  Four waves a seed with this list: calls
// 2.5 and 3.2 ms.  What is left is FP64 arithmetic (21 instructions a point)
// and, for the bulk of the seeds, the making of the list.
constexpr int kMsSeedWaves = 8;
constexpr int kMsKeep = 8;
constexpr double kMsSlack = 1.0 / 16;

template <int D>
__device__ __forceinline__ void ms_take_piece(const float4 &x, const double *s, double h2,
                                              double *acc, int &in) {
  const double xv[4] = {(double)x.x, (double)x.y, (double)x.z, (double)x.w};
  double d[D];
#pragma unroll
  for (int j = 0; j < D; ++j) d[j] = xv[j] - s[j];
  const bool t = sq_norm<D>(d) <= h2;   // (NaN: a lane past the cell's end)
  in += __popcll(__ballot(t));
  if (t) {
#pragma unroll
    for (int j = 0; j < D; ++j) acc[j] = acc[j] + xv[j];
  }
}

template <int D>
__global__ __launch_bounds__(64 * kMsSeedWaves, 4) void ms_shift_block_kernel(
    const float4 *__restrict__ ptsS, const int *__restrict__ cstart,
    const uint64_t *__restrict__ ckey, const int *__restrict__ ncp,
    const uint64_t *__restrict__ hk, const int *__restrict__ hv, uint64_t mask,
    double h, int max_iter, double *__restrict__ mode, int *__restrict__ weight,
    int *__restrict__ iters, int *__restrict__ max_it, int thr) {
  constexpr int NW = kMsSeedWaves;
  constexpr int NS = 1 << (2 * D), NR = NS / 64;
  static_assert(NS <= 64 * NW && (NW & (NW - 1)) == 0, "a thread per slot");
  __shared__ int2 list[NW][NS];   // a wave's pieces: first point, end of the cell
  __shared__ int num[NW][NR];     // of the slots of each wave
  __shared__ double part[2][NW][D + 1];
  const int ncells = *ncp;
  if (ncells > thr) return;                 // many seeds: ms_shift_kernel takes them
  const int c = blockIdx.x;
  if (c >= ncells) return;                  // uniform per block
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  // neighbouring cells to different waves
  const int home =
      ((tid & 3) + 3 * (tid >> 2 & 3) + 5 * (tid >> 4 & 3) + 7 * (tid >> 6 & 3)) & (NW - 1);
  double s[D];
  {
    int64_t b[D];
    unpack_key<D>(ckey[c], b);
#pragma unroll
    for (int j = 0; j < D; ++j) s[j] = (double)b[j] * h;
  }
  const double h2 = h * h;
  const double stop = 1e-3 * h;
  const double reach = kMsSlack * h * (1.0 - 1e-9);
  const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  uint64_t held = kNoKey;   // the bin whose cell is [cb, ce)
  int cb = 0, ce = 0;
  int it = 0, cnt = 0;
  for (bool more = true; more;) {
    if (tid < NS) {
      GridQuery<D> g;
      g.init(s, h, kMsSlack);
      int pieces = 0;
      uint64_t key;
      if (g.slot_key(tid, &key, kMsSlack)) {
        if (key != held) {
          held = key;
          const int id = hash_find(hk, hv, mask, key);
          cb = id >= 0 ? cstart[id] : 0;
          ce = id >= 0 ? cstart[id + 1] : 0;
        }
        pieces = (ce - cb + 63) >> 6;
      }
#pragma unroll
      for (int v = 0; v < NW; ++v) {
        const int p = (v - home) & (NW - 1);
        const uint64_t m = __ballot(p < pieces);
        if (p < pieces) list[v][64 * w + __popcll(m & below)] = make_int2(cb + 64 * p, ce);
        if (lane == 0) num[v][w] = __popcll(m);
      }
    }
    __syncthreads();
    int upto[NR];   // pieces of the slots of waves 0 .. r
#pragma unroll
    for (int r = 0; r < NR; ++r)
      upto[r] = __builtin_amdgcn_readfirstlane(num[w][r]) + (r ? upto[r ? r - 1 : 0] : 0);
    const int mine = upto[NR - 1];
    // cell k of this wave: its first point here, the cell's end
    auto cell = [&](int k) {
      int at = k;
#pragma unroll
      for (int r = 0; r + 1 < NR; ++r)
        if (k >= upto[r]) at = 64 * (r + 1) + k - upto[r];
      const int2 u = list[w][at];
      return make_int2(__builtin_amdgcn_readfirstlane(u.x), __builtin_amdgcn_readfirstlane(u.y));
    };
    // the wave's pieces in order: cell k, its piece [u.x, u.x + 64) of [.., u.y);
    // past the last one u is a piece of no points, whose loads are in range
    struct Cursor {
      int k;
      int2 u;
    };
    auto first = [&]() { return Cursor{0, mine > 0 ? cell(0) : make_int2(64, 1)}; };
    auto next = [&](Cursor &q) {
      q.u.x += 64 * NW;
      if (q.u.x >= q.u.y && q.k < mine && ++q.k < mine) q.u = cell(q.k);
    };
    float4 kept[kMsKeep];
    Cursor rest = first();
    int nk = 0;
    bool none[kMsKeep];
#pragma unroll
    for (int k = 0; k < kMsKeep; ++k) {
      const int p = rest.u.x + lane;
      kept[k] = ptsS[min(p, rest.u.y - 1)];
      none[k] = p >= rest.u.y;
      nk += rest.k < mine;
      next(rest);
    }
#pragma unroll
    for (int k = 0; k < kMsKeep; ++k)
      if (none[k]) kept[k].x = __builtin_nanf("");
    double s0[D];
#pragma unroll
    for (int j = 0; j < D; ++j) s0[j] = s[j];
    for (;;) {
      double acc[D];
#pragma unroll
      for (int j = 0; j < D; ++j) acc[j] = 0.0;
      int in = 0;
#pragma unroll
      for (int k = 0; k < kMsKeep; ++k)
        if (k < nk) {
          // (opaque, or the conversions to FP64 are kept too: 16 registers a piece)
          asm volatile("" : "+v"(kept[k].x), "+v"(kept[k].y), "+v"(kept[k].z), "+v"(kept[k].w));
          ms_take_piece<D>(kept[k], s, h2, acc, in);
        }
      for (Cursor q = rest; q.k < mine;) {
        float4 x[4];
        bool none[4];
        int m = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int p = q.u.x + lane;
          x[k] = ptsS[min(p, q.u.y - 1)];
          none[k] = p >= q.u.y;
          m += q.k < mine;
          next(q);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (k < m) {
            if (none[k]) x[k].x = __builtin_nanf("");
            ms_take_piece<D>(x[k], s, h2, acc, in);
          }
      }
      double (*pt)[D + 1] = part[it & 1];
#pragma unroll
      for (int j = 0; j < D; ++j) acc[j] = wave_sum_f64(acc[j]);
      if (lane == 0) {
#pragma unroll
        for (int j = 0; j < D; ++j) pt[w][j] = acc[j];
        pt[w][D] = (double)in;
      }
      __syncthreads();
      // lane j: coordinate j (the count in every lane)
      const int col = lane < D ? lane : D;
      double tot = pt[0][col], tin = pt[0][D];
#pragma unroll
      for (int v = 1; v < NW; ++v) {
        tot = tot + pt[v][col];
        tin += pt[v][D];
      }
      if (tin == 0.0) {   // uniform: every wave read the same sums
        more = false;
        break;
      }
      cnt = (int)tin;
      const double mean = tot / tin;
      double d[D], m[D];
#pragma unroll
      for (int j = 0; j < D; ++j) {
        const double v = readlane_f64(mean, j);
        d[j] = v - s[j];
        s[j] = v;
        m[j] = v - s0[j];
      }
      const double q = sq_norm<D>(d);
      // (the root only where it can decide)
      if ((q <= stop * stop * (1.0 + 1e-9) + 1e-300 && sqrt(q) <= stop) || it == max_iter) {
        more = false;
        break;
      }
      ++it;
      if (!(sq_norm<D>(m) <= reach * reach)) break;   // a new list
    }
  }
  if (tid == 0) {
#pragma unroll
    for (int j = 0; j < D; ++j) mode[(size_t)c * D + j] = s[j];
    weight[c] = cnt;
    iters[c] = it;
    atomicMax(max_it, it);
  }
}

// ------------------------------------------------------------------ merge
// status: 0 undecided, 1 kept, 2 removed by a kept mode, 3 dropped seed.
//
// The grid over the modes needs no order, so it is not sorted: every mode
// takes a place in its cell's hash slot, the slots take ranges, and the modes
// are written to them (three short launches; sorted like the points' it took
// thirty, 190 us at 76,800 points).
__global__ __launch_bounds__(kSortThreads) void ms_mode_clear_kernel(
    uint64_t *__restrict__ hk, int *__restrict__ hcount, uint64_t cap, int *__restrict__ used) {
  const uint64_t i = (uint64_t)blockIdx.x * kSortThreads + threadIdx.x;
  if (i == 0) *used = 0;
  if (i < cap) {
    hk[i] = kNoKey;
    hcount[i] = 0;
  }
}

// slot[i], rank[i]: mode i's place; rank -1 for a dropped seed.
template <int D>
__global__ __launch_bounds__(kSortThreads) void ms_mode_insert_kernel(
    const double *__restrict__ mode, const int *__restrict__ weight,
    const int *__restrict__ nsp, double h, uint64_t *__restrict__ hk, int *__restrict__ hcount,
    uint64_t mask, unsigned *__restrict__ slot, int *__restrict__ rank,
    int *__restrict__ status) {
  const int i = blockIdx.x * kSortThreads + threadIdx.x;
  if (i >= *nsp) return;
  const bool live = weight[i] > 0;
  status[i] = live ? 0 : 3;
  rank[i] = -1;
  int64_t b[D];
  uint64_t key;
#pragma unroll
  for (int j = 0; j < D; ++j) b[j] = (int64_t)rint(mode[(size_t)i * D + j] / h);
  if (!live || !pack_key<D>(b, &key)) return;   // (modes are means of points: in range)
  uint64_t s = mix64(key) & mask;
  for (;;) {
    const unsigned long long prev =
        atomicCAS(reinterpret_cast<unsigned long long *>(hk + s),
                  (unsigned long long)kNoKey, (unsigned long long)key);
    if (prev == (unsigned long long)kNoKey || prev == (unsigned long long)key) break;
    s = (s + 1) & mask;
  }
  slot[i] = (unsigned)s;
  rank[i] = atomicAdd(&hcount[s], 1);
}

// The first mode of a slot takes the slot's range.
__global__ __launch_bounds__(kSortThreads) void ms_mode_range_kernel(
    const int *__restrict__ nsp, const unsigned *__restrict__ slot, const int *__restrict__ rank,
    const int *__restrict__ hcount, int *__restrict__ hstart, int *__restrict__ used) {
  __shared__ unsigned wsum[kSortThreads / 64];
  __shared__ int base;
  const int i = blockIdx.x * kSortThreads + threadIdx.x;
  if ((int)blockIdx.x * kSortThreads >= *nsp) return;   // uniform
  const bool take = i < *nsp && rank[i] == 0;
  unsigned tot = 0;
  const unsigned off =
      gmm_dev::block_exclusive_scan256(take ? (unsigned)hcount[slot[i]] : 0u, wsum, &tot);
  if (threadIdx.x == 0) base = atomicAdd(used, (int)tot);
  __syncthreads();
  if (take) hstart[slot[i]] = base + (int)off;
}

__global__ __launch_bounds__(kSortThreads) void ms_mode_fill_kernel(
    const int *__restrict__ nsp, const unsigned *__restrict__ slot, const int *__restrict__ rank,
    const int *__restrict__ hstart, int *__restrict__ perm2) {
  const int i = blockIdx.x * kSortThreads + threadIdx.x;
  if (i < *nsp && rank[i] >= 0) perm2[hstart[slot[i]] + rank[i]] = i;
}

// cnt[0] = carry, cnt[1 .. kRoundBatch] = 0 (carry: the undecided count of
// the previous batch's last launch, or 1 before the first); the passes of
// each launch behind them.
__global__ void ms_round_clear_kernel(unsigned *__restrict__ cnt, int first) {
  const int t = threadIdx.x;
  const unsigned carry = first ? 1u : cnt[kRoundBatch];
  __syncthreads();
  if (t <= 2 * kRoundBatch) cnt[t] = (t == 0) ? carry : 0u;
}

// Does mode j come before mode i in the merge order?
template <int D>
__device__ __forceinline__ bool precedes(int j, int wj, const double *mj, int i, int wi,
                                         const double *mi) {
  if (wj != wi) return wj > wi;
#pragma unroll
  for (int k = 0; k < D; ++k)
    if (mj[k] != mi[k]) return mj[k] > mi[k];
  return j < i;
}

// Merge passes, one wave per undecided mode (wave k has modes k, k + waves,
// ...): a mode is removed if a kept predecessor lies within h, kept if every
// predecessor within h is decided and none is kept, else looked at again in
// the next pass.  A launch ends when its modes are decided or after
// kMergePasses (no wave waits for a block that has not started); what is
// left is counted in cnt[launch].
//
// The first pass spreads the modes of all the cells in reach over the lanes,
// and keeps the undecided predecessors of a wave's first kMergeOwn modes (up
// to kMergeList each) in LDS: a later pass reads their status alone.  One
// launch a round, a lane per cell, took 155, 89, 37, ... 14 us for the 17
// rounds of 10,972 modes (600 us with the idle launches to the host's check);
// this takes 73 us.
constexpr int kMergeBlocks = 1024;
constexpr int kMergePasses = 64;
constexpr int kMergeOwn = 4;
constexpr int kMergeList = 128;

__device__ __forceinline__ int ms_status_load(const int *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int D>
__global__ __launch_bounds__(kMsThreads) void ms_merge_kernel(
    const double *__restrict__ mode, const int *__restrict__ weight,
    const int *__restrict__ nsp, const int *__restrict__ perm2,
    const int *__restrict__ hstart, const int *__restrict__ hcount,
    const uint64_t *__restrict__ hk, uint64_t mask, double h, int *status,
    unsigned *__restrict__ cnt, int launch) {
  __shared__ int held[kMsWaves][kMergeOwn][kMergeList];
  __shared__ int nheld[kMsWaves][kMergeOwn];   // -1: too many
  if (cnt[launch - 1] == 0u) return;   // every mode decided already
  const int ns = *nsp;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  const double h2 = h * h;
  const int stride = (int)gridDim.x * kMsWaves;
  unsigned left = 0;
  int pass = 0;
  for (; pass < kMergePasses; ++pass) {
    left = 0;
    int own = 0;
    for (int64_t ii = (int64_t)blockIdx.x * kMsWaves + w; ii < ns; ii += stride, ++own) {
      const int i = (int)ii;
      if (ms_status_load(status + i) != 0) continue;
      bool kept = false, open = false;
      const int nl = pass > 0 && own < kMergeOwn ? nheld[w][own] : -1;
      if (nl >= 0) {
        for (int q = lane; q < nl; q += 64) {
          const int st = ms_status_load(status + held[w][own][q]);
          kept = kept || st == 1;
          open = open || st == 0;
        }
      } else {
        double mi[D];
#pragma unroll
        for (int k = 0; k < D; ++k) mi[k] = mode[(size_t)i * D + k];
        const int wi = weight[i];
        GridQuery<D> g;
        g.init(mi, h);
        int listed = 0;   // uniform
        for (int u0 = 0; u0 < (1 << (2 * D)); u0 += 64) {
          int b = 0, c = 0;
          uint64_t key;
          if (g.slot_key(u0 + lane, &key)) {
            uint64_t s = mix64(key) & mask;
            for (;;) {
              const uint64_t k = hk[s];
              if (k == key) {
                b = hstart[s];
                c = hcount[s];
                break;
              }
              if (k == kNoKey) break;
              s = (s + 1) & mask;
            }
          }
          int upto = c;   // inclusive running count
          for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(upto, off, 64);
            if (lane >= off) upto += o;
          }
          const int total = __builtin_amdgcn_readlane(upto, 63);
          for (int q0 = 0; q0 < total; q0 += 64) {
            const int q = q0 + lane;
            int o = 0;   // the slot of the q-th mode
#pragma unroll
            for (int step = 32; step > 0; step >>= 1)
              if (__shfl(upto, o + step - 1, 64) <= q) o += step;
            o &= 63;   // (q past the end)
            const int p = __shfl(b, o, 64) + q - (__shfl(upto, o, 64) - __shfl(c, o, 64));
            bool pre = false;
            int j = 0;
            if (q < total) {
              j = perm2[p];
              const int st = j == i ? 2 : ms_status_load(status + j);
              if (st < 2) {
                double mj[D], d[D];
#pragma unroll
                for (int k = 0; k < D; ++k) {
                  mj[k] = mode[(size_t)j * D + k];
                  d[k] = mi[k] - mj[k];
                }
                if (sq_norm<D>(d) <= h2 && precedes<D>(j, weight[j], mj, i, wi, mi)) {
                  kept = kept || st == 1;
                  pre = st == 0;
                }
              }
            }
            open = open || pre;
            const uint64_t m = __ballot(pre);
            if (own < kMergeOwn) {
              const int at = listed + __popcll(m & below);
              if (pre && at < kMergeList) held[w][own][at] = j;
            }
            listed += __popcll(m);
          }
          if (__ballot(kept)) break;
        }
        if (own < kMergeOwn && lane == 0) nheld[w][own] = listed <= kMergeList ? listed : -1;
        __builtin_amdgcn_wave_barrier();   // the list is read by other lanes of the wave
      }
      const bool any_kept = __ballot(kept) != 0ull, any_open = __ballot(open) != 0ull;
      if (!any_kept && any_open) {
        ++left;
        continue;
      }
      if (lane == 0)
        __hip_atomic_store(status + i, any_kept ? 2 : 1, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    if (left == 0) break;
  }
  if (lane == 0) {
    if (left) atomicAdd(&cnt[launch], left);
    const unsigned passes = (unsigned)(pass < kMergePasses ? pass + 1 : pass);
    if (passes > 1 || blockIdx.x == 0) atomicMax(&cnt[kRoundBatch + launch], passes);
  }
}

// The status word and the counters to the host's info block.
struct MsCounters {
  int ncells;    // seeds
  int nmodes;    // modes in the mode grid
  int kept;      // K
  int max_it;
  uint32_t status;
};

__global__ void ms_init_kernel(MsCounters *__restrict__ c) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    c->ncells = 0;
    c->nmodes = 0;
    c->kept = 0;
    c->max_it = 0;
    c->status = 0u;
  }
}

}  // namespace gbms_dev
