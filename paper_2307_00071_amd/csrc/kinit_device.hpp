// kinit_device.hpp - k-means++ seeding on the device (the initialisation
// that precedes EM; the paper starts EM from a randomised k-means step,
// Sec. V).  D^2 seeding after Arthur & Vassilvitskii (2007), one trial per
// centre, hard nearest-seed labels.
//
// With K draws u[j] in [0, 1):
//   centre 0 = floor(u[0] N) (at most N - 1);
//   D2_i = squared distance from x_i to the nearest centre so far;
//   centre j = the first index whose running sum of D2 exceeds u[j] W,
//     W = sum D2 (so index i is drawn with probability D2_i / W); when
//     W = 0 centre j repeats centre j - 1;
//   label_i = the nearest centre, the lowest index on ties.
// The running sums have a fixed order so that the choice is reproducible:
// sequential within chunks of kKppChunk points, chunk totals sequential in
// runs of 16 from offsets formed by a block scan (kpp_select_kernel); the
// pick is the first positive entry above u W, else the last positive entry.
// Squared distances are ((dx^2 + dy^2) + dz^2) in double with every
// operation rounded on its own (no contraction).
//
// Clouds of up to kKppRoundChunks chunks take one launch per round
// (kpp_round_kernel, kpp_round_cull_kernel).  Larger ones take two: kpp_update_kernel (D2 with
// centre j - 1, chunk totals; it streams 28 B per point) and
// kpp_select_kernel (one block: W, the chunk, the point), then
// kpp_label_kernel.  The work is a chain of K dependent steps; none does
// enough arithmetic to meet a compute roofline.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gmm_dev {

constexpr int kKppChunk = 256;      // points per chunk (running-sum order)
constexpr int kKppSelThreads = 1024;
constexpr int kKppLabelThreads = 256;

__device__ __forceinline__ double kpp_d2(double a0, double a1, double a2, double b0,
                                         double b1, double b2) {
#pragma clang fp contract(off)
  const double d0 = a0 - b0, d1 = a1 - b1, d2 = a2 - b2;
  return (d0 * d0 + d1 * d1) + d2 * d2;
}

// Checks the draws and places centre 0.  One block.
__global__ __launch_bounds__(256) void kpp_first_kernel(const double *__restrict__ u, int K,
                                                        int64_t n, int64_t *__restrict__ cidx,
                                                        uint32_t *status) {
  for (int j = threadIdx.x; j < K; j += 256) {
    const double v = u[j];
    if (!(v >= 0.0 && v < 1.0)) set_status(status, kStBadArg);
  }
  if (threadIdx.x == 0) {
    const double v = u[0];
    int64_t c = (v >= 0.0 && v < 1.0) ? (int64_t)(v * (double)n) : 0;
    cidx[0] = c > n - 1 ? n - 1 : c;
  }
}

// D2 with centre j (the first round sets it) and the chunk totals.  A
// block of kKppUpdThreads threads takes kKppUpdChunks chunks; the D2 values
// go to LDS (one padded row per chunk), then lane c of wave 0 sums chunk c
// sequentially (the chains run side by side in one wave).
constexpr int kKppUpdThreads = 256;
constexpr int kKppUpdChunks = 4;
constexpr int kKppRow = kKppChunk + 1;  // padded LDS row (bank spread)
__global__ __launch_bounds__(kKppUpdThreads) void kpp_update_kernel(
    const float *__restrict__ pts, int64_t n, const int64_t *__restrict__ cidx, int j,
    double *__restrict__ D, double *__restrict__ T, int64_t nch, uint32_t *status) {
  __shared__ double sh[kKppUpdChunks * kKppRow];
  const int64_t c = cidx[j];
  const double c0 = pts[3 * c], c1 = pts[3 * c + 1], c2 = pts[3 * c + 2];
  const int64_t base = (int64_t)blockIdx.x * kKppUpdChunks * kKppChunk;
  constexpr int PER = kKppUpdChunks * kKppChunk / kKppUpdThreads;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int l = q * kKppUpdThreads + threadIdx.x;
    const int64_t i = base + l;
    double v = 0.0;  // past the end: 0, which leaves the running sums as they are
    if (i < n) {
      const float x0 = pts[3 * i], x1 = pts[3 * i + 1], x2 = pts[3 * i + 2];
      const double d = kpp_d2(x0, x1, x2, c0, c1, c2);
      if (j == 0) {
        if (!isfinite(x0) || !isfinite(x1) || !isfinite(x2)) set_status(status, kStNonFinite);
        v = d;
      } else {
        const double o = D[i];
        v = d < o ? d : o;
      }
      D[i] = v;
    }
    sh[(l / kKppChunk) * kKppRow + (l % kKppChunk)] = v;
  }
  __syncthreads();
  const int64_t ch = (int64_t)blockIdx.x * kKppUpdChunks + threadIdx.x;
  if (threadIdx.x < kKppUpdChunks && ch < nch) {
    const double *a = sh + threadIdx.x * kKppRow;
    double s = 0.0;
    for (int k0 = 0; k0 < kKppChunk; k0 += 16) {
      double e[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) e[k] = a[k0 + k];
#pragma unroll
      for (int k = 0; k < 16; ++k) s += e[k];
    }
    T[ch] = s;
  }
}

// ---- centre j >= 1: one block of kKppSelThreads threads.
// The running sums in index order are formed as: chunk totals (sequential
// over 256 points, kpp_update_kernel); kKppSelPer consecutive chunk totals
// per thread of a stage of kKppSelThreads x kKppSelPer chunks, sequential
// from the thread's offset; the thread offsets by a block scan of the
// thread sums (a shuffle scan in each wave, the wave totals in order); the
// stages in order.  Inside the chosen chunk the 256 D2 by the same block
// scan from the chunk's running sum.  The pick is the first positive entry
// whose running sum exceeds t = u_j W (the exact running sum is flat over
// zero entries, so none of them is ever the first above a level); where
// rounding leaves no entry above t, the last positive entry.
constexpr int kKppSelPer = 16;

// Exclusive prefix of v over a block of NT threads and the block total
// (*tot).  wtot: NT / 64 + 1 doubles of LDS.  Three barriers.
template <int NT>
__device__ __forceinline__ double kpp_block_scan(double v, double *wtot, double *tot) {
  constexpr int NWV = NT / 64;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  double s = v;
  for (int off = 1; off < 64; off <<= 1) {
    const double o = __shfl_up(s, off, 64);
    if (lane >= off) s += o;
  }
  double e = __shfl_up(s, 1, 64);
  if (lane == 0) e = 0.0;
  __syncthreads();   // wtot free
  if (lane == 63) wtot[w] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    double acc = 0.0;
    for (int k = 0; k < NWV; ++k) {
      const double t = wtot[k];
      wtot[k] = acc;
      acc += t;
    }
    wtot[NWV] = acc;
  }
  __syncthreads();
  *tot = wtot[NWV];
  return wtot[w] + e;
}

// hit = min of the indices `a` >= 0, lastp = max of the indices `l` >= 0
// over the block; indices grow with the lane, so per wave the first (last)
// flagged lane holds the wave's minimum (maximum): one LDS atomic per wave.
__device__ __forceinline__ void kpp_wave_mark(long long a, long long l,
                                              unsigned long long *hit, long long *lastp) {
  const int lane = threadIdx.x & 63;
  const uint64_t ab = __ballot(a >= 0), lb = __ballot(l >= 0);
  if (ab && lane == __builtin_ctzll(ab)) atomicMin(hit, (unsigned long long)a);
  if (lb && lane == 63 - __builtin_clzll(lb)) atomicMax(lastp, l);
}

// The pick of one round by a block of NT threads (all of them call it; all
// get the index): D the n squared distances, T their chunk totals; prev
// is returned when W is not positive.
template <int NT>
__device__ int64_t kpp_pick(const double *__restrict__ D, const double *__restrict__ T,
                            int64_t n, double uj, int64_t prev) {
  constexpr int64_t STAGE = (int64_t)NT * kKppSelPer;
  static_assert(NT >= kKppChunk, "a block covers a chunk");
  __shared__ double wtot[NT / 64 + 1];
  __shared__ unsigned long long hit;   // smallest index above t (~0: none)
  __shared__ long long lastp;          // largest positive index (-1: none)
  __shared__ double hbefore, lbefore;  // running sum before the hit / last
  __shared__ int64_t result;
  const int tid = threadIdx.x;
  const int64_t nch = (n + kKppChunk - 1) / kKppChunk;
  const int64_t nst = (nch + STAGE - 1) / STAGE;
  double v[kKppSelPer];
  double off = 0.0, stot = 0.0;
  auto stage = [&](int64_t st) {   // v, this thread's offset in the stage, the stage total
    const int64_t c0 = st * STAGE + (int64_t)tid * kKppSelPer;
#pragma unroll
    for (int q = 0; q < kKppSelPer; ++q) v[q] = (c0 + q < nch) ? T[c0 + q] : 0.0;
    double sum = 0.0;
#pragma unroll
    for (int q = 0; q < kKppSelPer; ++q) sum += v[q];
    off = kpp_block_scan<NT>(sum, wtot, &stot);
  };
  // W: the stage totals in order
  double W = 0.0;
  for (int64_t st = 0; st < nst; ++st) {
    stage(st);
    W += stot;
  }
  if (!(W > 0.0)) return prev;   // uniform
  const double t = uj * W;
  // the chunk: first positive chunk total whose running sum exceeds t
  int64_t c = -1, cl = -1;
  double cbefore = 0.0, clbefore = 0.0, base = 0.0;
  for (int64_t st = 0; st < nst; ++st) {
    if (nst > 1) stage(st);
    __syncthreads();
    if (tid == 0) {
      hit = ~0ull;
      lastp = -1;
    }
    __syncthreads();
    double acc = base + off;
    long long mine = -1, myl = -1;
    double mb = 0.0, mlb = 0.0;
#pragma unroll
    for (int q = 0; q < kKppSelPer; ++q) {
      const double nxt = acc + v[q];
      if (v[q] > 0.0) {
        if (mine < 0 && nxt > t) {
          mine = (long long)tid * kKppSelPer + q;
          mb = acc;
        }
        myl = (long long)tid * kKppSelPer + q;
        mlb = acc;
      }
      acc = nxt;
    }
    kpp_wave_mark(mine, myl, &hit, &lastp);
    __syncthreads();
    if (mine >= 0 && (unsigned long long)mine == hit) hbefore = mb;
    if (myl >= 0 && myl == lastp) lbefore = mlb;
    __syncthreads();
    if (hit != ~0ull) {
      c = st * STAGE + (int64_t)hit;
      cbefore = hbefore;
      break;
    }
    if (lastp >= 0) {
      cl = st * STAGE + lastp;
      clbefore = lbefore;
    }
    base += stot;
  }
  if (c < 0) {
    c = cl;
    cbefore = clbefore;
  }
  if (c < 0) return prev;   // a guard: W > 0 has a positive chunk
  // the point: first positive D2 of chunk c whose running sum exceeds t
  const int64_t i0 = c * kKppChunk;
  const double x = (tid < kKppChunk && i0 + tid < n) ? D[i0 + tid] : 0.0;
  double ctot = 0.0;
  const double pre = cbefore + kpp_block_scan<NT>(x, wtot, &ctot);
  __syncthreads();
  if (tid == 0) {
    hit = ~0ull;
    lastp = -1;
  }
  __syncthreads();
  kpp_wave_mark((x > 0.0 && pre + x > t) ? (long long)tid : -1, x > 0.0 ? (long long)tid : -1,
                &hit, &lastp);
  __syncthreads();
  if (tid == 0) {
    const long long p = hit != ~0ull ? (long long)hit : lastp;
    result = p >= 0 ? i0 + p : prev;
  }
  __syncthreads();
  return result;
}

__device__ __forceinline__ double kpp_draw(const double *__restrict__ u, int j) {
  const double uj = u[j];
  return (uj >= 0.0 && uj < 1.0) ? uj : 0.0;  // reported by kpp_first_kernel
}

__global__ __launch_bounds__(kKppSelThreads) void kpp_select_kernel(
    const double *__restrict__ D, const double *__restrict__ T, int64_t n,
    const double *__restrict__ u, int j, int64_t *__restrict__ cidx) {
  const int64_t c = kpp_pick<kKppSelThreads>(D, T, n, kpp_draw(u, j), cidx[j - 1]);
  if (threadIdx.x == 0) cidx[j] = c;
}

// ---- one launch per round, for clouds of at most kKppRoundChunks chunks.
// Every block picks centre j itself from the distances and chunk totals of
// round j - 1 (the same result in every block, written by block 0), then
// brings its own chunks up to date with it.  Labels are written where a
// distance changes, which is where the nearest centre does (ties keep the
// lower index).  No block writes what another may still read.
//
// A round is bound by the chain pick -> centre -> distances -> totals:
// 8.1 us at the depth frame (307,200 points), 10.0 when the pick took fourteen
// barriers and the centre's coordinates and the block's points a load each
// after it.
constexpr int64_t kKppRoundChunks = (int64_t)kKppSelThreads * kKppSelPer;   // one stage

struct KppCentre {   // no array: one indexed in a loop would live in scratch
  int64_t i;
  double x, y, z;
};

// kpp_pick for totals that one stage covers: the same sums in the same
// order, four barriers.  A wave that has a candidate leaves its first hit
// and its last positive entry in LDS, and every thread reads them; the lanes
// of the chosen chunk load their point with their distance, so the centre's
// coordinates are there with its index.  D[side[c]] holds the distances of
// chunk c (D0 when side is NULL).
template <int NT>
__device__ KppCentre kpp_pick1(const double *__restrict__ D0, const double *__restrict__ D1,
                               const uint8_t *__restrict__ side,
                               const double *__restrict__ T, const float *__restrict__ pts,
                               int64_t n, double uj, int64_t prev) {
  constexpr int NWV = NT / 64;
  static_assert(NT >= kKppChunk, "a block covers a chunk");
  __shared__ double wt[2][NWV];
  __shared__ int idx[2][NWV][2];        // stage; wave; first hit, last positive
  __shared__ double before[NWV][2];
  __shared__ int which[NWV][2];
  __shared__ float cxyz[NWV][2][3];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int64_t nch = (n + kKppChunk - 1) / kKppChunk;
  const int64_t c0 = (int64_t)tid * kKppSelPer;
  // (totals padded with zeros to a multiple of kKppSelPer)
  double v[kKppSelPer];
#pragma unroll
  for (int q = 0; q < kKppSelPer; q += 2) {
    const double2 d = c0 < nch ? *reinterpret_cast<const double2 *>(T + c0 + q)
                               : make_double2(0.0, 0.0);
    v[q] = d.x;
    v[q + 1] = d.y;
  }
  uint32_t s0 = 0, s1 = 0, s2 = 0, s3 = 0;   // sides of the 16 chunks, a byte each
  if (side && c0 < nch) {
    const uint4 q = *reinterpret_cast<const uint4 *>(side + c0);
    s0 = q.x; s1 = q.y; s2 = q.z; s3 = q.w;
  }
  auto scan = [&](double x, double *wtot, double &tot) -> double {   // one barrier
    double s = x;
    for (int off = 1; off < 64; off <<= 1) {
      const double o = __shfl_up(s, off, 64);
      if (lane >= off) s += o;
    }
    double e = __shfl_up(s, 1, 64);
    if (lane == 0) e = 0.0;
    if (lane == 63) wtot[w] = s;
    __syncthreads();
    double acc = 0.0, mine = 0.0;
#pragma unroll 4
    for (int k = 0; k < NWV; ++k) {
      if (k == w) mine = acc;
      acc += wtot[k];
    }
    tot = acc;
    return mine + e;
  };
  auto at_point = [&](int64_t i) {
    return KppCentre{i, pts[3 * i], pts[3 * i + 1], pts[3 * i + 2]};
  };
  double sum = 0.0;
#pragma unroll
  for (int q = 0; q < kKppSelPer; ++q) sum += v[q];
  double W;
  const double off = scan(sum, wt[0], W);
  if (!(W > 0.0)) return at_point(prev);   // uniform
  const double t = uj * W;
  // the chunk: first positive chunk total whose running sum exceeds t
  {
    double acc = off;
    int mine = -1, myl = -1, ms = 0, mls = 0;
    double mb = 0.0, mlb = 0.0;
#pragma unroll
    for (int q = 0; q < kKppSelPer; ++q) {
      const uint32_t word = q < 4 ? s0 : q < 8 ? s1 : q < 12 ? s2 : s3;
      const int sq = (int)((word >> (8 * (q & 3))) & 255u);
      const double nxt = acc + v[q];
      if (v[q] > 0.0) {
        if (mine < 0 && nxt > t) {
          mine = q;
          mb = acc;
          ms = sq;
        }
        myl = q;
        mlb = acc;
        mls = sq;
      }
      acc = nxt;
    }
    const uint64_t hb = __ballot(mine >= 0), lb = __ballot(myl >= 0);
    if (lane == 0 && !hb) idx[0][w][0] = -1;
    if (lane == 0 && !lb) idx[0][w][1] = -1;
    if (hb && lane == __builtin_ctzll(hb)) {
      idx[0][w][0] = (int)c0 + mine;
      before[w][0] = mb;
      which[w][0] = ms;
    }
    if (lb && lane == 63 - __builtin_clzll(lb)) {
      idx[0][w][1] = (int)c0 + myl;
      before[w][1] = mlb;
      which[w][1] = mls;
    }
  }
  __syncthreads();
  // the first wave with a hit, else the last with a positive entry
  auto choose = [&](int st, int &wave, int &kind) -> int {
    const int h = lane < NWV ? idx[st][lane][0] : -1, l = lane < NWV ? idx[st][lane][1] : -1;
    const uint64_t hb = __ballot(h >= 0), lb = __ballot(l >= 0);
    kind = hb ? 0 : 1;
    wave = hb ? __builtin_ctzll(hb) : lb ? 63 - __builtin_clzll(lb) : 0;
    return (hb | lb) ? idx[st][wave][kind] : -1;
  };
  int cw, ck;
  const int c = choose(0, cw, ck);
  if (c < 0) return at_point(prev);   // a guard: W > 0 has a positive chunk
  // the point: first positive D2 of chunk c whose running sum exceeds t
  const int64_t i0 = (int64_t)c * kKppChunk;
  const double cbefore = before[cw][ck];
  const double *D = which[cw][ck] ? D1 : D0;
  double x = 0.0;
  float px = 0.0f, py = 0.0f, pz = 0.0f;
  if (tid < kKppChunk && i0 + tid < n) {
    const float *q = pts + 3 * (i0 + tid);
    x = D[i0 + tid];
    px = q[0]; py = q[1]; pz = q[2];
  }
  double ctot;
  const double pre = cbefore + scan(x, wt[1], ctot);
  {
    const uint64_t hb = __ballot(x > 0.0 && pre + x > t), lb = __ballot(x > 0.0);
    if (lane == 0 && !hb) idx[1][w][0] = -1;
    if (lane == 0 && !lb) idx[1][w][1] = -1;
    if (hb && lane == __builtin_ctzll(hb)) {
      idx[1][w][0] = tid;
      cxyz[w][0][0] = px; cxyz[w][0][1] = py; cxyz[w][0][2] = pz;
    }
    if (lb && lane == 63 - __builtin_clzll(lb)) {
      idx[1][w][1] = tid;
      cxyz[w][1][0] = px; cxyz[w][1][1] = py; cxyz[w][1][2] = pz;
    }
  }
  __syncthreads();
  int pw, ph;
  const int pt = choose(1, pw, ph);
  if (pt < 0) return at_point(prev);
  return KppCentre{i0 + pt, cxyz[pw][ph][0], cxyz[pw][ph][1], cxyz[pw][ph][2]};
}

// The total of a row of 256 distances, sequentially (one thread).
__device__ __forceinline__ double kpp_row_total(const double *a) {
  double s = 0.0;
  for (int k0 = 0; k0 < kKppChunk; k0 += 16) {
    double e[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) e[k] = a[k0 + k];
#pragma unroll
    for (int k = 0; k < 16; ++k) s += e[k];
  }
  return s;
}

// Clouds of at most kKppSmallChunks chunks: blocks of 256 threads and 4
// chunks, whose points and distances are loaded before the pick (they stay
// in cache from round to round); distances and totals double-buffered.
// The line to the culled form (us a round): 307,200 points 8.1 here, 8.9
// culled; 400,000 8.2, 8.9; 600,000 11.8, 9.6; 1,000,000 18.1, 10.6.
constexpr int64_t kKppSmallChunks = 2048;
static_assert(kKppSmallChunks <= (int64_t)kKppUpdThreads * kKppSelPer, "one stage");
__global__ __launch_bounds__(kKppUpdThreads) void kpp_round_kernel(
    const float *__restrict__ pts, int64_t n, const double *__restrict__ u, int j,
    int64_t *__restrict__ cidx, const double *__restrict__ Dp, const double *__restrict__ Tp,
    double *__restrict__ Dn, double *__restrict__ Tn, int64_t nch,
    int32_t *__restrict__ labels) {
  __shared__ double sh[kKppUpdChunks * kKppRow];
  const int64_t base = (int64_t)blockIdx.x * kKppUpdChunks * kKppChunk;
  constexpr int PER = kKppUpdChunks * kKppChunk / kKppUpdThreads;
  float x[PER][3];
  double o[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    // (clamped past the end, so that the loads need no branch)
    const int64_t i = base + q * kKppUpdThreads + threadIdx.x, ic = i < n ? i : n - 1;
#pragma unroll
    for (int k = 0; k < 3; ++k) x[q][k] = pts[3 * ic + k];
    o[q] = Dp[ic];
  }
  const KppCentre c = kpp_pick1<kKppUpdThreads>(Dp, Dp, nullptr, Tp, pts, n, kpp_draw(u, j),
                                                cidx[j - 1]);
  if (blockIdx.x == 0 && threadIdx.x == 0) cidx[j] = c.i;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int l = q * kKppUpdThreads + threadIdx.x;
    const int64_t i = base + l;
    double v = 0.0;  // past the end: 0, which leaves the running sums as they are
    if (i < n) {
      const double d = kpp_d2(x[q][0], x[q][1], x[q][2], c.x, c.y, c.z);
      const bool less = d < o[q];
      v = less ? d : o[q];
      Dn[i] = v;
      if (less && labels) labels[i] = j;
    }
    sh[(l / kKppChunk) * kKppRow + (l % kKppChunk)] = v;
  }
  __syncthreads();
  const int64_t ch = (int64_t)blockIdx.x * kKppUpdChunks + threadIdx.x;
  if (threadIdx.x < kKppUpdChunks && ch < nch) Tn[ch] = kpp_row_total(sh + threadIdx.x * kKppRow);
}

// Larger clouds: one block per compute unit (the pick costs every block the
// same), `per` chunks each, of 512 threads up to 8,192 chunks, else 1,024: the
// fewest whose stage covers the totals, since a pick's scans run over the
// waves (1,000,000 points: 10.7 us a round, 13.1 with 1,024 threads).
//
// A chunk whose bounding box lies further from the new centre than its
// largest D2 keeps every distance, so its total too: it is skipped.  (With
// lb the squared distance to the box, every computed d2 of the chunk is at
// least lb (1 - 2^-50), and lb is used with a margin of 1e-12.)  A scan's
// chunks are short runs of neighbouring points, so few are near a new
// centre.  The totals are double-buffered; a chunk's distances move to its
// other buffer when they change (`side`, itself double-buffered).
// Measured (LiDAR scans, us a round): 1,000,000 points 10.7, 2,000,000 14.4;
// 19.7 and 23.8 when every round read and wrote every distance.
constexpr int kKppMaxPer = 64;   // chunks per block

struct KppState {
  double *D[2];
  double *T[2];      // chunk totals
  uint8_t *side[2];  // which buffer holds a chunk's distances
  double *dmax;      // largest D2 of a chunk (its own block's)
  float *box;        // 6 per chunk: lo, hi
};

template <int NT>
__global__ __launch_bounds__(NT) void kpp_round_cull_kernel(
    const float *__restrict__ pts, int64_t n, int64_t nch, int per, const double *__restrict__ u,
    int j, int64_t *__restrict__ cidx, KppState s, int32_t *__restrict__ labels) {
  constexpr int SETS = NT / kKppChunk;
  extern __shared__ __align__(16) unsigned char kpp_smem[];
  double *rows = reinterpret_cast<double *>(kpp_smem);   // per x kKppRow
  __shared__ int act[kKppMaxPer];
  __shared__ double part[kKppMaxPer][4];
  __shared__ int nact;
  const int tid = threadIdx.x;
  const bool odd = (j & 1) != 0;
  double *Tp = odd ? s.T[0] : s.T[1], *Tn = odd ? s.T[1] : s.T[0];
  uint8_t *sp = odd ? s.side[0] : s.side[1], *sn = odd ? s.side[1] : s.side[0];
  const int64_t ch0 = (int64_t)blockIdx.x * per;
  const int mine = (int)((nch - ch0) < per ? (nch - ch0) : per);
  // chunk tid of this block: requested before the pick
  float lo0 = 0.f, lo1 = 0.f, lo2 = 0.f, hi0 = 0.f, hi1 = 0.f, hi2 = 0.f;
  double mx = 0.0, tp = 0.0;
  int sd = 0;
  if (tid < mine) {
    const float *b = s.box + 6 * (ch0 + tid);
    lo0 = b[0]; lo1 = b[1]; lo2 = b[2];
    hi0 = b[3]; hi1 = b[4]; hi2 = b[5];
    mx = s.dmax[ch0 + tid];
    tp = Tp[ch0 + tid];
    sd = sp[ch0 + tid];
  }
  const KppCentre c = kpp_pick1<NT>(s.D[0], s.D[1], sp, Tp, pts, n, kpp_draw(u, j),
                                    cidx[j - 1]);
  if (blockIdx.x == 0 && tid == 0) cidx[j] = c.i;
  if (tid < 64) {   // per <= 64
    bool on = false;
    if (tid < mine) {
      const double d0 = fmax(fmax(lo0 - c.x, c.x - hi0), 0.0);
      const double d1 = fmax(fmax(lo1 - c.y, c.y - hi1), 0.0);
      const double d2 = fmax(fmax(lo2 - c.z, c.z - hi2), 0.0);
      on = !((d0 * d0 + d1 * d1 + d2 * d2) * (1.0 - 1e-12) >= mx);
      sn[ch0 + tid] = (uint8_t)(on ? 1 - sd : sd);
      if (!on) Tn[ch0 + tid] = tp;
    }
    const uint64_t m = __ballot(on);
    if (on) act[__popcll(m & ((1ull << tid) - 1ull))] = tid | (sd << 8);
    if (tid == 0) nact = __popcll(m);
  }
  __syncthreads();
  const int na = nact;
  if (na == 0) return;
  const int set = tid / kKppChunk, t = tid % kKppChunk;
  for (int q0 = set; q0 < na; q0 += 4 * SETS) {
    float x[4][3];
    double o[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {   // four points of this thread in flight
      const int q = q0 + v * SETS;
      // (clamped, so that the loads need no branch)
      const int aq = act[q < na ? q : 0];
      const int64_t i = (ch0 + (aq & 255)) * kKppChunk + t, ic = i < n ? i : n - 1;
#pragma unroll
      for (int k = 0; k < 3; ++k) x[v][k] = pts[3 * ic + k];
      o[v] = (aq >> 8 ? s.D[1] : s.D[0])[ic];
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int q = q0 + v * SETS;
      if (q < na) {
        const int64_t i = (ch0 + (act[q] & 255)) * kKppChunk + t;
        double r = 0.0;   // past the end: 0, which leaves the running sums as they are
        if (i < n) {
          const double d = kpp_d2(x[v][0], x[v][1], x[v][2], c.x, c.y, c.z);
          const bool less = d < o[v];
          r = less ? d : o[v];
          (act[q] >> 8 ? s.D[0] : s.D[1])[i] = r;
          if (less && labels) labels[i] = j;
        }
        rows[q * kKppRow + t] = r;
        double m = r;
        for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
        if ((tid & 63) == 0) part[q][t >> 6] = m;
      }
    }
  }
  __syncthreads();
  if (tid < na) {
    const int64_t ch = ch0 + (act[tid] & 255);
    Tn[ch] = kpp_row_total(rows + tid * kKppRow);
    s.dmax[ch] = fmax(fmax(part[tid][0], part[tid][1]), fmax(part[tid][2], part[tid][3]));
  }
}

// The pick of the last centre alone (no labels wanted): one block.
__global__ __launch_bounds__(kKppSelThreads) void kpp_last_kernel(
    const float *__restrict__ pts, int64_t n, const double *__restrict__ u, int j,
    int64_t *__restrict__ cidx, const double *__restrict__ D0, const double *__restrict__ D1,
    const uint8_t *__restrict__ side, const double *__restrict__ T) {
  const KppCentre c =
      kpp_pick1<kKppSelThreads>(D0, D1, side, T, pts, n, kpp_draw(u, j), cidx[j - 1]);
  if (threadIdx.x == 0) cidx[j] = c.i;
}

// Round 0 of both: distances to centre 0, totals, labels 0; for the culled
// rounds (s.box) boxes, largest distances and sides.  A block of 256 threads
// per chunk.
__global__ __launch_bounds__(kKppChunk) void kpp_round0_kernel(
    const float *__restrict__ pts, int64_t n, const int64_t *__restrict__ cidx, KppState s,
    int32_t *__restrict__ labels, uint32_t *status) {
  __shared__ double row[kKppRow];
  __shared__ float ext[4][6];
  __shared__ double wm[4];
  const int tid = threadIdx.x, lane = tid & 63;
  const int64_t c = cidx[0], ch = blockIdx.x, i = ch * kKppChunk + tid;
  double v = 0.0;
  float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  if (i < n) {
    const float x0 = pts[3 * i], x1 = pts[3 * i + 1], x2 = pts[3 * i + 2];
    if (!isfinite(x0) || !isfinite(x1) || !isfinite(x2)) set_status(status, kStNonFinite);
    v = kpp_d2(x0, x1, x2, pts[3 * c], pts[3 * c + 1], pts[3 * c + 2]);
    s.D[0][i] = v;
    if (labels) labels[i] = 0;
    lo[0] = hi[0] = x0; lo[1] = hi[1] = x1; lo[2] = hi[2] = x2;
  }
  row[tid] = v;
  double m = v;
  if (s.box) {
    for (int off = 32; off > 0; off >>= 1) {
      m = fmax(m, __shfl_xor(m, off, 64));
      for (int k = 0; k < 3; ++k) {
        lo[k] = fminf(lo[k], __shfl_xor(lo[k], off, 64));
        hi[k] = fmaxf(hi[k], __shfl_xor(hi[k], off, 64));
      }
    }
    if (lane == 0) {
      wm[tid >> 6] = m;
      for (int k = 0; k < 3; ++k) {
        ext[tid >> 6][k] = lo[k];
        ext[tid >> 6][3 + k] = hi[k];
      }
    }
  }
  __syncthreads();
  if (s.box && tid < 6) {
    float e = ext[0][tid];
    for (int w = 1; w < 4; ++w) e = tid < 3 ? fminf(e, ext[w][tid]) : fmaxf(e, ext[w][tid]);
    s.box[6 * ch + tid] = e;
  }
  if (ch + 1 == (int64_t)gridDim.x && tid >= 128 && tid < 128 + kKppSelPer) {
    const int64_t pad = ch + 1 + tid - 128;   // zeros up to a multiple of kKppSelPer
    if (pad < (ch + kKppSelPer) / kKppSelPer * kKppSelPer) s.T[0][pad] = s.T[1][pad] = 0.0;
  }
  if (tid == 64) {
    s.T[0][ch] = kpp_row_total(row);
    if (s.box) {
      s.dmax[ch] = fmax(fmax(wm[0], wm[1]), fmax(wm[2], wm[3]));
      s.side[0][ch] = 0;
    }
  }
}

// Non-finite coordinates (for a call that forms no distances otherwise).
__global__ __launch_bounds__(256) void kpp_check_kernel(const float *__restrict__ pts,
                                                        int64_t n, uint32_t *status) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n && (!isfinite(pts[3 * i]) || !isfinite(pts[3 * i + 1]) || !isfinite(pts[3 * i + 2])))
    set_status(status, kStNonFinite);
}

// label_i = the nearest of the K centres (lowest index on ties).
__global__ __launch_bounds__(kKppLabelThreads) void kpp_label_kernel(
    const float *__restrict__ pts, int64_t n, const int64_t *__restrict__ cidx, int K,
    int32_t *__restrict__ labels, uint32_t *status) {
  extern __shared__ __align__(16) unsigned char kpp_smem[];
  double *cs = reinterpret_cast<double *>(kpp_smem);  // K x 3
  for (int k = threadIdx.x; k < K; k += kKppLabelThreads) {
    const int64_t c = cidx[k];
    cs[3 * k] = pts[3 * c];
    cs[3 * k + 1] = pts[3 * c + 1];
    cs[3 * k + 2] = pts[3 * c + 2];
  }
  __syncthreads();
  const int64_t i = (int64_t)blockIdx.x * kKppLabelThreads + threadIdx.x;
  if (i >= n) return;
  const float f0 = pts[3 * i], f1 = pts[3 * i + 1], f2 = pts[3 * i + 2];
  if (!isfinite(f0) || !isfinite(f1) || !isfinite(f2)) set_status(status, kStNonFinite);
  const double x0 = f0, x1 = f1, x2 = f2;
  double best = kpp_d2(x0, x1, x2, cs[0], cs[1], cs[2]);
  int l = 0;
  for (int k = 1; k < K; ++k) {
    const double d = kpp_d2(x0, x1, x2, cs[3 * k], cs[3 * k + 1], cs[3 * k + 2]);
    if (d < best) {
      best = d;
      l = k;
    }
  }
  labels[i] = l;
}

}  // namespace gmm_dev
