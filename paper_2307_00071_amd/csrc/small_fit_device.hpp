// Small fits in one launch: the label passes, every soft EM iteration (eq. 2
// E-step, the M-step of Sec. V: weights, means, covariances with lambda I,
// Cholesky) and the final log-likelihood of a fit with K <= 16 components
// and at most 256 tiles of 256 points.
//
// For such fits a launch pair per pass (tile pass, reduction + M-step) costs
// more than its arithmetic.  Here one block owns one 256-point tile for the
// whole fit and keeps its point in a register.  Per iteration:
//  E-phase  thread p: l'_pb for every component from the parameters in LDS,
//           e_pb = 2^l'_pb into the LDS row of b, s_p, lse_p (a point whose
//           s_p underflows is redone with its own maximum, as in the tile
//           kernel);
//  M-phase  thread (b, q): the ten shifted sums of component b over point
//           subset q (FP32 over at most 16 points, then FP64), the P
//           subsets added in order, and the block's log-likelihood sum:
//           one FP64 partial row of 10 K + 1 values;
//  exchange every block reads every row.  A value travels as two 8-byte
//           words, each 32 bits of it and the number of the exchange, stored
//           and loaded with relaxed agent-scope atomics: a reader that finds
//           the number has the data, so no fence, ticket or counter is
//           needed (rows alternate between two buffers; a block stores its
//           row of exchange t + 2 only after it has read every row of t + 1,
//           which their owners stored after reading all of t).  The wait is
//           bounded: after kSmallSpinLimit polls, or when another block gave
//           up, the block sets the device-error bit and returns, so every
//           wave exits;
//  update   every block adds all rows in the same fixed order and runs the
//           same FP64 M-step into its own LDS parameters, so no block reads
//           parameters another block wrote; block 0 also writes the
//           log-likelihood of the iteration and, at the end, the outputs;
//  stop     with a tolerance, every block makes the same decision from the
//           same L.
// The label passes add float32 groups of as many points as the tile kernel
// does (a.lab_trip), and the final pass adds a point's terms in its eight
// component groups, so that both give the same float32 values.
// All blocks must be resident at once: the host launches at most one
// block per compute unit.
//
// Measured, N = 10,000, K = 8, 50 iterations (40 blocks): with a ticket
// counter and device-scope fences an iteration took 8.3 us, 4.5 of them the
// exchange, and the label and final passes 54 us in six launches; now 6.9 us
// (E 0.6, M 0.85, column sums 0.6, exchange 3.0, update 1.8) and about 15 us
// inside the one launch: 518 -> 420 us a fit.
#pragma once

#include "em_device.hpp"

#include <type_traits>

namespace gmm_dev {

constexpr int kSmallThreads = 256;     // block = tile = 256 points
constexpr int kSmallMaxK = 16;
constexpr int kSmallMaxTiles = 256;    // blocks (one tile each)
constexpr int kSmallTS = kSmallThreads + 1;   // odd LDS row stride
constexpr unsigned kSmallSpinLimit = 1u << 20;
constexpr int kSmallLikGroups = 8;     // component groups of the dense log-likelihood pass
constexpr uint32_t kStDevice = 1u << GMM_ERR_DEVICE;

// Exchange words of a fit: two buffers of grid rows and a row of totals.
__host__ __device__ constexpr int64_t small_words(int64_t grid, int ncols) {
  return 2 * (grid + 1) * ncols * 2;
}
// One hop (every block reads every row) costs 2 us plus 0.47 ns per value of
// the grid x ncols rows (8 x 81: 2.05 us, 40 x 81: 3.03, 40 x 161: 5.4, 235 x
// 121: 15.2); two hops (an owner per column, then the totals) 3.6 to 5.0 us.
constexpr int kSmallOneHop = 4096;

struct SmallArgs {
  int64_t n;
  int K, P, trip, iters, ncols;
  int lab_trip;   // > 0: start from labels
  int fused;      // label start with the static bound (lambda > 0)
  int two_hops;   // the exchange goes by column totals
  double reg, lnZ, Ntot, Chdr;   // as FuseArgs
  // > 0: stopping rule; after the M-step of the first iteration t >= 1 with
  // |L_t - L_(t-1)| <= tol_abs the fit keeps theta_(t+1), and the L of the
  // skipped iterations is NaN
  double tol_abs;
  // tests of the give-up path: at this iteration block 0 raises the flag
  // instead of storing its row (-1: never)
  int give_up_at;
};

__global__ __launch_bounds__(kSmallThreads) void em_small_fit_kernel(
    const float *__restrict__ pts, const int32_t *__restrict__ labels,
    const float *__restrict__ cpar_in, const float4 *__restrict__ shift_in, uint64_t *words,
    unsigned *gave_up, double *__restrict__ loglik, float *__restrict__ out_w,
    float *__restrict__ out_mu, float *__restrict__ out_cov, uint32_t *__restrict__ status,
    SmallArgs a) {
  constexpr int NT = kSmallThreads, TS = kSmallTS;
  static_assert(NT == 256, "the log-likelihood sum adds four wave sums");
  constexpr int NPAR = (kSmallMaxK + 1) * kParStride;
  __shared__ __align__(16) float cp[2][NPAR];
  __shared__ float4 sh[2][kSmallMaxK];
  __shared__ float E[kSmallMaxK * TS];
  __shared__ float4 Xs[NT];
  __shared__ double D[NT * kNStat];
  __shared__ double gsum[NT];
  __shared__ double tot[kNStat * kSmallMaxK + 1];
  __shared__ double th[kSmallMaxK * kTh64Stride];
  __shared__ double scr[2 * NT / 64 + 2];
  __shared__ int abort_flag;

  const int tid = threadIdx.x, lane = tid & 63;
  const int K = a.K, P = a.P, trip = a.trip, ncols = a.ncols;
  const int grid = gridDim.x, blk = blockIdx.x;
  const int nf = (K + 1) * kParStride;
  if (a.lab_trip == 0)
    for (int i = tid; i < nf; i += NT) cp[0][i] = cpar_in[i];
  if (tid < K) sh[0][tid] = a.lab_trip ? make_float4(0.f, 0.f, 0.f, 0.f) : shift_in[tid];
  if (tid == 0) abort_flag = 0;
  float4 x = make_float4(0.f, 0.f, 0.f, __int_as_float(-1));
  {
    const int64_t i = (int64_t)blk * NT + tid;
    if (i < a.n) {
      x = make_float4(pts[3 * i], pts[3 * i + 1], pts[3 * i + 2], __int_as_float(0));
      if (!isfinite(x.x) || !isfinite(x.y) || !isfinite(x.z)) {
        set_status(status, kStNonFinite);
        x.x = x.y = x.z = 0.0f;
      }
      if (a.lab_trip) {
        int tag = labels[i];
        if (tag < 0 || tag >= K) {
          set_status(status, kStBadArg);
          tag = -1;
        }
        x.w = __int_as_float(tag);
      }
    }
  }
  const bool valid = __float_as_int(x.w) >= 0;
  const bool mact = tid < K * P;
  const int mb = mact ? tid % K : 0, mq = mact ? tid / K : 0;
  // a statistic column c = s K + b of the row; the P subset sums of
  // component b, statistic s are at D[(q K + b) kNStat + s]
  const int cs = tid / K, cb = tid - (tid / K) * K;
  int cur = 0, xchg = 0;
  double Lprev = 0.0;

  // FP64 sums of component mb over the points of subset mq, in float32
  // groups of `group` points, into D
  auto m_phase = [&](int group) {
    if (!mact) return;
    const float4 m = sh[cur][mb];
    const float *Eb = E + mb * TS + mq * trip;
    const float4 *Xb = Xs + mq * trip;
    double *d = D + (size_t)(mq * K + mb) * kNStat;
    double acc[kNStat];
#pragma unroll
    for (int j = 0; j < kNStat; ++j) acc[j] = 0.0;
    for (int j0 = 0; j0 < trip; j0 += group) {
      float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f, a4 = 0.f, a5 = 0.f,
            a6 = 0.f, a7 = 0.f, a8 = 0.f, a9 = 0.f;
#pragma unroll 4
      for (int j = j0; j < j0 + group; ++j) {
        const float4 xr = Xb[j];
        const float gm = Eb[j] * xr.w;
        const float d0 = xr.x - m.x, d1 = xr.y - m.y, d2 = xr.z - m.z;
        const float w0 = gm * d0, w1 = gm * d1, w2 = gm * d2;
        a0 += gm;
        a1 += w0; a2 += w1; a3 += w2;
        a4 = fmaf(w0, d0, a4);
        a5 = fmaf(w1, d0, a5);
        a6 = fmaf(w1, d1, a6);
        a7 = fmaf(w2, d0, a7);
        a8 = fmaf(w2, d1, a8);
        a9 = fmaf(w2, d2, a9);
      }
      acc[0] += a0; acc[1] += a1; acc[2] += a2; acc[3] += a3; acc[4] += a4;
      acc[5] += a5; acc[6] += a6; acc[7] += a7; acc[8] += a8; acc[9] += a9;
    }
#pragma unroll
    for (int j = 0; j < kNStat; ++j) d[j] = acc[j];
  };
  // this thread's column of the block's row: the P subset sums in order, or
  // the log-likelihood from the four wave sums
  auto column = [&]() -> double {
    double v = 0.0;
    if (tid < kNStat * K) {
#pragma unroll 8
      for (int q = 0; q < P; ++q) v += D[(size_t)(q * K + cb) * kNStat + cs];
    } else if (tid == kNStat * K) {
      v = (scr[0] + scr[1]) + (scr[2] + scr[3]);
    }
    return v;
  };
  auto put = [&](uint64_t *w, double v, uint32_t tag) {
    const uint64_t t64 = (uint64_t)tag << 32;
    __hip_atomic_store(w, t64 | (uint32_t)__double2loint(v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(w + 1, t64 | (uint32_t)__double2hiint(v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  };
  // The sum, in order, of the values at w, w + stride, ... that this thread
  // has (bit u of `have`), waiting for each; false: given up.
  auto take = [&](auto has, const uint64_t *w, size_t stride, uint32_t have, uint32_t tag,
                  double &acc) -> bool {
    constexpr int N = decltype(has)::value;
    uint64_t lo[N], hi[N];
    uint32_t todo = have;
    unsigned spins = 0;
#pragma unroll
    for (int u = 0; u < N; ++u) lo[u] = hi[u] = 0;
    while (todo) {
#pragma unroll
      for (int u = 0; u < N; ++u)
        if ((todo >> u) & 1u) {
          lo[u] = __hip_atomic_load(w + u * stride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          hi[u] =
              __hip_atomic_load(w + u * stride + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
      for (int u = 0; u < N; ++u)
        if ((uint32_t)(lo[u] >> 32) == tag && (uint32_t)(hi[u] >> 32) == tag) todo &= ~(1u << u);
      if (todo && (++spins > kSmallSpinLimit ||
                   ((spins & 63u) == 0 && __hip_atomic_load(gave_up, __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_AGENT)))) {
        __hip_atomic_store(gave_up, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return false;
      }
    }
#pragma unroll
    for (int u = 0; u < N; ++u)
      acc += ((have >> u) & 1u) ? __hiloint2double((int)(uint32_t)hi[u], (int)(uint32_t)lo[u])
                                : 0.0;
    return true;
  };
  // Columns [c0, ncols) of every block's row added into tot, identically in
  // every block.  v: this thread's column.  false: given up (the whole block
  // returns).
  auto exchange = [&](double v, int c0, bool give_up) -> bool {
    const uint32_t tag = (uint32_t)++xchg;
    uint64_t *rows = words + (size_t)(xchg & 1) * (grid + 1) * ncols * 2;
    uint64_t *sums = rows + (size_t)grid * ncols * 2;
    if (give_up) {
      if (tid == 0)
        __hip_atomic_store(gave_up, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else if (tid >= c0 && tid < ncols) {
      put(rows + ((size_t)blk * ncols + tid) * 2, v, tag);
    }
    const int nc = ncols - c0;
    bool ok = true;
    if (a.two_hops) {
      // block j adds the columns c0 + j, c0 + j + grid, ... (a wave each:
      // lane l the rows l, l + 64, ..., then the wave sum) and stores the
      // totals, which every block reads
      for (int c = c0 + blk + grid * (tid >> 6); c < ncols && ok; c += grid * (NT / 64)) {
        uint32_t have = 0;
#pragma unroll
        for (int u = 0; u < kSmallMaxTiles / 64; ++u)
          if (lane + 64 * u < grid) have |= 1u << u;
        double acc = 0.0;
        ok = take(std::integral_constant<int, kSmallMaxTiles / 64>{},
                  rows + ((size_t)lane * ncols + c) * 2, (size_t)64 * ncols * 2, have, tag, acc);
        const bool all = __ballot(!ok) == 0;
        acc = wave_sum_f64(acc);
        if (lane == 0 && all) put(sums + c * 2, acc, tag);
      }
      if (ok && tid < nc) {
        double acc = 0.0;
        ok = take(std::integral_constant<int, 1>{}, sums + (c0 + tid) * 2, 0, 1u, tag, acc);
        tot[c0 + tid] = acc;
      }
      if (!ok) abort_flag = 1;
      __syncthreads();
    } else {
      // G groups of threads, group g the rows g, g + G, ... in order (16 in
      // flight), then the G group sums in order
      const int G = NT / nc;
      const int g = tid / nc, c = c0 + tid - g * nc;
      if (g < G) {
        double acc = 0.0;
        for (int r0 = g; r0 < grid && ok; r0 += 16 * G) {
          uint32_t have = 0;
#pragma unroll
          for (int u = 0; u < 16; ++u)
            if (r0 + u * G < grid) have |= 1u << u;
          ok = take(std::integral_constant<int, 16>{}, rows + ((size_t)r0 * ncols + c) * 2,
                    (size_t)G * ncols * 2, have, tag, acc);
        }
        if (!ok) abort_flag = 1;
        gsum[tid] = acc;
      }
      __syncthreads();
      if (!abort_flag && tid < nc) {
        double acc = gsum[tid];
        for (int h = 1; h < G; ++h) acc += gsum[h * nc + tid];
        tot[c0 + tid] = acc;
      }
      __syncthreads();
    }
    if (abort_flag) {
      if (tid == 0) set_status(status, kStDevice);
      return false;
    }
    return true;
  };
  // block sum of the per-point log-normalisers: wave sums (DPP rows, then
  // rows in order) into scr
  auto lse_sums = [&](double lse) {
    const double wl = wave_sum_f64(lse);
    if (lane == 0) scr[tid >> 6] = wl;
  };
  __syncthreads();

  // ---- theta_0 from the labels: means about the origin, then the scatter
  // about them
  if (a.lab_trip) {
    const int tg = __float_as_int(x.w);
    for (int b = 0; b < K; ++b) E[b * TS + tid] = (b == tg) ? 1.0f : 0.0f;
    Xs[tid] = make_float4(x.x, x.y, x.z, valid ? 1.0f : 0.0f);
    if (lane == 0) scr[tid >> 6] = 0.0;
    __syncthreads();
    for (int pass = 0; pass < 2; ++pass) {
      m_phase(a.lab_trip);
      __syncthreads();
      if (!exchange(column(), 0, false)) return;
      const int nxt = 1 - cur;
      if (pass == 0) {
        if (tid < K) {
          double mu[3];
          if (!component_mean(tot + tid, K, sh[cur][tid], mu)) set_status(status, kStNonFinite);
          sh[nxt][tid] = make_float4((float)mu[0], (float)mu[1], (float)mu[2], 0.0f);
        }
      } else if (a.fused) {
        if (tid < K)
          update_component_static(tot + tid, K, sh[cur][tid], a.reg, a.lnZ, a.Ntot,
                                  cp[nxt] + tid * kParStride, &sh[nxt][tid],
                                  th + tid * kTh64Stride, status);
        if (tid == 0) *reinterpret_cast<double *>(cp[nxt] + (size_t)K * kParStride) = a.Chdr;
      } else {
        em_update_block<NT, true>(tot, K, kUpdFull, a.reg, cp[cur], sh[cur], cp[nxt], sh[nxt],
                                  th, scr, status);
      }
      cur = nxt;
      __syncthreads();
    }
  }

  for (int t = 0; t < a.iters; ++t) {
    const float *cq = cp[cur];
    // ---- E-phase
    const double Cb = *reinterpret_cast<const double *>(cq + (size_t)K * kParStride);
    float s = 0.0f;
#pragma unroll 4
    for (int b = 0; b < K; ++b) {
      const float e = __builtin_amdgcn_exp2f(
          comp_logterm(cq + b * kParStride, x.x, x.y, x.z));
      E[b * TS + tid] = e;
      s += e;
    }
    float mref = 0.0f;
    if (valid && !(s >= 0x1p-100f)) {
      float m = -INFINITY;
      for (int b = 0; b < K; ++b)
        m = fmaxf(m, comp_logterm(cq + b * kParStride, x.x, x.y, x.z));
      s = 0.0f;
      for (int b = 0; b < K; ++b) {
        const float e = __builtin_amdgcn_exp2f(
            comp_logterm(cq + b * kParStride, x.x, x.y, x.z) - m);
        E[b * TS + tid] = e;
        s += e;
      }
      mref = m;
    }
    Xs[tid] = make_float4(x.x, x.y, x.z, valid ? __builtin_amdgcn_rcpf(s) : 0.0f);
    const double lse =
        valid ? (Cb + (double)mref + (double)__builtin_amdgcn_logf(s)) * kLn2 : 0.0;
    __syncthreads();
    // ---- M-phase: subset q of component b
    m_phase(trip);
    lse_sums(lse);
    __syncthreads();
    if (!exchange(column(), 0, blk == 0 && t == a.give_up_at)) return;
    if (blk == 0 && tid == 0) {
      const double L = tot[kNStat * K];
      if (loglik) loglik[t] = L;
      if (!isfinite(L)) set_status(status, kStNonFinite);
    }
    const int nxt = 1 - cur;
    em_update_block<NT, true>(tot, K, kUpdFull, a.reg, cp[cur], sh[cur], cp[nxt], sh[nxt],
                        th, scr, status);
    cur = nxt;
    // every block holds the same L bits, so all stop at the same iteration
    const double L = tot[kNStat * K];
    const bool stop = a.tol_abs > 0.0 && t >= 1 && fabs(L - Lprev) <= a.tol_abs;
    Lprev = L;
    __syncthreads();
    if (stop) {
      if (blk == 0 && loglik)
        for (int u = t + 1 + tid; u < a.iters; u += NT) loglik[u] = (double)NAN;
      break;
    }
  }

  // ---- log-likelihood of the returned parameters, and the outputs
  {
    const float *cq = cp[cur];
    const double Cb = *reinterpret_cast<const double *>(cq + (size_t)K * kParStride);
    constexpr int G = kSmallLikGroups;
    float s = 0.0f;
    for (int g = 0; g < G; ++g) {
      float sg = 0.0f;
      for (int b = (g * K) / G; b < ((g + 1) * K) / G; ++b)
        sg += __builtin_amdgcn_exp2f(comp_logterm(cq + b * kParStride, x.x, x.y, x.z));
      s += sg;
    }
    float mref = 0.0f;
    if (valid && !(s >= 0x1p-100f)) {
      float m = -INFINITY;
      for (int b = 0; b < K; ++b)
        m = fmaxf(m, comp_logterm(cq + b * kParStride, x.x, x.y, x.z));
      s = 0.0f;
      for (int b = 0; b < K; ++b)
        s += __builtin_amdgcn_exp2f(comp_logterm(cq + b * kParStride, x.x, x.y, x.z) - m);
      mref = m;
    }
    lse_sums(valid ? (Cb + (double)mref + (double)__builtin_amdgcn_logf(s)) * kLn2 : 0.0);
    __syncthreads();
    if (!exchange(column(), kNStat * K, false)) return;
  }
  if (blk == 0) {
    if (tid < K) write_component(th + tid * kTh64Stride, tid, out_w, out_mu, out_cov);
    if (tid == 0) {
      const double L = tot[kNStat * K];
      if (loglik) loglik[a.iters] = L;
      if (!isfinite(L)) set_status(status, kStNonFinite);
    }
  }
}

}  // namespace gmm_dev
