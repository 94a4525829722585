// Device code of the registration likelihood: the launch before and the
// launches after its tile passes, and the culled backward pass.  Included
// once, by gmm.hip, after em_device.hpp.
//
// A forward call is three launches: lik_setup_kernel, a tile kernel of
// em_device.hpp in kSoftLogLik mode, lik_finish_kernel; a backward call
// lik_setup_kernel, em_bwd_cull_kernel (or em_bwd_kernel) and
// bwd_finish_kernel.
#pragma once

#include "em_device.hpp"

#include <type_traits>

namespace gmm_dev {

// ------------------------------------------------------------ setup launch
//
// Everything before the tile pass in one launch (it was six: status, pose,
// staging, tile spheres, parameters, each 3 us of launch for 1.5-3 us of
// work): block 0 clears the status word and forms the parameter block (and
// the pose in FP64); the other blocks move and stage the points (each with
// its own copy of the pose) and form the bounds of their tiles.  Blocks
// report through `flags`, one word each, since the status word is cleared in
// the same launch; the finishing launch collects them.
constexpr int kLikThreads = 256;
constexpr int kLikMaxBlocks = 2048;   // staging blocks (then grid-strided)

struct LikSetupArgs {
  int64_t n, npad;
  int K;
  int tpts;     // points per tile of the bounding spheres, 64 to 256; 0: none
};

// Block-wide status bits of one call (all threads call it).
__device__ __forceinline__ void lik_flag(uint32_t bits, uint32_t *flags) {
  __shared__ uint32_t any;
  if (threadIdx.x == 0) any = 0u;
  __syncthreads();
  if (bits) atomicOr(&any, bits);
  __syncthreads();
  if (threadIdx.x == 0) flags[blockIdx.x] = any;
}

// sph: bounding sphere per tpts points (tile_sphere_kernel's); box: bounding
// box per 64 points, (centre, 1 or -1 when only padding), (half extents, 0).
// Either may be NULL.
__global__ __launch_bounds__(kLikThreads) void lik_setup_kernel(
    const float *__restrict__ pts, const float *__restrict__ pose6,
    const float *__restrict__ w, const float *__restrict__ mu, const float *__restrict__ cov,
    float4 *__restrict__ out, float4 *__restrict__ sph, float4 *__restrict__ box,
    float *__restrict__ cpar, float4 *__restrict__ shift, double *__restrict__ th64,
    double *__restrict__ pose64, float *__restrict__ Rt32, uint32_t *__restrict__ status,
    uint32_t *__restrict__ flags, LikSetupArgs a) {
  const int tid = threadIdx.x;
  if (blockIdx.x == 0) {
    __shared__ double scratch[kLikThreads];
    __shared__ double sC[GMM_MAX_K];
    uint32_t bits = 0;
    if (tid == 0) {
      *status = 0u;
      if (pose6) pose_terms(pose6, pose64, Rt32);
    }
    for (int b = tid; b < a.K; b += kLikThreads)
      sC[b] = caller_component(b, w, mu, cov, cpar, shift, th64, &bits);
    apply_bound<kLikThreads>(a.K, sC, cpar, scratch);
    lik_flag(bits, flags);
    return;
  }
  __shared__ float R[12];
  __shared__ float wlo[4][3], whi[4][3];
  if (pose6) {
    if (tid == 0) {
      double p64[21];
      float r32[12];
      pose_terms(pose6, p64, r32);
      for (int j = 0; j < 12; ++j) R[j] = r32[j];
    }
    __syncthreads();
  }
  const int lane = tid & 63, wv = tid >> 6;
  uint32_t bits = 0;
  const int64_t step = (int64_t)(gridDim.x - 1) * kLikThreads;
  for (int64_t base = (int64_t)(blockIdx.x - 1) * kLikThreads; base < a.npad; base += step) {
    const int64_t i = base + tid;
    float x = 0.0f, y = 0.0f, z = 0.0f;
    const bool real = i < a.n;
    if (real) {
      x = pts[3 * i]; y = pts[3 * i + 1]; z = pts[3 * i + 2];
      if (!isfinite(x) || !isfinite(y) || !isfinite(z)) {
        bits = kStNonFinite;
        x = y = z = 0.0f;
      }
      if (pose6) {
        const float u = fmaf(R[0], x, fmaf(R[1], y, fmaf(R[2], z, R[9])));
        const float v = fmaf(R[3], x, fmaf(R[4], y, fmaf(R[5], z, R[10])));
        const float q = fmaf(R[6], x, fmaf(R[7], y, fmaf(R[8], z, R[11])));
        x = u; y = v; z = q;
      }
    }
    out[i] = make_float4(x, y, z, __int_as_float(real ? 0 : -1));
    if (!sph && !box) continue;
    float lo0 = real ? x : INFINITY, lo1 = real ? y : INFINITY, lo2 = real ? z : INFINITY;
    float hi0 = real ? x : -INFINITY, hi1 = real ? y : -INFINITY, hi2 = real ? z : -INFINITY;
    for (int off = 32; off > 0; off >>= 1) {
      lo0 = fminf(lo0, __shfl_xor(lo0, off, 64));
      lo1 = fminf(lo1, __shfl_xor(lo1, off, 64));
      lo2 = fminf(lo2, __shfl_xor(lo2, off, 64));
      hi0 = fmaxf(hi0, __shfl_xor(hi0, off, 64));
      hi1 = fmaxf(hi1, __shfl_xor(hi1, off, 64));
      hi2 = fmaxf(hi2, __shfl_xor(hi2, off, 64));
    }
    if (box && lane == 0) {
      const TileBox t = tile_box(lo0, lo1, lo2, hi0, hi1, hi2);
      box[2 * (i >> 6)] = t.c;
      box[2 * (i >> 6) + 1] = t.h;
    }
    if (sph) {
      if (lane == 0) {
        wlo[wv][0] = lo0; wlo[wv][1] = lo1; wlo[wv][2] = lo2;
        whi[wv][0] = hi0; whi[wv][1] = hi1; whi[wv][2] = hi2;
      }
      __syncthreads();
      const int per = a.tpts >> 6;       // waves per tile
      if (tid * a.tpts < kLikThreads) {  // thread q: tile q of the chunk
        for (int v = tid * per; v < (tid + 1) * per; ++v) {
          lo0 = fminf(v == tid * per ? INFINITY : lo0, wlo[v][0]);
          lo1 = fminf(v == tid * per ? INFINITY : lo1, wlo[v][1]);
          lo2 = fminf(v == tid * per ? INFINITY : lo2, wlo[v][2]);
          hi0 = fmaxf(v == tid * per ? -INFINITY : hi0, whi[v][0]);
          hi1 = fmaxf(v == tid * per ? -INFINITY : hi1, whi[v][1]);
          hi2 = fmaxf(v == tid * per ? -INFINITY : hi2, whi[v][2]);
        }
        sph[base / a.tpts + tid] = tile_sphere(lo0, lo1, lo2, hi0, hi1, hi2);
      }
      __syncthreads();
    }
  }
  lik_flag(bits, flags);
}

// The OR of the setup launch's block flags, by one wave or more (tid < nt).
__device__ __forceinline__ uint32_t lik_flags_or(const uint32_t *__restrict__ flags, int nflags,
                                                 int tid, int nt) {
  uint32_t f = 0;
  for (int i = tid; i < nflags; i += nt) f |= flags[i];
  return f;
}

// L of a forward pass: the last column of the partial rows, and the status
// of the whole call.  One block; thread t takes the rows t, t + 1024, ...,
// then block_sum_fast's order.
constexpr int kLikFinishThreads = 1024;
__global__ __launch_bounds__(kLikFinishThreads) void lik_finish_kernel(
    const double *__restrict__ part, int nrows, int ncols, int col,
    const uint32_t *__restrict__ flags, int nflags, double *__restrict__ out_L,
    uint32_t *__restrict__ status) {
  __shared__ double scratch[kLikFinishThreads / 64 + 1];
  double v = 0.0;
  for (int r = threadIdx.x; r < nrows; r += kLikFinishThreads)
    v += part[(size_t)r * ncols + col];
  uint32_t f = lik_flags_or(flags, nflags, threadIdx.x, kLikFinishThreads);
  const double L = block_sum_fast<kLikFinishThreads>(v, scratch);
  if (threadIdx.x == 0) {
    *out_L = L;
    if (!isfinite(L)) f |= kStNonFinite;
  }
  if (f) set_status(status, f);
}

// ------------------------------------------------ culled backward kernel
//
// The gradient of em_bwd_kernel (same formulas, same row layout) with the
// tile culling of the forward pass: a (tile, component) pair whose float32
// weight is exactly zero for the whole tile adds nothing to any gradient.
// Tiles are 64 points, not the forward's 128, and bounded by boxes: the
// source points of a registration are in the caller's order (raster rows of
// a depth image, not Morton order: one evaluation does not pay for a sort),
// and a run of them is long and thin.  At K = 200 and 100,000 of 307,200
// pixels 40 % of the pairs pass the box test at 64 points (53 % at 128),
// 52 % the sphere test (72 %).
//
// Per tile, NW waves, lanes = points:
//  E-phase    wave w takes slots w, w + NW, ... of the active list: e_pb to
//             LDS row `slot` (SCAP rows; a tile with more active components
//             recomputes later rows), s_p and G_p = sum e_pb P'^T z;
//  normaliser wave 0: s_p, G_p over the waves, then g_p = dL/dy_p, dL/dx_p
//             and the pose sums; meanwhile wave 1 + c lists chunk c of the
//             next tile;
//  M-phase    lanes = (slot, 8-point subset): N, A, B as the forward's, float32
//             over RUN points, then FP64;
//  far points (s_p below 2^-100): maxima and sums, each wave over its share
//             of all components, then a second M-phase over all components
//             with the weights of the far points alone.  With one thread
//             per far point walking the components twice, N = 100,000, K =
//             200 with 14 % far points took 216 us a launch (38 us without).
//
// Against em_bwd_kernel (us a call): 300,000 points of an image 337 and 1,216
// at K = 512, 150 and 375 at K = 200, 94 and 128 at K = 64; in random order 727
// and 2,262, 290 and 665, 131 and 172.  The other side of the line: components
// so wide that every pair is active and no point is far (sigma three times
// that of a fit), 166 and 149 at K = 200, 380 and 270 at K = 512; at 100,000
// points 97 and 99, 178 and 153.  There the dense kernel gains by 13 to 32
// points a thread and by rows that it need not form twice.  It is not chosen
// for them: on the host nothing tells such a call from a cloud in random
// order, every box of which is as active; a choice on the device, by sampled
// boxes, took 7 us more in every call and the dense kernel for those clouds.
// More rows cost blocks per CU: 128 of them 225 us instead of 164 at 100,000
// points, K = 512, all of them in blocks of 1,024 threads 96 instead of 90 at
// K = 200.
constexpr int kBwdCullT = 64;
constexpr int kBwdCullBlock = 512;
constexpr int kBwdCullP = 8;                        // point subsets per slot
constexpr int kBwdCullTrip = kBwdCullT / kBwdCullP;
constexpr int kBwdCullRow = (kBwdCullT + kBwdCullP) | 1;
constexpr int kBwdCullXs = kBwdCullT + kBwdCullP;

template <int SCAP>
__host__ __device__ constexpr size_t bwd_cull_lds_bytes(int K) {
  constexpr int NW = kBwdCullBlock / 64;
  return (((size_t)SCAP * kBwdCullRow * sizeof(float) + 15) & ~(size_t)15) +
         (size_t)kBwdCullXs * sizeof(float4) + (size_t)K * kNStat * sizeof(double) +
         32 * sizeof(uint64_t) + 6 * kBwdCullT * sizeof(double) +
         (size_t)4 * NW * kBwdCullT * sizeof(float) + (size_t)2 * K * sizeof(uint16_t) +
         4 * sizeof(int);
}

// s_p and G_p of one point over some components.
struct PairSums {
  float s = 0.0f, G0 = 0.0f, G1 = 0.0f, G2 = 0.0f;
  // one component: e = 2^(l' - m), s += e, G += e P'^T z; returns e
  __device__ __forceinline__ float add(const float *__restrict__ q, float4 x, float m) {
    const float d0 = x.x - q[0], d1 = x.y - q[1], d2 = x.z - q[2];
    const float z0 = q[4] * d0;
    const float z1 = fmaf(q[5], d0, q[6] * d1);
    const float z2 = fmaf(q[7], d0, fmaf(q[8], d1, q[9] * d2));
    const float l = fmaf(-z2, z2, fmaf(-z1, z1, fmaf(-z0, z0, q[3])));
    const float e = __builtin_amdgcn_exp2f(l - m);
    s += e;
    G0 = fmaf(e, fmaf(q[4], z0, fmaf(q[5], z1, q[7] * z2)), G0);
    G1 = fmaf(e, fmaf(q[6], z1, q[8] * z2), G1);
    G2 = fmaf(e, q[9] * z2, G2);
    return e;
  }
  // the sums of wave w into reds (4 x waves x T), and those of all waves
  __device__ __forceinline__ void store(float *reds, int w, int lane) const {
    constexpr int NW = kBwdCullBlock / 64, T = kBwdCullT;
    reds[w * T + lane] = s;
    reds[(NW + w) * T + lane] = G0;
    reds[(2 * NW + w) * T + lane] = G1;
    reds[(3 * NW + w) * T + lane] = G2;
  }
  __device__ __forceinline__ void load(const float *reds, int lane) {
    constexpr int NW = kBwdCullBlock / 64, T = kBwdCullT;
    s = G0 = G1 = G2 = 0.0f;
#pragma unroll
    for (int j = 0; j < NW; ++j) {
      s += reds[j * T + lane];
      G0 += reds[(NW + j) * T + lane];
      G1 += reds[(2 * NW + j) * T + lane];
      G2 += reds[(3 * NW + j) * T + lane];
    }
  }
};

// Ten statistics summed in FP64 over the 8 adjacent lanes of a slot as a
// reduce-scatter: half-mirror (q, 7 - q) keeps 0-4 in lanes 0-3 and 5-9 in
// lanes 4-7 (h = 0, 5); q ^ 2 keeps h, h + 1 where bit 1 of q is clear and
// h + 3, h + 4 where it is set; q ^ 1 the first or second of those.  *third:
// h + 2, in every lane.  float32 values travel as such to the first sum.
__device__ __forceinline__ double from_half_mirror(float v) {
  return (double)dpp_from_half_mirror(v);
}
__device__ __forceinline__ double from_half_mirror(double v) { return dpp_f64<0x141>(v); }

template <typename V>
__device__ __forceinline__ double scatter8_f64(const V *a, int q, double *third) {
  const bool hi = (q & 4) != 0, b2 = (q & 2) != 0, b1 = (q & 1) != 0;
  double k[5];
#pragma unroll
  for (int j = 0; j < 5; ++j) {
    k[j] = (double)(hi ? a[j + 5] : a[j]) + from_half_mirror(hi ? a[j] : a[j + 5]);
  }
  const double v0 = (b2 ? k[3] : k[0]) + dpp_f64<0x4E>(b2 ? k[0] : k[3]);
  const double v1 = (b2 ? k[4] : k[1]) + dpp_f64<0x4E>(b2 ? k[1] : k[4]);
  const double v2 = k[2] + dpp_f64<0x4E>(k[2]);
  *third = v2 + dpp_f64<0xB1>(v2);
  return (b1 ? v1 : v0) + dpp_f64<0xB1>(b1 ? v0 : v1);
}

// RUN: points that a thread adds in float32 before they reach FP64.  The
// dense kernel adds 1 (K <= 8) to 5 points in float32 below 40 components and
// at least 8 from there on; this one adds no more.  (A sum of a slot's eight
// lanes in float32 as well took the same time: 300,000 points, K = 200, all
// components active 166 us a call, 100,000 with 40 % of them 89 us.)
template <int SCAP, int RUN>
__global__ __launch_bounds__(kBwdCullBlock)
__attribute__((amdgpu_waves_per_eu(6, 8))) void em_bwd_cull_kernel(
    const float4 *__restrict__ pts, const float4 *__restrict__ box,
    const float *__restrict__ cpar, const float4 *__restrict__ shift,
    const float *__restrict__ Rt, const double *__restrict__ grad_L,
    double *__restrict__ part, float *__restrict__ g_pts, TileArgs a, int64_t n_real) {
  constexpr int BLOCK = kBwdCullBlock, NW = BLOCK / 64, T = kBwdCullT, P = kBwdCullP;
  constexpr int TRIP = kBwdCullTrip, RS = kBwdCullRow, SLOTS = BLOCK / P;
  extern __shared__ __align__(16) unsigned char smem[];
  const int K = a.K;
  float *E = reinterpret_cast<float *>(smem);
  float4 *Xs = reinterpret_cast<float4 *>(
      smem + (((size_t)SCAP * RS * sizeof(float) + 15) & ~(size_t)15));
  double *acc = reinterpret_cast<double *>(Xs + kBwdCullXs);
  uint64_t *masks = reinterpret_cast<uint64_t *>(acc + (size_t)K * kNStat);  // 2 x 16
  double *pgs = reinterpret_cast<double *>(masks + 32);    // 6 x T: pose sums
  float *reds = reinterpret_cast<float *>(pgs + 6 * T);     // 4 x NW x T
  uint16_t *list = reinterpret_cast<uint16_t *>(reds + 4 * NW * T);   // 2 x K
  int *nact_s = reinterpret_cast<int *>(list + 2 * K);                // 2
  __shared__ uint64_t fbmask;

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nchk = (K + 63) >> 6;   // <= NW
  const int tx = lane + lane / TRIP;
  const float inv_s2 = (float)(2.0 / kLog2e);
  const float gl = grad_L ? (float)grad_L[0] : 1.0f;
  for (int i = tid; i < K * kNStat; i += BLOCK) acc[i] = 0.0;
  const CullPar creg = cull_par(cpar, K, (w << 6) + lane);
  for (int i = tid; i < 6 * T; i += BLOCK) pgs[i] = 0.0;
  unsigned long long npairs = 0;

  // wave 0: dL/dx of this lane's point from s_p and G_p, and its share of
  // the pose sums
  auto finish_point = [&](float4 x, size_t idx, float st, float H0, float H1, float H2) {
    const float r = 1.0f / st;
    const float c = -r * inv_s2;
    const float g0 = c * H0, g1 = c * H1, g2 = c * H2;
    float tv0 = 0.0f, tv1 = 0.0f, tv2 = 0.0f;
    float o0 = g0, o1 = g1, o2 = g2;
    if (Rt) {
      o0 = Rt[0] * g0 + Rt[3] * g1 + Rt[6] * g2;
      o1 = Rt[1] * g0 + Rt[4] * g1 + Rt[7] * g2;
      o2 = Rt[2] * g0 + Rt[5] * g1 + Rt[8] * g2;
      tv0 = Rt[9]; tv1 = Rt[10]; tv2 = Rt[11];
    }
    if (g_pts && idx < (size_t)n_real) {
      g_pts[3 * idx + 0] = gl * o0;
      g_pts[3 * idx + 1] = gl * o1;
      g_pts[3 * idx + 2] = gl * o2;
    }
    const float rx = x.x - tv0, ry = x.y - tv1, rz = x.z - tv2;
    double *pg = pgs + lane;
    pg[0] += g0; pg[T] += g1; pg[2 * T] += g2;
    pg[3 * T] += (double)(ry * g2 - rz * g1);
    pg[4 * T] += (double)(rz * g0 - rx * g2);
    pg[5 * T] += (double)(rx * g1 - ry * g0);
  };
  // active list of a tile from masks buffer bf: chunk c by wave 1 + c (wave
  // 0 normalises meanwhile), by wave c when there are not that many waves
  const int wl = nchk < NW ? w - 1 : w;
  auto build_list = [&](int bf) {
    const uint64_t *mk = masks + 16 * bf;
    if (wl >= 0 && wl < nchk) {
      int off = 0;
      for (int c = 0; c < wl; ++c) off += __popcll(mk[c]);
      const uint64_t m = mk[wl];
      const unsigned below = __builtin_amdgcn_mbcnt_hi(
          (unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
      if ((m >> lane) & 1ull) list[K * bf + off + (int)below] = (uint16_t)((wl << 6) + lane);
      if (wl == nchk - 1 && lane == 0) nact_s[bf] = off + __popcll(m);
    }
  };

  // N, A, B of nloc slots (component comp(slot)) from the E rows and Xs
  static_assert(P == 8 && TRIP % RUN == 0, "scatter8_f64; whole runs");
  const int q = tid % P;
  auto m_phase = [&](int nloc, auto comp) {
    for (int sl = tid / P; sl < nloc; sl += SLOTS) {
      const int b = comp(sl);
      const float4 sh = shift[b];
      const float *Eb = E + sl * RS + q * (TRIP + 1);
      const float4 *Xb = Xs + q * (TRIP + 1);
      std::conditional_t<RUN == TRIP, float, double> av[kNStat];
#pragma unroll
      for (int r = 0; r < TRIP; r += RUN) {
        float f[kNStat];
#pragma unroll
        for (int j = 0; j < kNStat; ++j) f[j] = 0.0f;
#pragma unroll
        for (int j = r; j < r + RUN; ++j) {
          const float4 xr = Xb[j];
          const float gm = Eb[j] * xr.w;
          const float d0 = xr.x - sh.x, d1 = xr.y - sh.y, d2 = xr.z - sh.z;
          const float w0 = gm * d0, w1 = gm * d1, w2 = gm * d2;
          f[0] += gm;
          f[1] += w0; f[2] += w1; f[3] += w2;
          f[4] = fmaf(w0, d0, f[4]);
          f[5] = fmaf(w1, d0, f[5]);
          f[6] = fmaf(w1, d1, f[6]);
          f[7] = fmaf(w2, d0, f[7]);
          f[8] = fmaf(w2, d1, f[8]);
          f[9] = fmaf(w2, d2, f[9]);
          // (two points in flight: with all eight, 33 registers spill and a
          // call takes 4 to 5 us more)
          if (RUN == 1 || (j & 1)) __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int j = 0; j < kNStat; ++j) av[j] = r ? av[j] + f[j] : f[j];
      }
      double third;
      const double mine = scatter8_f64(av, q, &third);
      double *ab = acc + (size_t)b * kNStat + (q >> 2) * 5;
      ab[(q & 2) + (q >> 1 & 1) + (q & 1)] += mine;
      if ((q & 3) == 0) ab[2] += third;
    }
  };

  const int stride = gridDim.x;
  int tile = blockIdx.x, cur = 0;
  float4 xn = make_float4(0.f, 0.f, 0.f, __int_as_float(-1));
  TileBox bxn = {make_float4(0.f, 0.f, 0.f, -1.0f), make_float4(0.f, 0.f, 0.f, 0.f)};
  if (tile < a.ntiles) {
    xn = pts[(size_t)tile * T + lane];
    if (tile + stride < a.ntiles)
      bxn = {box[2 * (tile + stride)], box[2 * (tile + stride) + 1]};
    if (w < nchk) {
      const uint64_t m = box_ballot(creg, {box[2 * tile], box[2 * tile + 1]});
      if (lane == 0) masks[w] = m;
    }
  }
  __syncthreads();
  if (tile < a.ntiles) build_list(0);
  __syncthreads();
  for (; tile < a.ntiles; tile += stride) {
    const float4 x = xn;
    const bool more = tile + stride < a.ntiles;
    if (more) xn = pts[(size_t)(tile + stride) * T + lane];
    const bool valid = __float_as_int(x.w) >= 0;
    const int nxt = cur ^ 1;
    const int nact = nact_s[cur];
    const uint16_t *lst = list + K * cur;

    // ---- E-phase
    PairSums ps;
    {
      constexpr int EU = 4;
      int sl = w;
      for (; sl + (EU - 1) * NW < nact; sl += EU * NW) {
        float e[EU];
#pragma unroll
        for (int u = 0; u < EU; ++u) {
          const int b = __builtin_amdgcn_readfirstlane((int)lst[sl + u * NW]);
          e[u] = ps.add(cpar + (size_t)b * kParStride, x, 0.0f);
        }
#pragma unroll
        for (int u = 0; u < EU; ++u)
          if (sl + u * NW < SCAP) E[(sl + u * NW) * RS + tx] = e[u];
      }
      for (; sl < nact; sl += NW) {
        const int b = __builtin_amdgcn_readfirstlane((int)lst[sl]);
        const float e = ps.add(cpar + (size_t)b * kParStride, x, 0.0f);
        if (sl < SCAP) E[sl * RS + tx] = e;
      }
      ps.store(reds, w, lane);
    }
    if (more && w < nchk) {
      const uint64_t m = box_ballot(creg, bxn);
      if (lane == 0) masks[16 * nxt + w] = m;
    }
    if (tile + 2 * stride < a.ntiles)
      bxn = {box[2 * (tile + 2 * stride)], box[2 * (tile + 2 * stride) + 1]};
    __syncthreads();                                              // A

    // ---- normaliser and dL/dx
    if (w == 0) {
      ps.load(reds, lane);
      const bool fb = valid && !(ps.s >= 0x1p-100f);
      Xs[tx] = make_float4(x.x, x.y, x.z, (valid && !fb) ? 1.0f / ps.s : 0.0f);
      const uint64_t fm = __ballot(fb);
      if (lane == 0) fbmask = fm;
      if (valid && !fb)
        finish_point(x, (size_t)tile * T + lane, ps.s, ps.G0, ps.G1, ps.G2);
    }
    if (more) build_list(nxt);
    __syncthreads();                                              // B

    // ---- M-phase over the active list, SCAP slots at a time
    if (tid == 0) npairs += (unsigned)nact;
    for (int c0 = 0; c0 < nact; c0 += SCAP) {
      const int nloc = min(SCAP, nact - c0);
      if (c0 > 0) {
        __syncthreads();
        for (int sl = w; sl < nloc; sl += NW) {
          const int b = __builtin_amdgcn_readfirstlane((int)lst[c0 + sl]);
          E[sl * RS + tx] = __builtin_amdgcn_exp2f(
              comp_logterm(cpar + (size_t)b * kParStride, x.x, x.y, x.z));
        }
        __syncthreads();
      }
      m_phase(nloc, [&](int sl) { return (int)lst[c0 + sl]; });
    }

    // ---- far points: maxima, then sums, each wave over its share of the
    // components; then an M-phase over all components with their weights
    const uint64_t fball = fbmask;
    if (fball) {
      const bool fb = (fball >> lane) & 1ull;
      const int b_lo = (w * K) / NW, b_hi = ((w + 1) * K) / NW;
      float mx = -INFINITY;
      for (int b = b_lo; b < b_hi; ++b)
        mx = fmaxf(mx, comp_logterm(cpar + (size_t)b * kParStride, x.x, x.y, x.z));
      reds[w * T + lane] = mx;
      __syncthreads();
#pragma unroll
      for (int j = 0; j < NW; ++j) mx = fmaxf(mx, reds[j * T + lane]);
      // the other lanes' weights are 0, so their terms only have to be finite:
      // at padding's position every term may be -inf, less a maximum of -inf
      if (!fb) mx = 0.0f;
      __syncthreads();
      PairSums ps;
      for (int b = b_lo; b < b_hi; ++b) ps.add(cpar + (size_t)b * kParStride, x, mx);
      ps.store(reds, w, lane);
      __syncthreads();
      if (w == 0) {
        ps.load(reds, lane);
        Xs[tx] = make_float4(x.x, x.y, x.z, fb ? 1.0f / ps.s : 0.0f);
        if (fb) finish_point(x, (size_t)tile * T + lane, ps.s, ps.G0, ps.G1, ps.G2);
      }
      for (int c0 = 0; c0 < K; c0 += SCAP) {
        const int nloc = min(SCAP, K - c0);
        if (c0 > 0) __syncthreads();
        for (int sl = w; sl < nloc; sl += NW)
          E[sl * RS + tx] = __builtin_amdgcn_exp2f(
              comp_logterm(cpar + (size_t)(c0 + sl) * kParStride, x.x, x.y, x.z) - mx);
        __syncthreads();
        m_phase(nloc, [&](int sl) { return c0 + sl; });
      }
    }
    __syncthreads();                                                // C
    cur = nxt;
  }

  // ---- this block's partial row
  double *row = part + (size_t)blockIdx.x * a.ncols;
  for (int i = tid; i < K * kNStat; i += BLOCK) row[i] = acc[i];   // component-major
  if (w < kBwdExtra) {   // (the log-likelihood column before them is not used)
    const double v = wave_sum_f64(pgs[w * T + lane]);
    if (lane == 0) row[kNStat * K + 1 + w] = v;
  }
  if (tid == 0 && a.pairs) atomicAdd(a.pairs, npairs);
}

// ------------------------------------------------------ backward's last launch
// The gradients from the partial rows: block b < K sums the ten columns of
// component b (thread (g, s): statistic s of the rows g, g + 64, ...; wave s
// adds the 64 group sums) and thread 0 forms, from the FP32 mixture
// (Sigma^-1 = P^T P from an FP64 Cholesky),
//   dL/dpi_b = N_b / pi_b,  dL/dmu_b = Sigma^-1 A_b,
//   dL/dSigma_b = 1/2 Sigma^-1 B_b Sigma^-1 - 1/2 N_b Sigma^-1;
// block K sums the pose columns and forms dL/dt = sum g and dL/domega =
// J_l^T sum (y - t) x g.  All times grad_L.  One launch: as a row reduction
// and one finishing block these took 4.7 + 9.7 us at K = 200.
__global__ __launch_bounds__(kFuseThreads) void bwd_finish_kernel(
    const double *__restrict__ part, int nrows, int ncols, int K, int cmaj,
    const float *__restrict__ w, const float *__restrict__ cov,
    const double *__restrict__ pose64, const double *__restrict__ grad_L,
    const uint32_t *__restrict__ flags, int nflags, float *g_pose6, float *g_w, float *g_mu,
    float *g_cov, uint32_t *status) {
  __shared__ double sums[kFuseGroups * kNStat];
  __shared__ double tot[kNStat];
  const int tid = threadIdx.x, lane = tid & 63;
  const int b = blockIdx.x;
  const int ns = b < K ? kNStat : kBwdExtra;   // columns of this block
  if (tid < kFuseGroups * ns) {
    const int g = tid / ns, st = tid - g * ns;
    const double *src =
        part + (b == K ? kNStat * K + 1 + st : cmaj ? b * kNStat + st : st * K + b);
    double acc = 0.0;
    for (int r = g; r < nrows; r += 16 * kFuseGroups) {
      double v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u)
        v[u] = (r + u * kFuseGroups < nrows) ? src[(size_t)(r + u * kFuseGroups) * ncols] : 0.0;
#pragma unroll
      for (int u = 0; u < 16; ++u) acc += v[u];
    }
    sums[tid] = acc;
  }
  if (b == K) {
    const uint32_t f = lik_flags_or(flags, nflags, tid, kFuseThreads);
    if (f) set_status(status, f);
  }
  __syncthreads();
  if ((tid >> 6) < ns) {
    const double v = wave_sum_f64(sums[lane * ns + (tid >> 6)]);
    if (lane == 0) tot[tid >> 6] = v;
  }
  __syncthreads();
  if (tid != 0) return;
  const double gl = grad_L ? grad_L[0] : 1.0;
  if (b == K) {
    if (!g_pose6) return;
    double J[9] = {1, 0, 0, 0, 1, 0, 0, 0, 1};
    if (pose64)
      for (int i = 0; i < 9; ++i) J[i] = pose64[12 + i];
    double sum = 0.0;
    for (int i = 0; i < 6; ++i) sum += tot[i];
    for (int i = 0; i < 3; ++i) {
      g_pose6[i] = (float)(gl * (J[i] * tot[3] + J[3 + i] * tot[4] + J[6 + i] * tot[5]));
      g_pose6[3 + i] = (float)(gl * tot[i]);
    }
    if (!isfinite(sum)) set_status(status, kStNonFinite);
    return;
  }
  const double N = tot[0];
  const float *c = cov + 9 * b;
  const double C[6] = {c[0], c[3], c[4], c[6], c[7], c[8]};
  double L[6], P[6];
  if (!chol3(C, L)) {
    // no gradient exists: the component's outputs are NaN, not stale memory
    set_status(status, kStNotSpd);
    const float nan = __builtin_nanf("");
    if (g_w) g_w[b] = nan;
    if (g_mu)
      for (int i = 0; i < 3; ++i) g_mu[3 * b + i] = nan;
    if (g_cov)
      for (int i = 0; i < 9; ++i) g_cov[9 * b + i] = nan;
    return;
  }
  tri_inv3(L, P);
  // Sigma^-1 = P^T P (full symmetric)
  const double Pm[9] = {P[0], 0.0, 0.0, P[1], P[2], 0.0, P[3], P[4], P[5]};
  double Si[9];
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) {
      double v = 0.0;
      for (int k = 0; k < 3; ++k) v += Pm[k * 3 + i] * Pm[k * 3 + j];
      Si[i * 3 + j] = v;
    }
  const double *Bl = tot + 4;
  const double B[9] = {Bl[0], Bl[1], Bl[3], Bl[1], Bl[2], Bl[4], Bl[3], Bl[4], Bl[5]};
  if (g_w) g_w[b] = (float)(gl * N / (double)w[b]);
  if (g_mu)
    for (int i = 0; i < 3; ++i)
      g_mu[3 * b + i] =
          (float)(gl * (Si[i * 3] * tot[1] + Si[i * 3 + 1] * tot[2] + Si[i * 3 + 2] * tot[3]));
  if (g_cov) {
    double T1[9];
    for (int i = 0; i < 3; ++i)
      for (int j = 0; j < 3; ++j) {
        double v = 0.0;
        for (int k = 0; k < 3; ++k) v += Si[i * 3 + k] * B[k * 3 + j];
        T1[i * 3 + j] = v;
      }
    for (int i = 0; i < 3; ++i)
      for (int j = 0; j < 3; ++j) {
        double v = 0.0;
        for (int k = 0; k < 3; ++k) v += T1[i * 3 + k] * Si[k * 3 + j];
        g_cov[9 * b + i * 3 + j] = (float)(gl * (0.5 * v - 0.5 * N * Si[i * 3 + j]));
      }
  }
}

}  // namespace gmm_dev
