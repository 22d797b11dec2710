// Biot-Savart non-local superfluid velocity (paper Sec. II.A, Eq.
// Biot-Savart): every target point j sums the exact straight-segment
// integral over all segments k = (s_k, s_next(k)) except the two that touch
// it (k = prev(j) and k = j; their divergent contribution is the LIA term).
//
// Layout and decomposition:
//  * FP32: per point 32-bit grid coordinates X (3 x u32, SoA); the segment
//    vector d_k = s_next(k) - s_k is the wrapped grid difference.  FP64: the
//    sum reads the positions themselves (grid coordinates, residuals and
//    FP64 nearest-image segment vectors are formed while a tile is staged,
//    about 1% of the pair work, so that no kernel precedes the sum);
//  * a 2-D grid: blockIdx.x picks 64 consecutive targets (one per lane of
//    every wave), blockIdx.y one contiguous chunk of sources; the chunk is
//    staged through LDS in tiles of 256 sources, each of the block's 4
//    waves walks its own quarter of the tile, and the 4 wave sums are added
//    in LDS in a fixed order at the end (fewer, longer chunks than with one
//    wave per target, so fewer partial sums to write and to add);
//  * the separation R1 = s_k - r is the wrapped integer difference of the
//    grid coordinates, converted to floating point: exact nearest periodic
//    image and a relative (not absolute) rounding error for near pairs;
//  * each chunk writes one partial sum per target; the finalize kernel adds
//    the chunks in a fixed order (no atomics, bitwise reproducible).
#include "bs_pair.h"

#include <cmath>

namespace vlb {

namespace {

constexpr int kTile = 256;
constexpr int kTargets = 64;  // targets per block, one per lane of each wave
// Point count from which the FP64 sum takes two targets per lane: a record
// read from LDS then serves two pairs and two dependence chains overlap (2e4
// points 550 against 578 us, 6e4 points 4560 against 4710); with fewer points
// the blocks of half as many targets fill the chip better (1e4 points 159
// against 164 us).
constexpr long long kWideTargets = 16384;

// Point count up to which the FP32 stand-alone sum forms grid coordinates
// while it stages a tile (about 5% of the pair work) instead of in a launch
// before it: 1e3 points 13.4 against 16.9 us per call, 4e3 22.5 against 25.3,
// level from 8e3 on.
constexpr long long kDirectPoints = 4096;

// Point count up to which the stand-alone sum is one launch, each block with
// all sources for 8 targets (k_bs_few), in place of chunks and a launch that
// adds them: 300 points FP64 9.5 -> 6.9 us per call, 1000 FP32 13.3 -> 11.2,
// 1400 FP64 10.4 against 10.2, 1700 FP32 13.1 against 12.6; with 512 threads a
// block 11.5 at 1000 and 13.5 at 1700, with 256 (and 2000 points) half as fast
// as the chunks.
constexpr long long kFewPoints = 1280;

// Quarter of a staged tile of cnt sources walked by wave w: [lo, hi) (empty
// when lo >= hi), at most 64 of a tile of 256.
__device__ inline void wave_range(int cnt, int w, int& lo, int& hi) {
  const int q = (cnt + 3) >> 2;
  lo = w * q;
  hi = __builtin_amdgcn_readfirstlane(min(cnt, lo + q));
}

// FP32: grid coordinates X (stride nc) of the points (copy 0) and of their
// images in the wall planes (copies 1..).
__global__ void k_prep(BsPts in, const int32_t* __restrict__ cntp, int n_arg, long long nc,
                       BsAxes ax, uint32_t* __restrict__ X) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  const int n = cntp ? cntp[0] : n_arg;
  if (j >= n) return;
  double y[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) y[a] = in.Y[a * in.sa + j * in.sj];
  for (int c = 0; c < ax.copies; ++c) {
#pragma unroll
    for (int a = 0; a < 3; ++a)
      X[((long long)c * 3 + a) * nc + j] = bs_grid_f32(bs_mirror(y[a], ax.refl[c][a], ax.L[a]), ax, a);
  }
}

// Does one of the wave's sources [t0 + lo, t0 + hi) (at most 64, staged at
// src) start or end at one of the nt targets from j0 on?  Uniform per wave.
template <class Src>
__device__ inline bool bs_hit(const Src* src, int t0, int lo, int hi, int j0, int nt) {
  const int lane = threadIdx.x & 63;
  bool hit = false;
  if (lane < hi - lo)
    hit = (uint32_t)(t0 + lo + lane - j0) < (uint32_t)nt ||
          (uint32_t)(src[lo + lane].kn - j0) < (uint32_t)nt;
  return __any(hit);
}

template <bool kCheck, bool kUniform>
__device__ inline void bs_tile_f32(const BsSrc* src, int cnt, int t0, uint32_t xt, uint32_t yt,
                                   uint32_t zt, float iqx, float iqy, float iqz, int jj,
                                   float& ax, float& ay, float& az) {
  // unrolled twice: 8 waves per SIMD (four ways: 2% slower)
#pragma unroll 2
  for (int s = 0; s < cnt; ++s) {
    const BsSrc g = src[s];
    bs_pair_f32<kUniform>(g, xt, yt, zt, iqx, iqy, iqz,
                          kCheck && (t0 + s == jj || g.kn == jj), ax, ay, az);
  }
}

// Grid y: S chunks of every source copy (copy 0 the filaments, the others
// their wall images, which take no exclusion and carry the copy's sign).
// kDirect: grid coordinates from the positions (stand-alone sums of few
// points, one copy), else from X.
template <bool kUniform, bool kDirect>
__global__ __launch_bounds__(256) void k_bs_f32(BsPts in, const uint32_t* __restrict__ X,
                                               int32_t* __restrict__ cntp, int n_arg,
                                               long long nc, int S, float iqx, float iqy,
                                               float iqz, float* __restrict__ P, BsAxes bx) {
  const int n = cntp ? cntp[0] : n_arg;
  // work counter: (target, segment) pairs of this sum
  if (cntp && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0 && n > 2)
    *(long long*)(cntp + 16) += (long long)n * (n - 2) + (long long)(bx.copies - 1) * n * n;
  const int j0 = blockIdx.x * kTargets;
  if (j0 >= n) return;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform per wave
  const int j = j0 + lane;
  const bool valid = j < n;
  const int jc = min(j, n - 1);  // lanes beyond the points repeat the last one, unwritten
  const int copy = blockIdx.y / S;
  const uint32_t* __restrict__ Xs = X + (long long)copy * 3 * nc;  // this copy's sources
  const int per = (n + S - 1) / S;
  const int kb = (blockIdx.y - copy * S) * per;
  const int ke = min(n, kb + per);
  uint32_t xt, yt, zt;
  if (kDirect) {
    xt = bs_grid_f32(in.Y[jc * in.sj], bx, 0);
    yt = bs_grid_f32(in.Y[in.sa + jc * in.sj], bx, 1);
    zt = bs_grid_f32(in.Y[2 * in.sa + jc * in.sj], bx, 2);
  } else {
    xt = X[jc];
    yt = X[nc + jc];
    zt = X[2 * nc + jc];
  }
  // the target's own two segments are excluded in copy 0 and, for the end
  // of an open line, in the copy mirrored in its wall
  bool exl = valid && copy == 0;
  if (copy > 0 && valid && (in.nxt[jc] == jc || in.prv[jc] == jc)) {
    double y[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) y[a] = in.Y[a * in.sa + jc * in.sj];
    exl = bs_own_copy(y, bx) == copy;
  }
  const int jj = exl ? j : -1;
  const bool exany = __any(exl);
  __shared__ BsSrc src[kTile];
  __shared__ float red[3][3][kTargets];  // sums of waves 1..3
  float ax = 0.f, ay = 0.f, az = 0.f;
  for (int t0 = kb; t0 < ke; t0 += kTile) {
    const int k = t0 + threadIdx.x;
    if (k < ke)
      src[threadIdx.x] = bs_stage_f32<kUniform, kDirect>(in, Xs, nc, k, n, 0, iqx, iqy, iqz, bx);
    __syncthreads();
    int lo, hi;
    wave_range(min(kTile, ke - t0), w, lo, hi);
    if (lo < hi) {
      if (exany && bs_hit(src, t0, lo, hi, j0, kTargets))
        bs_tile_f32<true, kUniform>(src + lo, hi - lo, t0 + lo, xt, yt, zt, iqx, iqy, iqz, jj, ax,
                                    ay, az);
      else
        bs_tile_f32<false, kUniform>(src + lo, hi - lo, t0 + lo, xt, yt, zt, iqx, iqy, iqz, jj, ax,
                                     ay, az);
    }
    __syncthreads();
  }
  if (w > 0) {
    red[w - 1][0][lane] = ax;
    red[w - 1][1][lane] = ay;
    red[w - 1][2][lane] = az;
  }
  __syncthreads();
  if (w == 0 && valid) {
    const float sg = bx.sign[copy];
    float* out = P + (long long)blockIdx.y * 3 * nc;
    out[j] = sg * (((ax + red[0][0][lane]) + red[1][0][lane]) + red[2][0][lane]);
    out[nc + j] = sg * (((ay + red[0][1][lane]) + red[1][1][lane]) + red[2][1][lane]);
    out[2 * nc + j] = sg * (((az + red[0][2][lane]) + red[1][2][lane]) + red[2][2][lane]);
  }
}

template <int kPer, int NT, bool kCheck>
__device__ inline void bs_tile_f64(const BsSrcD* src, int cnt, int t0, BsTgtD* tg, double gx,
                                   double gy, double gz) {
#pragma unroll(NT == 1 ? 2 : 1)
  for (int s = 0; s < cnt; ++s) {
    const BsSrcD g = src[s];
#pragma unroll
    for (int m = 0; m < NT; ++m)
      bs_pair_f64<kPer>(g, tg[m], kCheck && (t0 + s == tg[m].jj || g.kn == tg[m].jj), gx, gy, gz);
  }
}

template <int kPer, int NT>
__global__ __launch_bounds__(256) void k_bs_f64(BsPts in, int32_t* __restrict__ cntp, int n_arg,
                                               long long nc, int S, double* __restrict__ P,
                                               BsAxes bx) {
  const int n = cntp ? cntp[0] : n_arg;
  if (cntp && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0 && n > 2)
    *(long long*)(cntp + 16) += (long long)n * (n - 2) + (long long)(bx.copies - 1) * n * n;
  constexpr int kT = kTargets * NT;  // targets per block
  const int j0 = blockIdx.x * kT;
  if (j0 >= n) return;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform per wave
  const int copy = blockIdx.y / S;
  const int per = (n + S - 1) / S;
  const int kb = (blockIdx.y - copy * S) * per;
  const int ke = min(n, kb + per);
  BsTgtD tg[NT];
  bool exl = false;
#pragma unroll
  for (int m = 0; m < NT; ++m) {
    const int j = j0 + m * kTargets + lane;
    const int jc = min(j, n - 1);  // lanes beyond the points repeat the last one, unwritten
    double y[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) y[a] = in.Y[a * in.sa + jc * in.sj];
    BsTgtD& t = tg[m];
    bs_target_f64<kPer>(y, bx, t);
    // the target's own two segments are excluded in copy 0 and, for the end
    // of an open line, in the copy mirrored in its wall
    bool ex = j < n && copy == 0;
    if (copy > 0 && j < n && (in.nxt[jc] == jc || in.prv[jc] == jc))
      ex = bs_own_copy(y, bx) == copy;
    t.jj = ex ? j : -1;
    exl = exl || ex;
  }
  const bool exany = __any(exl);
  __shared__ BsSrcD src[kTile];
  static_assert(sizeof(src) >= 9 * kT * sizeof(double), "the wave sums reuse the tile");
  for (int t0 = kb; t0 < ke; t0 += kTile) {
    const int k = t0 + threadIdx.x;
    if (k < ke) src[threadIdx.x] = bs_stage_f64<kPer>(in, k, n, copy, bx);
    __syncthreads();
    int lo, hi;
    wave_range(min(kTile, ke - t0), w, lo, hi);
    if (lo < hi) {
      if (exany && bs_hit(src, t0, lo, hi, j0, kT))
        bs_tile_f64<kPer, NT, true>(src + lo, hi - lo, t0 + lo, tg, bx.invq_d[0], bx.invq_d[1],
                                    bx.invq_d[2]);
      else
        bs_tile_f64<kPer, NT, false>(src + lo, hi - lo, t0 + lo, tg, bx.invq_d[0], bx.invq_d[1],
                                     bx.invq_d[2]);
    }
    __syncthreads();
  }
  double(*red)[3][kT] = reinterpret_cast<double(*)[3][kT]>(src);  // sums of waves 1..3
#pragma unroll
  for (int m = 0; m < NT; ++m)
    if (w > 0) {
      red[w - 1][0][m * kTargets + lane] = tg[m].ax;
      red[w - 1][1][m * kTargets + lane] = tg[m].ay;
      red[w - 1][2][m * kTargets + lane] = tg[m].az;
    }
  __syncthreads();
  const double sg = 0.5 * (double)bx.sign[copy];
  double* out = P + (long long)blockIdx.y * 3 * nc;
#pragma unroll
  for (int m = 0; m < NT; ++m) {
    const int e = m * kTargets + lane, j = j0 + e;
    if (w == 0 && j < n) {
      out[j] = sg * (((tg[m].ax + red[0][0][e]) + red[1][0][e]) + red[2][0][e]);
      out[nc + j] = sg * (((tg[m].ay + red[0][1][e]) + red[1][1][e]) + red[2][1][e]);
      out[2 * nc + j] = sg * (((tg[m].az + red[0][2][e]) + red[1][2][e]) + red[2][2][e]);
    }
  }
}

// ---- standalone sum (positions and links from the caller, no run)
//
// Few points: the whole sum and v in one launch, a block per kFewTargets
// targets.  What bounds it: latency, of the launch, of the links and positions
// (two dependent loads) and of the pairs of one slice in turn, for which the
// block has as many threads as there are.
constexpr int kFewThreads = 1024;
constexpr int kFewTile = 1024;

template <bool kF32, int kVar>
__global__ __launch_bounds__(kFewThreads) void k_bs_few(BsPts in, int n, double scale,
                                                        double* __restrict__ v, BsAxes bx) {
  using Src = std::conditional_t<kF32, BsSrc, BsSrcD>;
  __shared__ Src src[kFewTile];
  __shared__ double red[kFewThreads / 64][3][kFewTargets];
  const int j0 = blockIdx.x * kFewTargets;
  bs_few<kF32, kVar, kFewThreads, kFewTile>(in, n, n, (n + kFewTile - 1) / kFewTile,
                               j0 + (int)threadIdx.x % kFewTargets, bx, src, red);
  const int t = threadIdx.x, m = t / 3, a = t - 3 * m;
  if (t < 3 * kFewTargets && j0 + m < n) {
    double s = red[0][a][m];
#pragma unroll
    for (int w = 1; w < kFewThreads / 64; ++w) s += red[w][a][m];
    v[3LL * j0 + t] = s * scale;
  }
}

// v[j][a] = scale * (sum over the S chunk partials of target j, in chunk
// order, in FP64); one thread per (a, j).
template <class PT>
__global__ __launch_bounds__(256) void k_solo_sum(const PT* __restrict__ P, int S, int n,
                                                  double scale, double* __restrict__ v) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  const long long n3 = 3LL * n;
  if (i >= n3) return;
  double t = 0.0;
#pragma unroll 8
  for (int c = 0; c < S; ++c) t += (double)P[c * n3 + i];
  const long long a = i / n;
  v[3 * (i - a * n) + a] = t * scale;
}

}  // namespace

// Grid of the Biot-Savart sum on a box of n[a] nodes per axis (wall[a]: the
// axis is closed, positions in [-1/2, n - 1/2]; else periodic of length
// n[a]): periodic axes map [0, L) onto the whole 32-bit range, so that
// separations wrap exactly; wall axes use a power-of-two step with room
// for [-1, n + 1).
BsAxes bs_make_axes(const int n[3], const int wall[3], bool images) {
  BsAxes ax{};
  for (int a = 0; a < 3; ++a) {
    ax.L[a] = (double)n[a];
    ax.periodic[a] = !wall[a];
    if (ax.periodic[a]) {
      ax.q[a] = 4294967296.0 / (double)n[a];
      ax.off[a] = 0.0;
      ax.invq_d[a] = (double)n[a] / 4294967296.0;
    } else {
      // [-1, n + 1), or with wall images [-n - 1, 2n + 1)
      const double span = images ? 3.0 * n[a] + 2.0 : n[a] + 2.0;
      int k = 0;
      while (span * std::ldexp(1.0, k + 1) <= 2147483648.0) ++k;
      ax.q[a] = std::ldexp(1.0, k);
      ax.off[a] = images ? n[a] + 1.0 : 1.0;
      ax.invq_d[a] = std::ldexp(1.0, -k);
    }
    ax.invq_f[a] = (float)ax.invq_d[a];
  }
  {
    // one power-of-two grid step for all axes when every periodic axis has
    // the same power-of-two length and the wall axes fit that step
    double q = 0.0;
    for (int a = 0; a < 3; ++a)
      if (ax.periodic[a]) q = ax.q[a];
    if (q == 0.0)
      for (int a = 0; a < 3; ++a) q = (q == 0.0 || ax.q[a] < q) ? ax.q[a] : q;
    int ex = 0;
    bool ok = std::frexp(q, &ex) == 0.5;
    for (int a = 0; a < 3 && ok; ++a) {
      if (ax.periodic[a])
        ok = ax.q[a] == q;
      else
        ok = (images ? 3.0 * n[a] + 2.0 : n[a] + 2.0) * q <= 2147483648.0;
    }
    ax.uniform = ok ? 1 : 0;
    if (ok)
      for (int a = 0; a < 3; ++a) {
        ax.q[a] = q;
        ax.invq_d[a] = 1.0 / q;
        ax.invq_f[a] = (float)ax.invq_d[a];
      }
  }
  // source copies: every combination of no / lower / upper reflection on
  // the closed axes (the identity first)
  ax.copies = 0;
  for (int cz = 0; cz < 3; ++cz)
    for (int cy = 0; cy < 3; ++cy)
      for (int cx = 0; cx < 3; ++cx) {
        const int code[3] = {cx, cy, cz};
        bool ok = true;
        int refl = 0;
        for (int a = 0; a < 3; ++a) {
          if (code[a] && (!images || !wall[a])) ok = false;
          if (code[a]) ++refl;
        }
        if (!ok) continue;
        for (int a = 0; a < 3; ++a) ax.refl[ax.copies][a] = (int8_t)code[a];
        ax.sign[ax.copies] = (refl & 1) ? -1.0f : 1.0f;
        ++ax.copies;
      }
  return ax;
}

// Source chunks S of each of the sum's copies: about 16384 blocks over the
// target blocks, or up to 32768 while every chunk keeps at least 1024
// sources (large point counts: the launch's tail shortens), at least 256
// sources per chunk (64 per wave), at most 256 chunks; the chunk partials
// are added by the finalize kernel.  (At 1.2e4 points 512 and 1024 sources
// per chunk measured 1.5% and 6% slower per step, 128 and 192 no faster; at
// 1.0e5 points 14 chunks instead of 7 measured 1.1% faster, at 5e4 points 28
// instead of 14 0.9%.)  Few points leave the chip idle under that rule, and
// their time is the longest block's: up to 32 chunks in all (what the
// finalize kernel loads at once) while each keeps 32 sources (2000 points,
// the sum alone: 7 chunks 17.7 us, 13 12.0, 30 10.2, 60 9.4).
int bs_chunks(long long ncap, int copies) {
  const long long tb = (ncap + kTargets - 1) / kTargets;
  const long long t = tb > 0 ? tb : 1;
  long long S = 16384 / t;
  const long long wide = std::min(32768 / t, ncap / 1024);
  if (wide > S) S = wide;
  const long long maxS = std::max(ncap / 256, std::min<long long>(32 / copies, ncap / 32));
  if (S > maxS) S = maxS;
  if (S < 1) S = 1;
  if (S > 256) S = 256;
  return (int)S;
}

hipError_t bs_prep(Run& r, const double* Y) {
  if (r.prec == VLB_F64) return hipSuccess;  // that sum reads the positions
  const int nb = (int)((r.ncap + 255) / 256);
  hipLaunchKernelGGL(k_prep, dim3(nb), dim3(256), 0, r.stream,
                     BsPts{Y, r.ncap, 1, r.nxt, r.prv}, r.cnt, 0, r.ncap, r.bsax, r.bsX);
  return hipGetLastError();
}

namespace {

template <int NT>
hipError_t launch_bs_f64(const BsPts& in, int32_t* cnt, long long n, int S, double* P,
                         const BsAxes& ax, hipStream_t stream) {
  using K = void (*)(BsPts, int32_t*, int, long long, int, double*, BsAxes);
  static constexpr K kern[8] = {k_bs_f64<0, NT>, k_bs_f64<1, NT>, k_bs_f64<2, NT>,
                                k_bs_f64<3, NT>, k_bs_f64<4, NT>, k_bs_f64<5, NT>,
                                k_bs_f64<6, NT>, k_bs_f64<7, NT>};
  const int per = (ax.periodic[0] ? 1 : 0) | (ax.periodic[1] ? 2 : 0) | (ax.periodic[2] ? 4 : 0);
  const int tb = (int)((n + kTargets * NT - 1) / (kTargets * NT));
  hipLaunchKernelGGL(kern[per], dim3(tb, S * ax.copies), dim3(256), 0, stream, in, cnt, (int)n, n,
                     S, P, ax);
  return hipGetLastError();
}

// FP64 sum over n points (the capacity when the count is on the device).
hipError_t bs_f64(const BsPts& in, int32_t* cnt, long long n, int S, double* P, const BsAxes& ax,
                  hipStream_t stream) {
  return n >= kWideTargets ? launch_bs_f64<2>(in, cnt, n, S, P, ax, stream)
                           : launch_bs_f64<1>(in, cnt, n, S, P, ax, stream);
}

// FP32 sum; X the grid coordinates, or null: from the positions.
hipError_t bs_f32(const BsPts& in, const uint32_t* X, int32_t* cnt, long long n, int S, float* P,
                  const BsAxes& ax, hipStream_t stream) {
  const int tb = (int)((n + kTargets - 1) / kTargets);
  auto kern = ax.uniform ? (X ? k_bs_f32<true, false> : k_bs_f32<true, true>)
                         : (X ? k_bs_f32<false, false> : k_bs_f32<false, true>);
  hipLaunchKernelGGL(kern, dim3(tb, S * ax.copies), dim3(256), 0, stream, in, X, cnt, (int)n, n, S,
                     ax.invq_f[0], ax.invq_f[1], ax.invq_f[2], P, ax);
  return hipGetLastError();
}

}  // namespace

hipError_t bs_sum(Run& r, const double* Y) {
  hipEvent_t b = nullptr;
  time_begin(r, 0, &b);
  const BsPts in{Y, r.ncap, 1, r.nxt, r.prv};
  const hipError_t e =
      r.prec == VLB_F64
          ? bs_f64(in, r.cnt, r.ncap, r.bsS, (double*)r.bsP, r.bsax, r.stream)
          : bs_f32(in, r.bsX, r.cnt, r.ncap, r.bsS, (float*)r.bsP, r.bsax, r.stream);
  time_end(r, 0, b);
  return e;
}

int bs_check_desc(const vlb_bs_desc* d, int64_t n, std::string& msg) {
  if (!d) { msg = "null descriptor"; return VLB_EINVAL; }
  if (d->nx < 1 || d->ny < 1 || d->nz < 1 || d->nx > (1 << 24) || d->ny > (1 << 24) ||
      d->nz > (1 << 24)) { msg = "box dimensions must be in [1, 2^24]"; return VLB_EINVAL; }
  if (d->wall_axes & ~7u) { msg = "wall_axes uses bits 0..2 only"; return VLB_EINVAL; }
  if (d->precision < 0 || d->precision > 2) { msg = "precision must be VLB_F64, VLB_F32 or VLB_F16"; return VLB_EINVAL; }
  if (!(d->kappa > 0) || !std::isfinite(d->kappa)) { msg = "kappa must be positive and finite"; return VLB_EINVAL; }
  if (n < 0 || n > kSoloMaxPoints) { msg = "n_pts must be in [0, 2^26]"; return VLB_EINVAL; }
  return VLB_OK;
}

// Standalone sum: the chunk count, scratch layout and launches.  Up to the
// size of the largest allocation-free call (16384 points) the chunk partials
// are kept within 4 MB (FP64 10 chunks there, 32 from 5461 points down).
constexpr long long kSoloPartialBytes = 4LL << 20;

int bs_solo_chunks(long long n, size_t fe) {
  const int S = bs_chunks(n, 1);
  const long long most = std::max(1LL, kSoloPartialBytes / (3 * n * (long long)fe));
  return n <= 16384 && S > most ? (int)most : S;
}

size_t bs_solo_layout(int prec, long long n, char* base, BsSolo* b) {
  const size_t fe = prec == VLB_F64 ? 8 : 4;
  const int S = bs_solo_chunks(n, fe);
  size_t off = 0;
  auto take = [&](size_t bytes) -> void* {
    off = (off + 255) / 256 * 256;
    void* p = base ? base + off : nullptr;
    off += bytes;
    return p;
  };
  BsSolo s{};
  if (prec != VLB_F64 && n > kDirectPoints) s.X = (uint32_t*)take(3 * (size_t)n * sizeof(uint32_t));
  s.P = take((size_t)S * 3 * n * fe);
  s.S = S;
  if (b) *b = s;
  return (off + 255) / 256 * 256;
}

namespace {

// Do the m bytes at a and the k bytes at b share any?
bool overlap(const void* a, size_t m, const void* b, size_t k) {
  return (uintptr_t)a < (uintptr_t)b + k && (uintptr_t)b < (uintptr_t)a + m;
}

}  // namespace

hipError_t bs_solo(const BsAxes& ax, int prec, long long n, const double* xyz,
                   const int32_t* next, double kappa, double* v, const BsSolo& b,
                   hipStream_t stream) {
  const BsPts in{xyz, 1, 3, next, nullptr};
  const int nb3 = (int)((3 * n + 255) / 256);
  const double s = kappa / (4.0 * M_PI);
  hipError_t e;
  // (k_bs_few writes v while other blocks read the points: not for a caller
  // whose output takes the place of its inputs)
  const size_t bytes = 24 * (size_t)n;
  if (n <= kFewPoints && !overlap(v, bytes, xyz, bytes) && !overlap(v, bytes, next, 4 * (size_t)n)) {
    using K = void (*)(BsPts, int, double, double*, BsAxes);
    static constexpr K f64[8] = {k_bs_few<false, 0>, k_bs_few<false, 1>, k_bs_few<false, 2>,
                                 k_bs_few<false, 3>, k_bs_few<false, 4>, k_bs_few<false, 5>,
                                 k_bs_few<false, 6>, k_bs_few<false, 7>};
    const int per = (ax.periodic[0] ? 1 : 0) | (ax.periodic[1] ? 2 : 0) | (ax.periodic[2] ? 4 : 0);
    const K kern = prec == VLB_F64 ? f64[per] : (ax.uniform ? k_bs_few<true, 1> : k_bs_few<true, 0>);
    const double sc = prec != VLB_F64 && ax.uniform ? s * ax.q[0] : s;
    hipLaunchKernelGGL(kern, dim3((unsigned)((n + kFewTargets - 1) / kFewTargets)),
                       dim3(kFewThreads), 0, stream, in, (int)n, sc, v, ax);
    return hipGetLastError();
  }
  if (prec == VLB_F64) {
    e = bs_f64(in, nullptr, n, b.S, (double*)b.P, ax, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_solo_sum<double>, dim3(nb3), dim3(256), 0, stream, (const double*)b.P,
                       b.S, (int)n, s, v);
  } else {
    if (b.X)
      hipLaunchKernelGGL(k_prep, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, in,
                         nullptr, (int)n, n, ax, b.X);
    e = bs_f32(in, b.X, nullptr, n, b.S, (float*)b.P, ax, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_solo_sum<float>, dim3(nb3), dim3(256), 0, stream, (const float*)b.P, b.S,
                       (int)n, ax.uniform ? s * ax.q[0] : s, v);
  }
  return hipGetLastError();
}

}  // namespace vlb
