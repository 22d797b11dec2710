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
#include "vlb_internal.h"

#include <cmath>

namespace vlb {

namespace {

constexpr int kTile = 256;
constexpr int kTargets = 64;  // targets per block, one per lane of each wave
// Point count from which the FP64 sum takes two targets per lane: a record
// read from LDS then serves two pairs and two dependence chains overlap (2e4
// points 557 against 594 us, 6e4 points 4883 against 5010); with fewer points
// the blocks of half as many targets fill the chip better.
constexpr long long kWideTargets = 4096;

// Points of an FP64 sum: component a of point j at Y[a sa + j sj], links
// (entries of nxt are clamped into the points; prv is read with image
// copies only).
struct BsPts {
  const double* Y;
  long long sa, sj;
  const int32_t* nxt;
  const int32_t* prv;
};

// Quarter of a staged tile of cnt sources walked by wave w: [lo, hi) (empty
// when lo >= hi), lo a multiple of 4 so that the unrolled loop reads the
// tile with 16-byte loads.
__device__ inline void wave_range(int cnt, int w, int& lo, int& hi) {
  const int q = (((cnt + 3) >> 2) + 3) & ~3;
  lo = w * q;
  hi = __builtin_amdgcn_readfirstlane(min(cnt, lo + q));
}

// A coordinate mirrored for an image copy: 0 itself, 1 in the wall plane
// -1/2, 2 in the plane L - 1/2.
__device__ inline double bs_mirror(double y, int m, double L) {
  return m == 0 ? y : (m == 1 ? 2.0 * (-0.5) - y : 2.0 * (L - 0.5) - y);
}

// The image copy mirrored in the wall that the end of an open line at y is
// bound to (the lowest closed axis whose wall plane it lies on; nothing else
// reflected), 0 if none: in that copy the images of the end's two segments
// meet it and are excluded, as the real ones are in copy 0.
__device__ inline int bs_own_copy(const double* y, const BsAxes& ax) {
  int ea = -1, es = 0, oc = 0;
  for (int a = 2; a >= 0; --a)
    if (!ax.periodic[a] && (y[a] == -0.5 || y[a] == ax.L[a] - 0.5)) {
      ea = a;
      es = y[a] == -0.5 ? 1 : 2;
    }
  if (ea >= 0)
    for (int c = 1; c < ax.copies; ++c) {
      bool only = true;
      for (int a = 0; a < 3; ++a) only = only && ax.refl[c][a] == (a == ea ? es : 0);
      if (only) oc = c;
    }
  return oc;
}

// FP32: grid coordinates of the points at positions Y (copy 0) and of their
// images in the wall planes (copies 1..); with image copies (own non-null)
// the own copy of every open line's end (0 for other points).
__global__ void k_prep(const double* __restrict__ Y, const int32_t* __restrict__ nxt,
                       const int32_t* __restrict__ prv, const int32_t* __restrict__ cnt,
                       long long ncap, BsAxes ax, uint32_t* __restrict__ X,
                       int32_t* __restrict__ own) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  const int n = cnt[0];
  if (j >= n) return;
  double y[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) y[a] = Y[a * ncap + j];
  if (own) own[j] = (nxt[j] == j || prv[j] == j) ? bs_own_copy(y, ax) : 0;
  for (int c = 0; c < ax.copies; ++c) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const double s = floor((bs_mirror(y[a], ax.refl[c][a], ax.L[a]) + ax.off[a]) * ax.q[a]);
      X[((long long)c * 3 + a) * ncap + j] =
          ax.periodic[a] ? (uint32_t)(long long)s : (uint32_t)(int)(long long)s;
    }
  }
}

// FP32 pair sum.  Per pair, with R1 = s_k - r (from the grid difference),
// d = s_next(k) - s_k, q = |d|^2 and R2 = R1 + d:
//   R1 x R2 = R1 x d,  |R2|^2 = |R1|^2 + (2 R1.d + q),
//   (|R1| + |R2|)^2 - q = 2 (|R1||R2| + R1.R2),
// so the closed form (R1 x R2) (|R1| + |R2|) / (|R1||R2| (|R1||R2| + R1.R2))
// becomes (R1 x 2d) (i1 + i2) / (s^2 - q) with i_m = 1/|R_m| and
// s = |R1| + |R2| = |R1|^2 i1 + |R2|^2 i2: 27 ordinary and 3 transcendental
// instructions per pair (sources are staged as 2d and q).  Uniform grid: R1
// stays in grid units and the result is rescaled once per target (v is
// homogeneous of degree -1 in R).
//
// What bounds it: VALU issue.  Ordinary FP32 and integer instructions of two
// waves issue together (1.45 to 1.73 wave instructions per CU and cycle with
// 8 waves per SIMD; 0.89 when an operand is a scalar register, so the source
// data must come from vector registers), a transcendental one takes two
// cycles alone; the loop's mix takes 23.5 cycles per pair of wave and source
// by those rates, 25.7 measured.  Against the form with
// 1 + (R1.R2) i1 i2 in the denominator (29.5 ordinary): 1.45 -> 1.52 Tpairs/s
// at 1.0e5 points, the error against FP64 6.0e-7 -> 5.5e-7.  Two or four
// targets per lane measured 3% and 13% slower (fewer waves in flight).
struct __align__(16) BsSrc {
  uint32_t x, y, z;  // grid coordinates of the segment's start
  float q;           // |d|^2
  float dx, dy, dz;  // 2 d
  float pad;
};

template <bool kCheck, bool kUniform>
__device__ inline void bs_tile_f32(const BsSrc* src, int cnt, int t0, uint32_t xt, uint32_t yt,
                                   uint32_t zt, float iqx, float iqy, float iqz, int jj, int pj,
                                   float& ax, float& ay, float& az) {
  // unrolled twice: 8 waves per SIMD (four ways: 2% slower)
#pragma unroll 2
  for (int s = 0; s < cnt; ++s) {
    const BsSrc g = src[s];
    float r1x = (float)(int)(g.x - xt);
    float r1y = (float)(int)(g.y - yt);
    float r1z = (float)(int)(g.z - zt);
    if (!kUniform) {
      r1x *= iqx;
      r1y *= iqy;
      r1z *= iqz;
    }
    const float ex = g.dx, ey = g.dy, ez = g.dz;
    const float t = fmaf(r1x, ex, fmaf(r1y, ey, fmaf(r1z, ez, g.q)));
    const float n1 = fmaf(r1x, r1x, fmaf(r1y, r1y, r1z * r1z));
    const float n2 = n1 + t;
    const float i1 = __builtin_amdgcn_rsqf(n1);
    const float i2 = __builtin_amdgcn_rsqf(n2);
    const float sum = fmaf(n1, i1, n2 * i2);
    float f = (i1 + i2) * __builtin_amdgcn_rcpf(fmaf(sum, sum, -g.q));
    if (kCheck) {
      const int k = t0 + s;
      f = (k == jj || k == pj) ? 0.0f : f;
    }
    ax = fmaf(f, fmaf(r1y, ez, -(r1z * ey)), ax);
    ay = fmaf(f, fmaf(r1z, ex, -(r1x * ez)), ay);
    az = fmaf(f, fmaf(r1x, ey, -(r1y * ex)), az);
  }
}

// Grid y: S chunks of every source copy (copy 0 the filaments, the others
// their wall images, which take no exclusion and carry the copy's sign).
template <bool kUniform>
__global__ __launch_bounds__(256) void k_bs_f32(const uint32_t* __restrict__ X,
                                               const int32_t* __restrict__ nxt,
                                               const int32_t* __restrict__ prv,
                                               int32_t* __restrict__ cntp, long long ncap,
                                               int S, float iqx, float iqy, float iqz,
                                               float* __restrict__ P, BsAxes bx,
                                               const int32_t* __restrict__ own) {
  const int n = cntp[0];
  // work counter: (target, segment) pairs of this sum
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0 && n > 2)
    *(long long*)(cntp + 16) += (long long)n * (n - 2) + (long long)(bx.copies - 1) * n * n;
  const int j0 = blockIdx.x * kTargets;
  if (j0 >= n) return;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform per wave
  const int j = j0 + lane;
  const bool valid = j < n;
  const int copy = blockIdx.y / S;
  const uint32_t* __restrict__ Xs = X + (long long)copy * 3 * ncap;  // this copy's sources
  const int per = (n + S - 1) / S;
  const int kb = (blockIdx.y - copy * S) * per;
  const int ke = min(n, kb + per);
  const uint32_t xt = valid ? X[j] : 0u;
  const uint32_t yt = valid ? X[ncap + j] : 0u;
  const uint32_t zt = valid ? X[2 * ncap + j] : 0u;
  // the target's own two segments are excluded in copy 0 and, for the end
  // of an open line, in the copy mirrored in its wall
  const int oc = (valid && own) ? own[j] : 0;
  const bool exl = valid && (copy == 0 || copy == oc);
  const int pj = exl ? prv[j] : -1;
  const int jj = exl ? j : -1;
  __shared__ BsSrc src[kTile];
  __shared__ float red[3][3][kTargets];  // sums of waves 1..3
  float ax = 0.f, ay = 0.f, az = 0.f;
  for (int t0 = kb; t0 < ke; t0 += kTile) {
    const int k = t0 + threadIdx.x;
    if (k < ke) {
      // segment vector: wrapped grid difference to the successor
      const int kn = nxt[k];
      const uint32_t ax0 = Xs[k], ay0 = Xs[ncap + k], az0 = Xs[2 * ncap + k];
      float ex = (float)(int)(Xs[kn] - ax0);
      float ey = (float)(int)(Xs[ncap + kn] - ay0);
      float ez = (float)(int)(Xs[2 * ncap + kn] - az0);
      if (!kUniform) {
        ex *= iqx;
        ey *= iqy;
        ez *= iqz;
      }
      BsSrc g;
      g.x = ax0;
      g.y = ay0;
      g.z = az0;
      g.q = ex * ex + ey * ey + ez * ez;
      g.dx = 2.0f * ex;
      g.dy = 2.0f * ey;
      g.dz = 2.0f * ez;
      g.pad = 0.0f;
      src[threadIdx.x] = g;
    }
    __syncthreads();
    int lo, hi;
    wave_range(min(kTile, ke - t0), w, lo, hi);
    if (lo < hi) {
      const int s0 = t0 + lo, s1 = t0 + hi;
      const bool hit = exl && ((jj >= s0 && jj < s1) || (pj >= s0 && pj < s1));
      if (__any(hit))
        bs_tile_f32<true, kUniform>(src + lo, hi - lo, s0, xt, yt, zt, iqx, iqy, iqz, jj, pj, ax,
                                    ay, az);
      else
        bs_tile_f32<false, kUniform>(src + lo, hi - lo, s0, xt, yt, zt, iqx, iqy, iqz, jj, pj, ax,
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
    float* out = P + (long long)blockIdx.y * 3 * ncap;
    out[j] = sg * (((ax + red[0][0][lane]) + red[1][0][lane]) + red[2][0][lane]);
    out[ncap + j] = sg * (((ay + red[0][1][lane]) + red[1][1][lane]) + red[2][1][lane]);
    out[2 * ncap + j] = sg * (((az + red[0][2][lane]) + red[1][2][lane]) + red[2][2][lane]);
  }
}

// FP64 pair sum (plain path), with the FP32 sum's q, R2 and s^2:
//   s^2 = |R1|^2 + |R2|^2 + 2 p,  p = |R1||R2| = sqrt(|R1|^2 |R2|^2),
//   (|R1| + |R2|) / (p (p + R1.R2)) = 2 s / (p (s^2 - q))
//                                   = 2 s^2 / sqrt(s^2 p^2 (s^2 - q)^2),
// two inverse roots instead of two and a reciprocal.  Each is the hardware
// approximation (relative error up to about 5e-8) refined by one Newton step
// (which squares it), the first inside s^2, the second inside the factor:
// f = s^2 z (3 - arg z^2) with z ~ 1/sqrt(arg).  Sources are staged as 2 d;
// the partial sums take the 1/2.
//
// The separation R1: on a closed axis the difference of the positions; on a
// periodic axis (X_s - X_t) / q + (rho_s - rho_t), where the wrapped grid
// difference picks the image (the same decision as the FP32 sum) and the
// residuals rho = y - X / q restore the FP64 separation of that image to
// rounding.  The set of periodic axes is a template argument.
//
// What bounds it: VALU issue.  FP64 and conversions take one cycle per wave
// instruction and CU (no two waves issue together), an FP64 transcendental
// four; 62.5 cycles per pair with three of them and four instructions per
// axis of R1, 50 now (41 with two closed axes).  2e4 points, two closed axes:
// 0.61 -> 0.76 Tpairs/s with the error against 64 bits 5.9e-15 -> 1.3e-15.
struct __align__(16) BsSrcD {
  double rx, ry, rz;  // the segment's start: residual (periodic axis) or position (closed axis)
  double q;           // |d|^2
  double dx, dy, dz;  // 2 d
  uint32_t x, y, z;   // grid coordinates (periodic axes)
  int32_t kn;         // index of the segment's end
};

template <bool kPeriodic>
__device__ inline double bs_sep(uint32_t xs, uint32_t xt, double rs, double rt, double g) {
  return kPeriodic ? fma((double)(int)(xs - xt), g, rs - rt) : rs - rt;
}

// Targets per lane of the FP64 sum: index, exclusion index (-1: none),
// position data and the sums.
struct BsTgtD {
  uint32_t x, y, z;
  int jj;
  double rx, ry, rz, ax, ay, az;
};

template <int kPer, int NT, bool kCheck>
__device__ inline void bs_tile_f64(const BsSrcD* src, int cnt, int t0, BsTgtD* tg, double gx,
                                   double gy, double gz) {
#pragma unroll(NT == 1 ? 2 : 1)
  for (int s = 0; s < cnt; ++s) {
    const BsSrcD g = src[s];
#pragma unroll
    for (int m = 0; m < NT; ++m) {
      BsTgtD& t = tg[m];
      const double r1x = bs_sep<(kPer & 1) != 0>(g.x, t.x, g.rx, t.rx, gx);
      const double r1y = bs_sep<(kPer & 2) != 0>(g.y, t.y, g.ry, t.ry, gy);
      const double r1z = bs_sep<(kPer & 4) != 0>(g.z, t.z, g.rz, t.rz, gz);
      const double n1 = fma(r1x, r1x, fma(r1y, r1y, r1z * r1z));
      const double n2 = n1 + fma(r1x, g.dx, fma(r1y, g.dy, fma(r1z, g.dz, g.q)));
      const double n12 = n1 * n2;
      const double y = __builtin_amdgcn_rsq(n12);
      const double p = n12 * y;
      const double s2 = fma(p, fma(-p, y, 1.0), fma(2.0, p, n1 + n2));
      const double w = s2 - g.q;
      const double arg = (s2 * n12) * (w * w);
      const double z = __builtin_amdgcn_rsq(arg);
      double f = (s2 * z) * fma(-(arg * z), z, 3.0);
      if (kCheck) f = (t0 + s == t.jj || g.kn == t.jj) ? 0.0 : f;
      t.ax = fma(f, fma(r1y, g.dz, -(r1z * g.dy)), t.ax);
      t.ay = fma(f, fma(r1z, g.dx, -(r1x * g.dz)), t.ay);
      t.az = fma(f, fma(r1x, g.dy, -(r1y * g.dx)), t.az);
    }
  }
}

// Grid coordinate and residual of a coordinate on a periodic axis.
__device__ inline void bs_grid_f64(double y, double q, double invq, uint32_t& x, double& r) {
  const double s = floor(y * q);
  x = (uint32_t)(long long)s;
  r = y - s * invq;
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
    t.x = t.y = t.z = 0u;
    t.rx = y[0];
    t.ry = y[1];
    t.rz = y[2];
    if (kPer & 1) bs_grid_f64(y[0], bx.q[0], bx.invq_d[0], t.x, t.rx);
    if (kPer & 2) bs_grid_f64(y[1], bx.q[1], bx.invq_d[1], t.y, t.ry);
    if (kPer & 4) bs_grid_f64(y[2], bx.q[2], bx.invq_d[2], t.z, t.rz);
    t.ax = t.ay = t.az = 0.0;
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
    if (k < ke) {
      BsSrcD g;
      g.kn = min(max(in.nxt[k], 0), n - 1);
      double r[3], d[3];
      uint32_t x[3] = {0u, 0u, 0u};
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const double y = in.Y[a * in.sa + k * in.sj];
        d[a] = in.Y[a * in.sa + g.kn * in.sj] - y;
        if ((kPer >> a) & 1) {
          if (d[a] > 0.5 * bx.L[a])
            d[a] = d[a] - bx.L[a];
          else if (d[a] < -0.5 * bx.L[a])
            d[a] = d[a] + bx.L[a];
          bs_grid_f64(y, bx.q[a], bx.invq_d[a], x[a], r[a]);
        } else {
          const int rm = bx.refl[copy][a];
          r[a] = bs_mirror(y, rm, bx.L[a]);
          d[a] = rm ? -d[a] : d[a];
        }
      }
      g.rx = r[0];
      g.ry = r[1];
      g.rz = r[2];
      g.x = x[0];
      g.y = x[1];
      g.z = x[2];
      g.q = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
      g.dx = 2.0 * d[0];
      g.dy = 2.0 * d[1];
      g.dz = 2.0 * d[2];
      src[threadIdx.x] = g;
    }
    __syncthreads();
    int lo, hi;
    wave_range(min(kTile, ke - t0), w, lo, hi);
    if (lo < hi) {
      // does this wave's quarter (at most 64 sources) start or end at one of
      // the block's targets?
      bool hit = false;
      if (lane < hi - lo)
        hit = (uint32_t)(t0 + lo + lane - j0) < (uint32_t)kT ||
              (uint32_t)(src[lo + lane].kn - j0) < (uint32_t)kT;
      if (exany && __any(hit))
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

// FP32: links and grid coordinates of a caller's filaments: next is clamped
// into [0, n) (an invalid permutation gives meaningless velocities, never an
// access out of bounds) and inverted into prev; grid coordinates as k_prep,
// from [n][3] positions.  Thread 0 writes the point count and clears the pair
// counter.
// prv[j] = j: the first point of an open line keeps it (no real link to it)
__global__ void k_solo_init(int32_t* __restrict__ prv, int n) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j < n) prv[j] = j;
}

__global__ void k_solo_prep(const double* __restrict__ xyz, const int32_t* __restrict__ next,
                            int n, BsAxes ax, int32_t* __restrict__ cnt,
                            uint32_t* __restrict__ X, int32_t* __restrict__ nxt,
                            int32_t* __restrict__ prv) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j == 0) {
    cnt[0] = n;
    for (int i = 1; i < 32; ++i) cnt[i] = 0;
  }
  if (j >= n) return;
  const int k = min(max(next[j], 0), n - 1);
  nxt[j] = k;
  if (k != j) prv[k] = j;  // the last point of an open line links to itself
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double s = floor((xyz[3LL * j + a] + ax.off[a]) * ax.q[a]);
    X[(long long)a * n + j] = ax.periodic[a] ? (uint32_t)(long long)s
                                             : (uint32_t)(int)(long long)s;
  }
}

// v[j][a] = scale * (sum over the S chunk partials of target j, in chunk
// order, in FP64).
template <class PT>
__global__ void k_solo_sum(const PT* __restrict__ P, int S, int n, double scale,
                           double* __restrict__ v) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    double t = 0.0;
    for (int c = 0; c < S; ++c) t += (double)P[((long long)c * 3 + a) * n + j];
    v[3LL * j + a] = t * scale;
  }
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

// Source chunks S: about 16384 blocks over the target blocks, or up to
// 32768 while every chunk keeps at least 1024 sources (large point counts:
// the launch's tail shortens), at least 256 sources per chunk (64 per
// wave), at most 256 chunks; the chunk partials are added by the finalize
// kernel.  (At 1.2e4 points 512 and 1024 sources per chunk measured 1.5%
// and 6% slower per step, 128 and 192 no faster; at 1.0e5 points 14 chunks
// instead of 7 measured 1.1% faster, at 5e4 points 28 instead of 14 0.9%.)
int bs_chunks(long long ncap) {
  const long long tb = (ncap + kTargets - 1) / kTargets;
  const long long t = tb > 0 ? tb : 1;
  long long S = 16384 / t;
  const long long wide = std::min(32768 / t, ncap / 1024);
  if (wide > S) S = wide;
  const long long maxS = ncap / 256;
  if (S > maxS) S = maxS;
  if (S < 1) S = 1;
  if (S > 256) S = 256;
  return (int)S;
}

hipError_t bs_prep(Run& r, const double* Y) {
  if (r.prec == VLB_F64) return hipSuccess;  // that sum reads the positions
  const int nb = (int)((r.ncap + 255) / 256);
  hipLaunchKernelGGL(k_prep, dim3(nb), dim3(256), 0, r.stream, Y, r.nxt, r.prv, r.cnt, r.ncap,
                     r.bsax, r.bsX, r.bsax.copies > 1 ? r.bsown : nullptr);
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

}  // namespace

hipError_t bs_sum(Run& r, const double* Y) {
  const int tb = (int)((r.ncap + kTargets - 1) / kTargets);
  dim3 grid(tb, r.bsS * r.bsax.copies);
  hipEvent_t b = nullptr;
  time_begin(r, 0, &b);
  const int32_t* own = r.bsax.copies > 1 ? r.bsown : nullptr;
  hipError_t e = hipSuccess;
  if (r.prec == VLB_F64)
    e = bs_f64(BsPts{Y, r.ncap, 1, r.nxt, r.prv}, r.cnt, r.ncap, r.bsS, (double*)r.bsP, r.bsax,
               r.stream);
  else if (r.bsax.uniform)
    hipLaunchKernelGGL(k_bs_f32<true>, grid, dim3(256), 0, r.stream, r.bsX, r.nxt,
                       r.prv, r.cnt, r.ncap, r.bsS, r.bsax.invq_f[0], r.bsax.invq_f[1],
                       r.bsax.invq_f[2], (float*)r.bsP, r.bsax, own);
  else
    hipLaunchKernelGGL(k_bs_f32<false>, grid, dim3(256), 0, r.stream, r.bsX, r.nxt,
                       r.prv, r.cnt, r.ncap, r.bsS, r.bsax.invq_f[0], r.bsax.invq_f[1],
                       r.bsax.invq_f[2], (float*)r.bsP, r.bsax, own);
  time_end(r, 0, b);
  return e == hipSuccess ? hipGetLastError() : e;
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

// Standalone sum: the chunk count, scratch layout and launches.  The
// chunks are capped at kSoloChunks, so that the scratch of the largest
// allocation-free call stays small.
constexpr int kSoloChunks = 8;

int bs_solo_chunks(long long n) {
  const int S = bs_chunks(n);
  return S < kSoloChunks ? S : kSoloChunks;
}

size_t bs_solo_layout(int prec, long long n, char* base, BsSolo* b) {
  const size_t fe = prec == VLB_F64 ? 8 : 4;
  const int S = bs_solo_chunks(n);
  size_t off = 0;
  auto take = [&](size_t bytes) -> void* {
    off = (off + 255) / 256 * 256;
    void* p = base ? base + off : nullptr;
    off += bytes;
    return p;
  };
  BsSolo s{};
  s.cnt = (int32_t*)take(32 * sizeof(int32_t));
  if (prec != VLB_F64) {
    s.X = (uint32_t*)take(3 * (size_t)n * sizeof(uint32_t));
    s.nxt = (int32_t*)take((size_t)n * sizeof(int32_t));
    s.prv = (int32_t*)take((size_t)n * sizeof(int32_t));
  }
  s.P = take((size_t)S * 3 * n * fe);
  s.S = S;
  if (b) *b = s;
  return (off + 255) / 256 * 256;
}

hipError_t bs_solo(const BsAxes& ax, int prec, long long n, const double* xyz,
                   const int32_t* next, double kappa, double* v, const BsSolo& b,
                   hipStream_t stream) {
  const int nb = (int)((n + 255) / 256);
  const int tb = (int)((n + kTargets - 1) / kTargets);
  const dim3 grid(tb, b.S);
  const double s = kappa / (4.0 * M_PI);
  if (prec == VLB_F64) {
    const hipError_t e = bs_f64(BsPts{xyz, 1, 3, next, nullptr}, nullptr, n, b.S, (double*)b.P, ax,
                                stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_solo_sum<double>, dim3(nb), dim3(256), 0, stream, (const double*)b.P,
                       b.S, (int)n, s, v);
  } else {
    hipLaunchKernelGGL(k_solo_init, dim3(nb), dim3(256), 0, stream, b.prv, (int)n);
    hipLaunchKernelGGL(k_solo_prep, dim3(nb), dim3(256), 0, stream, xyz, next, (int)n, ax, b.cnt,
                       b.X, b.nxt, b.prv);
    if (ax.uniform)
      hipLaunchKernelGGL(k_bs_f32<true>, grid, dim3(256), 0, stream, b.X, b.nxt, b.prv, b.cnt,
                         n, b.S, ax.invq_f[0], ax.invq_f[1], ax.invq_f[2], (float*)b.P, ax,
                         nullptr);
    else
      hipLaunchKernelGGL(k_bs_f32<false>, grid, dim3(256), 0, stream, b.X, b.nxt, b.prv, b.cnt,
                         n, b.S, ax.invq_f[0], ax.invq_f[1], ax.invq_f[2], (float*)b.P, ax,
                         nullptr);
    hipLaunchKernelGGL(k_solo_sum<float>, dim3(nb), dim3(256), 0, stream, (const float*)b.P,
                       b.S, (int)n, ax.uniform ? s * ax.q[0] : s, v);
  }
  return hipGetLastError();
}

}  // namespace vlb
