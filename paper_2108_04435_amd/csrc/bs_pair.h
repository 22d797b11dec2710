// Device pieces of the Biot-Savart sum shared by the sum's kernels (bs.hip)
// and the stage kernel of small runs (filament.hip): staged source records,
// targets, and one (target, segment) pair in FP32 and FP64.
#pragma once

#include "vlb_internal.h"

#include <type_traits>

namespace vlb {

// Points of a sum: component a of point j at Y[a sa + j sj], links (entries
// of nxt are clamped into the points; prv is read with image copies only).
struct BsPts {
  const double* Y;
  long long sa, sj;
  const int32_t* nxt;
  const int32_t* prv;
};

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

// FP32 grid coordinate of a coordinate on axis a.
__device__ inline uint32_t bs_grid_f32(double y, const BsAxes& ax, int a) {
  const double s = floor((y + ax.off[a]) * ax.q[a]);
  return ax.periodic[a] ? (uint32_t)(long long)s : (uint32_t)(int)(long long)s;
}

// FP32 pair sum.  Per pair, with R1 = s_k - r (from the grid difference),
// d = s_next(k) - s_k, q = |d|^2 and R2 = R1 + d:
//   R1 x R2 = R1 x d,  R1.R2 = |R1|^2 + R1.d,  |R2|^2 = |R1|^2 + 2 R1.d + q,
//   v = (R1 x R2) (i1 + i2) i1 i2 / (1 + (R1.R2) i1 i2),  i_m = 1/|R_m|,
// the closed form (|R1| + |R2|) / (|R1||R2| (|R1||R2| + R1.R2)) rewritten with
// inverse norms.  Uniform grid: R1 stays in grid units and the result is
// rescaled once per target (v is homogeneous of degree -1 in R).
//
// The denominator is 1 + cos of the angle between R1 and R2, not the
// (|R1| + |R2|)^2 - q that it is a multiple of and that takes two instructions
// less (1.0e5 points: 6.48 against 6.86 ms): beside the segment's start that
// difference cancels, and a q added into 2 R1.d before |R1|^2 is rounds at the
// size of q.
// Error of the factor beside the start of a segment of 0.7 to 0.95, rms, at 0.3,
// 0.1 and 0.01 from it: 9.5e-8, 8.6e-8 and 8.4e-8 so, 1.9e-7, 4.1e-7 and 3.5e-6
// with the difference.
//
// What bounds it: VALU issue.  Ordinary FP32 and integer instructions of two
// waves issue together (1.45 to 1.73 wave instructions per CU and cycle with
// 8 waves per SIMD; 0.89 when an operand is a scalar register, so the source
// data must come from vector registers), a transcendental one takes two
// cycles alone: 29 ordinary and 3 transcendental per pair, 24.5 cycles per pair
// of wave and source by those rates, 26.7 measured (1.46 Tpairs/s at 1.0e5
// points).  Two or four targets per lane measured 3% and 13% slower (fewer
// waves in flight).
struct __align__(16) BsSrc {
  uint32_t x, y, z;  // grid coordinates of the segment's start
  float q;           // |d|^2
  float dx, dy, dz;  // d
  int32_t kn;        // index of the segment's end
};

// Record of segment k: grid coordinates from X (stride nc), or from the
// positions, mirrored for the image copy (kDirect).  Segment vector: the
// wrapped grid difference to the successor.
template <bool kUniform, bool kDirect>
__device__ inline BsSrc bs_stage_f32(const BsPts& in, const uint32_t* __restrict__ X, long long nc,
                                     int k, int n, int copy, float iqx, float iqy, float iqz,
                                     const BsAxes& bx) {
  const int kn = min(max(in.nxt[k], 0), n - 1);
  uint32_t x0[3], x1[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if (kDirect) {
      const int rm = bx.refl[copy][a];
      x0[a] = bs_grid_f32(bs_mirror(in.Y[a * in.sa + k * in.sj], rm, bx.L[a]), bx, a);
      x1[a] = bs_grid_f32(bs_mirror(in.Y[a * in.sa + kn * in.sj], rm, bx.L[a]), bx, a);
    } else {
      x0[a] = X[a * nc + k];
      x1[a] = X[a * nc + kn];
    }
  }
  float ex = (float)(int)(x1[0] - x0[0]);
  float ey = (float)(int)(x1[1] - x0[1]);
  float ez = (float)(int)(x1[2] - x0[2]);
  if (!kUniform) {
    ex *= iqx;
    ey *= iqy;
    ez *= iqz;
  }
  BsSrc g;
  g.x = x0[0];
  g.y = x0[1];
  g.z = x0[2];
  g.q = ex * ex + ey * ey + ez * ez;
  g.dx = ex;
  g.dy = ey;
  g.dz = ez;
  g.kn = kn;
  return g;
}

template <bool kUniform>
__device__ __forceinline__ void bs_pair_f32(const BsSrc& g, uint32_t xt, uint32_t yt, uint32_t zt,
                                            float iqx, float iqy, float iqz, bool excluded,
                                            float& ax, float& ay, float& az) {
  float r1x = (float)(int)(g.x - xt);
  float r1y = (float)(int)(g.y - yt);
  float r1z = (float)(int)(g.z - zt);
  if (!kUniform) {
    r1x *= iqx;
    r1y *= iqy;
    r1z *= iqz;
  }
  const float ex = g.dx, ey = g.dy, ez = g.dz;
  const float t = r1x * ex + r1y * ey + r1z * ez;
  const float n1 = r1x * r1x + r1y * r1y + r1z * r1z;
  const float n2 = fmaf(2.0f, t, n1 + g.q);
  const float i1 = __builtin_amdgcn_rsqf(n1);
  const float i2 = __builtin_amdgcn_rsqf(n2);
  const float crx = r1y * ez - r1z * ey;
  const float cry = r1z * ex - r1x * ez;
  const float crz = r1x * ey - r1y * ex;
  const float a = i1 * i2;
  const float den = fmaf(n1 + t, a, 1.0f);
  float f = (i1 + i2) * a * __builtin_amdgcn_rcpf(den);
  f = excluded ? 0.0f : f;
  ax = fmaf(f, crx, ax);
  ay = fmaf(f, cry, ay);
  az = fmaf(f, crz, az);
}

// FP64 pair sum (plain path), with q and R2 as above, s = |R1| + |R2| and
// p = |R1||R2| = sqrt(|R1|^2 |R2|^2):
//   w = 2 (p + R1.R2),  s^2 = w + q,
//   (|R1| + |R2|) / (p (p + R1.R2)) = 2 s / (p w) = 2 s^2 / sqrt(s^2 p^2 w^2),
// two inverse roots instead of two and a reciprocal.  Each is the hardware
// approximation (relative error up to about 5e-8) refined by one Newton step
// (which squares it), the first inside w, the second inside the factor:
// f = s^2 z (3 - arg z^2) with z ~ 1/sqrt(arg).  Sources are staged as 2 d;
// the partial sums take the 1/2.  (w as s^2 - q, as many instructions, cancels
// beside the segment's start: the factor's error there, rms, at 0.001 from a
// segment of 0.7 to 0.95: 5.6e-14, 1.6e-15 so.)
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
// 0.59 -> 0.76 Tpairs/s; relative error against the sum in 80-bit arithmetic, L2
// over 150 targets, 1.7e-15 -> 0.8e-15.
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

// Grid coordinate and residual of a coordinate on a periodic axis.
__device__ inline void bs_grid_f64(double y, double q, double invq, uint32_t& x, double& r) {
  const double s = floor(y * q);
  x = (uint32_t)(long long)s;
  r = y - s * invq;
}

template <int kPer>
__device__ inline void bs_target_f64(const double y[3], const BsAxes& bx, BsTgtD& t) {
  t.x = t.y = t.z = 0u;
  t.rx = y[0];
  t.ry = y[1];
  t.rz = y[2];
  if (kPer & 1) bs_grid_f64(y[0], bx.q[0], bx.invq_d[0], t.x, t.rx);
  if (kPer & 2) bs_grid_f64(y[1], bx.q[1], bx.invq_d[1], t.y, t.ry);
  if (kPer & 4) bs_grid_f64(y[2], bx.q[2], bx.invq_d[2], t.z, t.rz);
  t.ax = t.ay = t.az = 0.0;
}

template <int kPer>
__device__ inline BsSrcD bs_stage_f64(const BsPts& in, int k, int n, int copy, const BsAxes& bx) {
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
  return g;
}

template <int kPer>
__device__ __forceinline__ void bs_pair_f64(const BsSrcD& g, BsTgtD& t, bool excluded, double gx,
                                            double gy, double gz) {
  const double r1x = bs_sep<(kPer & 1) != 0>(g.x, t.x, g.rx, t.rx, gx);
  const double r1y = bs_sep<(kPer & 2) != 0>(g.y, t.y, g.ry, t.ry, gy);
  const double r1z = bs_sep<(kPer & 4) != 0>(g.z, t.z, g.rz, t.rz, gz);
  const double n1 = fma(r1x, r1x, fma(r1y, r1y, r1z * r1z));
  const double v = n1 + fma(r1x, g.dx, fma(r1y, g.dy, r1z * g.dz));
  const double n2 = v + g.q;
  const double n12 = n1 * n2;
  const double y = __builtin_amdgcn_rsq(n12);
  const double p = n12 * y;
  const double w = fma(p, fma(-p, y, 3.0), n1 + v);
  const double s2 = w + g.q;
  const double arg = (s2 * n12) * (w * w);
  const double z = __builtin_amdgcn_rsq(arg);
  double f = (s2 * z) * fma(-(arg * z), z, 3.0);
  f = excluded ? 0.0 : f;
  t.ax = fma(f, fma(r1y, g.dz, -(r1z * g.dy)), t.ax);
  t.ay = fma(f, fma(r1z, g.dx, -(r1x * g.dz)), t.ay);
  t.az = fma(f, fma(r1x, g.dy, -(r1y * g.dx)), t.az);
}

// The whole sum for kFewTargets targets by kThreads threads: thread (slice,
// target) adds every slice-th segment of the staged tiles (kTile records at
// src) for its target j; the slices are added in FP64 in a fixed tree, to a
// part per wave and target (red).  n: the points, lim >= n: what may be read;
// the first tile's loads do not wait for n.
constexpr int kFewTargets = 8;

template <bool kF32, int kVar, int kThreads, int kTile, class Src>
__device__ __forceinline__ void bs_few(const BsPts& in, int n, int lim, int tiles, int j,
                                       const BsAxes& bx, Src* src,
                                       double (*red)[3][kFewTargets]) {
  constexpr int kSlices = kThreads / kFewTargets;
  const int lane = threadIdx.x & 63;
  const int sl = threadIdx.x / kFewTargets;
  const int jc = min(j, lim - 1);  // (lanes beyond the points write nothing)
  double y[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) y[a] = in.Y[a * in.sa + jc * in.sj];
  int oc = 0;  // the image copy whose own segments are excluded too
  if (bx.copies > 1 && (in.nxt[jc] == jc || in.prv[jc] == jc)) oc = bs_own_copy(y, bx);
  uint32_t xt[3] = {0u, 0u, 0u};
  BsTgtD td;
  if constexpr (kF32) {
#pragma unroll
    for (int a = 0; a < 3; ++a) xt[a] = bs_grid_f32(y[a], bx, a);
  } else {
    bs_target_f64<kVar>(y, bx, td);
  }
  double v[3] = {0.0, 0.0, 0.0};
  for (int copy = 0; copy < bx.copies; ++copy) {
    const int jj = copy == 0 || copy == oc ? jc : -1;
    float fx = 0.f, fy = 0.f, fz = 0.f;
    td.ax = td.ay = td.az = 0.0;
    for (int tile = 0; tile == 0 || tile < tiles; ++tile) {
      const int t0 = tile * kTile;
#pragma unroll
      for (int u = 0; u < kTile; u += kThreads) {
        const int k = t0 + u + threadIdx.x;
        if (k < lim) {
          if constexpr (kF32)
            src[u + threadIdx.x] = bs_stage_f32<kVar != 0, true>(
                in, nullptr, 0, k, lim, copy, bx.invq_f[0], bx.invq_f[1], bx.invq_f[2], bx);
          else
            src[u + threadIdx.x] = bs_stage_f64<kVar>(in, k, lim, copy, bx);
        }
      }
      __syncthreads();
      const int cnt = min(kTile, n - t0);
#pragma unroll 2
      for (int s = sl; s < cnt; s += kSlices) {
        const Src g = src[s];
        const bool ex = t0 + s == jj || g.kn == jj;
        if constexpr (kF32)
          bs_pair_f32<kVar != 0>(g, xt[0], xt[1], xt[2], bx.invq_f[0], bx.invq_f[1], bx.invq_f[2],
                                 ex, fx, fy, fz);
        else
          bs_pair_f64<kVar>(g, td, ex, bx.invq_d[0], bx.invq_d[1], bx.invq_d[2]);
      }
      __syncthreads();
    }
    const double sg = (kF32 ? 1.0 : 0.5) * (double)bx.sign[copy];
    v[0] += sg * (kF32 ? (double)fx : td.ax);
    v[1] += sg * (kF32 ? (double)fy : td.ay);
    v[2] += sg * (kF32 ? (double)fz : td.az);
  }
#pragma unroll
  for (int off = kFewTargets; off < 64; off <<= 1)
#pragma unroll
    for (int a = 0; a < 3; ++a) v[a] += __shfl_xor(v[a], off);
  if (lane < kFewTargets)
    for (int a = 0; a < 3; ++a) red[threadIdx.x >> 6][a][lane] = v[a];
  __syncthreads();
}

}  // namespace vlb
