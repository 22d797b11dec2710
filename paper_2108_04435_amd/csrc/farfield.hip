// Far-field approximation of the non-local Biot-Savart sum (an extension of
// Sec. II.A, Eq. Biot-Savart, for large tangles): periodic box, uniform
// cells of edge h, monopole to quadrupole moments of each cell's segment
// vorticity about its centre, evaluated per (target, cell) where the cell
// is far, the exact straight-segment integral where it is near.
//
// Definitions (the decisions are those of the FP64 reference of the same
// approximation, taken in FP64 and on the 32-bit position grid):
//  * positions are reduced into [0, L) per axis; segment k belongs to the
//    cell of its midpoint; y_k = m_k - c at the nearest image, d_k the
//    segment vector at the nearest image; rad = max_k (|y_k| + |d_k| / 2);
//  * per target r, each segment sits at the image of its start that the
//    direct sum takes (the wrapped difference of 32-bit grid coordinates);
//    with delta_k = X(s_k) - X(c) (wrapped, small) and u = X(c) - X(r),
//    the segment's image places the centre at (c - r) + K L with
//    K = (wrap(u + delta_k) - delta_k - (X(c) - X(r))) / 2^32, so the class
//    of a cell's segments changes only where u + delta crosses 2^31 (the
//    plane half a box from the target);
//  * one class: far when |R|^2 theta^2 >= rad^2 at R = (c - r) + K L;
//    classes differing on one axis (delta_min and delta_max on opposite
//    sides): split when both images pass, the class below the crossing
//    taking the prefix moments of the cell's segments sorted by delta on
//    that axis, the other the rest; otherwise direct;
//  * with two levels the cells of edge 2h are classified first and an
//    opened one (neither far nor split) hands its 8 children of edge h to
//    the same rule, the lanes that opened it taking part.
//
// Layout (workspace, all per call):
//  * per point: wrapped FP64 positions, grid coordinates, links, y and d
//    (FP64), cell key;
//  * segments sorted by cell (stable radix sort, so ascending index inside
//    a cell; with two levels the key is coarse cell * 8 + child, so each
//    coarse cell's children are consecutive), one 32-byte record each for
//    the direct loop;
//  * one 256-byte record per cell (range, rad^2, centre, grid centre,
//    delta extremes, 42 moments), read with scalar loads;
//  * per axis: each cell's deltas in ascending order and the prefix sums of
//    the 42 moment components over that order (cnt + 1 rows per cell);
//  * the evaluation grid: blockIdx.x picks 256 targets, 64 per wave
//    (consecutive in the cell order, so a wave's targets are close),
//    blockIdx.y one of S cell chunks (cells y modulo S of the coarsest level);
//    the chunk partials are added in FP64 in chunk order (bitwise
//    reproducible).
#include "vlb_internal.h"

#include <cmath>

namespace vlb {

namespace {

constexpr int kMom = 42;       // moment components per cell or class
constexpr int kFfTargets = 256;  // targets per block, 64 per wave

// Moment components (no kappa: the caller scales the sum), each linear in
// the segments and combined so that the expansion takes them as they are.
// With A = d x y and Q_n,jk = d_n (y_j y_k + d_j d_k / 12), tr_n its trace:
//   0..2    M0_n = d_n;
//   3..5    -A_m (the antisymmetric part of the dipole);
//   6..14   3 d_n y_p (the dipole);
//   15..32  7.5 (Q_n,jk - delta_jk tr_n / 5) for jk = 00 01 02 11 12 22, the
//           off-diagonal ones doubled (both orders of a symmetric pair);
//   33..41  -3 A_m y_k (what the curl of the quadrupole leaves beside Q).
__device__ inline double comp_value(int comp, const double* y, const double* d) {
#pragma clang fp contract(off)
  if (comp < 3) return d[comp];
  const auto cross = [&](int m) {
    const int a = (m + 1) % 3, b = (m + 2) % 3;
    return d[a] * y[b] - d[b] * y[a];
  };
  if (comp < 6) return -cross(comp - 3);
  if (comp < 15) {
    const int i = comp - 6;
    return 3.0 * (d[i / 3] * y[i % 3]);
  }
  if (comp < 33) {
    const int i = comp - 15;
    const int nn = i / 6, jk = i % 6;
    const int j = jk < 3 ? 0 : (jk < 5 ? 1 : 2);
    const int k = jk < 3 ? jk : (jk < 5 ? jk - 2 : 2);
    const double q = y[j] * y[k] + d[j] * d[k] / 12.0;
    if (j != k) return 15.0 * (d[nn] * q);
    const double tr = (y[0] * y[0] + y[1] * y[1] + y[2] * y[2]) +
                      (d[0] * d[0] + d[1] * d[1] + d[2] * d[2]) / 12.0;
    return 7.5 * (d[nn] * (q - tr / 5.0));
  }
  const int i = comp - 33;
  return -3.0 * (cross(i / 3) * y[i % 3]);
}

struct FfAxes {
  double L[3], q[3], th2;
  double h[2];   // cell edge per level (level 0 the finest)
  float iqf[3];  // lattice units per grid step
  float qf;      // one grid step count per lattice unit when uniform
  int nc[2][3];  // cells per axis per level
  int C[2];      // cells per level
  int levels;    // 1 or 2
  int uniform;
};

// Cell coordinates at a level from its record index: one level, x fastest;
// two levels, the coarse cell x fastest and, at the fine level, index =
// coarse * 8 + child with child bits x | y << 1 | z << 2.
__device__ inline void ff_coords(const FfAxes& ax, int level, int idx, int* ci) {
  if (ax.levels == 1 || level == 1) {
    const int* nc = ax.nc[level];
    ci[0] = idx % nc[0];
    ci[1] = (idx / nc[0]) % nc[1];
    ci[2] = idx / (nc[0] * nc[1]);
  } else {
    const int t = idx >> 3, ch = idx & 7;
    const int* nc = ax.nc[1];
    ci[0] = 2 * (t % nc[0]) + (ch & 1);
    ci[1] = 2 * ((t / nc[0]) % nc[1]) + ((ch >> 1) & 1);
    ci[2] = 2 * (t / (nc[0] * nc[1])) + ((ch >> 2) & 1);
  }
}

__device__ inline double ff_min_image(double x, double L) {
#pragma clang fp contract(off)
  if (x > 0.5 * L) return x - L;
  if (x < -0.5 * L) return x + L;
  return x;
}

struct __align__(256) FfCell {
  int32_t start, count;      // range in the sorted order
  double rad2;               // rad * rad
  double c[3];               // centre
  uint32_t xc[3];            // centre on the 32-bit grid
  int32_t dmin[3], dmax[3];  // extremes of the wrapped grid offset start - centre
  int32_t pad;
  float m[kMom];
};

struct __align__(32) FfSeg {
  uint32_t x[3];  // start on the grid
  float d[3];     // segment vector: wrapped grid difference (uniform) or lattice units
  float dq;       // |d|^2
  int32_t idx;    // segment (point) index
};

__device__ inline double ff_wrap(double x, double L) {
#pragma clang fp contract(off)
  if (x < 0.0) x = x + L;
  if (x >= L) x = x - L;
  if (x >= L) x = 0.0;  // x + L rounded up to L
  return x;
}

__global__ void k_ff_init(int32_t* __restrict__ prv, int n) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j < n) prv[j] = j;
}

// Point j with successor k (positions y_j, y_k): wrapped position, grid
// coordinate, segment vector, midpoint and the sort key of its finest cell.
__device__ inline void ff_point(const double* yj, const double* yk, int j, long long nc,
                                const FfAxes& ax, double* __restrict__ P,
                                uint32_t* __restrict__ X, double* __restrict__ M,
                                double* __restrict__ D, uint32_t* __restrict__ keys,
                                int32_t* __restrict__ kidx, int32_t* __restrict__ vals) {
#pragma clang fp contract(off)
  int idx[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double L = ax.L[a];
    const double p = ff_wrap(yj[a], L);
    const double pk = ff_wrap(yk[a], L);
    P[(long long)a * nc + j] = p;
    X[(long long)a * nc + j] = (uint32_t)(long long)floor(p * ax.q[a]);
    const double d = ff_min_image(pk - p, L);
    double mid = p + 0.5 * d;
    mid = mid - L * floor(mid / L);
    int i = (int)floor(mid / ax.h[0]);
    idx[a] = min(max(i, 0), ax.nc[0][a] - 1);
    M[(long long)a * nc + j] = mid;
    D[(long long)a * nc + j] = d;
  }
  int key;
  if (ax.levels == 1) {
    key = (idx[2] * ax.nc[0][1] + idx[1]) * ax.nc[0][0] + idx[0];
  } else {
    const int t = ((idx[2] >> 1) * ax.nc[1][1] + (idx[1] >> 1)) * ax.nc[1][0] + (idx[0] >> 1);
    key = t * 8 + ((idx[0] & 1) | ((idx[1] & 1) << 1) | ((idx[2] & 1) << 2));
  }
  keys[j] = (uint32_t)key;
  kidx[j] = key;
  vals[j] = j;
}

// Stand-alone sum: links sanitised from the caller's (clamped into
// [0, n), inverted into prv, which k_ff_init set to self), positions
// [n][3]; thread 0 writes the point count.
__global__ void k_ff_prep(const double* __restrict__ xyz, const int32_t* __restrict__ next, int n,
                          FfAxes ax, int32_t* __restrict__ cnt, double* __restrict__ P,
                          uint32_t* __restrict__ X, int32_t* __restrict__ nxt,
                          int32_t* __restrict__ prv, double* __restrict__ M,
                          double* __restrict__ D, uint32_t* __restrict__ keys,
                          int32_t* __restrict__ kidx, int32_t* __restrict__ vals) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j == 0) {
    cnt[0] = n;
    for (int i = 1; i < 32; ++i) cnt[i] = 0;
  }
  if (j >= n) return;
  const int k = min(max(next[j], 0), n - 1);
  nxt[j] = k;
  if (k != j) prv[k] = j;
  const double yj[3] = {xyz[3LL * j], xyz[3LL * j + 1], xyz[3LL * j + 2]};
  const double yk[3] = {xyz[3LL * k], xyz[3LL * k + 1], xyz[3LL * k + 2]};
  ff_point(yj, yk, j, n, ax, P, X, M, D, keys, kidx, vals);
}

// In a run: positions Y (3 x nc, SoA) and the run's links, the live count
// cnt[0]; slots beyond it get the largest key (they sort last).
__global__ void k_ff_prep_run(const double* __restrict__ Y, const int32_t* __restrict__ nxt,
                              const int32_t* __restrict__ cnt, long long nc, FfAxes ax,
                              double* __restrict__ P, uint32_t* __restrict__ X,
                              double* __restrict__ M, double* __restrict__ D,
                              uint32_t* __restrict__ keys, int32_t* __restrict__ kidx,
                              int32_t* __restrict__ vals) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= nc) return;
  if (j >= cnt[0]) {
    keys[j] = 0xffffffffu;
    kidx[j] = 0;
    vals[j] = j;
    return;
  }
  const int k = nxt[j];
  const double yj[3] = {Y[j], Y[nc + j], Y[2 * nc + j]};
  const double yk[3] = {Y[k], Y[nc + k], Y[2 * nc + k]};
  ff_point(yj, yk, j, nc, ax, P, X, M, D, keys, kidx, vals);
}

// Cell ranges in the sorted keys (binary search; empty cells get count 0).
__device__ inline int lower_bound_u32(const uint32_t* a, int n, uint32_t v) {
  int lo = 0, hi = n;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (a[mid] < v)
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo;
}

// Level records cover the sorted keys [c << shift, (c + 1) << shift).
__global__ void k_ff_bounds(const uint32_t* __restrict__ sk, int n, int C, int shift,
                            FfCell* __restrict__ cells) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= C) return;
  const int lo = lower_bound_u32(sk, n, (uint32_t)c << shift);
  const int hi = lower_bound_u32(sk, n, ((uint32_t)c + 1u) << shift);
  cells[c].start = lo;
  cells[c].count = hi - lo;
}

// Per sorted position: the direct loop's segment record.
__global__ void k_ff_seg(const int32_t* __restrict__ so, const uint32_t* __restrict__ X,
                         const int32_t* __restrict__ nxt, const int32_t* __restrict__ cntp,
                         long long nc, FfAxes ax, FfSeg* __restrict__ recs) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= cntp[0]) return;
  const int k = so[p];
  const int kn = nxt[k];
  FfSeg r;
  for (int a = 0; a < 3; ++a) {
    const uint32_t x0 = X[(long long)a * nc + k];
    float e = (float)(int)(X[(long long)a * nc + kn] - x0);
    if (!ax.uniform) e *= ax.iqf[a];
    r.x[a] = x0;
    r.d[a] = e;
  }
  r.dq = r.d[0] * r.d[0] + r.d[1] * r.d[1] + r.d[2] * r.d[2];
  r.idx = k;
  recs[p] = r;
}

// Per segment, at one level: the 42 moment components about its cell's
// centre (FP64, row k of comps) and |y| + |d| / 2 (srad).
__global__ void k_ff_comps(const double* __restrict__ M, const double* __restrict__ D,
                           const int32_t* __restrict__ kidx, const int32_t* __restrict__ cntp,
                           long long nc, FfAxes ax, int level, double* __restrict__ comps,
                           double* __restrict__ srad) {
#pragma clang fp contract(off)
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= cntp[0]) return;
  int ci[3];
  ff_coords(ax, level, kidx[k] >> (3 * level), ci);
  double y[3], d[3];
  for (int b = 0; b < 3; ++b) {
    y[b] = ff_min_image(M[(long long)b * nc + k] - ((double)ci[b] + 0.5) * ax.h[level], ax.L[b]);
    d[b] = D[(long long)b * nc + k];
  }
  double* row = comps + (long long)k * kMom;
#pragma unroll
  for (int i = 0; i < kMom; ++i) row[i] = comp_value(i, y, d);
  const double ny = sqrt(y[0] * y[0] + y[1] * y[1] + y[2] * y[2]);
  const double nd = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
  srad[k] = ny + 0.5 * nd;
}

// One block of kOrder threads per (cell of a level, axis): the cell's start
// offsets on the axis in ascending order (ties by sorted position) with
// their segment indices (sdel, sidx), the prefix sums of the 42 moment
// components over that order (FP64 sums stored FP32, rows
// a (nc + C) + start + c + i for i = 0 .. count, row 0 zero; nc the
// capacity of the point arrays), and the
// record's fields for the axis (centre, grid centre, offset extremes); the
// axis-0 block also writes the radius and the moments (its prefix totals).
// The ranks compare offsets staged in LDS; the prefix sums add the components
// of k_ff_comps, one lane per component, each wave over its share of the
// order: the shares' sums first, then the rows from the sum of the shares
// before.  What bounds it is the latency of the dependent loads and of the
// sums' chain: one wave per cell took 240 us for 512 cells of 195 points,
// four waves take 84 us.
template <int kOrder>
__global__ __launch_bounds__(kOrder) void k_ff_order(const int32_t* __restrict__ so,
                                                     const double* __restrict__ comps,
                                                     const double* __restrict__ srad,
                                                     const uint32_t* __restrict__ X, long long nc,
                                                     FfAxes ax, int level,
                                                     FfCell* __restrict__ cells,
                                                     int32_t* __restrict__ sdel,
                                                     int32_t* __restrict__ sidx,
                                                     float* __restrict__ pre) {
#pragma clang fp contract(off)
  constexpr int kWaves = kOrder / 64;
  const int c = blockIdx.x / 3, a = blockIdx.x - 3 * (blockIdx.x / 3);
  const int t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int C = ax.C[level];
  const int s = cells[c].start, cnt = cells[c].count;
  int ci[3];
  ff_coords(ax, level, c, ci);
  double cen[3];
  for (int b = 0; b < 3; ++b) cen[b] = ((double)ci[b] + 0.5) * ax.h[level];
  const uint32_t xc = (uint32_t)(long long)floor(cen[a] * ax.q[a]);
  const uint32_t* Xa = X + (long long)a * nc;
  int32_t* sd = sdel + (long long)a * nc + s;
  int32_t* si = sidx + (long long)a * nc + s;
  __shared__ int32_t off[kOrder];
  __shared__ double part[kWaves][kMom];
  __shared__ int32_t lo[kWaves], hi[kWaves];
  __shared__ double far[kWaves];
  int dmn = 0x7fffffff, dmx = -0x7fffffff - 1;
  double rad = 0.0;
  for (int b0 = 0; b0 < cnt; b0 += kOrder) {
    const int i = b0 + t;
    const bool vi = i < cnt;
    const int ki = vi ? so[s + i] : 0;
    const int di = vi ? (int)(Xa[ki] - xc) : 0;
    if (vi) {
      dmn = min(dmn, di);
      dmx = max(dmx, di);
      if (a == 0) rad = fmax(rad, srad[ki]);
    }
    int rank = 0;
    for (int j0 = 0; j0 < cnt; j0 += kOrder) {
      __syncthreads();  // the offsets of the previous round have been read
      off[t] = j0 == b0 ? di : (j0 + t < cnt ? (int)(Xa[so[s + j0 + t]] - xc) : 0);
      __syncthreads();
      const int m = min(kOrder, cnt - j0);
#pragma unroll 4
      for (int k = 0; k < m; ++k) {
        const int dk = off[k];
        rank += (dk < di || (dk == di && j0 + k < i)) ? 1 : 0;
      }
    }
    if (vi) {
      sd[rank] = di;
      si[rank] = ki;
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    dmn = min(dmn, __shfl_xor(dmn, o));
    dmx = max(dmx, __shfl_xor(dmx, o));
    rad = fmax(rad, __shfl_xor(rad, o));
  }
  if (lane == 0) {
    lo[w] = dmn;
    hi[w] = dmx;
    far[w] = rad;
  }
  __syncthreads();  // the sorted order, written above, is read below
  float* row = pre + ((long long)a * (nc + C) + s + c) * kMom;
  const int per = (cnt + kWaves - 1) / kWaves;
  const int i0 = min(w * per, cnt), i1 = min(i0 + per, cnt);
  double acc = 0.0;
  if (kWaves > 1) {
    if (lane < kMom && w + 1 < kWaves) {
#pragma unroll 8
      for (int i = i0; i < i1; ++i) acc = acc + comps[(long long)si[i] * kMom + lane];
      part[w][lane] = acc;
    }
    __syncthreads();
    acc = 0.0;
    if (lane < kMom)
      for (int u = 0; u < w; ++u) acc = acc + part[u][lane];
  }
  if (lane < kMom) {
    if (w == 0) row[lane] = 0.f;
#pragma unroll 8
    for (int i = i0; i < i1; ++i) {
      acc = acc + comps[(long long)si[i] * kMom + lane];
      row[(long long)(i + 1) * kMom + lane] = (float)acc;
    }
  }
  FfCell& o = cells[c];
  if (t == 0) {
    for (int u = 1; u < kWaves; ++u) {
      dmn = min(dmn, lo[u]);
      dmx = max(dmx, hi[u]);
      rad = fmax(rad, far[u]);
    }
    o.c[a] = cen[a];
    o.xc[a] = xc;
    o.dmin[a] = cnt > 0 ? dmn : 0;
    o.dmax[a] = cnt > 0 ? dmx : 0;
    if (a == 0) {
      o.rad2 = rad * rad;
      o.pad = 0;
    }
  }
  if (a == 0 && w == kWaves - 1 && lane < kMom) o.m[lane] = (float)acc;
}

// Moments: one array, or the difference of two (the upper class of a split
// cell: the cell's totals minus the prefix of the lower class).
struct MomA {
  const float* p;
  __device__ float operator()(int i) const { return p[i]; }
};
struct MomD {
  const float* t;
  const float* p;
  __device__ float operator()(int i) const { return t[i] - p[i]; }
};

// The expansion of a cell (or class) of moments m at separation R (target
// less centre): 69 ordinary instructions.
template <class M>
__device__ __forceinline__ void m2p_f32(float Rx, float Ry, float Rz, const M& m, float& vx,
                                        float& vy, float& vz) {
  const float r2 = fmaf(Rx, Rx, fmaf(Ry, Ry, Rz * Rz));
  const float ir = __builtin_amdgcn_rsqf(r2);
  const float i2 = ir * ir;
  const float r3 = ir * i2;
  const float r5 = r3 * i2;
  const float xx = Rx * Rx, xy = Rx * Ry, xz = Rx * Rz, yy = Ry * Ry, yz = Ry * Rz, zz = Rz * Rz;
  float W[3], B[3];  // both to be scaled by r5
#pragma unroll
  for (int n = 0; n < 3; ++n) {
    const int q = 15 + 6 * n;
    const float Q = fmaf(m(q), xx, fmaf(m(q + 1), xy, fmaf(m(q + 2), xz, fmaf(m(q + 3), yy,
                    fmaf(m(q + 4), yz, m(q + 5) * zz)))));
    const float a = fmaf(m(6 + 3 * n), Rx, fmaf(m(7 + 3 * n), Ry, m(8 + 3 * n) * Rz));
    W[n] = fmaf(i2, Q, a);
    B[n] = fmaf(m(33 + 3 * n), Rx, fmaf(m(34 + 3 * n), Ry, m(35 + 3 * n) * Rz));
  }
  const float V0 = fmaf(m(1), Rz, fmaf(-m(2), Ry, m(3)));
  const float V1 = fmaf(m(2), Rx, fmaf(-m(0), Rz, m(4)));
  const float V2 = fmaf(m(0), Ry, fmaf(-m(1), Rx, m(5)));
  vx = fmaf(r3, V0, fmaf(r5, fmaf(W[1], Rz, fmaf(-W[2], Ry, B[0])), vx));
  vy = fmaf(r3, V1, fmaf(r5, fmaf(W[2], Rx, fmaf(-W[0], Rz, B[1])), vy));
  vz = fmaf(r3, V2, fmaf(r5, fmaf(W[0], Ry, fmaf(-W[1], Rx, B[2])), vz));
}

// One (target, segment) pair of the exact straight-segment integral, in the
// direct FP32 sum's form (bs_pair_f32) with the products nested from the last
// axis.
template <bool kUniform>
__device__ __forceinline__ void ff_pair(const FfSeg& g, uint32_t xt, uint32_t yt, uint32_t zt,
                                        const FfAxes& ax, float& vx, float& vy, float& vz,
                                        bool zero) {
  float r1x = (float)(int)(g.x[0] - xt);
  float r1y = (float)(int)(g.x[1] - yt);
  float r1z = (float)(int)(g.x[2] - zt);
  if (!kUniform) {
    r1x *= ax.iqf[0];
    r1y *= ax.iqf[1];
    r1z *= ax.iqf[2];
  }
  const float ex = g.d[0], ey = g.d[1], ez = g.d[2];
  const float t = fmaf(r1x, ex, fmaf(r1y, ey, r1z * ez));
  const float n1 = fmaf(r1x, r1x, fmaf(r1y, r1y, r1z * r1z));
  const float n2 = fmaf(2.0f, t, n1 + g.dq);
  const float i1 = __builtin_amdgcn_rsqf(n1);
  const float i2 = __builtin_amdgcn_rsqf(n2);
  const float crx = fmaf(r1y, ez, -r1z * ey);
  const float cry = fmaf(r1z, ex, -r1x * ez);
  const float crz = fmaf(r1x, ey, -r1y * ex);
  const float a = i1 * i2;
  const float den = fmaf(n1 + t, a, 1.0f);
  float f = (i1 + i2) * a * __builtin_amdgcn_rcpf(den);
  f = zero ? 0.0f : f;
  vx = fmaf(f, crx, vx);
  vy = fmaf(f, cry, vy);
  vz = fmaf(f, crz, vz);
}

// Per-lane decision for one cell (FP64 and integers, no contraction).
struct FfDecision {
  double R0[3];  // (c - r) + K L of the class of the smallest start offset
  int ncross;    // axes on which the start offsets cross the half-box plane
  int axis;      // the crossed axis (ncross == 1)
  int kc;        // K of that class on the crossed axis
  bool ok0;      // R0 passes the opening test
};

__device__ inline void ff_decide(const FfCell* __restrict__ cm, const double* r, const uint32_t* xt,
                                 const FfAxes& ax, FfDecision& o) {
#pragma clang fp contract(off)
  o.ncross = 0;
  o.axis = 0;
  o.kc = 0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const uint32_t xc = cm->xc[a];
    const int dmin = cm->dmin[a], dmax = cm->dmax[a];
    const uint32_t u = xc - xt[a];
    const int wmin = (int)(u + (uint32_t)dmin);
    const int wmax = (int)(u + (uint32_t)dmax);
    const long long rawc = (long long)xc - (long long)xt[a];
    const int k = (int)(((long long)wmin - (long long)dmin - rawc) >> 32);
    const bool cr = wmax < wmin;
    o.ncross += cr ? 1 : 0;
    o.axis = cr ? a : o.axis;
    o.kc = cr ? k : o.kc;
    o.R0[a] = (cm->c[a] - r[a]) + (double)k * ax.L[a];
  }
  const double d2 = (o.R0[0] * o.R0[0] + o.R0[1] * o.R0[1]) + o.R0[2] * o.R0[2];
  o.ok0 = d2 * ax.th2 >= cm->rad2;
}

// The class of the largest offset on the crossed axis: its wrapped offset
// dropped by 2^32 at the crossing, so its K there is one less.  Returns
// whether that image passes the opening test.
__device__ inline bool ff_other(const FfCell* __restrict__ cm, const FfDecision& o, const double* r,
                                const FfAxes& ax, double* R1) {
#pragma clang fp contract(off)
#pragma unroll
  for (int a = 0; a < 3; ++a)
    R1[a] = a == o.axis ? (cm->c[a] - r[a]) + (double)(o.kc - 1) * ax.L[a] : o.R0[a];
  const double d2 = (R1[0] * R1[0] + R1[1] * R1[1]) + R1[2] * R1[2];
  return d2 * ax.th2 >= cm->rad2;
}

// Far and split contributions of one cell for the active lanes; returns
// whether this lane opens the cell (active, neither far nor split).
__device__ inline bool ff_cell_eval(const FfCell* __restrict__ cm, int c,
                                    const int32_t* __restrict__ sdel,
                                    const float* __restrict__ pre, long long nc, int C,
                                    bool active,
                                    const double* r, const uint32_t* xt, const FfAxes& ax,
                                    float& fx, float& fy, float& fz) {
  FfDecision dc;
  ff_decide(cm, r, xt, ax, dc);
  const bool far = active && dc.ncross == 0 && dc.ok0;
  bool split = false;
  double R1[3] = {0.0, 0.0, 0.0};
  if (active && dc.ncross == 1 && dc.ok0) split = ff_other(cm, dc, r, ax, R1);
  if (__any(far)) {
    if (far)
      m2p_f32((float)-dc.R0[0], (float)-dc.R0[1], (float)-dc.R0[2], MomA{cm->m}, fx, fy, fz);
  }
  if (__any(split)) {
    if (split) {
      // offsets below the crossing: u + delta < 2^31
      const int a = dc.axis;
      const uint32_t u = cm->xc[a] - xt[a];
      const int db = (int)(0x80000000u - u);
      const int32_t* dl = sdel + (long long)a * nc + cm->start;
      int lo = 0, hi = cm->count;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (dl[mid] < db)
          lo = mid + 1;
        else
          hi = mid;
      }
      const float* pr = pre + ((long long)a * (nc + C) + cm->start + c + lo) * kMom;
      m2p_f32((float)-dc.R0[0], (float)-dc.R0[1], (float)-dc.R0[2], MomA{pr}, fx, fy, fz);
      m2p_f32((float)-R1[0], (float)-R1[1], (float)-R1[2], MomD{cm->m, pr}, fx, fy, fz);
    }
  }
  return active && !far && !split;
}

// The exact pairs of a finest cell for the lanes in `near`; the target's
// own two segments excluded where the cell holds them (kCheck).  The
// cell's records are staged 64 at a time in the wave's own LDS slots
// (lds, 64 records) and read back with broadcast LDS loads, so the loop
// waits on no scalar load.
template <bool kUniform, bool kCheck>
__device__ inline void ff_direct_loop(int s0, int e, const FfSeg* __restrict__ recs,
                                      FfSeg* lds, bool near, int jj, int pj, const uint32_t* xt,
                                      const FfAxes& ax, float& dx, float& dy, float& dz) {
  const int lane = threadIdx.x & 63;
  for (int c0 = s0; c0 < e; c0 += 64) {
    const int m = min(64, e - c0);
    if (lane < m) lds[lane] = recs[c0 + lane];
    __builtin_amdgcn_wave_barrier();
    if (near) {
#pragma unroll 2
      for (int k = 0; k < m; ++k) {
        const FfSeg g = lds[k];
        ff_pair<kUniform>(g, xt[0], xt[1], xt[2], ax, dx, dy, dz,
                          kCheck && (g.idx == jj || g.idx == pj));
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
}

template <bool kUniform>
__device__ inline void ff_direct(int s0, int count, int c, const FfSeg* __restrict__ recs,
                                 FfSeg* lds, bool near, int kj, int kp, int jj, int pj,
                                 const uint32_t* xt, const FfAxes& ax, float& dx, float& dy,
                                 float& dz) {
  const int e = s0 + count;
  if (__any(kj == c || kp == c))
    ff_direct_loop<kUniform, true>(s0, e, recs, lds, near, jj, pj, xt, ax, dx, dy, dz);
  else
    ff_direct_loop<kUniform, false>(s0, e, recs, lds, near, jj, pj, xt, ax, dx, dy, dz);
}

// The wave's targets: grid coordinates of lane 0 and the extremes of the
// targets' offsets from it; one: no target lies beyond the box boundary from
// lane 0 on any axis, so that a cell's image is the same grid distance for
// all of them.
struct FfBox {
  uint32_t x0[3];
  int emin[3], emax[3];
  bool one;
};

__device__ inline void ff_box(const uint32_t* xt, bool valid, FfBox& b) {
  b.one = true;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    b.x0[a] = (uint32_t)__builtin_amdgcn_readfirstlane((int)xt[a]);
    const int e = valid ? (int)(xt[a] - b.x0[a]) : 0;
    int lo = e, hi = e;
    for (int off = 32; off > 0; off >>= 1) {
      lo = min(lo, __shfl_xor(lo, off));
      hi = max(hi, __shfl_xor(hi, off));
    }
    b.emin[a] = __builtin_amdgcn_readfirstlane(lo);
    b.emax[a] = __builtin_amdgcn_readfirstlane(hi);
    b.one = b.one && (long long)b.x0[a] + b.emin[a] >= 0 &&
            (long long)b.x0[a] + b.emax[a] < (1LL << 32);
  }
}

// What the per-lane decision (ff_decide) comes to for all of the wave's
// targets at once, one cell per lane: far for all of them at the image K, or
// opened by all, or one of the two at that image with no crossing (each lane
// tests its distance), or mixed (each lane decides).  A target at offset e has
// wmin = a - e and wmax = b - e where that neither wraps (no crossing), and
// the image of the centre lies a - dmin - e grid steps away (one more at most
// for the positions' parts below the grid); the bounds on its distance over
// the box decide with a margin of 1e-9.
enum FfClass { kEmpty = 0, kFar = 1, kRing = 2, kOpen = 3, kMixed = 4 };

__device__ inline int ff_class(const FfCell* __restrict__ cm, const FfBox& b, const FfAxes& ax,
                               int K[3]) {
  K[0] = K[1] = K[2] = 0;
  if (cm->count == 0) return kEmpty;
  bool ok = b.one;
  double near2 = 0.0, far2 = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int dmin = cm->dmin[a], dmax = cm->dmax[a];
    const uint32_t xc = cm->xc[a];
    const long long lo = (int)(xc - b.x0[a] + (uint32_t)dmin);
    const long long hi = lo + ((long long)dmax - dmin);
    ok = ok && lo - b.emax[a] >= -(1LL << 31) && hi - b.emin[a] < (1LL << 31);
    const long long at = lo - dmin;
    K[a] = (int)((at - ((long long)xc - (long long)b.x0[a])) >> 32);
    const double iq = ax.L[a] / 4294967296.0;
    const double rlo = (double)(at - b.emax[a] - 1) * iq, rhi = (double)(at - b.emin[a] + 1) * iq;
    const double m = fmax(0.0, fmax(rlo, -rhi)), M = fmax(fabs(rlo), fabs(rhi));
    near2 += m * m;
    far2 += M * M;
  }
  const double rad2 = cm->rad2;
  if (!ok) return kMixed;
  if (near2 * ax.th2 > rad2 * (1.0 + 1e-9)) return kFar;
  return far2 * ax.th2 < rad2 * (1.0 - 1e-9) ? kOpen : kRing;
}

// A cell at the image K for all lanes: the expansion for the active lanes it
// is far for (kTest: those that pass the opening test of ff_decide; else all).
// Returns whether this lane opens the cell.
template <bool kTest>
__device__ __forceinline__ bool ff_far(const FfCell* __restrict__ cm, const int K[3], bool active,
                                       const double* r, const FfAxes& ax, float& fx, float& fy,
                                       float& fz) {
#pragma clang fp contract(off)
  double R[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) R[a] = (cm->c[a] - r[a]) + (double)K[a] * ax.L[a];
  bool far = active;
  if (kTest) {
    const double d2 = (R[0] * R[0] + R[1] * R[1]) + R[2] * R[2];
    far = active && d2 * ax.th2 >= cm->rad2;
  }
  if (far) m2p_f32((float)-R[0], (float)-R[1], (float)-R[2], MomA{cm->m}, fx, fy, fz);
  return active && !far;
}

// Cell c of a level, of class cls (ff_class; its K in lane i): the far and
// split contributions for the active lanes; returns whether this lane opens
// the cell.
__device__ __forceinline__ bool ff_take(const FfCell* __restrict__ cells, int c, int cls,
                                        const int K[3], int i, const int32_t* __restrict__ sdel,
                                        const float* __restrict__ pre, long long nc, int C,
                                        bool active, const double* r, const uint32_t* xt,
                                        const FfAxes& ax, float& fx, float& fy, float& fz) {
  const FfCell* __restrict__ cm = cells + c;
  if (cls == kOpen) return active;
  if (cls == kMixed) return ff_cell_eval(cm, c, sdel, pre, nc, C, active, r, xt, ax, fx, fy, fz);
  const int Ki[3] = {__builtin_amdgcn_readlane(K[0], i), __builtin_amdgcn_readlane(K[1], i),
                     __builtin_amdgcn_readlane(K[2], i)};
  return cls == kFar ? ff_far<false>(cm, Ki, active, r, ax, fx, fy, fz)
                     : ff_far<true>(cm, Ki, active, r, ax, fx, fy, fz);
}

// What bounds it: the vector units, at 1.09 wave instructions per cycle and CU
// (an FMA with a scalar operand, as 42 of the expansion's are, issues at 0.89,
// one of vector registers at 1.6).  So the decision, 50 instructions per target
// and cell, is taken once per wave and cell, 64 cells at a time, where all of
// the wave's targets agree, and costs a distance where only the opening test
// differs.  The waves of a block, and the blocks that run beside it, walk the
// same cells, so that their records are read from the scalar cache.  Five
// waves per SIMD (96 VGPRs, 15 spilled) beat four by 4% and six by 5%.  1e5
// points of a 256^3 tangle, cells of 16 and 32, theta 0.25: 2.55 ms before
// (each lane deciding each cell, a block's four waves on four cells), 1.84 ms.
template <bool kUniform, int kLevels>
__global__ __launch_bounds__(256, 5) void k_ff_eval(
    const FfCell* __restrict__ cells0, const FfCell* __restrict__ cells1,
    const FfSeg* __restrict__ recs, const int32_t* __restrict__ so,
    const int32_t* __restrict__ kidx, const int32_t* __restrict__ prv,
    const double* __restrict__ Pw, const uint32_t* __restrict__ X,
    const int32_t* __restrict__ sdel0, const int32_t* __restrict__ sdel1,
    const float* __restrict__ pre0, const float* __restrict__ pre1,
    const int32_t* __restrict__ cntp, long long nc, int S, FfAxes ax, float* __restrict__ Pout) {
  const int n = cntp[0];
  if (blockIdx.x * kFfTargets >= n) return;  // whole block beyond the live points
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int t = blockIdx.x * kFfTargets + threadIdx.x;
  if (t - lane >= n) return;  // the wave's targets
  const bool valid = t < n;
  const int j = so[valid ? t : n - 1];  // lanes beyond the points repeat the last one, unwritten
  double r[3];
  uint32_t xt[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    r[a] = Pw[(long long)a * nc + j];
    xt[a] = X[(long long)a * nc + j];
  }
  const int pj = valid ? prv[j] : -1;
  const int jj = valid ? j : -1;
  const int kj = valid ? kidx[j] : -1;
  const int kp = valid ? kidx[pj] : -1;
  float fx = 0.f, fy = 0.f, fz = 0.f;  // expansions (lattice units)
  float dx = 0.f, dy = 0.f, dz = 0.f;  // direct pairs (grid units when uniform)
  const FfCell* __restrict__ top = kLevels == 2 ? cells1 : cells0;
  const int32_t* __restrict__ sdt = kLevels == 2 ? sdel1 : sdel0;
  const float* __restrict__ prt = kLevels == 2 ? pre1 : pre0;
  const int Ct = ax.C[kLevels - 1];
  const int step = S;
  __shared__ FfSeg stage[4][64];  // each wave's staged segment records
  FfSeg* lds = stage[w];
  FfBox box;
  ff_box(xt, valid, box);
  // The wave's coarsest cells, in groups of one per lane (one level) or of 8,
  // whose 64 children are then one per lane.
  constexpr int kGroup = kLevels == 2 ? 8 : 64;
  for (int c0 = blockIdx.y; c0 < Ct; c0 += step * kGroup) {
    int K[3] = {0, 0, 0};
    int cls = kEmpty;
    if (lane < kGroup && c0 + lane * step < Ct) cls = ff_class(top + c0 + lane * step, box, ax, K);
    uint32_t open_lo = 0u, open_hi = 0u;  // two levels, lane i: the lanes that open cell i
    for (uint64_t todo = __ballot(cls != kEmpty); todo; todo &= todo - 1) {
      const int i = __ffsll((unsigned long long)todo) - 1;
      const int c = c0 + i * step;
      const bool op = ff_take(top, c, __builtin_amdgcn_readlane(cls, i), K, i, sdt, prt, nc, Ct,
                              valid, r, xt, ax, fx, fy, fz);
      if (kLevels == 2) {
        const uint64_t m = __ballot(op);
        if (lane == i) {
          open_lo = (uint32_t)m;
          open_hi = (uint32_t)(m >> 32);
        }
      } else if (__any(op)) {
        ff_direct<kUniform>(top[c].start, top[c].count, c, recs, lds, op, kj, kp, jj, pj, xt, ax,
                            dx, dy, dz);
      }
    }
    if (kLevels == 1) continue;
    // lane: child lane & 7 of the group's cell lane >> 3
    const int f0 = (c0 + (lane >> 3) * step) * 8 + (lane & 7);
    cls = kEmpty;
    if (__shfl((int)(open_lo | open_hi), lane >> 3) != 0) cls = ff_class(cells0 + f0, box, ax, K);
    for (uint64_t todo = __ballot(cls != kEmpty); todo; todo &= todo - 1) {
      const int i = __ffsll((unsigned long long)todo) - 1;
      const int f = (c0 + (i >> 3) * step) * 8 + (i & 7);
      const uint64_t m = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)open_lo, i >> 3) |
                         (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)open_hi, i >> 3) << 32;
      const bool near = ff_take(cells0, f, __builtin_amdgcn_readlane(cls, i), K, i, sdel0, pre0,
                                nc, ax.C[0], (m >> lane) & 1u, r, xt, ax, fx, fy, fz);
      if (__any(near))
        ff_direct<kUniform>(cells0[f].start, cells0[f].count, f, recs, lds, near, kj, kp, jj, pj,
                            xt, ax, dx, dy, dz);
    }
  }
  if (kUniform) {
    fx = fmaf(dx, ax.qf, fx);
    fy = fmaf(dy, ax.qf, fy);
    fz = fmaf(dz, ax.qf, fz);
  } else {
    fx += dx;
    fy += dy;
    fz += dz;
  }
  if (valid) {
    float* out = Pout + (long long)blockIdx.y * 3 * nc;
    out[j] = fx;
    out[nc + j] = fy;
    out[2 * nc + j] = fz;
  }
}

// v[j][a] = scale * (sum over the S chunk partials of target j, in chunk
// order, in FP64); a thread per component.
__global__ void k_ff_sum(const float* __restrict__ P, int S, int n, double scale,
                         double* __restrict__ v) {
  const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= 3LL * n) return;
  double t = 0.0;
#pragma unroll 8
  for (int c = 0; c < S; ++c) t += (double)P[3LL * c * n + q];
  const int a = (int)(q / n);
  v[3 * (q - (long long)a * n) + a] = t * scale;
}

FfAxes ff_axes(const vlb_bs_desc* d, const vlb_ff_params* p) {
  FfAxes ax{};
  const int nn[3] = {d->nx, d->ny, d->nz};
  ax.levels = p->levels == 2 ? 2 : 1;
  bool uniform = true;
  for (int a = 0; a < 3; ++a) {
    ax.L[a] = (double)nn[a];
    ax.q[a] = 4294967296.0 / (double)nn[a];
    ax.iqf[a] = (float)((double)nn[a] / 4294967296.0);
    ax.nc[0][a] = nn[a] / p->cell;
    ax.nc[1][a] = ax.levels == 2 ? nn[a] / (2 * p->cell) : 0;
    uniform = uniform && nn[a] == nn[0];
  }
  // one grid step for all axes: equal power-of-two lengths
  int ex = 0;
  uniform = uniform && std::frexp((double)nn[0], &ex) == 0.5;
  ax.uniform = uniform ? 1 : 0;
  ax.qf = (float)ax.q[0];
  ax.h[0] = (double)p->cell;
  ax.h[1] = 2.0 * p->cell;
  ax.th2 = p->theta * p->theta;
  for (int l = 0; l < 2; ++l) ax.C[l] = ax.nc[l][0] * ax.nc[l][1] * ax.nc[l][2];
  return ax;
}

// Chunks of the coarsest cells: about 8192 blocks over the target blocks (a
// 256^3 tangle of 1e5 points: 21; with 4096 blocks its sum takes 4% longer,
// with 16384 the same), at most a chunk per cell and 64 chunks.  Few points
// need the short chunks: 3637 points over 90 cells take 137 us with 64 chunks
// and 167 us with 22 (22118 points over 324 cells: 473 us with 64 chunks, 481
// us with 95).
int ff_chunks(long long n, int Ctop) {
  const long long tb = (n + kFfTargets - 1) / kFfTargets;
  long long S = (8192 + tb - 1) / tb;
  if (S > Ctop) S = Ctop;
  if (S > 64) S = 64;
  if (S < 1) S = 1;
  return (int)S;
}

struct FfBufs {
  int32_t* cnt;
  double* Pw;
  uint32_t* X;
  int32_t* nxt;
  int32_t* prv;
  double* M;
  double* D;
  uint32_t* ka;
  uint32_t* kb;
  int32_t* va;
  int32_t* vb;
  int32_t* kidx;
  void* stmp;
  FfSeg* recs;
  double* comps;  // per segment, one level at a time
  double* srad;
  FfCell* cells[2];
  int32_t* sdel[2];
  int32_t* sidx[2];
  float* pre[2];
  float* P;
  int S;
};

// Workspace of the sum for n points (the capacity in a run).  solo: the
// stand-alone call, which also needs the sanitised links, the point count
// and its own chunk partials (a run has its own and writes into its
// Biot-Savart partials).
size_t ff_layout(long long n, const FfAxes& ax, bool solo, char* base, FfBufs* b) {
  size_t off = 0;
  auto take = [&](size_t bytes) -> void* {
    off = (off + 255) / 256 * 256;
    void* q = base ? base + off : nullptr;
    off += bytes;
    return q;
  };
  FfBufs s{};
  s.S = ff_chunks(n, ax.C[ax.levels - 1]);
  if (solo) {
    s.cnt = (int32_t*)take(32 * sizeof(int32_t));
    s.nxt = (int32_t*)take((size_t)n * sizeof(int32_t));
    s.prv = (int32_t*)take((size_t)n * sizeof(int32_t));
  }
  s.Pw = (double*)take(3 * (size_t)n * sizeof(double));
  s.X = (uint32_t*)take(3 * (size_t)n * sizeof(uint32_t));
  s.M = (double*)take(3 * (size_t)n * sizeof(double));
  s.D = (double*)take(3 * (size_t)n * sizeof(double));
  s.ka = (uint32_t*)take((size_t)n * sizeof(uint32_t));
  s.kb = (uint32_t*)take((size_t)n * sizeof(uint32_t));
  s.va = (int32_t*)take((size_t)n * sizeof(int32_t));
  s.vb = (int32_t*)take((size_t)n * sizeof(int32_t));
  s.kidx = (int32_t*)take((size_t)n * sizeof(int32_t));
  s.stmp = take(sort_tmp_bytes(n));
  s.recs = (FfSeg*)take((size_t)n * sizeof(FfSeg));
  s.comps = (double*)take((size_t)n * kMom * sizeof(double));
  s.srad = (double*)take((size_t)n * sizeof(double));
  for (int l = 0; l < ax.levels; ++l) {
    const size_t C = (size_t)ax.C[l];
    s.cells[l] = (FfCell*)take(C * sizeof(FfCell));
    s.sdel[l] = (int32_t*)take(3 * (size_t)n * sizeof(int32_t));
    s.sidx[l] = (int32_t*)take(3 * (size_t)n * sizeof(int32_t));
    s.pre[l] = (float*)take(3 * ((size_t)n + C) * kMom * sizeof(float));
  }
  if (ax.levels == 1) {
    s.cells[1] = s.cells[0];
    s.sdel[1] = s.sdel[0];
    s.sidx[1] = s.sidx[0];
    s.pre[1] = s.pre[0];
  }
  // (for as many chunks as a box of more cells takes, so that finer cells and
  // a second level never need less)
  if (solo) s.P = (float*)take((size_t)ff_chunks(n, 64) * 3 * n * sizeof(float));
  if (b) *b = s;
  return (off + 255) / 256 * 256;
}

// The order of a level's cells: a wave per (cell, axis) where a cell holds
// fewer than 64 points on average (4096 cells of 24: 42 us), else 4 waves (512
// cells of 195: 84 us, with one wave 240 us).
void ff_order(const FfBufs& b, const int32_t* so, long long n, const FfAxes& ax, int l,
              hipStream_t stream) {
  const auto kernel = n < 64LL * ax.C[l] ? k_ff_order<64> : k_ff_order<256>;
  const int threads = n < 64LL * ax.C[l] ? 64 : 256;
  hipLaunchKernelGGL(kernel, dim3((unsigned)(3 * ax.C[l])), dim3(threads), 0, stream, so, b.comps,
                     b.srad, b.X, n, ax, l, b.cells[l], b.sdel[l], b.sidx[l], b.pre[l]);
}

}  // namespace

int ff_check(const vlb_bs_desc* d, const vlb_ff_params* p, int64_t n, std::string& msg) {
  const int c = bs_check_desc(d, n, msg);
  if (c != VLB_OK) return c;
  if (!p) { msg = "null far-field parameters"; return VLB_EINVAL; }
  if (d->wall_axes != 0) { msg = "the far-field sum needs a periodic box (wall_axes 0)"; return VLB_EINVAL; }
  if (d->precision != VLB_F32) { msg = "the far-field sum is FP32 (precision VLB_F32)"; return VLB_EINVAL; }
  if (!(p->theta > 0.0 && p->theta < 1.0)) { msg = "theta must lie in (0, 1)"; return VLB_EINVAL; }
  if (p->levels < 0 || p->levels > 2) { msg = "levels must be 0, 1 or 2"; return VLB_EINVAL; }
  const int top = p->levels == 2 ? 2 * p->cell : p->cell;
  if (p->cell < 1 || d->nx % top || d->ny % top || d->nz % top) {
    msg = p->levels == 2 ? "the cell edge must be >= 1 and twice the cell edge divide nx, ny and nz"
                         : "the cell edge must be >= 1 and divide nx, ny and nz";
    return VLB_EINVAL;
  }
  const long long C = (long long)(d->nx / p->cell) * (d->ny / p->cell) * (d->nz / p->cell);
  if (C > (1LL << 22)) { msg = "more than 2^22 cells"; return VLB_EINVAL; }
  return VLB_OK;
}

size_t ff_workspace(const vlb_bs_desc* d, const vlb_ff_params* p, long long n) {
  return ff_layout(n, ff_axes(d, p), true, nullptr, nullptr);
}

hipError_t ff_solo(const vlb_bs_desc* d, const vlb_ff_params* p, long long n, const double* xyz,
                   const int32_t* next, double* v, void* ws, hipStream_t stream) {
  const FfAxes ax = ff_axes(d, p);
  FfBufs b;
  ff_layout(n, ax, true, (char*)ws, &b);
  const int nb = (int)((n + 255) / 256);
  hipLaunchKernelGGL(k_ff_init, dim3(nb), dim3(256), 0, stream, b.prv, (int)n);
  hipLaunchKernelGGL(k_ff_prep, dim3(nb), dim3(256), 0, stream, xyz, next, (int)n, ax, b.cnt, b.Pw,
                     b.X, b.nxt, b.prv, b.M, b.D, b.ka, b.kidx, b.va);
  int bits = 1;
  while ((1LL << bits) < ax.C[0]) ++bits;
  uint32_t* sk = nullptr;
  int32_t* so = nullptr;
  hipError_t e = sort_pairs(n, bits, b.stmp, b.ka, b.kb, b.va, b.vb, stream, &sk, &so);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_ff_seg, dim3(nb), dim3(256), 0, stream, so, b.X, b.nxt, b.cnt, n, ax,
                     b.recs);
  for (int l = 0; l < ax.levels; ++l) {
    const int C = ax.C[l];
    hipLaunchKernelGGL(k_ff_bounds, dim3((C + 255) / 256), dim3(256), 0, stream, sk, (int)n, C,
                       3 * l, b.cells[l]);
    hipLaunchKernelGGL(k_ff_comps, dim3(nb), dim3(256), 0, stream, b.M, b.D, b.kidx, b.cnt, n,
                       ax, l, b.comps, b.srad);
    ff_order(b, so, n, ax, l, stream);
  }
  const dim3 grid((unsigned)((n + kFfTargets - 1) / kFfTargets), b.S);
#define FF_EVAL(U, LV)                                                                         \
  hipLaunchKernelGGL((k_ff_eval<U, LV>), grid, dim3(256), 0, stream, b.cells[0], b.cells[1],   \
                     b.recs, so, b.kidx, b.prv, b.Pw, b.X, b.sdel[0], b.sdel[1], b.pre[0],     \
                     b.pre[1], b.cnt, n, b.S, ax, b.P)
  if (ax.uniform) {
    if (ax.levels == 2) FF_EVAL(true, 2); else FF_EVAL(true, 1);
  } else {
    if (ax.levels == 2) FF_EVAL(false, 2); else FF_EVAL(false, 1);
  }
#undef FF_EVAL
  hipLaunchKernelGGL(k_ff_sum, dim3((unsigned)((3 * n + 255) / 256)), dim3(256), 0, stream, b.P, b.S, (int)n,
                     d->kappa / (4.0 * M_PI), v);
  return hipGetLastError();
}

namespace {

FfAxes ff_run_axes(const Run& r) {
  const vlb_bs_desc bd{r.lat.nx, r.lat.ny, r.lat.nz, 0u, VLB_F32, 0, r.vor.kappa};
  const vlb_ff_params fp{r.vor.ff_cell, r.vor.ff_levels, r.vor.ff_theta};
  return ff_axes(&bd, &fp);
}

}  // namespace

size_t ff_run_bytes(const Run& r) {
  return ff_layout(r.ncap, ff_run_axes(r), false, nullptr, nullptr);
}

int ff_run_chunks(const Run& r) {
  const FfAxes ax = ff_run_axes(r);
  return ff_chunks(r.ncap, ax.C[ax.levels - 1]);
}

hipError_t ff_run_sum(Run& r, const double* Y) {
  const FfAxes ax = ff_run_axes(r);
  const long long nc = r.ncap;
  hipStream_t stream = r.stream;
  FfBufs b;
  ff_layout(nc, ax, false, (char*)r.ffws, &b);
  hipEvent_t t0 = nullptr;
  time_begin(r, 0, &t0);
  const int nb = (int)((nc + 255) / 256);
  hipLaunchKernelGGL(k_ff_prep_run, dim3(nb), dim3(256), 0, stream, Y, r.nxt, r.cnt, nc, ax, b.Pw,
                     b.X, b.M, b.D, b.ka, b.kidx, b.va);
  int bits = 1;
  while ((1LL << bits) < ax.C[0]) ++bits;
  uint32_t* sk = nullptr;
  int32_t* so = nullptr;
  hipError_t e = sort_pairs(nc, bits, b.stmp, b.ka, b.kb, b.va, b.vb, stream, &sk, &so);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_ff_seg, dim3(nb), dim3(256), 0, stream, so, b.X, r.nxt, r.cnt, nc, ax,
                     b.recs);
  for (int l = 0; l < ax.levels; ++l) {
    const int C = ax.C[l];
    hipLaunchKernelGGL(k_ff_bounds, dim3((C + 255) / 256), dim3(256), 0, stream, sk, (int)nc, C,
                       3 * l, b.cells[l]);
    hipLaunchKernelGGL(k_ff_comps, dim3(nb), dim3(256), 0, stream, b.M, b.D, b.kidx, r.cnt, nc,
                       ax, l, b.comps, b.srad);
    ff_order(b, so, nc, ax, l, stream);
  }
  const dim3 grid((unsigned)((nc + kFfTargets - 1) / kFfTargets), r.ffS);
#define FF_EVAL(U, LV)                                                                         \
  hipLaunchKernelGGL((k_ff_eval<U, LV>), grid, dim3(256), 0, stream, b.cells[0], b.cells[1],   \
                     b.recs, so, b.kidx, r.prv, b.Pw, b.X, b.sdel[0], b.sdel[1], b.pre[0],     \
                     b.pre[1], r.cnt, nc, r.ffS, ax, (float*)r.bsP)
  if (ax.uniform) {
    if (ax.levels == 2) FF_EVAL(true, 2); else FF_EVAL(true, 1);
  } else {
    if (ax.levels == 2) FF_EVAL(false, 2); else FF_EVAL(false, 1);
  }
#undef FF_EVAL
  time_end(r, 0, t0);
  return hipGetLastError();
}

}  // namespace vlb
