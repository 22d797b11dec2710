// Per-point filament kernels (paper Sec. II.A and II.B):
//  * finalize: sum of the Biot-Savart partials, local geometry and LIA term,
//    mass-balance superflow, two-point-delta interpolation of the normal
//    fluid, Schwarz line velocity, mutual-friction force and the RK4
//    bookkeeping of one stage;
//  * spreading of the point forces onto the lattice, without atomics on
//    the forces: the stage-1 finalize pushes every point on the list of the
//    cell of its stencil's lower corner (its bin); each touched node is then
//    owned by exactly one bin and gathers the contributions of the (at most
//    8) bins around it, each bin's points in ascending order.
#include "bs_pair.h"
#include "lbm_node.h"

#include <type_traits>

namespace vlb {

namespace {

// Spreading bins: the lattice cell of the stencil's lower corner.
struct SpreadGeom {
  int n[3];
  int wall[3];
  int ext[3];  // bins per axis: n (periodic) or n + 1 (wall: lower corner -1..n-1)
};

// floor of a coordinate as an int; 0 for a non-finite or absurd value, so
// that a position that blew up still yields an index inside the lattice
// (the non-finite line velocity is reported by its own flag)
__device__ inline int ifloor_safe(double x) {
  const double f = floor(x);
  return (f > -1.0e9 && f < 1.0e9) ? (int)f : 0;
}

__device__ inline uint32_t base_key(const SpreadGeom& sg, const double p[3], int b[3]) {
  for (int a = 0; a < 3; ++a) {
    int c = ifloor_safe(p[a]);
    if (sg.wall[a]) {
      c += 1;  // lower corner -1 .. n-1 -> 0 .. n
      c = c < 0 ? 0 : (c > sg.n[a] ? sg.n[a] : c);
    } else {
      c = ((c % sg.n[a]) + sg.n[a]) % sg.n[a];
    }
    b[a] = c;
  }
  return (uint32_t)(((long long)b[2] * sg.ext[1] + b[1]) * sg.ext[0] + b[0]);
}

SpreadGeom spread_geom(const Run& r) {
  SpreadGeom sg;
  const int n[3] = {r.geom.nx, r.geom.ny, r.geom.nz};
  for (int a = 0; a < 3; ++a) {
    sg.n[a] = n[a];
    sg.wall[a] = r.geom.wall[a];
    sg.ext[a] = n[a] + (r.geom.wall[a] ? 1 : 0);
  }
  return sg;
}

struct FinArgs {
  const void* ub;  // bare normal-fluid velocity field of the step
  Geom g;
  const double* Y;
  double* Ynext;
  double* pos;
  double* ksum;
  const int32_t* nxt;
  const int32_t* prv;
  int32_t* cnt;
  const void* P;
  int S;
  long long ncap;
  const double* Vs;
  int mass_balance;
  int mb_axis;      // flow axis of the superflow
  int stage;        // stage of the Runge-Kutta method, 1..rk
  int rk;           // stages of the method: 1, 2 or 4
  int first;        // first stage of the step's first substep: stage-1 outputs
  double h, hh;     // substep length 1/m and half of it
  int eval_only;
  int coupling;
  int force_model;  // 0: s' x (ds/dt - v_s) (Magnus balance); 1: ds/dt - v_s
  double kappa;
  double bs_scale;    // kappa / (4 pi)
  double nl_scale;    // kappa / (4 pi) times the grid step when the sum ran in grid units
  double ln2_ea;      // ln(2 / (e^C a))
  double alpha, alpha_p;
  // mutual-friction profiles along z: alpha at [0, nz), alpha' at
  // [nz, 2 nz), and at [2 nz] 1.0 when they replace the constants (read at
  // run time, so that a captured graph follows the current setting)
  const double* fric;
  double rs_rn;
  double vs_app[3];
  double* vs1;
  double* vn1;
  double* sd1;
  double* gpt;
  uint32_t* X;      // grid coordinates of the next stage's positions (FP32 sum), or null
  BsAxes ax;
  // stage 1 with spreading: per point, the bin key, the fractional stencil
  // offsets of the step's positions and its place on the bin's list (which
  // lists are empty before: the moments kernel clears them), and the point
  // count
  SpreadGeom sg;
  uint32_t* skeys;  // or null
  double* sfrac;
  int32_t* bins;    // per bin the last point pushed (-1: none)
  int32_t* bnext;   // per point the one pushed before it
};

// Nearest-image separation on the filament axes (wall axes: plain).
__device__ inline double mimg(double d, double L, int periodic) {
  if (periodic) {
    if (d > 0.5 * L)
      d = d - L;
    else if (d < -0.5 * L)
      d = d + L;
  }
  return d;
}

// Periodic axes wrap into [0, L); wall axes mirror a point that crossed
// the wall plane at -1/2 or n - 1/2.
__device__ inline double wrap_coord(double x, double L, int periodic) {
  if (periodic) {
    if (x < 0.0) x = x + L;
    if (x >= L) x = x - L;
    if (x >= L) x = 0.0;
  } else {
    const double lo = -0.5, hi = L - 0.5;
    if (x < lo) x = 2.0 * lo - x;
    if (x > hi) x = 2.0 * hi - x;
  }
  return x;
}

// Normal-fluid velocity at a point: delta_2pt weights on the 8 surrounding
// nodes of the step's bare-velocity field; nodes beyond a wall carry zero.
// All 24 loads are in flight together (a node beyond a wall reads another and
// adds nothing): with a branch around each node's loads they followed one
// another, and 20 steps of a ring of 64 points took 1220 us instead of 1140.
template <class UT>
__device__ void interp_vn(const UT* __restrict__ ub, const Geom& g, double px, double py,
                          double pz, double v[3]) {
  const double fr[3] = {px - floor(px), py - floor(py), pz - floor(pz)};
  const int ib[3] = {ifloor_safe(px), ifloor_safe(py), ifloor_safe(pz)};
  const int n[3] = {g.nx, g.ny, g.nz};
  int node[3][2];
  bool ghost[3][2];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      int c = ib[a] + s;
      const bool out = c < 0 || c >= n[a];
      ghost[a][s] = out && g.wall[a];
      if (out) c = g.wall[a] ? 0 : ((c % n[a]) + n[a]) % n[a];
      node[a][s] = c;
    }
  UT u[8][3];
#pragma unroll
  for (int o = 0; o < 8; ++o) {
    const long long c =
        ((long long)node[2][o >> 2] * g.ny + node[1][(o >> 1) & 1]) * g.nx + node[0][o & 1];
#pragma unroll
    for (int a = 0; a < 3; ++a) u[o][a] = ub[a * g.cells + c];
  }
  v[0] = v[1] = v[2] = 0.0;
#pragma unroll
  for (int o = 0; o < 8; ++o) {
    const int off[3] = {o & 1, (o >> 1) & 1, o >> 2};
    double w = 1.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) w *= off[a] ? fr[a] : 1.0 - fr[a];
    const bool in = !(ghost[0][off[0]] || ghost[1][off[1]] || ghost[2][off[2]]);
#pragma unroll
    for (int a = 0; a < 3; ++a) v[a] = in ? v[a] + w * (double)u[o][a] : v[a];
  }
}

// What waves 1 to 3 of a block find for its N points, one lane per point.
template <int N>
struct FinShared {
  double vn[3][N];   // wave 1: normal-fluid velocity
  double geo[8][N];  // wave 2: s' (3), LIA (3), real l+, l-
  int end[N];        // wave 2: wall axis of an open line's end, or -1
  double rk[9][N];   // wave 3: s^n (3), ksum (3), superflow, alpha, alpha'
};

// Wave 1 interpolates the normal-fluid velocity (and, at the step's first
// stage, pushes the point on its spreading bin), wave 2 evaluates the local
// geometry and the LIA term, wave 3 loads the RK4 state, so that these load
// chains overlap.  slot: j is below the capacity (every load is in bounds,
// non-finite values are harmless); live: j is a point.
template <class UT, int N>
__device__ __forceinline__ void fin_roles(const FinArgs& A, int grp, int lane, int j, bool slot,
                                          bool live, FinShared<N>& sh) {
  const long long nc = A.ncap;
  const Geom& g = A.g;
  const double L[3] = {(double)g.nx, (double)g.ny, (double)g.nz};
  const int per[3] = {!g.wall[0], !g.wall[1], !g.wall[2]};
  if (slot && grp == 1) {
    const double p[3] = {A.Y[j], A.Y[nc + j], A.Y[2 * nc + j]};
    double vn[3];
    int below = 0;  // the point pushed upon
    const bool push = live && A.skeys;
    if (push) {
      int b[3];
      const uint32_t key = base_key(A.sg, p, b);
      A.skeys[j] = key;
      below = atomicExch(&A.bins[key], j);
      for (int a = 0; a < 3; ++a) A.sfrac[a * nc + j] = p[a] - floor(p[a]);
    }
    interp_vn<UT>((const UT*)A.ub, g, p[0], p[1], p[2], vn);
    for (int a = 0; a < 3; ++a) sh.vn[a][lane] = vn[a];
    if (push) A.bnext[j] = below;
  }
  if (slot && grp == 2) {
    // local geometry (three-point derivatives on a non-uniform arc length)
    const int jn = min(max(A.nxt[j], 0), (int)nc - 1), jp = min(max(A.prv[j], 0), (int)nc - 1);
    double dp[3], dm[3], pj[3];
    for (int a = 0; a < 3; ++a) {
      const double pa = A.Y[a * nc + j];
      pj[a] = pa;
      dp[a] = mimg(A.Y[a * nc + jn] - pa, L[a], per[a]);
      dm[a] = mimg(pa - A.Y[a * nc + jp], L[a], per[a]);
    }
    // the lengths of the segments that exist (the line length carried)
    const double lp_real = sqrt(dp[0] * dp[0] + dp[1] * dp[1] + dp[2] * dp[2]);
    const double lm_real = sqrt(dm[0] * dm[0] + dm[1] * dm[1] + dm[2] * dm[2]);
    // An end of an open line lies on a wall plane (the lowest such closed
    // axis); the line continues into its mirror image there, so the
    // missing neighbour is the mirrored existing one: the missing segment
    // vector is the existing one with its components along the wall negated.
    int ea = -1;
    if (jn == j || jp == j)
      for (int a = 2; a >= 0; --a)
        if (!per[a] && (pj[a] == -0.5 || pj[a] == L[a] - 0.5)) ea = a;
    double lp = lp_real, lm = lm_real;
    if (ea >= 0) {
      if (jn == j) {
        for (int a = 0; a < 3; ++a) dp[a] = a == ea ? dm[a] : -dm[a];
      } else {
        for (int a = 0; a < 3; ++a) dm[a] = a == ea ? dp[a] : -dp[a];
      }
      lp = sqrt(dp[0] * dp[0] + dp[1] * dp[1] + dp[2] * dp[2]);
      lm = sqrt(dm[0] * dm[0] + dm[1] * dm[1] + dm[2] * dm[2]);
    }
    sh.end[lane] = ea;
    const double iden = 1.0 / (lp * lm * (lp + lm));
    double sp[3], spp[3];
    for (int a = 0; a < 3; ++a) {
      sp[a] = (lm * lm * dp[a] + lp * lp * dm[a]) * iden;
      spp[a] = 2.0 * (lm * dp[a] - lp * dm[a]) * iden;
    }
    const double isn = 1.0 / sqrt(sp[0] * sp[0] + sp[1] * sp[1] + sp[2] * sp[2]);
    for (int a = 0; a < 3; ++a) sp[a] *= isn;
    // LIA: beta s' x s'', beta = kappa/(4 pi) ln(2 sqrt(l+ l-) / (e^C a))
    //                          = kappa/(4 pi) (ln(l+ l-) / 2 + ln(2 / (e^C a)))
    const double beta = A.bs_scale * fma(0.5, log(lp * lm), A.ln2_ea);
    sh.geo[3][lane] = beta * (sp[1] * spp[2] - sp[2] * spp[1]);
    sh.geo[4][lane] = beta * (sp[2] * spp[0] - sp[0] * spp[2]);
    sh.geo[5][lane] = beta * (sp[0] * spp[1] - sp[1] * spp[0]);
    for (int a = 0; a < 3; ++a) sh.geo[a][lane] = sp[a];
    sh.geo[6][lane] = lp_real;
    sh.geo[7][lane] = lm_real;
  }
  if (slot && grp == 3) {
    if (!A.eval_only)
      for (int a = 0; a < 3; ++a) {
        sh.rk[a][lane] = A.pos[a * nc + j];
        sh.rk[3 + a][lane] = A.stage > 1 ? A.ksum[a * nc + j] : 0.0;
      }
    if (A.mass_balance) {
      const int ma = A.mb_axis;
      const int nm = ma == 0 ? g.nx : (ma == 1 ? g.ny : g.nz);
      const double pz = A.Y[ma * nc + j];
      const double fz = floor(pz);
      const double t = pz - fz;
      int i0 = ifloor_safe(pz), i1 = i0 + 1;
      i0 = ((i0 % nm) + nm) % nm;
      i1 = ((i1 % nm) + nm) % nm;
      sh.rk[6][lane] = (1.0 - t) * A.Vs[i0] + t * A.Vs[i1];
    }
    // mutual-friction coefficients at the point's height: the constants,
    // or the slice profiles linear between floor(z) and floor(z) + 1
    // (periodic z wraps; a wall z axis extends its end values)
    double al = A.alpha, alp = A.alpha_p;
    if (A.fric[2 * g.nz] != 0.0) {
      const double pz = A.Y[2 * nc + j];
      const double t = pz - floor(pz);
      int i0 = ifloor_safe(pz), i1 = i0 + 1;
      if (g.wall[2]) {
        i0 = min(max(i0, 0), g.nz - 1);
        i1 = min(max(i1, 0), g.nz - 1);
      } else {
        i0 = ((i0 % g.nz) + g.nz) % g.nz;
        i1 = ((i1 % g.nz) + g.nz) % g.nz;
      }
      al = (1.0 - t) * A.fric[i0] + t * A.fric[i1];
      alp = (1.0 - t) * A.fric[g.nz + i0] + t * A.fric[g.nz + i1];
    }
    sh.rk[7][lane] = al;
    sh.rk[8][lane] = alp;
  }
}

// The rest of a stage for live point j from its non-local velocity vs.
template <int N>
__device__ __forceinline__ void fin_combine(const FinArgs& A, int lane, int j, double vs[3],
                                            const FinShared<N>& sh) {
  const long long nc = A.ncap;
  const Geom& g = A.g;
  const double L[3] = {(double)g.nx, (double)g.ny, (double)g.nz};
  const int per[3] = {!g.wall[0], !g.wall[1], !g.wall[2]};
  double sp[3];
  for (int a = 0; a < 3; ++a) {
    sp[a] = sh.geo[a][lane];
    vs[a] += sh.geo[3 + a][lane];
  }
  const double lp = sh.geo[6][lane], lm = sh.geo[7][lane];
  for (int a = 0; a < 3; ++a) vs[a] += A.vs_app[a];
  if (A.mass_balance) vs[A.mb_axis] += sh.rk[6][lane];

  // normal-fluid velocity at the point
  const double vn[3] = {sh.vn[0][lane], sh.vn[1][lane], sh.vn[2][lane]};

  // Schwarz equation of motion (Sec. II.A, Eq. E of M)
  const double w[3] = {vn[0] - vs[0], vn[1] - vs[1], vn[2] - vs[2]};
  const double sxw[3] = {sp[1] * w[2] - sp[2] * w[1], sp[2] * w[0] - sp[0] * w[2],
                         sp[0] * w[1] - sp[1] * w[0]};
  const double ssw[3] = {sp[1] * sxw[2] - sp[2] * sxw[1], sp[2] * sxw[0] - sp[0] * sxw[2],
                         sp[0] * sxw[1] - sp[1] * sxw[0]};
  const double al = sh.rk[7][lane], alp = sh.rk[8][lane];
  double sd[3];
  for (int a = 0; a < 3; ++a) sd[a] = vs[a] + al * sxw[a] - alp * ssw[a];
  // an open line's end slides on its wall: no velocity normal to it
  const int ea = sh.end[lane];
  if (ea >= 0) sd[ea] = 0.0;
  if (!(isfinite(sd[0]) && isfinite(sd[1]) && isfinite(sd[2])))
    atomicOr(&A.cnt[7], kFlagNumeric);

  if (A.first) {
    for (int a = 0; a < 3; ++a) {
      A.vs1[a * nc + j] = vs[a];
      A.vn1[a * nc + j] = vn[a];
      A.sd1[a * nc + j] = sd[a];
    }
    // reaction on the normal fluid (Magnus balance), per point, with the
    // line length (l+ + l-)/2 carried by the point (the real segments)
    const double r[3] = {sd[0] - vs[0], sd[1] - vs[1], sd[2] - vs[2]};
    const double sxr[3] = {sp[1] * r[2] - sp[2] * r[1], sp[2] * r[0] - sp[0] * r[2],
                           sp[0] * r[1] - sp[1] * r[0]};
    const double dxi = 0.5 * (lp + lm);
    for (int a = 0; a < 3; ++a) {
      const double w = A.force_model ? r[a] : sxr[a];  // literal reading: for ablation
      A.gpt[a * nc + j] = A.coupling ? A.rs_rn * A.kappa * w * dxi : 0.0;
    }
  }
  if (A.eval_only) return;

  // Runge-Kutta over a substep of length h from s0 (the substep's start):
  // classical (4 stages): ksum = k1 + 2 k2 + 2 k3 + k4, stage positions
  // s0 + (h/2) k1, s0 + (h/2) k2, s0 + h k3, result s0 + h ksum / 6;
  // midpoint (2): s0 + (h/2) k1, result s0 + h k2; Euler (1): s0 + h k1
  for (int a = 0; a < 3; ++a) {
    const double s0 = sh.rk[a][lane];
    const double kp = sh.rk[3 + a][lane];
    double ks = sd[a];
    double y;
    if (A.rk == 4) {
      switch (A.stage) {
        case 1:
          y = s0 + A.hh * sd[a];
          break;
        case 2:
          ks = kp + 2.0 * sd[a];
          y = s0 + A.hh * sd[a];
          break;
        case 3:
          ks = kp + 2.0 * sd[a];
          y = s0 + A.h * sd[a];
          break;
        default:
          ks = kp + sd[a];
          y = s0 + A.h * (ks / 6.0);
          break;
      }
    } else if (A.rk == 2 && A.stage == 1) {
      y = s0 + A.hh * sd[a];
    } else {
      y = s0 + A.h * sd[a];
    }
    A.ksum[a * nc + j] = ks;
    const double yw = wrap_coord(y, L[a], per[a]);
    A.Ynext[a * nc + j] = yw;
    if (A.X) {
      const double sgrid = floor((yw + A.ax.off[a]) * A.ax.q[a]);
      A.X[a * nc + j] = A.ax.periodic[a] ? (uint32_t)(long long)sgrid : (uint32_t)(int)(long long)sgrid;
    }
  }
}

// 64 points per block of kFinWaves waves.  The waves add the Biot-Savart
// chunk partials of the block's points (wave g takes chunks g, g + kFinWaves,
// ..., eight chunks' loads in flight at a time); before its share, each wave
// but the first has its own role (fin_roles).  Wave 0 then combines the parts
// in a fixed order and does the rest per point.
constexpr int kFinPts = 64;
constexpr int kFinWaves = 4;

template <class UT, class PT>
__global__ __launch_bounds__(kFinWaves * 64) void k_finalize(FinArgs A) {
  __shared__ double red[kFinWaves - 1][3][kFinPts];  // chunk sums of waves 1..kFinWaves-1
  __shared__ FinShared<kFinPts> sh;
  const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
  const int j = blockIdx.x * kFinPts + lane;
  const int n = A.cnt[0];
  const bool live = j < n;
  const long long nc = A.ncap;
  // The loads do not wait for the point count: every slot below the
  // capacity is read (indices clamped into the arrays, non-finite values
  // harmless), and only live points write.
  const bool slot = j < nc;
  // the first batch of this wave's Biot-Savart chunk partials (chunks grp,
  // grp + kFinWaves, ..., up to 8 of them; beyond S they read as zero, which
  // adds nothing), loaded before the wave's own work so that the latencies
  // overlap
  const PT* __restrict__ P = (const PT*)A.P;
  const long long jc = slot ? j : 0;  // in-bounds index for the unconditional loads
  PT v0[8][3];
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const bool ok = slot && grp + kFinWaves * u < A.S;
    const long long c = ok ? grp + kFinWaves * u : 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const PT x = P[(c * 3 + a) * nc + jc];
      v0[u][a] = ok ? x : (PT)0;
    }
  }
  if (A.skeys && blockIdx.x == 0 && threadIdx.x == 0) A.cnt[11] = n;
  fin_roles<UT>(A, grp, lane, j, slot, live, sh);

  // non-local Biot-Savart: chunk partials added in a fixed order
  double vs[3] = {0.0, 0.0, 0.0};
  if (slot) {
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int a = 0; a < 3; ++a) vs[a] += (double)v0[u][a];
    for (int s = grp + 8 * kFinWaves; s < A.S; s += 8 * kFinWaves) {
      PT v[8][3];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const bool ok = s + kFinWaves * u < A.S;
        const long long c = ok ? s + kFinWaves * u : 0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          const PT x = P[(c * 3 + a) * nc + j];
          v[u][a] = ok ? x : (PT)0;
        }
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int a = 0; a < 3; ++a) vs[a] += (double)v[u][a];
    }
  }
  if (grp > 0)
    for (int a = 0; a < 3; ++a) red[grp - 1][a][lane] = vs[a];
  __syncthreads();
  if (grp > 0 || !live) return;
  for (int a = 0; a < 3; ++a) {
    double t = vs[a];
#pragma unroll
    for (int w = 0; w < kFinWaves - 1; ++w) t += red[w][a][lane];
    vs[a] = t * A.nl_scale;
  }
  fin_combine(A, lane, j, vs, sh);
}

// ----------------------------------------------------------- spreading

// Sum of the contributions to one node of the m points of a bin's list,
// whose order depends on timing, as a fixed function of the points: up to
// kOrdered points are taken in ascending order; more are added as 64-bit
// integers in units of 2^-(62 - log2 m) of the largest (exact sums, so the
// order is irrelevant; infinities and NaNs add as they would).  Eight:
// the line velocity of 5e3 points ten to a cell takes 118 us so, 112 with four
// and 105 with sixteen, which takes 117 against 110 at twenty to a cell and 207
// against 200 at a hundred; few cells hold more than three at the remeshed
// spacing.
constexpr int kOrdered = 8;

struct BinPoint {
  const double* sfrac;
  const double* gpt;
  long long ncap;
  int q;  // the node is corner q of the bin's stencil
  __device__ void operator()(int j, double c[3]) const {
    double w = 1.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const double fr = sfrac[a * ncap + j];
      w *= ((q >> a) & 1) ? fr : 1.0 - fr;
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) c[a] = w * gpt[a * ncap + j];
  }
};

__device__ inline void add_many(int head, int m, int n, const int32_t* __restrict__ bnext,
                                const BinPoint& at, double f[3]) {
  double c[3], big[3] = {0.0, 0.0, 0.0};
  bool bad[3] = {false, false, false};
  int j = head;
  for (int k = 0; k < m && (uint32_t)j < (uint32_t)n; ++k, j = bnext[j]) {
    at(j, c);
    for (int a = 0; a < 3; ++a) {
      bad[a] = bad[a] || !isfinite(c[a]);
      big[a] = fmax(big[a], fabs(c[a]));
    }
  }
  int e[3];
  const int room = 62 - (32 - __clz(m));
  for (int a = 0; a < 3; ++a) {
    e[a] = 0;
    if (big[a] > 0.0 && !bad[a]) e[a] = room - 1 - ilogb(big[a]);
  }
  long long s[3] = {0, 0, 0};
  j = head;
  for (int k = 0; k < m && (uint32_t)j < (uint32_t)n; ++k, j = bnext[j]) {
    at(j, c);
    for (int a = 0; a < 3; ++a)
      if (!bad[a]) s[a] += __double2ll_rn(ldexp(c[a], e[a]));
  }
  for (int a = 0; a < 3; ++a)
    if (!bad[a]) f[a] += ldexp((double)s[a], -e[a]);
  if (!(bad[0] || bad[1] || bad[2])) return;
  // what is not finite decides its sum, the same in any order
  j = head;
  for (int k = 0; k < m && (uint32_t)j < (uint32_t)n; ++k, j = bnext[j]) {
    at(j, c);
    for (int a = 0; a < 3; ++a)
      if (!isfinite(c[a])) f[a] += c[a];
  }
}

// Adds to f the contributions of the points on a bin's list to the node.
__device__ __forceinline__ void add_bin(int head, int n, const int32_t* __restrict__ bnext,
                                        const BinPoint& at, double f[3]) {
  int first[kOrdered];  // the smallest indices on the list, ascending
#pragma unroll
  for (int s = 0; s < kOrdered; ++s) first[s] = 0x7fffffff;
  int m = 0;
  for (int j = head; (uint32_t)j < (uint32_t)n && m < n; j = bnext[j], ++m) {
    int v = j;
#pragma unroll
    for (int s = 0; s < kOrdered; ++s) {
      const int t = min(first[s], v);
      v = max(first[s], v);
      first[s] = t;
    }
  }
  if (m > kOrdered) {
    add_many(head, m, n, bnext, at, f);
    return;
  }
#pragma unroll
  for (int s = 0; s < kOrdered; ++s)
    if (s < m) {
      double c[3];
      at(first[s], c);
      for (int a = 0; a < 3; ++a) f[a] += c[a];
    }
}

// Corner o of the stencil of bin `me`: the node in lattice coordinates (lat)
// and bin coordinates (e); false beyond a wall.
__device__ inline bool bin_corner(uint32_t me, int o, const SpreadGeom& sg, int e[3], int lat[3]) {
  e[0] = (int)(me % (uint32_t)sg.ext[0]);
  e[1] = (int)((me / (uint32_t)sg.ext[0]) % (uint32_t)sg.ext[1]);
  e[2] = (int)(me / ((uint32_t)sg.ext[0] * (uint32_t)sg.ext[1]));
  bool inside = true;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    e[a] += (o >> a) & 1;
    if (sg.wall[a]) {
      lat[a] = e[a] - 1;
      inside = inside && lat[a] >= 0 && lat[a] < sg.n[a];
    } else {
      if (e[a] >= sg.n[a]) e[a] -= sg.n[a];
      lat[a] = e[a];
    }
  }
  return inside;
}

// Bin q around node e, whose corner q the node is; false if there is none.
__device__ inline bool bin_around(const int e[3], int q, const SpreadGeom& sg, uint32_t& key) {
  int c[3];
  bool ok = true;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    c[a] = e[a] - ((q >> a) & 1);
    if (c[a] < 0) {
      if (sg.wall[a])
        ok = false;
      else
        c[a] += sg.n[a];
    }
  }
  key = (uint32_t)(((long long)c[2] * sg.ext[1] + c[1]) * sg.ext[0] + c[0]);
  return ok;
}

// Only the point at the head of its bin's list acts: the node at a corner of
// the bin's stencil is written by the occupied bin of smallest key among the
// (up to 8) bins whose stencils contain it, which adds those bins' points in a
// fixed order.  The nodes written are listed; the next moments kernel zeroes
// them.  A wave takes a head's eight nodes together, lane (corner, bin) adding
// one bin and the eight lanes of a node then added in the order of the bins, or
// a lane per node walks the bins in turn, eight heads to a wave.
//
// What bounds it: latency (list heads, links, offsets: dependent loads).
// With a stable sort of the points by bin in place of the lists, the
// spreading was ten launches, 65 us of a served step (128x128x256, 2e3
// points); this is one of 13.  A ring of 64 points, alone on the chip: 12 us
// by lanes walking the eight bins in turn, 4.8 by waves; beside the pair
// sums of a large run the eight times more waves wait for their slots (9.4e3
// points: 27 against 33 us), so a wave has one point in small runs
// (kStagePoints) and, up to kGatherWaves points, in a gather with nothing
// beside it (the line velocity of 700 points 73 -> 65 us, of 9.4e3 196 -> 193,
// of 2e4 619 -> 621), else eight.
//
// Of a wave's eight points, kManyHeads heads at the most are taken one after
// another by the wave together: that many or fewer mean crowded bins, whose
// lists a lane would walk eight times over.  Ten steps of about 5e3 points 0.02
// apart (FP32) 3620 -> 1770 us, 0.05 apart 2010 -> 1290, 0.1 apart 1625 ->
// 1540; always together, 2e3 points 0.95 apart take 955 against 938 and the
// served steps 1.3% more.  With a line at two heads 0.05 apart takes 1515, at
// six the served steps 0.4% more.
constexpr int kManyHeads = 4;

struct GatherArgs {
  const uint32_t* skeys;
  const int32_t* bins;
  const int32_t* bnext;
  const double* sfrac;
  const double* gpt;
  int32_t* touched;
};

// One node of the bin me that point r heads, written by this lane: corner o.
template <class FT>
__device__ __forceinline__ void gather_node(int r, int o, uint32_t me, int n, const GatherArgs& s,
                                            long long ncap, const SpreadGeom& sg, long long cells,
                                            FT* __restrict__ F) {
  int32_t* const mine = s.touched + 8LL * r + o;
  int e[3], lat[3];
  if (!bin_corner(me, o, sg, e, lat)) {
    *mine = -1;
    return;
  }
  int head[8];
  bool owner = true;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    uint32_t key;
    head[q] = bin_around(e, q, sg, key) ? s.bins[key] : -1;
    owner = owner && !(head[q] >= 0 && key < me);
  }
  if (!owner) {
    *mine = -1;
    return;
  }
  double f[3] = {0.0, 0.0, 0.0};
  for (int q = 0; q < 8; ++q)
    if (head[q] >= 0) add_bin(head[q], n, s.bnext, BinPoint{s.sfrac, s.gpt, ncap, q}, f);
  const long long node = ((long long)lat[2] * sg.n[1] + lat[1]) * sg.n[0] + lat[0];
#pragma unroll
  for (int a = 0; a < 3; ++a) F[a * cells + node] = (FT)f[a];
  *mine = (int32_t)node;
}

// All eight of them, written by the wave: lane (o, q) adds bin q.
template <class FT>
__device__ __forceinline__ void gather_nodes(int r, uint32_t me, int n, const GatherArgs& s,
                                             long long ncap, const SpreadGeom& sg,
                                             long long cells, FT* __restrict__ F) {
  const int lane = threadIdx.x & 63, o = lane >> 3, q = lane & 7;
  int e[3], lat[3];
  const bool inside = bin_corner(me, o, sg, e, lat);
  uint32_t key;
  const int head = bin_around(e, q, sg, key) && inside ? s.bins[key] : -1;
  const uint64_t smaller = __ballot(head >= 0 && key < me);
  const bool owner = inside && ((smaller >> (8 * o)) & 0xffu) == 0;
  double f[3] = {0.0, 0.0, 0.0};
  if (owner && head >= 0) add_bin(head, n, s.bnext, BinPoint{s.sfrac, s.gpt, ncap, q}, f);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    double t = __shfl(f[a], 8 * o);
#pragma unroll
    for (int k = 1; k < 8; ++k) t += __shfl(f[a], 8 * o + k);
    f[a] = t;
  }
  if (q != 0) return;
  int32_t* const mine = s.touched + 8LL * r + o;
  if (!owner) {
    *mine = -1;
    return;
  }
  const long long node = ((long long)lat[2] * sg.n[1] + lat[1]) * sg.n[0] + lat[0];
#pragma unroll
  for (int a = 0; a < 3; ++a) F[a * cells + node] = (FT)f[a];
  *mine = (int32_t)node;
}

// kPts points per wave, lanes (point, corner) or the one point's.
template <class FT, int kPts>
__device__ __forceinline__ void spread_gather(long long id, const GatherArgs& s,
                                              int32_t* __restrict__ cnt, long long ncap,
                                              const SpreadGeom& sg, long long cells,
                                              FT* __restrict__ F) {
  const int lane = threadIdx.x & 63;
  const int r0 = (int)(id >> 6) * kPts;
  const int r = r0 + (kPts > 1 ? lane >> 3 : 0);
  const uint32_t me = r < ncap ? s.skeys[r] : 0u;  // (beyond the points: unused)
  const int n = cnt[11];
  if (id == 0) cnt[1] = 8 * n;
  if (r0 >= n) return;
  const bool heads = r < n && s.bins[me] == r;
  if (r < n && !heads && (kPts > 1 || lane < 8)) s.touched[8LL * r + (lane & 7)] = -1;
  if constexpr (kPts == 1) {
    if (heads) gather_nodes<FT>(r, me, n, s, ncap, sg, cells, F);  // (uniform)
  } else {
    uint64_t todo = __ballot(heads && (lane & 7) == 0);
    if (__popcll(todo) > kManyHeads) {
      if (heads) gather_node<FT>(r, lane & 7, me, n, s, ncap, sg, cells, F);
      return;
    }
    for (; todo; todo &= todo - 1) {
      const int p = __ffsll((unsigned long long)todo) - 1;
      gather_nodes<FT>(r0 + (p >> 3), (uint32_t)__builtin_amdgcn_readlane((int)me, p), n, s, ncap,
                       sg, cells, F);
    }
  }
}

// The work a stage carries, in blocks of kSideThreads (two items of 256
// threads each for the moments, whose sums keep their tree).
template <class UT, class S>
__device__ __forceinline__ void side_work(const SideWork& w, const FinArgs& A,
                                          const GatherArgs& ga, int block, double (*red)[256]) {
  const Geom& g = A.g;
  const int tid = threadIdx.x;
  if (w.kind == SideWork::kGather) {
    spread_gather<UT, 1>((long long)block * kSideThreads + tid, ga, A.cnt, A.ncap, A.sg, g.cells,
                            (UT*)w.force);
  } else if (w.kind == SideWork::kUpdate) {
    const int c = block * kSideThreads + tid;
    if (c >= (int)g.cells) return;
    const int t = c / g.nx, z = t / g.ny;
    if (w.parity == 0)
      collide_node<S, 0, false, true>((S*)w.pops, (const UT*)w.force, g, c - t * g.nx, t - z * g.ny, z);
    else
      collide_node<S, 1, false, true>((S*)w.pops, (const UT*)w.force, g, c - t * g.nx, t - z * g.ny, z);
  } else {
    const SpreadClear<UT> sc{w.clear ? A.cnt : nullptr, ga.touched, ga.skeys, (int32_t*)ga.bins,
                             (UT*)w.force};
    spread_clear(sc, g.cells, block * kSideThreads + tid, w.blocks * kSideThreads);
    const int half = tid >> 8, t = tid & 255, nt = w.bx * w.by;
    const int it = 2 * block + half;
    double uzv = 0.0;
    if (it < w.items && t < nt) {
      const int ty = t / w.bx, tx = t - ty * w.bx;
      uzv = w.parity == 0
                ? moments_item<S, UT, 0, true, false>((const S*)w.pops, g, (UT*)w.ub, it, w.parts, tx, ty, w.bx, w.by)
                : moments_item<S, UT, 1, true, false>((const S*)w.pops, g, (UT*)w.ub, it, w.parts, tx, ty, w.bx, w.by);
    }
    if (!w.Ps) return;
    red[half][t] = uzv;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
      if (t < s && t + s < nt) red[half][t] += red[half][t + s];
      __syncthreads();
    }
    if (t == 0 && it < w.items) w.Ps[it] = w.parts == 1 ? w.scale * red[half][0] : red[half][0];
  }
}

// One stage of a small run in one launch: the pair sum and the finalize of 8
// points per block.  Waves 0 to 3: thread (slice, target) adds every 32nd
// segment of the staged tiles for its target; the 32 slices are added in
// FP64 in a fixed tree.  Waves 5 to 7 meanwhile take the roles of the
// finalize (fin_roles; wave 4 has none).  Source records come from the
// positions Y (other blocks may already write the next stage's), in FP32
// too.
//
// What bounds it: latency.  A ring of 64 points spent 4.4 us in the sum, 7.9
// in the finalize and about 4 between them per stage; with the roles before
// the sum on the same waves this kernel took 10.4, this way 8.6, and 7.2 with
// no load waiting for the point count and the loads of the velocity field in
// flight together.  It pays while the chip is not filled by the sum
// (kStagePoints).
//
// Blocks from `blocks` on do the work it carries (side_work): latency bound
// as well, it costs nothing beside the stage, where the gather, the update and
// the moments took 15 us of a ring's 56 us step as launches of their own.
constexpr int kStTargets = kFewTargets;
constexpr int kStThreads = 256;  // threads of the sum

template <bool kF32, int kVar, class UT, class S>
__global__ __launch_bounds__(512) void k_stage(FinArgs A, BsPts in, BsAxes bx, SideWork side,
                                               GatherArgs ga, int blocks) {
  using Src = std::conditional_t<kF32, BsSrc, BsSrcD>;
  __shared__ Src src[kStThreads];
  __shared__ FinShared<kStTargets> sh;
  __shared__ double red[4][3][kStTargets];
  if ((int)blockIdx.x >= blocks) {
    __shared__ double sums[2][256];
    side_work<UT, S>(side, A, ga, blockIdx.x - blocks, sums);
    return;
  }
  const int n = A.cnt[0];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (A.skeys) A.cnt[11] = n;
    if (n > 2)
      *(long long*)(A.cnt + 16) += (long long)n * (n - 2) + (long long)(bx.copies - 1) * n * n;
  }
  // The loads of the first tile and of the roles do not wait for the point
  // count: slots below the capacity are read (links clamped, values beyond the
  // points unused), and a block beyond the points writes nothing.
  const int nc = (int)A.ncap;
  const int tiles = max(1, (n + kStThreads - 1) / kStThreads);
  const int j0 = blockIdx.x * kStTargets;
  const int lane = threadIdx.x & 63, grp = threadIdx.x >> 6;
  if (grp >= 4) {
    if (lane < kStTargets)
      fin_roles<UT>(A, grp - 4, lane, j0 + lane, j0 + lane < nc, j0 + lane < n, sh);
    // the barriers of the sum
    for (int t = 0; t < bx.copies * tiles; ++t) {
      __syncthreads();
      __syncthreads();
    }
    __syncthreads();
    return;
  }

  const int j = j0 + (int)threadIdx.x % kStTargets;
  bs_few<kF32, kVar, kStThreads, kStThreads>(in, n, nc, tiles, j, bx, src, red);
  if (threadIdx.x >= kStTargets || j >= n) return;
  double vs[3];
  for (int a = 0; a < 3; ++a)
    vs[a] = (((red[0][a][lane] + red[1][a][lane]) + red[2][a][lane]) + red[3][a][lane]) * A.nl_scale;
  fin_combine(A, lane, j, vs, sh);
}

template <class FT, int kPts>
__global__ __launch_bounds__(256) void k_spread_gather(GatherArgs s, int32_t* __restrict__ cnt,
                                                       long long ncap, SpreadGeom sg,
                                                       long long cells, FT* __restrict__ F) {
  spread_gather<FT, kPts>((long long)blockIdx.x * blockDim.x + threadIdx.x, s, cnt, ncap, sg,
                           cells, F);
}

inline int nblocks(long long n, int b) { return (int)((n + b - 1) / b); }

}  // namespace

namespace {

FinArgs fin_args(Run& r, int stage, int first, int last, const double* Y, double* Ynext,
                 int eval_only) {
  FinArgs A;
  A.ub = r.ub;
  A.g = r.geom;
  A.Y = Y;
  A.Ynext = Ynext;
  A.pos = r.pos;
  A.ksum = r.ksum;
  A.nxt = r.nxt;
  A.prv = r.prv;
  A.cnt = r.cnt;
  A.P = r.bsP;
  A.S = r.vor.ff_cell > 0 ? r.ffS : r.bsS * r.bsax.copies;
  A.ncap = r.ncap;
  A.Vs = r.Vs;
  A.mass_balance = r.vor.mass_balance;
  A.mb_axis = r.vor.mass_balance_axis;
  A.stage = stage;
  A.rk = r.vor.rk_stages;
  A.first = first;
  A.h = 1.0 / r.vor.vfm_substeps;
  A.hh = 0.5 * A.h;
  A.eval_only = eval_only;
  A.coupling = r.vor.coupling;
  A.kappa = r.vor.kappa;
  A.bs_scale = r.vor.kappa / (4.0 * M_PI);
  // the direct FP32 sum on a uniform grid leaves grid units; the far-field
  // sum lattice units
  A.nl_scale = (r.prec != VLB_F64 && r.bsax.uniform && r.vor.ff_cell <= 0)
                   ? A.bs_scale * r.bsax.q[0]
                   : A.bs_scale;
  A.ln2_ea = log(2.0 / (exp(r.vor.core_c) * r.vor.core_a));
  A.alpha = r.vor.alpha;
  A.alpha_p = r.vor.alpha_p;
  A.fric = r.fric;
  A.force_model = r.vor.force_model;
  A.rs_rn = r.vor.rho_s_over_rho_n;
  for (int a = 0; a < 3; ++a) A.vs_app[a] = r.vor.vs_applied[a];
  A.vs1 = r.vs1;
  A.vn1 = r.vn1;
  A.sd1 = r.sd1;
  A.gpt = r.gpt;
  // the FP32 sum of the next stage reads grid coordinates written here
  A.X = (r.prec != VLB_F64 && !last && !eval_only) ? r.bsX : nullptr;
  A.ax = r.bsax;
  A.sg = spread_geom(r);
  A.skeys = (first && r.vor.coupling) ? r.skeys : nullptr;
  A.sfrac = r.sfrac;
  A.bins = r.bins;
  A.bnext = r.bnext;
  return A;
}

GatherArgs gather_args(const Run& r) {
  return GatherArgs{r.skeys, r.bins, r.bnext, r.sfrac, r.gpt, r.touched};
}

using StageKernel = void (*)(FinArgs, BsPts, BsAxes, SideWork, GatherArgs, int);

template <int... V>
StageKernel stage_f64(int per, std::integer_sequence<int, V...>) {
  static constexpr StageKernel kern[] = {k_stage<false, V, double, double>...};
  return kern[per];
}

}  // namespace

SideWork fil_ride_gather(const Run& r) {
  SideWork w;
  w.kind = SideWork::kGather;
  w.blocks = nblocks(64 * r.ncap, kSideThreads);
  w.force = r.force;
  return w;
}

hipError_t fil_stage(Run& r, int stage, int first, int last, const double* Y, double* Ynext,
                     const SideWork& side) {
  FinArgs A = fin_args(r, stage, first, last, Y, Ynext, 0);
  A.X = nullptr;  // the next stage reads the positions
  const BsPts in{Y, r.ncap, 1, r.nxt, r.prv};
  const int nb = nblocks(r.ncap, kStTargets);
  hipEvent_t b = nullptr;
  time_begin(r, 0, &b);  // timed with the pair sums
  const BsAxes& ax = r.bsax;
  const int per = (ax.periodic[0] ? 1 : 0) | (ax.periodic[1] ? 2 : 0) | (ax.periodic[2] ? 4 : 0);
  StageKernel kern;
  if (r.prec == VLB_F64)
    kern = stage_f64(per, std::make_integer_sequence<int, 8>{});
  else if (r.prec == VLB_F32)
    kern = ax.uniform ? k_stage<true, 1, float, float> : k_stage<true, 0, float, float>;
  else
    kern = ax.uniform ? k_stage<true, 1, float, __half> : k_stage<true, 0, float, __half>;
  hipLaunchKernelGGL(kern, dim3(nb + side.blocks), dim3(2 * kStThreads), 0, r.stream, A, in, ax,
                     side, gather_args(r), nb);
  time_end(r, 0, b);
  return hipGetLastError();
}

hipError_t fil_finalize(Run& r, int stage, int first, int last, const double* Y, double* Ynext,
                        int eval_only) {
  const FinArgs A = fin_args(r, stage, first, last, Y, Ynext, eval_only);
  const int nb = nblocks(r.ncap, kFinPts);
  switch (r.prec) {
    case VLB_F64: hipLaunchKernelGGL((k_finalize<double, double>), dim3(nb), dim3(kFinWaves * 64), 0, r.stream, A); break;
    default: hipLaunchKernelGGL((k_finalize<float, float>), dim3(nb), dim3(kFinWaves * 64), 0, r.stream, A); break;
  }
  return hipGetLastError();
}

// Positions copied slot by slot (3 n_cap values): forward Euler writes its
// result beside the positions it reads and copies it back.
__global__ void k_copy_pos(const double* __restrict__ src, double* __restrict__ dst, long long n) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

hipError_t fil_copy_positions(Run& r, const double* src, double* dst) {
  const long long n = 3 * r.ncap;
  hipLaunchKernelGGL(k_copy_pos, dim3(nblocks(n, 256)), dim3(256), 0, r.stream, src, dst, n);
  return hipGetLastError();
}

namespace {

struct HostArrays {
  const double* p[4];
};

// Threads walk the values in the order of the host's arrays, so that a wave
// writes (or reads) whole lines across the bus.
__global__ __launch_bounds__(256) void k_export(HostArrays src, int k,
                                                const int32_t* __restrict__ nxt,
                                                const int32_t* __restrict__ cnt, long long nc,
                                                char* __restrict__ host, size_t bytes) {
  const int n = cnt[0];
  const uint32_t t0 = blockIdx.x * 256u + threadIdx.x, step = gridDim.x * 256u;
  if (t0 == 0) {
    ((int32_t*)host)[0] = n;
    ((int32_t*)host)[1] = cnt[7];
  }
  if (host_io_need(n, k, nxt ? 1 : 0) > bytes) return;
  double* out = (double*)(host + kHostIoHeader);
  const uint32_t per = 3u * (uint32_t)n;
  for (uint32_t q = t0; q < per * k; q += step) {
    const uint32_t m = q / per, i = q - m * per;
    const double* s = m == 0 ? src.p[0] : (m == 1 ? src.p[1] : (m == 2 ? src.p[2] : src.p[3]));
    out[q] = s[(long long)(i % 3u) * nc + i / 3u];
  }
  if (nxt)
    for (uint32_t j = t0; j < (uint32_t)n; j += step) ((int32_t*)(out + (size_t)per * k))[j] = nxt[j];
}

__global__ __launch_bounds__(256) void k_import(const char* __restrict__ host, int n, long long nc,
                                                double* __restrict__ pos,
                                                int32_t* __restrict__ nxt,
                                                int32_t* __restrict__ prv,
                                                int32_t* __restrict__ cnt) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j == 0) cnt[0] = n;
  if (j >= n) return;
  const double* xyz = (const double*)(host + kHostIoHeader);
  const int32_t* links = (const int32_t*)(xyz + 3 * (size_t)n);
#pragma unroll
  for (int a = 0; a < 3; ++a) pos[a * nc + j] = xyz[(size_t)a * n + j];
  nxt[j] = links[j];
  prv[j] = links[n + j];
}

}  // namespace

hipError_t fil_export(Run& r, const double* const* src, int k, bool links) {
  HostArrays a{};
  for (int m = 0; m < k; ++m) a.p[m] = src[m];
  long long work = k > 0 ? 3 * k * r.ncap : (links ? r.ncap : 1);
  if (work > 65536) work = 65536;
  hipLaunchKernelGGL(k_export, dim3(nblocks(work, 256)), dim3(256), 0, r.stream, a, k,
                     links ? r.nxt : nullptr, r.cnt, r.ncap, r.host, r.host_bytes);
  return hipGetLastError();
}

hipError_t fil_import(Run& r, int n) {
  hipLaunchKernelGGL(k_import, dim3(nblocks(n > 0 ? n : 1, 256)), dim3(256), 0, r.stream, r.host, n,
                     r.ncap, r.pos, r.nxt, r.prv, r.cnt);
  return hipGetLastError();
}

namespace {

constexpr long long kGatherWaves = 16384;

template <class FT>
void launch_gather(Run& r, bool waves) {
  auto kern = waves ? k_spread_gather<FT, 1> : k_spread_gather<FT, 8>;
  hipLaunchKernelGGL(kern, dim3(nblocks((waves ? 64 : 8) * r.ncap, 256)), dim3(256), 0, r.stream,
                     gather_args(r), r.cnt, r.ncap, spread_geom(r), r.cells, (FT*)r.force);
}

}  // namespace

hipError_t fil_spread(Run& r, bool alone) {
  const bool waves = r.small || (alone && r.ncap <= kGatherWaves);
  if (r.prec == VLB_F64)
    launch_gather<double>(r, waves);
  else
    launch_gather<float>(r, waves);
  return hipGetLastError();
}

}  // namespace vlb
