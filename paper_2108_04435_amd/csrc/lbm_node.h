// Device code of the lattice update and of the moments, per node: shared by
// the lattice kernels (lbm.hip) and by the stages of small runs that carry
// lattice work beside them (filament.hip).
#pragma once

#include "vlb_internal.h"

// Multiplies and adds fuse only within one source expression, so that every
// variant of a kernel (even or odd pass, any addressing) rounds the same
// arithmetic the same way, whatever the surrounding control flow: a run
// resumed in the natural layout continues bit for bit.
#pragma clang fp contract(on)

namespace vlb {

// 32-bit slot offsets: the population array spans less than 4 GiB.
template <class S>
bool slots32(const Geom& g) {
  return g.cells < (1LL << 29) && 19.0 * (double)g.cells * sizeof(S) < 4294967296.0;
}

// The forced BGK collision of one node (Sec. II.B, Eqs. LBM 1-3 collapsed)
// from its 19 raw stored values D (deviations times kScale; overwritten on a
// velocity plane) and the spread force (fx, fy, fz) when has_f: the 19
// post-collision values in the storage format.  Every kernel variant calls
// this one function, so every variant rounds the update identically.
template <class S>
__device__ __forceinline__ void collide_values(typename Store<S>::T* D, bool has_f,
                                               typename Store<S>::T fx,
                                               typename Store<S>::T fy,
                                               typename Store<S>::T fz, const Geom& g,
                                               bool on_plane, S* En) {
  using T = typename Store<S>::T;
  const T kS = T(Raw<S>::kScale);
  const T kInvS = T(1) / kS;  // a power of two: exact
  T om, pref, body[3], plane[3];
  geom_params<T>(g, om, pref, body, plane);
  if (on_plane) {
#pragma unroll
    for (int i = 0; i < 19; ++i) D[i] = kS * eq_dev<T>(i, T(0), T(1), plane[0], plane[1], plane[2]);
  }
  T gx = body[0], gy = body[1], gz = body[2];
  if (has_f) {
    gx += fx;
    gy += fy;
    gz += fz;
  }
  T sD, sx, sy, sz;
  moments<T>(D, sD, sx, sy, sz);
  const T drho = kInvS * sD;
  const T rho = T(1) + drho;
  T inv;
  if constexpr (sizeof(T) == 4) {
    // hardware reciprocal refined by one Newton step (within an ulp of 1/rho)
    const T r0 = __builtin_amdgcn_rcpf(rho);
    inv = fmaf(r0, fmaf(-rho, r0, 1.0f), r0);
  } else {
    inv = T(1) / rho;
  }
  const T ux = (kInvS * sx + T(0.5) * gx) * inv;
  const T uy = (kInvS * sy + T(0.5) * gy) * inv;
  const T uz = (kInvS * sz + T(0.5) * gz) * inv;
  const T ug = ux * gx + uy * gy + uz * gz;
  // Post-collision value f - (f - f^eq)/tau + F_i with f^eq and the
  // Cheng-Li/Guo term F_i built from rho and u = (sum c f + g/2)/rho
  // (Sec. II.B, Eqs. LBM 1-3 collapsed).  It is (1 - 1/tau) d_i +
  // [d^eq_i/tau + F_i], and the bracket splits into parts even and odd in
  // c_i, shared by each pair (i, opp(i)): with cu = c_i.u and cg = c_i.g it
  // is w_i (P + Q) for i and w_i (P - Q) for opp(i),
  //   P = om (drho - 1.5 rho u.u) - 3 pref u.g + cu (4.5 om rho cu + 9 pref cg),
  //   Q = 3 om rho cu + 3 pref cg,
  // all of it times kScale, the storage scale.  Half the directional terms
  // of the direct form; it matters with FP16 storage, where the arithmetic
  // is a large share of the update.
  T Dn[19];
  {
    const T uu = ux * ux + uy * uy + uz * uz;
    const T om1 = T(1) - om;
    const T Kp = om * (drho - T(1.5) * rho * uu) - T(3) * pref * ug;
    const T a1 = T(4.5) * om * rho, a2 = T(9) * pref;
    const T b1 = T(3) * om * rho, b2 = T(3) * pref;
    Dn[0] = fma(om1, D[0], (T(wq(0)) * kS) * Kp);
#pragma unroll
    for (int k = 1; k <= 9; ++k) {
      const int i = 2 * k - 1;  // i and opp(i) = i + 1
      const T ws = T(wq(i)) * kS;
      const T cu = cdot<T>(i, ux, uy, uz);
      const T cg = cdot<T>(i, gx, gy, gz);
      const T Pk = ws * fma(cu, fma(a1, cu, a2 * cg), Kp);
      const T Qk = ws * fma(b1, cu, b2 * cg);
      Dn[i] = fma(om1, D[i], Pk + Qk);
      Dn[i + 1] = fma(om1, D[i + 1], Pk - Qk);
    }
  }
  // Values in the storage format, encoded here, before the passes'
  // addressing branches: a conversion to FP16 that the compiler fuses with
  // the last multiply-add rounds once, and it must do so in every variant.
#pragma unroll
  for (int i = 0; i < 19; ++i) En[i] = Raw<S>::enc(Dn[i]);
}

// Post-collision deviation (Sec. II.B, Eqs. LBM 1-3 collapsed):
// f''' = f - (f - f^eq)/tau + F, with f^eq and the Cheng-Li/Guo term F built
// from rho and u = (sum c f + g/2)/rho.
//
// I32: the lattice has fewer than 2^29 nodes and its population array
// spans less than 4 GiB, so a slot has a 32-bit byte offset.  With FP16
// storage, where the vector arithmetic is a large share of the update, the
// array is accessed as a raw buffer: a slot's byte offset is a per-lane part
// plus a uniform part.  Even passes use the node's own offset for all 38
// accesses and the slot's slab as the uniform part.  Odd passes of a tile
// that is periodic in x and y and has both z neighbours (a tile is one z
// slice: the choice is uniform) use nine per-lane offsets, one per (dx, dy)
// in {-1, 0, 1}^2, and the slab plus the neighbour slice as the uniform
// part, so that no access costs vector arithmetic (256^3: odd pass 626 ->
// 395 VALU instructions per wave, 308 -> 247 us).  Other tiles, and FP32
// and FP64 storage (bound by HBM, and 1-3% faster with plain global
// accesses), find each neighbour's slot (or the bounce-back slot) per lane
// from one base.
template <class S, int P, bool NT, bool I32>
__device__ __forceinline__ void collide_node(S* __restrict__ M,
                                             const typename Store<S>::T* __restrict__ F,
                                             const Geom& g, int x, int y, int z) {
  using T = typename Store<S>::T;
  const long long c = ((long long)z * g.ny + y) * g.nx + x;
  const uint32_t c32 = (uint32_t)c;
  const uint32_t cells32 = (uint32_t)g.cells;
  constexpr uint32_t kSz = sizeof(S);
  constexpr bool kBuf = I32 && sizeof(S) == 2;
  const bool fast = P == 1 && kBuf && !g.wall[0] && !g.wall[1] &&
                    (!g.wall[2] || (z > 0 && z < g.nz - 1));
  __amdgpu_buffer_rsrc_t rs;
  if (kBuf) rs = pop_rsrc(M, (uint32_t)(19ull * g.cells * kSz));

  // raw stored values (deviations times kScale)
  T D[19];
  Nbr nb;
  Nbr32 nb32;
  uint32_t off[3][3];  // [dy + 1][dx + 1]: byte offset of (x + dx, y + dy) in a slice
  uint32_t zo[3];      // [dz + 1]: byte offset of slice z + dz (periodic)
  if (P == 1 && fast) {
    const uint32_t nx = (uint32_t)g.nx, ny = (uint32_t)g.ny, nz = (uint32_t)g.nz;
    const uint32_t ux = (uint32_t)x, uy = (uint32_t)y, uz = (uint32_t)z;
    const uint32_t xo[3] = {ux == 0 ? nx - 1 : ux - 1, ux, ux + 1 == nx ? 0u : ux + 1};
    const uint32_t yo[3] = {(uy == 0 ? ny - 1 : uy - 1) * nx, uy * nx,
                            (uy + 1 == ny ? 0u : uy + 1) * nx};
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) off[a][b] = (yo[a] + xo[b]) * kSz;
    const uint32_t sl = nx * ny * kSz;
    zo[0] = (uz == 0 ? nz - 1 : uz - 1) * sl;
    zo[1] = uz * sl;
    zo[2] = (uz + 1 == nz ? 0u : uz + 1) * sl;
  } else if (P == 1) {
    if (I32)
      make_nbr32(g, x, y, z, nb32);
    else
      make_nbr(g, x, y, z, nb);
  }
  if (P == 0 && kBuf) {
    const uint32_t vo = c32 * kSz;
#pragma unroll
    for (int i = 0; i < 19; ++i) D[i] = Buf<S>::template ld<NT>(rs, vo, (uint32_t)i * cells32 * kSz);
  } else if (P == 0) {
#pragma unroll
    for (int i = 0; i < 19; ++i) D[i] = Raw<S>::template ld<NT>(M + (long long)i * g.cells + c);
  } else if (fast) {
    // slot opp(i) of x - c_i
#pragma unroll
    for (int i = 0; i < 19; ++i) {
      const uint32_t o = off[1 - cy(i)][1 - cx(i)];
      const uint32_t so = (uint32_t)opp(i) * cells32 * kSz + zo[1 - cz(i)];
      // FP64: the x-shifted loads (a wave spans five lines instead of
      // four) go through L2, where the neighbouring wave finds the shared
      // line (256^3: 0.940 -> 0.932 ms per update; no gain for FP32/FP16)
      if (NT && (sizeof(S) < 8 || cx(i) == 0))
        D[i] = Buf<S>::template ld<true>(rs, o, so);
      else
        D[i] = Buf<S>::template ld<false>(rs, o, so);
    }
  } else if (I32) {
#pragma unroll
    for (int i = 0; i < 19; ++i) {
      const int s = nbr_index32(nb32, -cx(i), -cy(i), -cz(i));
      const uint32_t e = (s >= 0) ? (uint32_t)opp(i) * cells32 + (uint32_t)s
                                  : (uint32_t)i * cells32 + c32;
      if (NT && (sizeof(S) < 8 || cx(i) == 0))
        D[i] = Raw<S>::template ld<true>(at_byte(M, e * kSz));
      else
        D[i] = Raw<S>::template ld<false>(at_byte(M, e * kSz));
    }
  } else {
#pragma unroll
    for (int i = 0; i < 19; ++i) {
      const long long s = nbr_index(nb, -cx(i), -cy(i), -cz(i));
      D[i] = (s >= 0) ? Raw<S>::template ld<NT>(M + (long long)opp(i) * g.cells + s)
                      : Raw<S>::template ld<NT>(M + (long long)i * g.cells + c);
    }
  }
  T fxv = T(0), fyv = T(0), fzv = T(0);
  if (F) {
    if (I32) {
      const uint32_t fo = c32 * (uint32_t)sizeof(T);
      fxv = *at_byte(F, fo);
      fyv = *at_byte(F + g.cells, fo);
      fzv = *at_byte(F + 2 * g.cells, fo);
    } else {
      fxv = F[c];
      fyv = F[g.cells + c];
      fzv = F[2 * g.cells + c];
    }
  }
  S En[19];
  collide_values<S>(D, F != nullptr, fxv, fyv, fzv, g, is_plane(g, z), En);
#pragma unroll
  for (int i = 0; i < 19; ++i) {
    const S dn = En[i];
    // Odd passes store to the neighbours' slots: a direction with an x
    // component stores each wave's values one element off the cache lines,
    // and those partial lines must meet their other part in L2, so only the
    // directions without an x component bypass it with non-temporal stores
    // (256^3 FP32: 7% fewer bytes written, odd pass 537 -> 460 us).
    const bool nt_st = NT && (P == 0 || cx(i) == 0);
    if (P == 0 && kBuf) {
      Buf<S>::template st<NT>(rs, c32 * kSz, (uint32_t)opp(i) * cells32 * kSz, dn);
    } else if (P == 0) {
      Raw<S>::template st_enc<NT>(M + (long long)opp(i) * g.cells + c, dn);
    } else if (fast) {
      // slot i of x + c_i
      const uint32_t o = off[1 + cy(i)][1 + cx(i)];
      const uint32_t so = (uint32_t)i * cells32 * kSz + zo[1 + cz(i)];
      if (nt_st)
        Buf<S>::template st<true>(rs, o, so, dn);
      else
        Buf<S>::template st<false>(rs, o, so, dn);
    } else if (I32) {
      const int s = nbr_index32(nb32, cx(i), cy(i), cz(i));
      const uint32_t e = (s >= 0) ? (uint32_t)i * cells32 + (uint32_t)s
                                  : (uint32_t)opp(i) * cells32 + c32;
      if (nt_st)
        Raw<S>::template st_enc<true>(at_byte(M, e * kSz), dn);
      else
        Raw<S>::template st_enc<false>(at_byte(M, e * kSz), dn);
    } else {
      const long long s = nbr_index(nb, cx(i), cy(i), cz(i));
      S* p = (s >= 0) ? M + (long long)i * g.cells + s : M + (long long)opp(i) * g.cells + c;
      if (nt_st)
        Raw<S>::template st_enc<true>(p, dn);
      else
        Raw<S>::template st_enc<false>(p, dn);
    }
  }
}

// Effective density and bare velocity of node c (velocity planes applied).
template <class S>
__device__ inline void node_rho_u(const S* M, const Geom& g, int parity, int x, int y, int z,
                                  double& rho, double& ux, double& uy, double& uz) {
  using T = typename Store<S>::T;
  if (is_plane(g, z)) {
    rho = 1.0;
    ux = g.plane_u[0];
    uy = g.plane_u[1];
    uz = g.plane_u[2];
    return;
  }
  T d[19];
  load_node<S>(M, g, parity, x, y, z, d);
  T drho, jx, jy, jz;
  moments<T>(d, drho, jx, jy, jz);
  rho = 1.0 + (double)drho;
  ux = (double)jx / rho;
  uy = (double)jy / rho;
  uz = (double)jz / rho;
}

// The same for one AA parity, with 32-bit slot offsets where the population
// array spans less than 4 GiB (I32) and non-temporal loads of all slots (NT:
// lattices above the last-level cache; 128x128x256 FP32, even parity 76 -> 63
// us).  In odd parity a wave shares the lines of the x-shifted slots with its
// neighbour, but the hint pays there too: a line velocity of 16 points, mostly
// its moments, in 256^3 FP32 342 -> 310 us, 328 with the hint on the other
// slots alone; FP16 221, 208, 216; 128x128x512 FP32 195, 181, 187; only
// 128x128x256 by itself is faster that way (117, 113, 101), and its steps are
// level (2716 against 2720 us).
template <class S, int P, bool I32, bool NT>
__device__ inline void node_u(const S* __restrict__ M, const Geom& g, int x, int y, int z,
                              double u[3]) {
  using T = typename Store<S>::T;
  if constexpr (!I32) {
    double rho;
    node_rho_u<S>(M, g, P, x, y, z, rho, u[0], u[1], u[2]);
  } else {
    if (is_plane(g, z)) {
#pragma unroll
      for (int a = 0; a < 3; ++a) u[a] = g.plane_u[a];
      return;
    }
    const uint32_t cells = (uint32_t)g.cells;
    const uint32_t c = (uint32_t)((z * g.ny + y) * g.nx + x);
    T d[19];
    if (P == 0) {
#pragma unroll
      for (int i = 0; i < 19; ++i)
        d[i] = pop_ld<S, NT>(at_byte(M + (long long)i * g.cells, c * (uint32_t)sizeof(S)));
    } else {
      Nbr32 nb;
      make_nbr32(g, x, y, z, nb);
#pragma unroll
      for (int i = 0; i < 19; ++i) {
        const int s = nbr_index32(nb, -cx(i), -cy(i), -cz(i));
        const uint32_t e = s >= 0 ? (uint32_t)opp(i) * cells + (uint32_t)s : (uint32_t)i * cells + c;
        d[i] = pop_ld<S, NT>(at_byte(M, e * (uint32_t)sizeof(S)));
      }
    }
    T drho, j[3];
    moments<T>(d, drho, j[0], j[1], j[2]);
    const double rho = 1.0 + (double)drho;
#pragma unroll
    for (int a = 0; a < 3; ++a) u[a] = (double)j[a] / rho;
  }
}

// What the previous spreading left, cleared by the moments kernel: the force
// at the nodes it wrote and the heads of the bin lists it used (it precedes
// the finalize that pushes on them).
template <class UT>
struct SpreadClear {
  const int32_t* cnt;      // null: no spreading in this run
  const int32_t* touched;  // cnt[1] nodes (-1: none)
  const uint32_t* skeys;   // cnt[11] bins
  int32_t* bins;
  UT* F;
};

// Clears it, thread t of a grid of `step`.
template <class UT>
__device__ __forceinline__ void spread_clear(const SpreadClear<UT>& sc, long long cells, int t,
                                             int step) {
  if (!sc.cnt) return;
  const int nf = sc.cnt[1], nk = sc.cnt[11];
  for (int i = t; i < nf; i += step) {
    const int node = sc.touched[i];
    if (node >= 0) {
      sc.F[node] = UT(0);
      sc.F[cells + node] = UT(0);
      sc.F[2 * cells + node] = UT(0);
    }
  }
  for (int i = t; i < nk; i += step) sc.bins[sc.skeys[i]] = -1;
}

// Item `it` of the moments (a range of rows of one z slice) for thread
// (tx, ty) of a tile (bx, by): writes its nodes' velocities, returns the sum
// of their u_z.
template <class S, class UT, int P, bool I32, bool NT>
__device__ __forceinline__ double moments_item(const S* __restrict__ M, const Geom& g,
                                               UT* __restrict__ ub, int it, int parts, int tx,
                                               int ty, int bx, int by) {
  const int rows = (g.ny + parts - 1) / parts;
  const int z = it / parts;
  const int yb = (it - z * parts) * rows, ye = min(g.ny, yb + rows);
  double uzv = 0.0;
  for (int y = yb + ty; y < ye; y += by)
    for (int x = tx; x < g.nx; x += bx) {
      double u[3];
      node_u<S, P, I32, NT>(M, g, x, y, z, u);
      const long long c = ((long long)z * g.ny + y) * g.nx + x;
#pragma unroll
      for (int a = 0; a < 3; ++a) ub[a * g.cells + c] = (UT)u[a];
      uzv += u[2];
    }
  return uzv;
}

}  // namespace vlb

#pragma clang fp contract(fast)
