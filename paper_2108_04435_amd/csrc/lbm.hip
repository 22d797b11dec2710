// Normal fluid on the D3Q19 lattice (paper Sec. II.B): forced BGK
// collision and streaming in one pass, AA access pattern in a single
// structure-of-arrays population array.
//
// Memory holds deviations d_i = f_i - w_i.  An even pass reads the
// populations of a node from its own slots and writes the post-collision
// values into the opposite slots of the same node; an odd pass reads
// population i of x from slot opp(i) of x - c_i and writes the new
// population i to slot i of x + c_i, which restores the natural layout.  A
// neighbour beyond a wall is replaced by the node itself with the reflected
// slot (halfway bounce-back).  Each node's 19 slots are read and written by
// that node's thread only, so the update is in place and race-free.
#include "lbm_node.h"

// Multiplies and adds fuse only within one source expression, so that every
// variant of a kernel (even or odd pass, any addressing) rounds the same
// arithmetic the same way, whatever the surrounding control flow: a run
// resumed in the natural layout continues bit for bit.
#pragma clang fp contract(on)

namespace vlb {

namespace {

// Tiles of (bx, 256 / bx) nodes (x, y) of one z slice; hardware blocks are mapped
// so that the blocks of one XCD cover one contiguous range of tiles.  The
// grid may be smaller than the tile count (a multiple of 8): each block
// then walks tiles b, b + grid, ..., which stay on its XCD's range.  The
// tile id splits into (x tile, y tile, z) by divisions by the launch's
// tile counts.
template <class S, int P, bool NT, bool I32>
__global__ __launch_bounds__(256) void k_collide_stream(S* __restrict__ M,
                                                        const typename Store<S>::T* __restrict__ F,
                                                        Geom g, FastDiv fbx, FastDiv fby, int nblk) {
  for (int it = blockIdx.x; it < nblk; it += gridDim.x) {
    const uint32_t t = (uint32_t)xcd_remap(it, nblk);
    const uint32_t rr = fdiv(t, fbx);
    const uint32_t zq = fdiv(rr, fby);
    const int bxi = (int)(t - rr * fbx.d);
    const int byi = (int)(rr - zq * fby.d);
    const int z = (int)zq;
    const int x = bxi * blockDim.x + threadIdx.x;
    const int y = byi * blockDim.y + threadIdx.y;
    if (x < g.nx && y < g.ny) collide_node<S, P, NT, I32>(M, F, g, x, y, z);
  }
}

// FP16 storage on rows of exactly 256 nodes, periodic in x and y: one wave
// per row (z, y), four x-consecutive nodes per lane, every slot of the
// four read or written with one aligned 8-byte buffer access (2-byte
// accesses cap the pattern at about 0.71 of the HBM peak, 8-byte ones at
// about 0.77: pure-memory probes on this chip).  The lane's byte offset in
// a row is the same for all 38 accesses; rows and slabs are uniform.  The
// x-shifted directions of odd passes move one node across lanes: the
// element entering from the previous lane (or, for -x, from the next) comes
// with a one-lane rotation of the whole wave, which also wraps x
// periodically (lane 0 takes lane 63's last node).  Each slot is still read
// and written by its own node's lane only.  Odd passes of the slices next
// to z walls take the per-node path (collide_node) for the lane's four
// nodes.
__device__ inline uint32_t rot_prev(uint32_t v) {  // lane L gets lane L - 1's value (wave_ror:1)
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x13C, 0xF, 0xF, false);
}
__device__ inline uint32_t rot_next(uint32_t v) {  // lane L gets lane L + 1's value (wave_rol:1)
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x134, 0xF, 0xF, false);
}
// The lane's four nodes (halves e0..e3 in lo/hi of .x, .y) as seen one
// node to the left: [e3 of lane L - 1, e0, e1, e2]; and to the right:
// [e1, e2, e3, e0 of lane L + 1].
__device__ inline vlb_u32x2 shift_in_prev(vlb_u32x2 g) {
  const uint32_t p3 = rot_prev(g.y) >> 16;
  vlb_u32x2 o;
  o.x = (g.x << 16) | p3;
  o.y = (g.y << 16) | (g.x >> 16);
  return o;
}
__device__ inline vlb_u32x2 shift_in_next(vlb_u32x2 g) {
  const uint32_t n0 = rot_next(g.x) & 0xffffu;
  vlb_u32x2 o;
  o.x = (g.x >> 16) | (g.y << 16);
  o.y = (g.y >> 16) | (n0 << 16);
  return o;
}

template <int P, bool NT>
__global__ __launch_bounds__(256) void k_collide_rows4(__half* __restrict__ M,
                                                       const float* __restrict__ F, Geom g,
                                                       int nblk) {
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rows = g.ny * g.nz;
  const uint32_t cells32 = (uint32_t)g.cells;
  const uint32_t slab = cells32 * 2u;
  const __amdgpu_buffer_rsrc_t rs = pop_rsrc(M, 19u * slab);
  const uint32_t vo = (uint32_t)lane * 8u;  // byte offset of the lane's nodes in a row
  for (int it = blockIdx.x; it < nblk; it += gridDim.x) {
    const int row = __builtin_amdgcn_readfirstlane(xcd_remap(it, nblk) * 4 + w);
    if (row >= rows) continue;
    const int z = row / g.ny, y = row - z * g.ny;
    if (P == 1 && g.wall[2] && (z == 0 || z == g.nz - 1)) {
#pragma unroll 1
      for (int k = 0; k < 4; ++k) collide_node<__half, 1, NT, true>(M, F, g, 4 * lane + k, y, z);
      continue;
    }
    // byte offsets of the rows (y + dy, z + dz), periodic
    uint32_t ro[3][3];  // [dz + 1][dy + 1]
#pragma unroll
    for (int dz = -1; dz <= 1; ++dz)
#pragma unroll
      for (int dy = -1; dy <= 1; ++dy) {
        int zz = z + dz, yy = y + dy;
        zz = zz < 0 ? zz + g.nz : (zz >= g.nz ? zz - g.nz : zz);
        yy = yy < 0 ? yy + g.ny : (yy >= g.ny ? yy - g.ny : yy);
        ro[dz + 1][dy + 1] = (uint32_t)(zz * g.ny + yy) * 512u;
      }
    vlb_u32x2 G[19];
#pragma unroll
    for (int i = 0; i < 19; ++i) {
      if (P == 0) {
        G[i] = __builtin_bit_cast(vlb_u32x2, __builtin_amdgcn_raw_buffer_load_b64(
                                                 rs, vo, (uint32_t)i * slab + ro[1][1], NT ? 2 : 0));
      } else {
        // slot opp(i) of x - c_i
        const vlb_u32x2 v = __builtin_bit_cast(
            vlb_u32x2, __builtin_amdgcn_raw_buffer_load_b64(
                           rs, vo, (uint32_t)opp(i) * slab + ro[1 - cz(i)][1 - cy(i)], NT ? 2 : 0));
        G[i] = cx(i) == 1 ? shift_in_prev(v) : (cx(i) == -1 ? shift_in_next(v) : v);
      }
    }
    const long long fo = (long long)row * 256 + 4 * lane;  // the lane's first node
    const bool pl = is_plane(g, z);
    vlb_u32x2 O[19];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float D[19];
#pragma unroll
      for (int i = 0; i < 19; ++i) {
        const uint32_t word = (k < 2) ? G[i].x : G[i].y;
        const unsigned short h = (unsigned short)((k & 1) ? (word >> 16) : (word & 0xffffu));
        D[i] = __half2float(__ushort_as_half(h));
      }
      float fx = 0.f, fy = 0.f, fz = 0.f;
      if (F) {
        fx = F[fo + k];
        fy = F[g.cells + fo + k];
        fz = F[2 * g.cells + fo + k];
      }
      __half En[19];
      collide_values<__half>(D, F != nullptr, fx, fy, fz, g, pl, En);
#pragma unroll
      for (int i = 0; i < 19; ++i) {
        const uint32_t h = (uint32_t)__half_as_ushort(En[i]);
        if (k == 0) O[i].x = h;
        else if (k == 1) O[i].x |= h << 16;
        else if (k == 2) O[i].y = h;
        else O[i].y |= h << 16;
      }
    }
#pragma unroll
    for (int i = 0; i < 19; ++i) {
      if (P == 0) {
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(vlb_u32x2, O[i]), rs, vo,
                                              (uint32_t)opp(i) * slab + ro[1][1], NT ? 2 : 0);
      } else {
        // slot i of x + c_i: the lane's group holds the values of the nodes
        // one to the left (+x) or right (-x)
        const vlb_u32x2 v = cx(i) == 1 ? shift_in_prev(O[i]) : (cx(i) == -1 ? shift_in_next(O[i]) : O[i]);
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(vlb_u32x2, v), rs, vo,
                                              (uint32_t)i * slab + ro[1 + cz(i)][1 + cy(i)],
                                              NT ? 2 : 0);
      }
    }
  }
}

template <class S>
__global__ void k_init_eq(S* __restrict__ M, const double* __restrict__ rho,
                          const double* __restrict__ u, Geom g) {
  const long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= g.cells) return;
  const double r = rho[c];
  const double ux = u[c], uy = u[g.cells + c], uz = u[2 * g.cells + c];
  const double uu = ux * ux + uy * uy + uz * uz;
#pragma unroll
  for (int i = 0; i < 19; ++i) {
    const double cu = cx(i) * ux + cy(i) * uy + cz(i) * uz;
    const double feq = wq(i) * r * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * uu);
    Store<S>::st(M + (long long)i * g.cells + c, (typename Store<S>::T)(feq - wq(i)));
  }
}

template <class S>
__global__ void k_read_fields(const S* __restrict__ M, Geom g, int parity, double* rho_out,
                              double* u_out) {
  const long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= g.cells) return;
  const int x = (int)(c % g.nx);
  const int y = (int)((c / g.nx) % g.ny);
  const int z = (int)(c / ((long long)g.nx * g.ny));
  double rho, ux, uy, uz;
  node_rho_u<S>(M, g, parity, x, y, z, rho, ux, uy, uz);
  if (rho_out) rho_out[c] = rho;
  if (u_out) {
    u_out[c] = ux;
    u_out[g.cells + c] = uy;
    u_out[2 * g.cells + c] = uz;
  }
}

template <class S>
__global__ void k_read_pops(const S* __restrict__ M, Geom g, int parity, double* f) {
  using T = typename Store<S>::T;
  const long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= g.cells) return;
  const int x = (int)(c % g.nx);
  const int y = (int)((c / g.nx) % g.ny);
  const int z = (int)(c / ((long long)g.nx * g.ny));
  T d[19];
  load_node<S>(M, g, parity, x, y, z, d);
#pragma unroll
  for (int i = 0; i < 19; ++i) f[(long long)i * g.cells + c] = wq(i) + (double)d[i];
}

// n16 words of 16 bytes, four per thread in flight (both sides 16-byte
// aligned), and the rest (< 16) bytes behind them.  What bounds it: HBM.  128 x
// 128 x 512 FP32 (638 MB read, as much written): 246 us with a value per thread
// and ordinary accesses, 190 so; below the last-level cache ordinary accesses
// are the faster ones (61x67x129 FP64, ten steps and a read: 318 against 325).
typedef uint32_t vlb_u32x4 __attribute__((ext_vector_type(4)));

template <bool NT>
__global__ __launch_bounds__(256) void k_copy16(const vlb_u32x4* __restrict__ in,
                                                vlb_u32x4* __restrict__ out, long long n16,
                                                int rest) {
  const long long b = (long long)blockIdx.x * 1024 + threadIdx.x;
  if (b < rest) ((uint8_t*)(out + n16))[b] = ((const uint8_t*)(in + n16))[b];
  vlb_u32x4 v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (b + 256 * k < n16) v[k] = NT ? __builtin_nontemporal_load(in + b + 256 * k) : in[b + 256 * k];
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (b + 256 * k < n16) {
      if (NT)
        __builtin_nontemporal_store(v[k], out + b + 256 * k);
      else
        out[b + 256 * k] = v[k];
    }
}

// The stored values (deviations in the storage format) of every node's
// populations in natural layout (population i of node c in slot i of c),
// gathered from the current AA layout.
template <class S>
__global__ void k_read_state(const S* __restrict__ M, Geom g, int parity, S* __restrict__ out) {
  const long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= g.cells) return;
  if (parity == 0) {
#pragma unroll
    for (int i = 0; i < 19; ++i) out[(long long)i * g.cells + c] = M[(long long)i * g.cells + c];
    return;
  }
  const int x = (int)(c % g.nx);
  const int y = (int)((c / g.nx) % g.ny);
  const int z = (int)(c / ((long long)g.nx * g.ny));
  Nbr nb;
  make_nbr(g, x, y, z, nb);
#pragma unroll
  for (int i = 0; i < 19; ++i) {
    const long long s = nbr_index(nb, -cx(i), -cy(i), -cz(i));
    out[(long long)i * g.cells + c] = (s >= 0) ? M[(long long)opp(i) * g.cells + s]
                                               : M[(long long)i * g.cells + c];
  }
}

template <class T>
__global__ void k_read_force(const T* __restrict__ F, long long n, double* out) {
  const long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (c < n) out[c] = F ? (double)F[c] : 0.0;
}

// Bare normal-fluid velocity u_b = sum(c f)/sum(f) of every node (velocity
// planes applied), written once per step for the interpolation onto the
// filaments, fused (flow along z) with the sum of u_z over each z slice that
// the mass-balance superflow needs (Sec. III.C, Eq. mass cons).  Item
// (z, part) is a range of y rows of slice z: the block of 256 threads walks
// it in tiles (x fastest), each thread adds its nodes' u_z in order and the
// block adds the threads in a fixed tree.  The parts depend on the lattice
// alone, so the sums do not depend on the grid, which may be narrower than
// the items.  One part per slice: Ps[z] = scale * sum is the superflow; else
// Ps[z * parts + part] the part's sum (k_mb_total adds them).  Ps is null
// without mass balance along z.
//
// What bounds it: HBM (19 populations read, three velocities written), given
// enough waves in flight: with one block per slice, 128x128x256 FP32 took
// 94 to 110 us beside the filament kernels (3.4 TB/s); parts of about
// kMomentNodes nodes take 63 (even parity) to 73 us (5.1 to 5.9 TB/s); longer
// parts (2048 nodes) fill every CU at once and hold up the filament kernels.
constexpr int kMomentNodes = 512;

inline int moment_parts(const Geom& g) {
  const long long ns = (long long)g.nx * g.ny;
  const long long p = (ns + kMomentNodes - 1) / kMomentNodes;
  return (int)(p > g.ny ? g.ny : p);
}

template <class S, class UT, int P, bool I32, bool NT>
__global__ __launch_bounds__(256) void k_moments(const S* __restrict__ M, Geom g,
                                                UT* __restrict__ ub, double scale, int parts,
                                                int items, double* __restrict__ Ps,
                                                SpreadClear<UT> sc) {
  __shared__ double red[256];
  const int tid = threadIdx.y * blockDim.x + threadIdx.x;
  const int nt = blockDim.x * blockDim.y;
  spread_clear(sc, g.cells, blockIdx.x * nt + tid, gridDim.x * nt);
  for (int hw = blockIdx.x; hw < items; hw += gridDim.x) {
    const int it = xcd_remap(hw, items);
    const double uzv = moments_item<S, UT, P, I32, NT>(M, g, ub, it, parts, threadIdx.x,
                                                       threadIdx.y, blockDim.x, blockDim.y);
    if (!Ps) continue;
    red[tid] = uzv;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
      if (tid < s && tid + s < nt) red[tid] += red[tid + s];
      __syncthreads();
    }
    if (tid == 0) Ps[it] = parts == 1 ? scale * red[0] : red[0];
    __syncthreads();  // the next item writes red
  }
}

// Mass balance along x or y (flow axis a): for each z slice and each node
// position i along a, the sum of u_a over the slice's other axis in
// ascending order (one thread per (i, z)); then for each i the slice sums
// in ascending z, Vs[i] = scale * total.  u_a is the bare velocity the
// moments kernel wrote.
template <class UT>
__global__ void k_mb_partial(const UT* __restrict__ ua, Geom g, int axis, double* __restrict__ P) {
  const int z = blockIdx.y;
  const int n = axis == 0 ? g.nx : g.ny;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const long long slice = (long long)z * g.ny * g.nx;
  double s = 0.0;
  if (axis == 0)
    for (int y = 0; y < g.ny; ++y) s += (double)ua[slice + (long long)y * g.nx + i];
  else
    for (int x = 0; x < g.nx; ++x) s += (double)ua[slice + (long long)i * g.nx + x];
  P[(long long)z * n + i] = s;
}

// Vs[i] = scale * the sum of k values P[i si + j sj] in ascending j.
__global__ void k_mb_total(const double* __restrict__ P, int k, int n, int si, int sj,
                           double scale, double* __restrict__ Vs) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double s = 0.0;
  for (int j = 0; j < k; ++j) s += P[(long long)i * si + (long long)j * sj];
  Vs[i] = scale * s;
}

// Sum of v[0..2] over the 1024 threads of a block in a fixed tree; every
// thread returns the three totals.
__device__ inline void block_sum3_1024(double v[3], double (*red)[1024]) {
  const int t = threadIdx.x;
  for (int a = 0; a < 3; ++a) red[a][t] = v[a];
  __syncthreads();
  for (int s = 512; s > 0; s >>= 1) {
    if (t < s)
      for (int a = 0; a < 3; ++a) red[a][t] += red[a][t + s];
    __syncthreads();
  }
  for (int a = 0; a < 3; ++a) v[a] = red[a][0];
  __syncthreads();
}

// Statistics of the bare velocity over each z slice (diagnostics of the
// mean flow and its fluctuations, Sec. III.C): one block of 1024 threads
// per slice; the slice mean of each component, then the sum of the squared
// deviations from that mean (the nodes' velocities are recomputed from the
// populations in the second pass).  Each thread adds its nodes in order,
// the block adds the threads in a fixed tree.  out[6 z + a] = mean of
// component a, out[6 z + 3 + a] = sum of squared deviations.
template <class S>
__global__ __launch_bounds__(1024) void k_flow_stats(const S* __restrict__ M, Geom g, int parity,
                                                    double* __restrict__ out) {
  __shared__ double red[3][1024];
  const int z = blockIdx.x;
  const long long ns = (long long)g.nx * g.ny;
  double v[3] = {0.0, 0.0, 0.0};
  for (long long k = threadIdx.x; k < ns; k += 1024) {
    double rho, u[3];
    node_rho_u<S>(M, g, parity, (int)(k % g.nx), (int)(k / g.nx), z, rho, u[0], u[1], u[2]);
    for (int a = 0; a < 3; ++a) v[a] += u[a];
  }
  block_sum3_1024(v, red);
  const double m[3] = {v[0] / (double)ns, v[1] / (double)ns, v[2] / (double)ns};
  double q[3] = {0.0, 0.0, 0.0};
  for (long long k = threadIdx.x; k < ns; k += 1024) {
    double rho, u[3];
    node_rho_u<S>(M, g, parity, (int)(k % g.nx), (int)(k / g.nx), z, rho, u[0], u[1], u[2]);
    for (int a = 0; a < 3; ++a) q[a] += (u[a] - m[a]) * (u[a] - m[a]);
  }
  block_sum3_1024(q, red);
  if (threadIdx.x == 0)
    for (int a = 0; a < 3; ++a) {
      out[6 * z + a] = m[a];
      out[6 * z + 3 + a] = q[a];
    }
}

inline int blocks_for(long long n, int b) { return (int)((n + b - 1) / b); }

// Population arrays above this size are streamed with non-temporal hints
// (the last-level cache is 256 MB; smaller lattices stay resident in it
// from one step to the next).
constexpr double kStreamBytes = 192.0 * (1 << 20);

// Grid of a lattice kernel beside longer filament kernels: two blocks per CU.
constexpr int kNarrowBlocks = 512;

template <class S>
hipError_t launch_collide(Run& r) {
  using T = typename Store<S>::T;
  const Geom& g = r.geom;
  // one x row of up to 256 nodes per block: the x-shifted accesses of odd
  // passes stay inside the block's row (measured 4% faster than 64 x 4)
  const int bx = g.nx < 256 ? g.nx : 256;
  const int by = 256 / bx;
  const int nbx = (g.nx + bx - 1) / bx;
  const int nby = (g.ny + by - 1) / by;
  const int nblk = nbx * nby * g.nz;
  // the spread force field exists once filaments were seeded into a coupled run
  const T* F = (r.vor.coupling && r.has_points) ? (const T*)r.force : nullptr;
  dim3 blk(bx, by);
  // beside the filament kernels the update runs on a narrow grid, leaving
  // most CU slots to the other stream
  int grid = nblk;
  if (r.lbm_narrow && grid > kNarrowBlocks) grid = kNarrowBlocks;
  // populations far above the last-level cache: non-temporal accesses
  const bool nt = 19.0 * (double)g.cells * sizeof(S) > kStreamBytes;
  const bool i32 = slots32<S>(g);
  if constexpr (sizeof(S) == 2) {
    // rows of 256 nodes periodic in x and y: four nodes per lane
    if (i32 && g.nx == 256 && !g.wall[0] && !g.wall[1]) {
      const int nrb = (g.ny * g.nz + 3) / 4;  // blocks of four rows
      int grid4 = nrb;
      if (r.lbm_narrow && grid4 > kNarrowBlocks) grid4 = kNarrowBlocks;
      auto k4 = r.parity == 0 ? (nt ? k_collide_rows4<0, true> : k_collide_rows4<0, false>)
                              : (nt ? k_collide_rows4<1, true> : k_collide_rows4<1, false>);
      hipLaunchKernelGGL(k4, dim3(grid4), dim3(256), 0, r.stream, (__half*)r.pops, (const float*)F,
                         g, nrb);
      return hipGetLastError();
    }
  }
  auto kern = r.parity == 0
                  ? (i32 ? (nt ? k_collide_stream<S, 0, true, true> : k_collide_stream<S, 0, false, true>)
                         : (nt ? k_collide_stream<S, 0, true, false> : k_collide_stream<S, 0, false, false>))
                  : (i32 ? (nt ? k_collide_stream<S, 1, true, true> : k_collide_stream<S, 1, false, true>)
                         : (nt ? k_collide_stream<S, 1, true, false> : k_collide_stream<S, 1, false, false>));
  hipLaunchKernelGGL(kern, dim3(grid), blk, 0, r.stream, (S*)r.pops, F, g, make_fastdiv(nbx),
                     make_fastdiv(nby), nblk);
  return hipGetLastError();
}

}  // namespace

hipError_t lbm_step(Run& r) {
  hipEvent_t b = nullptr;
  time_begin(r, 1, &b);
  hipError_t e;
  switch (r.prec) {
    case VLB_F64: e = launch_collide<double>(r); break;
    case VLB_F32: e = launch_collide<float>(r); break;
    default: e = launch_collide<__half>(r); break;
  }
  time_end(r, 1, b);
  r.parity ^= 1;
  return e;
}

hipError_t lbm_init_eq(Run& r, const double* rho, const double* u) {
  const int nb = blocks_for(r.cells, 256);
  switch (r.prec) {
    case VLB_F64:
      hipLaunchKernelGGL(k_init_eq<double>, dim3(nb), dim3(256), 0, r.stream, (double*)r.pops, rho, u, r.geom);
      break;
    case VLB_F32:
      hipLaunchKernelGGL(k_init_eq<float>, dim3(nb), dim3(256), 0, r.stream, (float*)r.pops, rho, u, r.geom);
      break;
    default:
      hipLaunchKernelGGL(k_init_eq<__half>, dim3(nb), dim3(256), 0, r.stream, (__half*)r.pops, rho, u, r.geom);
      break;
  }
  r.parity = 0;
  return hipGetLastError();
}

hipError_t lbm_read_fields(Run& r, double* rho, double* u) {
  const int nb = blocks_for(r.cells, 256);
  switch (r.prec) {
    case VLB_F64:
      hipLaunchKernelGGL(k_read_fields<double>, dim3(nb), dim3(256), 0, r.stream, (const double*)r.pops, r.geom, r.parity, rho, u);
      break;
    case VLB_F32:
      hipLaunchKernelGGL(k_read_fields<float>, dim3(nb), dim3(256), 0, r.stream, (const float*)r.pops, r.geom, r.parity, rho, u);
      break;
    default:
      hipLaunchKernelGGL(k_read_fields<__half>, dim3(nb), dim3(256), 0, r.stream, (const __half*)r.pops, r.geom, r.parity, rho, u);
      break;
  }
  return hipGetLastError();
}

hipError_t lbm_read_pops(Run& r, double* f) {
  const int nb = blocks_for(r.cells, 256);
  switch (r.prec) {
    case VLB_F64:
      hipLaunchKernelGGL(k_read_pops<double>, dim3(nb), dim3(256), 0, r.stream, (const double*)r.pops, r.geom, r.parity, f);
      break;
    case VLB_F32:
      hipLaunchKernelGGL(k_read_pops<float>, dim3(nb), dim3(256), 0, r.stream, (const float*)r.pops, r.geom, r.parity, f);
      break;
    default:
      hipLaunchKernelGGL(k_read_pops<__half>, dim3(nb), dim3(256), 0, r.stream, (const __half*)r.pops, r.geom, r.parity, f);
      break;
  }
  return hipGetLastError();
}

namespace {

// Populations in natural layout between two aligned buffers.
hipError_t copy_state(Run& r, const void* in, void* out) {
  const size_t bytes = 19 * (size_t)r.cells * elt_size(r.prec);
  const long long n16 = (long long)(bytes / 16);
  auto kern = (double)bytes > kStreamBytes ? k_copy16<true> : k_copy16<false>;
  hipLaunchKernelGGL(kern, dim3(blocks_for(n16 + 1, 1024)), dim3(256), 0, r.stream,
                     (const vlb_u32x4*)in, (vlb_u32x4*)out, n16, (int)(bytes & 15));
  return hipGetLastError();
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

// The GPU whose memory p points into, or -1.
int gpu_of(const void* p) {
  hipPointerAttribute_t at;
  if (hipPointerGetAttributes(&at, p) != hipSuccess) {
    (void)hipGetLastError();
    return -1;
  }
  return at.type == hipMemoryTypeDevice ? at.device : -1;
}

}  // namespace

// By a kernel where it may read the input, which is memory of the run's GPU;
// the runtime's copy takes memory of any kind.
hipError_t lbm_write_state(Run& r, const void* in) {
  const int gpu = gpu_of(in);
  if (aligned16(in) && gpu >= 0 && gpu == gpu_of(r.pops)) return copy_state(r, in, r.pops);
  return hipMemcpyAsync(r.pops, in, 19 * (size_t)r.cells * elt_size(r.prec),
                        hipMemcpyDeviceToDevice, r.stream);
}

hipError_t lbm_read_state(Run& r, void* out) {
  if (r.parity == 0 && aligned16(out)) return copy_state(r, r.pops, out);
  const int nb = blocks_for(r.cells, 256);
  switch (r.prec) {
    case VLB_F64:
      hipLaunchKernelGGL(k_read_state<double>, dim3(nb), dim3(256), 0, r.stream, (const double*)r.pops, r.geom, r.parity, (double*)out);
      break;
    case VLB_F32:
      hipLaunchKernelGGL(k_read_state<float>, dim3(nb), dim3(256), 0, r.stream, (const float*)r.pops, r.geom, r.parity, (float*)out);
      break;
    default:
      hipLaunchKernelGGL(k_read_state<__half>, dim3(nb), dim3(256), 0, r.stream, (const __half*)r.pops, r.geom, r.parity, (__half*)out);
      break;
  }
  return hipGetLastError();
}

hipError_t lbm_flow_stats(Run& r, double* out) {
  const int nz = r.geom.nz;
  switch (r.prec) {
    case VLB_F64:
      hipLaunchKernelGGL(k_flow_stats<double>, dim3(nz), dim3(1024), 0, r.stream, (const double*)r.pops, r.geom, r.parity, out);
      break;
    case VLB_F32:
      hipLaunchKernelGGL(k_flow_stats<float>, dim3(nz), dim3(1024), 0, r.stream, (const float*)r.pops, r.geom, r.parity, out);
      break;
    default:
      hipLaunchKernelGGL(k_flow_stats<__half>, dim3(nz), dim3(1024), 0, r.stream, (const __half*)r.pops, r.geom, r.parity, out);
      break;
  }
  return hipGetLastError();
}

hipError_t lbm_read_force(Run& r, double* out) {
  const long long n = 3 * r.cells;
  const int nb = blocks_for(n, 256);
  if (r.prec == VLB_F64)
    hipLaunchKernelGGL(k_read_force<double>, dim3(nb), dim3(256), 0, r.stream, (const double*)r.force, n, out);
  else
    hipLaunchKernelGGL(k_read_force<float>, dim3(nb), dim3(256), 0, r.stream, (const float*)r.force, n, out);
  return hipGetLastError();
}

size_t lbm_mb_doubles(const Run& r) {
  if (!r.vor.mass_balance) return 0;
  const int axis = r.vor.mass_balance_axis;
  const Geom& g = r.geom;
  return (size_t)g.nz * (axis == 0 ? g.nx : (axis == 1 ? g.ny : moment_parts(g)));
}

namespace {

template <class S, class UT>
void launch_moments(Run& r, dim3 blk, int grid, double scale, int parts, int items, double* Ps) {
  const Geom& g = r.geom;
  const SpreadClear<UT> sc{r.vor.coupling ? r.cnt : nullptr, r.touched, r.skeys, r.bins,
                           (UT*)r.force};
  const bool i32 = slots32<S>(g);
  const bool nt = i32 && 19.0 * (double)g.cells * sizeof(S) > kStreamBytes;
  auto kern = r.parity == 0 ? (nt    ? k_moments<S, UT, 0, true, true>
                               : i32 ? k_moments<S, UT, 0, true, false>
                                     : k_moments<S, UT, 0, false, false>)
                            : (nt    ? k_moments<S, UT, 1, true, true>
                               : i32 ? k_moments<S, UT, 1, true, false>
                                     : k_moments<S, UT, 1, false, false>);
  hipLaunchKernelGGL(kern, dim3(grid), blk, 0, r.stream, (const S*)r.pops, g, (UT*)r.ub, scale,
                     parts, items, Ps, sc);
}

}  // namespace

namespace {

struct MomentsPlan {
  int bx, by, parts, items;
  double scale;
  double* Ps;
};

MomentsPlan moments_plan(const Run& r) {
  const Geom& g = r.geom;
  MomentsPlan p;
  // one x row of up to 256 nodes, as the update (odd parity 76 -> 73 us
  // against rows of 64)
  p.bx = g.nx < 256 ? g.nx : 256;
  p.by = 256 / p.bx;
  if (p.by < 1) p.by = 1;
  if (p.by > g.ny) p.by = g.ny;
  p.parts = moment_parts(g);
  p.items = g.nz * p.parts;
  // flow along z: the slice sums come with the moments; along x or y: two
  // small passes over u_a afterwards
  const int axis = r.vor.mass_balance_axis;
  const int n = axis == 0 ? g.nx : (axis == 1 ? g.ny : g.nz);
  const bool mbz = r.vor.mass_balance && axis == 2;
  p.Ps = mbz ? (p.parts == 1 ? r.Vs : r.mbP) : nullptr;
  p.scale = -(1.0 / r.vor.rho_s_over_rho_n) / ((double)g.cells / n);
  return p;
}

// What the superflow needs after the moments.
hipError_t moments_after(Run& r, const MomentsPlan& p) {
  const Geom& g = r.geom;
  const int axis = r.vor.mass_balance_axis;
  const int n = axis == 0 ? g.nx : (axis == 1 ? g.ny : g.nz);
  if (p.Ps && p.parts > 1)
    hipLaunchKernelGGL(k_mb_total, dim3((n + 63) / 64), dim3(64), 0, r.stream, (const double*)r.mbP, p.parts, n, p.parts, 1, p.scale, r.Vs);
  if (r.vor.mass_balance && axis != 2) {
    const dim3 pg((n + 63) / 64, g.nz);
    if (r.prec == VLB_F64)
      hipLaunchKernelGGL(k_mb_partial<double>, pg, dim3(64), 0, r.stream, (const double*)r.ub + (long long)axis * g.cells, g, axis, r.mbP);
    else
      hipLaunchKernelGGL(k_mb_partial<float>, pg, dim3(64), 0, r.stream, (const float*)r.ub + (long long)axis * g.cells, g, axis, r.mbP);
    hipLaunchKernelGGL(k_mb_total, dim3((n + 63) / 64), dim3(64), 0, r.stream, (const double*)r.mbP, g.nz, n, 1, n, p.scale, r.Vs);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t lbm_moments(Run& r) {
  const MomentsPlan p = moments_plan(r);
  dim3 blk(p.bx, p.by);
  int grid = p.items;
  if (r.lbm_narrow && grid > kNarrowBlocks) grid = kNarrowBlocks;
  switch (r.prec) {
    case VLB_F64: launch_moments<double, double>(r, blk, grid, p.scale, p.parts, p.items, p.Ps); break;
    case VLB_F32: launch_moments<float, float>(r, blk, grid, p.scale, p.parts, p.items, p.Ps); break;
    default: launch_moments<__half, float>(r, blk, grid, p.scale, p.parts, p.items, p.Ps); break;
  }
  return moments_after(r, p);
}

bool lbm_can_ride(const Run& r) {
  switch (r.prec) {
    case VLB_F64: return slots32<double>(r.geom);
    case VLB_F32: return slots32<float>(r.geom);
    default: return slots32<__half>(r.geom);
  }
}

SideWork lbm_ride_update(Run& r) {
  SideWork w;
  w.kind = SideWork::kUpdate;
  w.parity = r.parity;
  w.blocks = blocks_for(r.cells, kSideThreads);
  w.pops = r.pops;
  w.force = (r.vor.coupling && r.has_points) ? r.force : nullptr;
  r.parity ^= 1;
  return w;
}

SideWork lbm_ride_moments(Run& r) {
  const MomentsPlan p = moments_plan(r);
  SideWork w;
  w.kind = SideWork::kMoments;
  w.parity = r.parity;
  w.blocks = (p.items + 1) / 2;
  w.pops = r.pops;
  w.ub = r.ub;
  w.force = r.force;
  w.clear = r.vor.coupling;
  w.bx = p.bx;
  w.by = p.by;
  w.parts = p.parts;
  w.items = p.items;
  w.scale = p.scale;
  w.Ps = p.Ps;
  return w;
}

hipError_t lbm_moments_after(Run& r) { return moments_after(r, moments_plan(r)); }

}  // namespace vlb
