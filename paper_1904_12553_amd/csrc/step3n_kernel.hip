// step3n_kernel.hip -- the D3Q15 time step by node kernels (gfx950): the phi
// pass of step3d_kernel.hip, then chemical potentials and collision with one
// thread per node, phi and C passing through dense arrays.
//
// The node order of every kernel is the dense order of a plane whose rows
// are rounded up to whole cache lines (W columns), 64 nodes to a wave, so
// short or ragged rows fill the lanes (the marching kernel's tiles are 64
// columns wide), every row of stores covers whole lines, and the grid has as
// many waves as the lattice has nodes / 64.  The lanes past the end of a row
// repeat its last node and store into the padding of the row pitch.
//
// k_chem3n writes C_i of each node from the phi array (eq:N18, eq:N31b); the
// 14 neighbours come from L1 / L2.  k_step3n forms the eq:N31a gradients of
// phi and C the same way and collides.  Against the marching kernel this
// moves 2 (N - 1) words a node more (C written and read), and keeps no LDS
// rings: registers alone set the occupancy.
#include "node_math3.h"

namespace nplbm {

namespace {

constexpr int kT3n = 256;  // threads of a workgroup

// The node of a thread and how to reach its neighbours.  Blocks are numbered
// for the 8 XCDs as in the phi pass: XCD x takes the x-th contiguous eighth
// of the plane-ordered block list, so planes share an L2.
template <typename Real>
struct Node3 {
  int y, z;              // row and plane (z uniform over the workgroup)
  int x;                 // column, up to W - 1 (past nx - 1: padding)
  bool live;
  uint32_t cx[3];        // byte offsets of columns x - 1, x, x + 1
  uint32_t own;          // byte offset of column x itself, padding included
  int ry[3];             // rows y - 1, y, y + 1
  int pz[3];             // planes z - 1, z, z + 1: periodic, or mirrored at a wall
};

template <typename Real>
__device__ __forceinline__ Node3<Real> node3(const NPL_CONST DomDesc *D, int W, uint32_t nblk,
                                             uint32_t per_plane) {
  Node3<Real> n;
  constexpr uint32_t SZ = sizeof(Real);
  const int nx = D->nx, ny = D->ny, nz = D->nz;
  const bool wall = D->wall != 0;
  const uint32_t per = (nblk + 7) / 8;
  const uint32_t t = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  n.live = t < nblk;
  if (!n.live) return n;
  n.z = (int)(t / per_plane);
  const uint32_t q = (t - (uint32_t)n.z * per_plane) * kT3n + threadIdx.x;
  n.y = (int)(q / (uint32_t)W);
  n.x = (int)(q - (uint32_t)n.y * (uint32_t)W);
  n.live = n.y < ny;
  if (!n.live) return n;
  const int xs = n.x < nx ? n.x : nx - 1;
  n.own = (uint32_t)n.x * SZ;
  n.cx[0] = (uint32_t)(xs == 0 ? nx - 1 : xs - 1) * SZ;
  n.cx[1] = (uint32_t)xs * SZ;
  n.cx[2] = (uint32_t)(xs == nx - 1 ? 0 : xs + 1) * SZ;
  n.ry[0] = n.y == 0 ? ny - 1 : n.y - 1;
  n.ry[1] = n.y;
  n.ry[2] = n.y == ny - 1 ? 0 : n.y + 1;
  n.pz[0] = n.z == 0 ? (wall ? 0 : nz - 1) : n.z - 1;
  n.pz[1] = n.z;
  n.pz[2] = n.z == nz - 1 ? (wall ? nz - 1 : 0) : n.z + 1;
  return n;
}

struct Step3nArgs {
  StepArgs s;
  int32_t W;
  uint32_t nblk, per_plane;
};

template <int N, typename Real>
__global__ void __launch_bounds__(kT3n) k_chem3n(Step3nArgs a) {
  constexpr uint32_t SZ = sizeof(Real);
  const NPL_CONST DomDesc *D = (const NPL_CONST DomDesc *)a.s.doms;
  const Node3<Real> n = node3<Real>(D, a.W, a.nblk, a.per_plane);
  if (!n.live) return;
  const NPL_CONST Consts<Real> &K = *consts_of<Real>(D);
  const uint32_t pb = (uint32_t)D->ps[0] * SZ, rbf = (uint32_t)D->rsf * SZ,
                 plf = (uint32_t)D->ny * rbf;
  const Rsrc r[3] = {row_rsrc(D->phi3, plf, n.pz[0]), row_rsrc(D->phi3, plf, n.pz[1]),
                     row_rsrc(D->phi3, plf, n.pz[2])};
  uint32_t o[3][3];
#pragma unroll
  for (int j = 0; j < 3; ++j)
#pragma unroll
    for (int c = 0; c < 3; ++c) o[j][c] = (uint32_t)n.ry[j] * rbf + n.cx[c];
  const Rsrc w = row_rsrc(D->c3, plf, n.z);
  const uint32_t ow = (uint32_t)n.y * rbf + n.own;
  chem_node3<N, Real>(
      K,
      [&](int i, int dx, int dy, int dz) {
        return bld<Real>(r[dz + 1], o[dy + 1][dx + 1], (uint32_t)i * pb);
      },
      [&](int i, Real v) { bst<Real, false>(w, ow, (uint32_t)i * pb, v); });
}

// kNT: nontemporal stores of the new state, for states that do not fit the
// Infinity Cache (112^3 FP32 N = 5 326 us a step against 346 with plain
// stores); states that do are read back from it (64^3 FP32 N = 5 53 us with
// plain stores against 57, FP64 N = 3 55 against 62).
template <int N, typename Real, bool kNT>
__global__ void __launch_bounds__(kT3n) k_step3n(Step3nArgs a) {
  constexpr int M = N - 1;
  constexpr uint32_t SZ = sizeof(Real);
  const NPL_CONST DomDesc *D = (const NPL_CONST DomDesc *)a.s.doms;
  const Node3<Real> n = node3<Real>(D, a.W, a.nblk, a.per_plane);
  if (!n.live) return;
  const NPL_CONST Consts<Real> &K = *consts_of<Real>(D);
  const NPL_CONST Consts<double> &KD = *consts_of<double>(D);
  const int par = (a.s.substep + D->parity0) & 1;
  const int ny = D->ny, nz = D->nz;
  const bool wall = D->wall != 0;
  const uint32_t pb = (uint32_t)D->ps[0] * SZ;
  const uint32_t rbh = (uint32_t)D->rs[0] * SZ, rbg = (uint32_t)D->rs[1] * SZ,
                 rbp = (uint32_t)D->rs[2] * SZ, rbf = (uint32_t)D->rsf * SZ;
  const uint32_t plh = (uint32_t)ny * rbh, plg = (uint32_t)ny * rbg, plp = (uint32_t)ny * rbp,
                 plf = (uint32_t)ny * rbf;
  // bounce-back: populations that would come from beyond a wall are the
  // node's own opposite ones (uniform over the workgroup)
  const bool bS = wall && n.z == 0, bN = wall && n.z == nz - 1;

  // NS populations and previous u
  Real g[15], pu[3];
  const uint32_t op = (uint32_t)n.y * rbp + n.cx[1];
  const Rsrc rp = row_rsrc(D->prev[par], plp, n.z);
  auto pull = [&](const Rsrc (&r)[3], uint32_t rb, int k, int q0) {
    const int cx = ex3(k), cy = ey3(k), cz = ez3(k);
    const bool b = (cz == 1 && bS) || (cz == -1 && bN);
    if (b)
      return bld<Real>(r[1], (uint32_t)n.y * rb + n.cx[1], (uint32_t)(q0 + opp3(k)) * pb);
    return bld<Real>(r[1 - cz], (uint32_t)n.ry[1 - cy] * rb + n.cx[1 - cx],
                     (uint32_t)(q0 + k) * pb);
  };
  {
    const Rsrc r[3] = {row_rsrc(D->g[par], plg, n.pz[0]), row_rsrc(D->g[par], plg, n.pz[1]),
                       row_rsrc(D->g[par], plg, n.pz[2])};
#pragma unroll
    for (int k = 1; k < 15; ++k) g[k] = pull(r, rbg, k, -1);
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) pu[d] = bld<Real>(rp, op, (uint32_t)(M + d) * pb);

  // phi, C and their gradients
  Real phi[M], Cv[M];
  Sums3<Real> S = sums3_begin<N, Real>(KD);
  {
    const Rsrc rf[3] = {row_rsrc(D->phi3, plf, n.pz[0]), row_rsrc(D->phi3, plf, n.pz[1]),
                        row_rsrc(D->phi3, plf, n.pz[2])};
    const Rsrc rc[3] = {row_rsrc(D->c3, plf, n.pz[0]), row_rsrc(D->c3, plf, n.pz[1]),
                        row_rsrc(D->c3, plf, n.pz[2])};
    uint32_t o[3][3];
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int c = 0; c < 3; ++c) o[j][c] = (uint32_t)n.ry[j] * rbf + n.cx[c];
#pragma unroll
    for (int i = 0; i < M; ++i) {
      phi[i] = bld<Real>(rf[1], o[1][1], (uint32_t)i * pb);
      Cv[i] = bld<Real>(rc[1], o[1][1], (uint32_t)i * pb);
      Real gp[3], gc[3];
      grad_node3<Real>(
          [&](int dx, int dy, int dz) {
            return bld<Real>(rf[dz + 1], o[dy + 1][dx + 1], (uint32_t)i * pb);
          },
          gp);
      grad_node3<Real>(
          [&](int dx, int dy, int dz) {
            return bld<Real>(rc[dz + 1], o[dy + 1][dx + 1], (uint32_t)i * pb);
          },
          gc);
      sums3_add<Real>(K, KD, i, phi[i], Cv[i], gp, gc, S);
    }
  }

  const Rsrc rh[3] = {row_rsrc(D->h[par], plh, n.pz[0]), row_rsrc(D->h[par], plh, n.pz[1]),
                      row_rsrc(D->h[par], plh, n.pz[2])};
  const Rsrc wh = row_rsrc(D->h[par ^ 1], plh, n.z), wg = row_rsrc(D->g[par ^ 1], plg, n.z),
             wp = row_rsrc(D->prev[par ^ 1], plp, n.z);
  const uint32_t oh = (uint32_t)n.y * rbh + n.own, og = (uint32_t)n.y * rbg + n.own,
                 ow = (uint32_t)n.y * rbp + n.own;
  collide_node3<N, Real>(
      K, KD, S, g, pu,
      [&](int i, auto collide) {
        Real h[15];
#pragma unroll
        for (int k = 0; k < 15; ++k) h[k] = pull(rh, rbh, k, i * 15);
        const Real hi = bld<Real>(rp, op, (uint32_t)i * pb);
        collide(h, hi, phi[i], Cv[i]);
      },
      [&](int plane, Real v) { bst<Real, kNT>(wg, og, (uint32_t)plane * pb, v); },
      [&](int plane, Real v) { bst<Real, kNT>(wh, oh, (uint32_t)plane * pb, v); },
      [&](int plane, Real v) { bst<Real, kNT>(wp, ow, (uint32_t)plane * pb, v); });
}

template <int N, typename Real>
hipError_t launch3n(const Step3nArgs &a, bool cached, hipStream_t st) {
  const dim3 grid((a.nblk + 7) / 8 * 8);
  hipLaunchKernelGGL((k_chem3n<N, Real>), grid, dim3(kT3n), 0, st, a);
  if (cached)
    hipLaunchKernelGGL((k_step3n<N, Real, false>), grid, dim3(kT3n), 0, st, a);
  else
    hipLaunchKernelGGL((k_step3n<N, Real, true>), grid, dim3(kT3n), 0, st, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_step3n(int N, int precision, const StepArgs &s, int nx, int ny, int nz,
                         hipStream_t st) {
  Step3nArgs a{};
  a.s = s;
  const int line = 128 / (precision / 8);
  a.W = (nx + line - 1) / line * line;
  const int64_t per = ((int64_t)a.W * ny + kT3n - 1) / kT3n;
  if (per * nz > (int64_t)1 << 30) return hipErrorInvalidValue;
  a.per_plane = (uint32_t)per;
  a.nblk = (uint32_t)(per * nz);
  // both copies of the state in the Infinity Cache
  const bool cached = 2 * (int64_t)(16 * N + 1) * (precision / 8) * nx * ny * nz <= kCacheBytes;
  switch (N) {
    case 2:
      return precision == 64 ? launch3n<2, double>(a, cached, st) : launch3n<2, float>(a, cached, st);
    case 3:
      return precision == 64 ? launch3n<3, double>(a, cached, st) : launch3n<3, float>(a, cached, st);
    case 4:
      return precision == 64 ? launch3n<4, double>(a, cached, st) : launch3n<4, float>(a, cached, st);
    case 5:
      return precision == 64 ? launch3n<5, double>(a, cached, st) : launch3n<5, float>(a, cached, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace nplbm
