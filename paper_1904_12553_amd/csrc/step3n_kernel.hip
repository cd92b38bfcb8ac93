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
//
// The 15 reads of a stencil come from the same few rows, and read singly they
// cost more than their bytes (100 x 84 x 60 FP64 N = 4: with the centre read
// in their place the two kernels took 112 us a step, not 141).  While a
// workgroup holds two rows and more (W <= 128) it therefore copies the rows
// it needs into LDS, 3 (R + 2) / R reads a node and field, and forms the
// stencils from there (k_chem3r, kRows): that lattice 187 -> 171 us a step,
// FP64 N = 3 64^3 54 -> 51, FP32 N = 3 64^3 31.6 -> 29.8, FP32 N = 5 40 x 64 x 50
// 50 -> 44.  With one row a workgroup (180 x 60 x 60, 130 x 70 x 70) the copy is
// as long as the reads it saves, and LDS leaves fewer workgroups: FP64 N = 4
// 228 -> 239 us, N = 5 FP32 172 -> 187.
// What bounds them: HBM where the state exceeds the Infinity Cache (that
// lattice: 0.73 GB a step in three passes, 4.3 TB/s), else latency.
#include "node_math3.h"

#include <algorithm>

namespace nplbm {

namespace {

constexpr int kT3n = 256;  // threads of a workgroup
static_assert(2 * kRows3Width == kT3n, "two rows to a workgroup");
constexpr int kT3r = 512;  // and of one of k_chem3r

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

// The node of a thread where a workgroup owns R whole rows of a plane (R W
// threads in use), and its place in their LDS copy.  Blocks are numbered for
// the XCDs as above.
template <typename Real>
struct Rows3 {
  Node3<Real> n;
  bool use;     // holds a column of the rows
  int ly, col;  // row and column within the workgroup
  int cx[3];    // LDS columns x - 1, x, x + 1
};

template <typename Real>
__device__ __forceinline__ Rows3<Real> rows3(const NPL_CONST DomDesc *D, int W, int R,
                                             uint32_t nblk, uint32_t per_plane) {
  Rows3<Real> q;
  constexpr uint32_t SZ = sizeof(Real);
  const int nx = D->nx, ny = D->ny, nz = D->nz;
  const bool wall = D->wall != 0;
  const uint32_t per = (nblk + 7) / 8;
  const uint32_t t = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  Node3<Real> &n = q.n;
  n.live = t < nblk;
  if (!n.live) return q;
  n.z = (int)(t / per_plane);
  const int y0 = (int)(t - (uint32_t)n.z * per_plane) * R;
  q.ly = (int)threadIdx.x / W;
  q.col = (int)threadIdx.x - q.ly * W;
  q.use = q.ly < R;
  n.x = q.col;
  n.y = y0 + q.ly;
  const int xs = n.x < nx ? n.x : nx - 1;
  q.cx[0] = xs == 0 ? nx - 1 : xs - 1;
  q.cx[1] = xs;
  q.cx[2] = xs == nx - 1 ? 0 : xs + 1;
  n.own = (uint32_t)n.x * SZ;
  for (int c = 0; c < 3; ++c) n.cx[c] = (uint32_t)q.cx[c] * SZ;
  n.ry[0] = n.y == 0 ? ny - 1 : n.y - 1;
  n.ry[1] = n.y;
  n.ry[2] = n.y == ny - 1 ? 0 : n.y + 1;
  n.pz[0] = n.z == 0 ? (wall ? 0 : nz - 1) : n.z - 1;
  n.pz[1] = n.z;
  n.pz[2] = n.z == nz - 1 ? (wall ? nz - 1 : 0) : n.z + 1;
  return q;
}

// Copies M dense fields' rows into s[(i * 3 + plane) * (R + 2) + row][W].
template <int M, typename Real>
__device__ __forceinline__ void copy_rows3(const Rows3<Real> &q, const Rsrc (&r)[3], uint32_t rbf,
                                           uint32_t pb, int ny, int W, int R, Real *s) {
  if (!q.use) return;
  for (int rr = q.ly; rr < R + 2; rr += R) {
    int y = q.n.y - q.ly - 1 + rr;
    y = y < 0 ? y + ny : (y >= ny ? y - ny : y);  // R <= ny: one turn suffices
    const uint32_t o = (uint32_t)y * rbf + q.n.own;
#pragma unroll
    for (int i = 0; i < M; ++i)
#pragma unroll
      for (int p = 0; p < 3; ++p)
        s[((i * 3 + p) * (R + 2) + rr) * W + q.col] = bld<Real>(r[p], o, (uint32_t)i * pb);
  }
}

struct Step3nArgs {
  StepArgs s;
  int32_t W, R;
  int32_t cs;  // node3_stride
  uint32_t nblk, per_plane;
};

template <int N, typename Real>
__global__ void __launch_bounds__(kT3r) k_chem3r(Step3nArgs a) {
  constexpr uint32_t SZ = sizeof(Real);
  extern __shared__ __align__(16) char lds3[];
  Real *s = (Real *)lds3;
  const NPL_CONST DomDesc *D = (const NPL_CONST DomDesc *)a.s.doms;
  const int W = a.W, R = a.R, ny = D->ny;
  const Rows3<Real> q = rows3<Real>(D, W, R, a.nblk, a.per_plane);
  if (!q.n.live) return;
  const NPL_CONST Consts<Real> &K = *consts_of<Real>(D);
  const uint32_t pb = (uint32_t)D->ps[0] * SZ, rbf = (uint32_t)D->rsf * SZ,
                 plf = (uint32_t)ny * rbf;
  const Rsrc r[3] = {row_rsrc(D->phi3, plf, q.n.pz[0]), row_rsrc(D->phi3, plf, q.n.pz[1]),
                     row_rsrc(D->phi3, plf, q.n.pz[2])};
  copy_rows3<N - 1, Real>(q, r, rbf, pb, ny, W, R, s);
  __syncthreads();
  if (!q.use || q.n.y >= ny) return;
  const uint32_t pbc = (uint32_t)a.cs * SZ, rbc = (N - 1) * pbc;
  const Rsrc w = row_rsrc(D->c3, (uint32_t)ny * rbc, q.n.z);
  const uint32_t ow = (uint32_t)q.n.y * rbc + q.n.own;
  chem_node3<N, Real>(
      K,
      [&](int i, int dx, int dy, int dz) {
        return s[((i * 3 + dz + 1) * (R + 2) + q.ly + 1 + dy) * W + q.cx[dx + 1]];
      },
      [&](int i, Real v) { bst<Real, false>(w, ow, (uint32_t)i * pbc, v); });
}

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
// Infinity Cache (112^3 FP32 N = 5, stencils not yet read through LDS: 326 us a
// step against 346 with plain stores); states that do are read back from it
// (likewise 64^3 FP32 N = 5 53 us with plain stores against 57, FP64 N = 3 55
// against 62).
template <int N, typename Real, bool kNT, bool kRows>
__global__ void __launch_bounds__(kT3n) k_step3n(Step3nArgs a) {
  constexpr int M = N - 1;
  constexpr uint32_t SZ = sizeof(Real);
  const NPL_CONST DomDesc *D = (const NPL_CONST DomDesc *)a.s.doms;
  extern __shared__ __align__(16) char lds3[];
  Real *sf = (Real *)lds3, *sc = sf + M * 3 * (a.R + 2) * a.W;
  Rows3<Real> q;
  if constexpr (kRows)
    q = rows3<Real>(D, a.W, a.R, a.nblk, a.per_plane);
  else
    q.n = node3<Real>(D, a.W, a.nblk, a.per_plane);
  const Node3<Real> &n = q.n;
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

  if constexpr (kRows) {
    const Rsrc rf[3] = {row_rsrc(D->phi3, plf, n.pz[0]), row_rsrc(D->phi3, plf, n.pz[1]),
                        row_rsrc(D->phi3, plf, n.pz[2])};
    const uint32_t pbc = (uint32_t)a.cs * SZ, rbc = M * pbc, plc = (uint32_t)ny * rbc;
    const Rsrc rc[3] = {row_rsrc(D->c3, plc, n.pz[0]), row_rsrc(D->c3, plc, n.pz[1]),
                        row_rsrc(D->c3, plc, n.pz[2])};
    copy_rows3<M, Real>(q, rf, rbf, pb, ny, a.W, a.R, sf);
    copy_rows3<M, Real>(q, rc, rbc, pbc, ny, a.W, a.R, sc);
    __syncthreads();
    if (!q.use || n.y >= ny) return;
  }
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
      Real gp[3], gc[3];
      if constexpr (kRows) {
        auto at = [&](const Real *f, int dx, int dy, int dz) {
          return f[((i * 3 + dz + 1) * (a.R + 2) + q.ly + 1 + dy) * a.W + q.cx[dx + 1]];
        };
        phi[i] = at(sf, 0, 0, 0);
        Cv[i] = at(sc, 0, 0, 0);
        grad_node3<Real>([&](int dx, int dy, int dz) { return at(sf, dx, dy, dz); }, gp);
        grad_node3<Real>([&](int dx, int dy, int dz) { return at(sc, dx, dy, dz); }, gc);
        sums3_add<Real>(K, KD, i, phi[i], Cv[i], gp, gc, S);
        continue;
      }
      phi[i] = bld<Real>(rf[1], o[1][1], (uint32_t)i * pb);
      Cv[i] = bld<Real>(rc[1], o[1][1], (uint32_t)i * pb);
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

template <int N, typename Real, bool kRows>
void launch_step3_nodes(const Step3nArgs &a, bool cached, int threads, size_t lds,
                        hipStream_t st) {
  const dim3 grid((a.nblk + 7) / 8 * 8);
  if (cached)
    hipLaunchKernelGGL((k_step3n<N, Real, false, kRows>), grid, dim3(threads), lds, st, a);
  else
    hipLaunchKernelGGL((k_step3n<N, Real, true, kRows>), grid, dim3(threads), lds, st, a);
}

template <int N, typename Real>
hipError_t launch3n(Step3nArgs a, bool cached, int ny, int nz, hipStream_t st) {
  const size_t row = (size_t)a.W * sizeof(Real) * 3 * (N - 1);
  Step3nArgs b = a;
  auto rows = [&](int T) {
    b.R = std::min(T / b.W, ny);
    b.per_plane = (uint32_t)((ny + b.R - 1) / b.R);
    b.nblk = b.per_plane * (uint32_t)nz;
    return (b.R * b.W + 63) / 64 * 64;
  };
  // whole rows while two and more of them are a workgroup of kT3n threads
  if (a.W <= kRows3Width) {
    const int tc = rows(kT3r);
    hipLaunchKernelGGL((k_chem3r<N, Real>), dim3((b.nblk + 7) / 8 * 8), dim3(tc),
                       row * (b.R + 2), st, b);
    const int ts = rows(kT3n);
    launch_step3_nodes<N, Real, true>(b, cached, ts, 2 * row * (b.R + 2), st);
  } else {
    hipLaunchKernelGGL((k_chem3n<N, Real>), dim3((a.nblk + 7) / 8 * 8), dim3(kT3n), 0, st, a);
    launch_step3_nodes<N, Real, false>(a, cached, kT3n, 0, st);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_step3n(int N, int precision, const StepArgs &s, int nx, int ny, int nz, int pitch,
                         hipStream_t st) {
  Step3nArgs a{};
  a.s = s;
  a.W = node3_width(nx, precision);
  a.cs = node3_stride(nx, precision, pitch);
  const int64_t per = ((int64_t)a.W * ny + kT3n - 1) / kT3n;
  if (per * nz > (int64_t)1 << 30) return hipErrorInvalidValue;
  a.per_plane = (uint32_t)per;
  a.nblk = (uint32_t)(per * nz);
  // both copies of the state in the Infinity Cache
  const bool cached = 2 * (int64_t)(16 * N + 1) * (precision / 8) * nx * ny * nz <= kCacheBytes;
  switch (N) {
    case 2:
      return precision == 64 ? launch3n<2, double>(a, cached, ny, nz, st) : launch3n<2, float>(a, cached, ny, nz, st);
    case 3:
      return precision == 64 ? launch3n<3, double>(a, cached, ny, nz, st) : launch3n<3, float>(a, cached, ny, nz, st);
    case 4:
      return precision == 64 ? launch3n<4, double>(a, cached, ny, nz, st) : launch3n<4, float>(a, cached, ny, nz, st);
    case 5:
      return precision == 64 ? launch3n<5, double>(a, cached, ny, nz, st) : launch3n<5, float>(a, cached, ny, nz, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace nplbm
