// step3d_kernel.hip -- one time step of the N-phase phase-field LB model
// (arXiv:1904.12553) on the D3Q15 lattice of Sec. 3.1, for gfx950.
//
// The arithmetic per node is that of the 2-D kernel (step_kernel.hip) with
// three velocity components: pull streaming, phi_i by eq:N28 (the stored
// k = 0 value is the deviation h_0 - phi_prev, phi carried as the unevaluated
// sum phi_prev + (d + sum h_k)), closure eq:N18, C_i with the eq:N31b
// Laplacian, F and J~ from the eq:N31a gradients, u by eq:N22_1, p by
// eq:N23, NS collision eq:24 / eq:25 / eq:N20_1, CH collisions
// eq:N24-N27.  Only eq:N31a's central stencils and eq:N20_1 are built in 3-D.
//
// Two passes per step.  The phi pass (k_phi3) pulls the CH populations of
// every node once -- streaming fused into the load, bounce-back at z walls
// -- and writes phi_i to a dense array.  The step pass (k_step3) then owns
// a tile of interior nodes [x0, x1) x [y0, y1) (at most 64 x TY, x0 a
// multiple of 64, so loads and stores are whole cache lines) and marches
// through the planes [z0, z1) with one 64-lane wave per interior row; four
// lanes of each row bring in the 2-column x-halos and four waves the 2-row
// y-halos, so every wave collides.  Each iteration copies phi of plane mA
// from the array into a 5-plane LDS ring (all threads; the next plane's
// values are loaded right after, so they are in flight during the rest of
// the iteration); computes C of plane mA - 1 on the tile plus a ring of one
// into a 4-plane ring; and collides plane mA - 2 on the interior with the
// populations it pulls for that node, issued at the start of the iteration.
// The halo rings thus cost (N - 1) reads per node of the phi array (mostly
// from the 256 MB MALL, where the phi pass left it) instead of 16 (N - 1)
// population reads, and no population is read twice by the step pass.
// D3Q15 stencils reach the six faces and eight corners of a node, so the
// halo is two nodes for phi and one for C, as in 2-D.
#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "node_math3.h"

namespace nplbm {

namespace {

constexpr int k3W = 64;   // threads per tile row (one wave) = interior columns of a tile
constexpr int k3L = 68;   // LDS row: the 64 columns plus 2 halo columns each side
constexpr int k3PR = 5;   // phi ring planes
constexpr int k3CR = 4;   // C ring planes

// what the collision of one node reads: CH populations pulled (k = 0: the
// stored deviation), stored previous phi, NS populations k = 1..14 pulled,
// stored previous u
template <int M, typename Real>
struct Col3 {
  Real h[M][15];
  Real hi[M];
  Real g[15];
  Real pu[3];
};

__device__ __forceinline__ int wrap_i(int a, int n) {
  a %= n;
  return a < 0 ? a + n : a;
}

template <int N, typename Real, int TY>
__global__ void __launch_bounds__(k3W * TY) k_step3(StepArgs a) {
  constexpr int M = N - 1;
  // FP64 at N = 4 on 8-row tiles: the LDS rings (163 200 B) leave room for
  // one 8-wave workgroup per CU, two waves per SIMD, if the registers fit in
  // 256.  To get there this variant keeps fewer values live: each phase's
  // previous phi is loaded with its CH pulls, the collision re-reads phi_i
  // and C_i from LDS rather than holding them, the chemical-potential
  // stencil is one inline copy, and the next plane's phi values are loaded
  // after the collision rather than held through it.  Three moving spheres
  // at 192^3: 2.04 ms (45.0% of the HBM roofline) against 2.26 ms (40.7%)
  // on 4-row tiles at one wave per SIMD.  The same changes measured slower
  // on every other variant (up to 9%), which keep the plain code.
  constexpr bool kLean = sizeof(Real) == 8 && N == 4 && TY == 8;
  const NPL_CONST TileDesc3 *tp = (const NPL_CONST TileDesc3 *)a.strips + blockIdx.x;
  const int dom = tp->dom;
  if (dom < 0) return;
  const int x0 = tp->x0, x1 = tp->x1, y0 = tp->y0, y1 = tp->y1, z0 = tp->z0, z1 = tp->z1;
  const int dir = tp->dir;
  const NPL_CONST DomDesc *D = (const NPL_CONST DomDesc *)a.doms + dom;
  if (a.substep >= D->steps_left) return;
  const int par = (a.substep + D->parity0) & 1;
  const void *hs = D->h[par], *hd = D->h[par ^ 1];
  const void *gs = D->g[par], *gd = D->g[par ^ 1];
  const void *pvs = D->prev[par], *pvd = D->prev[par ^ 1];
  const NPL_CONST Consts<Real> &K = *consts_of<Real>(D);
  const NPL_CONST Consts<double> &KD = *consts_of<double>(D);
  const int nx = D->nx, ny = D->ny, nz = D->nz;
  const bool wall = D->wall != 0;
  constexpr uint32_t SZ = sizeof(Real);
  const uint32_t pb = (uint32_t)D->ps[0] * SZ;
  const uint32_t rbh = (uint32_t)D->rs[0] * SZ, rbg = (uint32_t)D->rs[1] * SZ,
                 rbp = (uint32_t)D->rs[2] * SZ;

  // rows of the rings: phi on the TY interior rows and 2 halo rows each
  // side, C on the interior rows and 1 each side
  constexpr int kPRows = TY + 4, kCRows = TY + 2;
  __shared__ Real sphi[k3PR][M][kPRows][k3L];
  __shared__ Real sC[k3CR][M][kCRows][k3L];

  const int lane = threadIdx.x & (k3W - 1);
  const int ty = __builtin_amdgcn_readfirstlane(threadIdx.x / k3W);  // uniform
  const int nxi = x1 - x0, nyi = y1 - y0;
  // Columns: lane l owns interior column x0 + l (tiles start on whole
  // cache lines, so every row of loads and stores is line-aligned) at LDS
  // column l + 2; lanes 0..3 also bring the halo columns x0 - 2, x0 - 1,
  // x0 + 64, x0 + 65 (LDS columns 0, 1, 66, 67) into the phi ring.
  const int xc = wrap_i(x0 + lane, nx);
  const int col = lane + 2;
  const int hcol = lane < 2 ? lane : 64 + lane;  // halo LDS column (lanes < 4)
  const uint32_t xh = (uint32_t)wrap_i(lane < 2 ? x0 - 2 + lane : x0 + 62 + lane, nx) * SZ;
  const uint32_t xcu = (uint32_t)xc * SZ;
  const uint32_t xw = (uint32_t)(xc == 0 ? nx - 1 : xc - 1) * SZ;  // x - 1
  const uint32_t xe = (uint32_t)(xc == nx - 1 ? 0 : xc + 1) * SZ;  // x + 1
  // Rows: wave w owns interior row y0 + w (phi ring row w + 2, C ring row
  // w + 1); waves 0..3 also bring the halo rows y0 - 2, y0 - 1, y0 + TY,
  // y0 + TY + 1 (phi ring rows 0, 1, TY + 2, TY + 3), and waves 0, 1
  // compute C of rows y0 - 1 and y0 + TY.  In a ragged tile (nyi < TY) the
  // waves past the interior hold the halo rows below it, as the lanes past
  // a ragged x end do.
  const int yc = wrap_i(y0 + ty, ny);                                // uniform
  const int yS = yc == 0 ? ny - 1 : yc - 1, yN = yc == ny - 1 ? 0 : yc + 1;
  const int pr = ty + 2, cr = ty + 1;                                // ring rows
  const bool lane_int = lane < nxi;
  const bool row_int = ty < nyi;                                     // uniform
  const bool hrow = ty < 4;                                          // uniform
  const int yh = wrap_i(ty < 2 ? y0 - 2 + ty : y0 + TY - 2 + ty, ny);
  const int prh = ty < 2 ? ty : TY + ty;                             // its ring row
  const int H = z1 - z0;

  auto plane_of = [&](int m) { return dir > 0 ? z0 + m : z1 - 1 - m; };
  // physical plane of a (possibly ghost) plane index: mirror beyond a wall,
  // periodic otherwise
  auto phys_plane = [&](int z) {
    if (wall) {
      if (z < 0) z = -1 - z;
      if (z >= nz) z = 2 * nz - 1 - z;
      z = z < 0 ? 0 : (z >= nz ? nz - 1 : z);
    } else {
      z = wrap_i(z, nz);
    }
    return z;
  };
  auto ring5 = [](int m) { return (m + 16 * k3PR) % k3PR; };
  auto ring4 = [](int m) { return (m + 16 * k3CR) % k3CR; };

  // Addressing.  A buffer resource spans one plane block of a group (its ny
  // row blocks); the row is a scalar byte offset fixed for the whole march
  // (the tile's rows do not change), the plane offset another scalar, and
  // the column the per-lane offset.
  const uint32_t ybh[3] = {(uint32_t)yS * rbh, (uint32_t)yc * rbh, (uint32_t)yN * rbh};
  const uint32_t ybg[3] = {(uint32_t)yS * rbg, (uint32_t)yc * rbg, (uint32_t)yN * rbg};
  const uint32_t ybp = (uint32_t)yc * rbp;
  const uint32_t plh = (uint32_t)ny * rbh, plg = (uint32_t)ny * rbg, plp = (uint32_t)ny * rbp;

  // Sources of the populations arriving at plane zp: plane zp - c_z, or the
  // node itself with the opposite direction when that plane lies beyond a
  // wall (bounce-back).  Index 0 / 1 / 2 = plane zp - 1 / zp / zp + 1.
  struct Planes {
    Rsrc r[3];
    bool bS, bN;  // bounce for c_z = +1 / c_z = -1
  };
  auto planes_of = [&](const void *base, uint32_t pl, int zp) {
    Planes P;
    P.bS = wall && zp == 0;
    P.bN = wall && zp == nz - 1;
    P.r[0] = row_rsrc(base, pl, zp == 0 ? nz - 1 : zp - 1);
    P.r[1] = row_rsrc(base, pl, zp);
    P.r[2] = row_rsrc(base, pl, zp == nz - 1 ? 0 : zp + 1);
    return P;
  };
  // load plane q0 + kk of direction k (kk = k, or its opposite when
  // bounced).  Bounce-back happens only on the two planes next to a wall,
  // so the callers take a branch-free path (kWall false) everywhere else.
  auto pull = [&](const Planes &P, const uint32_t (&yb)[3], int k, int q0, auto kWall) {
    const int cx = ex3(k), cy = ey3(k), cz = ez3(k);
    const uint32_t col = cx == 1 ? xw : (cx == -1 ? xe : xcu);
    if (!decltype(kWall)::value || cz == 0)
      return bld<Real>(P.r[1 - cz], col, yb[1 - cy] + (uint32_t)(q0 + k) * pb);
    const bool b = cz == 1 ? P.bS : P.bN;
    const Rsrc r = b ? P.r[1] : P.r[cz == 1 ? 0 : 2];
    const uint32_t so = b ? yb[1] + (uint32_t)(q0 + opp3(k)) * pb
                          : yb[1 - cy] + (uint32_t)(q0 + k) * pb;
    return bld<Real>(r, b ? xcu : col, so);
  };
  // run f(kWall) with kWall a compile-time flag: does plane zp border a wall?
  auto by_wall = [&](const Planes &P, auto f) {
    if (P.bS || P.bN)
      f(std::true_type());
    else
      f(std::false_type());
  };

  // ---- pull what the collision of march index m reads ----
  // CH populations of phase i
  auto pull_phase = [&](int m, int i, Col3<M, Real> &C) {
    const Planes P = planes_of(hs, plh, phys_plane(plane_of(m)));
    by_wall(P, [&](auto kWall) {
#pragma unroll
      for (int k = 0; k < 15; ++k) C.h[i][k] = pull(P, ybh, k, i * 15, kWall);
    });
    if constexpr (kLean)
      C.hi[i] = bld<Real>(row_rsrc(pvs, plp, phys_plane(plane_of(m))), xcu,
                          ybp + (uint32_t)i * pb);
  };
  // NS populations (planes k - 1), stored previous phi and u
  auto pull_ns = [&](int m, Col3<M, Real> &C) {
    const int zp = phys_plane(plane_of(m));
    const Planes P = planes_of(gs, plg, zp);
    by_wall(P, [&](auto kWall) {
#pragma unroll
      for (int k = 1; k < 15; ++k) C.g[k] = pull(P, ybg, k, -1, kWall);
    });
    const Rsrc rp = row_rsrc(pvs, plp, zp);
    if constexpr (!kLean)
#pragma unroll
      for (int i = 0; i < M; ++i) C.hi[i] = bld<Real>(rp, xcu, ybp + (uint32_t)i * pb);
#pragma unroll
    for (int d = 0; d < 3; ++d) C.pu[d] = bld<Real>(rp, xcu, ybp + (uint32_t)(M + d) * pb);
  };
  auto pull_col = [&](int m, Col3<M, Real> &C) {
#pragma unroll
    for (int i = 0; i < M; ++i) pull_phase(m, i, C);
    pull_ns(m, C);
  };

  // ---- stage A: phi of march index mA (from the phi pass) -> LDS ----
  // all threads; the values of plane mA + 1 are loaded right after, so they
  // are in flight during the rest of the iteration
  const uint32_t rbf = (uint32_t)D->rsf * SZ, plf = (uint32_t)ny * rbf;
  const uint32_t ybf = (uint32_t)yc * rbf, ybfh = (uint32_t)yh * rbf;
  const void *phi3 = D->phi3;
  // the values of the own row (f: column, fh: x-halo column of lanes < 4)
  // and of the halo row of waves 0..3 (g, gh)
  struct PhiRow {
    Real f[M], fh[M], g[M], gh[M];
  };
  auto load_phi = [&](int mA, PhiRow &F) {
    const Rsrc r = row_rsrc(phi3, plf, phys_plane(plane_of(mA)));
#pragma unroll
    for (int i = 0; i < M; ++i) {
      F.f[i] = bld<Real>(r, xcu, ybf + (uint32_t)i * pb);
      F.fh[i] = bld<Real>(r, xh, ybf + (uint32_t)i * pb);
    }
    if (hrow)
#pragma unroll
      for (int i = 0; i < M; ++i) {
        F.g[i] = bld<Real>(r, xcu, ybfh + (uint32_t)i * pb);
        F.gh[i] = bld<Real>(r, xh, ybfh + (uint32_t)i * pb);
      }
  };
  auto stageA = [&](int mA, const PhiRow &F) {
    const int slot = ring5(mA);
#pragma unroll
    for (int i = 0; i < M; ++i) sphi[slot][i][pr][col] = F.f[i];
    if (lane < 4)
#pragma unroll
      for (int i = 0; i < M; ++i) sphi[slot][i][pr][hcol] = F.fh[i];
    if (hrow) {
#pragma unroll
      for (int i = 0; i < M; ++i) sphi[slot][i][prh][col] = F.g[i];
      if (lane < 4)
#pragma unroll
        for (int i = 0; i < M; ++i) sphi[slot][i][prh][hcol] = F.gh[i];
    }
  };

  // ---- stage B: chemical potentials of march index mB -> LDS ----
  // On the tile plus a ring of one: LDS columns 1 .. nxi + 2, taken as
  // lane + 1 and, for the last two, 65 + lane.  Planes beyond a wall are
  // skipped: the collision next to the wall reads its own plane for the
  // mirror ghost.
  constexpr bool kOneCopy = N >= 5 || kLean;
  auto chem_at = [&](int q, int c, int s0, int sU, int sD, int sc) {
    const int ty = q + 1;  // phi ring row of C ring row q
    chem_node3<N, Real>(
        K,
        [&](int i, int dx, int dy, int dz) {
          return sphi[dz == 0 ? s0 : (dz > 0 ? sU : sD)][i][ty + dy][c + dx];
        },
        [&](int i, Real v) { sC[sc][i][q][c] = v; });
  };
  // the C ring rows of a wave: its own (row y0 + w) while w <= nyi, and for
  // waves 0 / 1 rows y0 - 1 / y0 + TY
  //
  // At N = 5 the stencil code is kept to one inline copy (loops over the
  // rows and columns to evaluate): left to itself the compiler called it
  // out of line, and the call and its stack frame cost 16% of the step
  // (256^3 FP32: 3.56 against 3.00 ms).  Smaller N inline three copies.
  auto chem_row = [&](int q, int s0, int sU, int sD, int sc) __attribute__((always_inline)) {
    if constexpr (kOneCopy) {
#pragma unroll 1
      for (int pass = 0; pass < 2; ++pass) {
        const int c = pass == 0 ? lane + 1 : 65 + lane;
        if (c <= nxi + 2 && (pass == 0 || lane < 2)) chem_at(q, c, s0, sU, sD, sc);
      }
    } else {
      if (lane + 1 <= nxi + 2) chem_at(q, lane + 1, s0, sU, sD, sc);
      if (lane < 2 && 65 + lane <= nxi + 2) chem_at(q, 65 + lane, s0, sU, sD, sc);
    }
  };
  auto stageB = [&](int mB) {
    if (wall) {
      const int z = plane_of(mB);
      if (z < 0 || z >= nz) return;
    }
    const int s0 = ring5(mB), sU = ring5(mB + dir), sD = ring5(mB - dir), sc = ring4(mB);
    if constexpr (kOneCopy) {
      // this wave's C rows: its own while it has one, and a halo row for
      // waves 0 and 1 (uniform over the wave)
      const int qa = ty <= nyi ? cr : -1;
      const int qb = ty == 0 ? 0 : (ty == 1 && nyi == TY ? TY + 1 : -1);
#pragma unroll 1
      for (int pass = 0; pass < 2; ++pass) {
        const int q = pass == 0 ? qa : qb;
        if (q >= 0) chem_row(q, s0, sU, sD, sc);
      }
    } else {
      if (ty <= nyi) chem_row(cr, s0, sU, sD, sc);
      if (ty == 0) chem_row(0, s0, sU, sD, sc);
      if (ty == 1 && nyi == TY) chem_row(TY + 1, s0, sU, sD, sc);
    }
  };

  // ---- stage C: collide march index mC (interior rows) ----
  // With kLate the NS pulls are issued here and the CH populations of each
  // phase right before its collision, behind a compiler barrier, so only one
  // phase's populations are live at a time.
  auto stageC = [&](int mC, Col3<M, Real> &P, auto kLate) {
    if constexpr (decltype(kLate)::value) pull_ns(mC, P);
    const int zp = plane_of(mC);
    // ghost planes beyond a wall mirror the boundary plane, which is the
    // collision plane itself; march index mC + dir is plane zp + 1
    const bool gU = wall && zp + 1 >= nz, gD = wall && zp - 1 < 0;
    const int s0 = ring5(mC), c0 = ring4(mC);
    const int sU = gU ? s0 : ring5(mC + dir), sD = gD ? s0 : ring5(mC - dir);
    const int cU = gU ? c0 : ring4(mC + dir), cD = gD ? c0 : ring4(mC - dir);
    // lanes past a ragged tile end compute on their (valid) columns and do
    // not store
    int ln = col;
    Real phi[M], Cv[M];
    Sums3<Real> S = sums3_begin<N, Real>(KD);
#pragma unroll
    for (int i = 0; i < M; ++i) {
      // (not with kLean, whose stencils leave registers enough: 192^3 N = 4
      // FP64 2050 us a step with it, 2031 without; N = 5 FP64 2878 / 2916,
      // FP32 1257 / 1264)
      if constexpr (!kLean) sums3_order(ln, S);
      phi[i] = sphi[s0][i][pr][ln];
      Cv[i] = sC[c0][i][cr][ln];
      Real gp[3], gc[3];
      grad_node3<Real>(
          [&](int dx, int dy, int dz) {
            return sphi[dz == 0 ? s0 : (dz > 0 ? sU : sD)][i][pr + dy][ln + dx];
          },
          gp);
      grad_node3<Real>(
          [&](int dx, int dy, int dz) {
            return sC[dz == 0 ? c0 : (dz > 0 ? cU : cD)][i][cr + dy][ln + dx];
          },
          gc);
      sums3_add<Real>(K, KD, i, phi[i], Cv[i], gp, gc, S);
    }
    if (!lane_int) return;
    const Rsrc wh = row_rsrc(hd, plh, zp), wg = row_rsrc(gd, plg, zp),
               wp = row_rsrc(pvd, plp, zp);
    collide_node3<N, Real>(
        K, KD, S, P.g, P.pu,
        [&](int i, auto collide) {
          Real phii = phi[i], Cvi = Cv[i];
          if constexpr (decltype(kLate)::value) {
            asm volatile("" ::: "memory");
            pull_phase(mC, i, P);
            // plane mC's slots of the phi and C rings are rewritten only two
            // iterations later, so these are the values read above
            if constexpr (kLean) {
              phii = sphi[s0][i][pr][ln];
              Cvi = sC[c0][i][cr][ln];
            }
          }
          collide(P.h[i], P.hi[i], phii, Cvi);
        },
        [&](int plane, Real v) { bst<Real, true>(wg, xcu, ybg[1] + (uint32_t)plane * pb, v); },
        [&](int plane, Real v) { bst<Real, true>(wh, xcu, ybh[1] + (uint32_t)plane * pb, v); },
        [&](int plane, Real v) { bst<Real, true>(wp, xcu, ybp + (uint32_t)plane * pb, v); });
  };

  // March: iteration j pulls plane mA = j - 2, computes C of mA - 1 and
  // collides mA - 2, so J = H + 4 iterations cover the interior planes.
  // The collision's own pulls are issued before stage A where the registers
  // allow it (held through two barriers); FP64 with N >= 3 spills that way,
  // so there they are issued at the collision (256^3 N = 3 FP64: 49.9%
  // against 44.9% of the HBM roofline; FP32 measured slower late).
  constexpr bool kEarly = !(sizeof(Real) == 8 && N >= 3);
  const int J = H + 4;
  PhiRow fr;
  load_phi(-2, fr);
  for (int j = 0; j < J; ++j) {  // j is uniform over the block
    const int mA = j - 2;
    const int mC = mA - 2;
    const bool collide = row_int && mC >= 0 && mC < H;  // uniform
    Col3<M, Real> col;
    if constexpr (kEarly)
      if (collide) pull_col(mC, col);
    stageA(mA, fr);
    if constexpr (!kLean) load_phi(mA + 1, fr);
    __syncthreads();
    stageB(mA - 1);
    __syncthreads();
    if (collide) stageC(mC, col, std::integral_constant<bool, !kEarly>());
    if constexpr (kLean) load_phi(mA + 1, fr);
  }
}

// The phi pass: phi_i = phi_prev + (d + sum_{k>=1} h_k) (eq:N28, the
// pulled populations and the stored deviation of h_0) of every node of the
// domain into the phi array.  One 64-lane wave per row segment of 64 nodes,
// four rows per workgroup; no halo, so every population is read once.
//
// Blocks are numbered for the 8 XCDs: hardware block b runs on XCD b % 8,
// and XCD x takes the x-th contiguous eighth of the (x, y, z)-ordered block
// list, in order.  Blocks next to each other in x then run on one XCD at
// about the same time, so the cache line that two of them pull from (the
// one holding the column left or right of a 64-column segment) comes from
// that XCD's L2 the second time.
template <int N, typename Real>
__global__ void __launch_bounds__(256) k_phi3(StepArgs a) {
  constexpr int M = N - 1;
  const NPL_CONST DomDesc *D = (const NPL_CONST DomDesc *)a.doms;
  if (a.substep >= D->steps_left) return;
  const int par = (a.substep + D->parity0) & 1;
  const void *hs = D->h[par], *pvs = D->prev[par];
  const int nx = D->nx, ny = D->ny, nz = D->nz;
  const bool wall = D->wall != 0;
  constexpr uint32_t SZ = sizeof(Real);
  const uint32_t pb = (uint32_t)D->ps[0] * SZ;
  const uint32_t rbh = (uint32_t)D->rs[0] * SZ, rbp = (uint32_t)D->rs[2] * SZ,
                 rbf = (uint32_t)D->rsf * SZ;
  const int gx = (nx + k3W - 1) / k3W, gy = (ny + 3) / 4;
  const int nblk = gx * gy * nz, per = (nblk + 7) / 8;
  const int t = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if (t >= nblk) return;
  const int bx = t % gx, by = (t / gx) % gy;
  const int lane = threadIdx.x & (k3W - 1);
  const int y = by * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / k3W);  // uniform
  const int z = t / (gx * gy);
  const int x = bx * k3W + lane;
  if (y >= ny || x >= nx) return;
  const uint32_t xcu = (uint32_t)x * SZ;
  const uint32_t xw = (uint32_t)(x == 0 ? nx - 1 : x - 1) * SZ;
  const uint32_t xe = (uint32_t)(x == nx - 1 ? 0 : x + 1) * SZ;
  const int yS = y == 0 ? ny - 1 : y - 1, yN = y == ny - 1 ? 0 : y + 1;
  const uint32_t yb[3] = {(uint32_t)yS * rbh, (uint32_t)y * rbh, (uint32_t)yN * rbh};
  const uint32_t plh = (uint32_t)ny * rbh;
  const bool bS = wall && z == 0, bN = wall && z == nz - 1;
  const Rsrc r0 = row_rsrc(hs, plh, z == 0 ? nz - 1 : z - 1);
  const Rsrc r1 = row_rsrc(hs, plh, z);
  const Rsrc r2 = row_rsrc(hs, plh, z == nz - 1 ? 0 : z + 1);
  const Rsrc rp = row_rsrc(pvs, (uint32_t)ny * rbp, z);
  Real f[M];
#pragma unroll
  for (int i = 0; i < M; ++i) {
    Real lo = Real(0);
#pragma unroll
    for (int k = 0; k < 15; ++k) {
      const int cx = ex3(k), cy = ey3(k), cz = ez3(k);
      const bool b = (cz == 1 && bS) || (cz == -1 && bN);
      const Rsrc r = b ? r1 : (cz == 1 ? r0 : (cz == -1 ? r2 : r1));
      const uint32_t col = b ? xcu : (cx == 1 ? xw : (cx == -1 ? xe : xcu));
      const uint32_t so = b ? yb[1] + (uint32_t)(i * 15 + opp3(k)) * pb
                            : yb[1 - cy] + (uint32_t)(i * 15 + k) * pb;
      lo += bld<Real>(r, col, so);
    }
    f[i] = bld<Real>(rp, xcu, (uint32_t)y * rbp + (uint32_t)i * pb) + lo;
  }
  const Rsrc wf = row_rsrc(D->phi3, (uint32_t)ny * rbf, z);
#pragma unroll
  for (int i = 0; i < M; ++i) bst<Real, true>(wf, xcu, (uint32_t)y * rbf + (uint32_t)i * pb, f[i]);
}

template <int N, int TY>
constexpr int lds3_bytes(int bytes) {
  return (k3PR * (TY + 4) + k3CR * (TY + 2)) * (N - 1) * k3L * bytes;
}

template <int N>
hipError_t launch_phi3(int precision, const StepArgs &a, dim3 grid, hipStream_t st) {
  if (precision == 64)
    hipLaunchKernelGGL((k_phi3<N, double>), grid, dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL((k_phi3<N, float>), grid, dim3(256), 0, st, a);
  return hipGetLastError();
}

// LDS asked for beyond the rings of an FP32 workgroup so that two of them
// fill a compute unit: three (at N <= 3 registers and rings would allow
// them) march more tiles at once, each over fewer planes (256^3 N = 2 996 us
// a step against 1131, 192^3 446 against 485; N = 3 256^3 1584 against 1787,
// 192^3 710 against 767).
template <int N, int TY>
constexpr int pad3_bytes() {
  return std::max(0, 56 * 1024 - lds3_bytes<N, TY>(4));
}

template <int N, int TY>
hipError_t launch3(int precision, const StepArgs &a, int nblocks, hipStream_t st) {
  if (precision == 64) {
    if constexpr (lds3_bytes<N, TY>(8) <= 160 * 1024)
      hipLaunchKernelGGL((k_step3<N, double, TY>), dim3(nblocks), dim3(k3W * TY), 0, st, a);
    else
      return hipErrorInvalidValue;
  } else {
    if constexpr (lds3_bytes<N, TY>(4) <= 160 * 1024)
      hipLaunchKernelGGL((k_step3<N, float, TY>), dim3(nblocks), dim3(k3W * TY),
                         (pad3_bytes<N, TY>()), st, a);
    else
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int N, int TY>
int occ3(int precision) {
  int nb = 0;
  hipError_t e = hipErrorInvalidValue;
  if (precision == 64) {
    if constexpr (lds3_bytes<N, TY>(8) <= 160 * 1024)
      e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_step3<N, double, TY>, k3W * TY, 0);
  } else {
    if constexpr (lds3_bytes<N, TY>(4) <= 160 * 1024)
      e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_step3<N, float, TY>, k3W * TY,
                                                       (pad3_bytes<N, TY>()));
  }
  return e == hipSuccess ? nb : 0;
}

}  // namespace

// Interior rows of a marching tile = waves of a workgroup: 4 in FP32, where two or
// more 4-row workgroups per CU measured faster than one of 8 (256^3: N = 3
// 48.3% against 44.9% of the HBM roofline, N = 5 38.2% against 35.6%); in
// FP64 8 for N <= 4 (N = 3: 44.9% against 43.9%; N = 4, with the leaner
// register use of that variant: 45.0% against 40.7%) and 4 for N = 5, where
// FP64 rings of 8 rows would not fit in LDS.
int step3_march_ty(int N, int precision) { return precision == 64 && N <= 4 ? 8 : 4; }

// The node kernels (0) take lattices of up to 900 000 nodes, where the
// marching tiles leave compute units idle, and those whose rows fill less
// than 77% of the marching kernel's 64-column tiles; the marching kernel the
// others, where it moves 2 (N - 1) words a node less.  A step, node /
// marching: 64^3 FP32 N = 3 30 / 69 us, FP64 N = 4 76 / 182; 100 x 84 x 60
// FP64 N = 4 171 / 246; 96^3 FP32 N = 3 100 / 117; 72 x 160^2 FP64 N = 3
// 461 / 500; 96 x 200^2 FP64 N = 3 836 / 895; 112^3 FP32 N = 3 171 / 166;
// 128^3 230 / 213; 200^3 (78%) FP32 N = 3 1016 / 952.
// NPLBM_TY3 = 0, 4 or 8 overrides; NPLBM_TARGET_BLOCKS asks for the marching
// kernel.
int step3_ty(int N, int precision, int nx, int ny, int nz) {
  if (const char *e = std::getenv("NPLBM_TY3")) {
    const int t = std::atoi(e);
    if (t == 0) return 0;
    const int bytes = precision == 64 ? 8 : 4;
    const int lds = (k3PR * (t + 4) + k3CR * (t + 2)) * (N - 1) * k3L * bytes;
    if (t == 4 || (t == 8 && lds <= 160 * 1024)) return t;
  }
  const int tiles = (nx + k3W - 1) / k3W * k3W;
  if (std::getenv("NPLBM_TARGET_BLOCKS") == nullptr &&
      ((int64_t)nx * ny * nz <= 900000 || nx * 100 < tiles * 77))
    return 0;
  return step3_march_ty(N, precision);
}

hipError_t launch_step3(int N, int precision, int ty, const StepArgs &a, int nblocks, int nx,
                        int ny, int nz, int pitch, hipStream_t st) {
  if (nblocks <= 0) return hipSuccess;
  // one block per 64 x 4 row segments of a plane, in a 1-D grid whose
  // size is a multiple of 8 (the phi pass maps block numbers to XCDs)
  const int64_t nphi = (int64_t)((nx + k3W - 1) / k3W) * ((ny + 3) / 4) * nz;
  if (nphi > (int64_t)1 << 30) return hipErrorInvalidValue;
  const dim3 pg((unsigned)((nphi + 7) / 8 * 8));
  hipError_t e;
  switch (N) {
    case 2: e = launch_phi3<2>(precision, a, pg, st); break;
    case 3: e = launch_phi3<3>(precision, a, pg, st); break;
    case 4: e = launch_phi3<4>(precision, a, pg, st); break;
    case 5: e = launch_phi3<5>(precision, a, pg, st); break;
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  if (ty == 0) return launch_step3n(N, precision, a, nx, ny, nz, pitch, st);
  if (ty == 4) {
    switch (N) {
      case 2: return launch3<2, 4>(precision, a, nblocks, st);
      case 3: return launch3<3, 4>(precision, a, nblocks, st);
      case 4: return launch3<4, 4>(precision, a, nblocks, st);
      case 5: return launch3<5, 4>(precision, a, nblocks, st);
      default: return hipErrorInvalidValue;
    }
  }
  switch (N) {
    case 2: return launch3<2, 8>(precision, a, nblocks, st);
    case 3: return launch3<3, 8>(precision, a, nblocks, st);
    case 4: return launch3<4, 8>(precision, a, nblocks, st);
    case 5: return launch3<5, 8>(precision, a, nblocks, st);
    default: return hipErrorInvalidValue;
  }
}

int step3_blocks_per_cu(int N, int precision, int ty) {
  if (ty == 4) {
    switch (N) {
      case 2: return occ3<2, 4>(precision);
      case 3: return occ3<3, 4>(precision);
      case 4: return occ3<4, 4>(precision);
      case 5: return occ3<5, 4>(precision);
      default: return 0;
    }
  }
  switch (N) {
    case 2: return occ3<2, 8>(precision);
    case 3: return occ3<3, 8>(precision);
    case 4: return occ3<4, 8>(precision);
    case 5: return occ3<5, 8>(precision);
    default: return 0;
  }
}

}  // namespace nplbm
