// tile_kernel.hip -- the time step of a 2-D domain (D2Q9) by tiles, for
// lattices too small to fill the chip with marching strips (gfx950).
//
// The marching kernel (step_kernel.hip) reads every population once but
// walks its strip two rows at a time, and one iteration is a serial chain of
// loads, LDS stages and two barriers (about 4 us with few workgroups on the
// chip), so a small lattice -- a few strips of 16 rows and more -- leaves
// most compute units idle and is bound by that chain: 44 us a step on the
// 100 x 100 N = 3 FP64 droplet, seven workgroups; 5.5 us here.  One launch
// gives every node a thread of its own, or two, and goes through the chain
// once: a workgroup owns a tile of 32 x TY nodes (one cache line of FP32
// wide) and
//
//   stage A: each thread pulls the CH populations of its node (kept in
//            registers for the collision) and the workgroup shares out the
//            halo nodes around the tile, one (node, phase) pair per thread,
//            so all loads of the step, the NS populations too, are in flight
//            together; phi_i (eq:N28) -> LDS;
//   stage B: chemical potentials (eq:N18, eq:N17 with eq:N31b) on the tile
//            and the ring the gradients need -> LDS;
//   stage J: Remark 1 only, the products J~_b u_a on the tile and a ring
//            of one -> LDS;
//   stage C: gradients, forces, both collisions, store.
//
// The halo populations are pulled again by the neighbouring tiles (1.7 times
// the CH reads at TY = 8, 2.3 at TY = 4), from L2 or MALL at the sizes this
// kernel runs at.  What bounds it: with a tile or less per compute unit the
// chain of latencies, half of it in stage A (N = 8 FP32 on 128^2: 10 of 21
// thousand cycles, 3 in B, 7 in C) on top of 1.6 us a launch; with many, the
// traffic of L2 and MALL (512^2 N = 4 FP32: 106 MB in 18.9 us, 5.6 TB/s).
// Wider tiles (64 x 4, 64 x 8, 128 x 4) were slower, but for FP32 with N <= 5
// at 512^2 (64 x 8: 5 - 7%).  Every node's arithmetic is that of node_math.h, as in the
// marching kernel, and a halo phi is summed in the order its own tile sums
// it, so the state does not depend on which kernel or tile advanced a node.
#include "node_math.h"

#include <climits>

namespace nplbm {

// This translation unit instantiates the kernel for one scheme, NPL_GS (0
// central, 1 mixed, 2 Remark 1), as step_kernel.hip does.
#ifndef NPL_GS
#define NPL_GS 0
#endif

namespace {

constexpr int kTW = kTileWidth;  // columns of a tile

// Position q of the frame of width H around the tile, q < 2 H (kTW + 2 H + TY),
// counted from the frame's corner: the rows below and above, then the columns
// beside the tile.
template <int H, int TY>
__device__ __forceinline__ void frame_at(int q, int &px, int &py) {
  constexpr int kW = kTW + 2 * H, kTop = H * kW;
  if (q < 2 * kTop) {
    const int r = q / kW;
    px = q % kW;
    py = r < H ? r : r + TY;
  } else {
    const int s = q - 2 * kTop, c = s % (2 * H);
    px = c < H ? c : c + kTW;
    py = s / (2 * H) + H;
  }
}

// One word of each 64-byte line of the constants in use, kept alive by an
// empty asm.
template <int N, typename Real>
__device__ __forceinline__ void touch_consts(const NPL_CONST Consts<Real> &K) {
  constexpr int kLine = 64 / (int)sizeof(Real);
  Real s = K.gx;
  auto range = [&](const NPL_CONST Real *p, int n) {
#pragma unroll
    for (int i = 0; i < n + kLine - 1; i += kLine) s += p[i < n ? i : n - 1];
  };
  range(&K.ca[0], N);
  range(&K.cA[0][0], (N - 1) * kMaxM + N - 1);
  range(&K.ra, 2);
  range(&K.rA[0], N - 1);
  range(&K.lam[0][0], (N - 2) * kMaxM + N - 1);
  range(&K.KH[0][0], (N - 1) * kMaxM + N - 1);
  range(&K.Jc[0], 4 * kMaxM);
  asm volatile("" ::"v"(s));
}

// kHelp: the workgroup has a second set of kTW x TY threads (helpers) that
// takes the rings of stages B and J and the halo items of stage A, so that a
// node's own thread goes through its own part only.  kSplit: the sets share
// the halo items, and a node's collision too: the first set takes the NS
// populations and the CH phases below kOwn (the NS collision weighs as two
// phases), the helpers the other phases and the gradients of C.
template <int N, typename Real, int TY, int kGS, bool kHelp,
          bool kSplit = kHelp && tile_split(N, (int)sizeof(Real), kGS, TY)>
__global__ void __launch_bounds__(kTW * TY * (kHelp ? 2 : 1)) k_tile(TileArgs a) {
  constexpr int M = N - 1;
  constexpr bool kTwoHop = kGS == kSchemeMixed;  // eq:N40 first derivatives
  constexpr bool kR1 = kGS == kSchemeRemark1;    // Remark 1 force distribution
  constexpr int kNT = kTW * TY;
  constexpr int kHT = kNT * (kSplit ? 2 : 1);  // threads that bring the halo
  constexpr int kOwn = kSplit ? (M > 2 ? (M - 2) / 2 : 0) : M;
  constexpr int kPh = M - kOwn > kOwn ? M - kOwn : kOwn;  // most phases of a thread
  // Many phases in FP64 on one thread: the own populations, three and more
  // rounds of halo items and the NS ones together exceed the registers of two
  // waves per SIMD.  These variants finish the own phi before the halo and
  // take the halo three items at a time (512^2 FP64 Remark 1 N = 6: 63 us a
  // step against 78, 360^2 mixed N = 6: 39 against 46; up to N = 5 it costs a
  // few percent).
  constexpr bool kGrouped = !kSplit && sizeof(Real) == 8 && M * 8 + (kGS ? 8 : 0) >= 48;
  // phi is needed kHalo nodes around a node that collides, C kHalo - 1
  constexpr int kHalo = kGS ? 3 : 2, kRing = kHalo - 1;
  constexpr int kPW = kTW + 2 * kHalo, kPR = TY + 2 * kHalo;
  constexpr int kCW = kTW + 2 * kRing, kCR = TY + 2 * kRing;
  constexpr int kQW = kTW + 2, kQR = TY + 2;
  __shared__ Real sphi[M][kPR][kPW];
  __shared__ Real sC[M][kCR][kCW];
  __shared__ Acc sU[kSplit ? 2 : 1][kSplit ? kNT : 1];  // new velocity
  __shared__ Real sJ[kSplit && !kR1 ? 2 : 1][kSplit && !kR1 ? kNT : 1];  // G.Jxs, G.Jys
  __shared__ Real sQ[kR1 ? 4 : 1][kR1 ? kQR : 1][kQW];  // J~_x u_x, J~_y u_x, J~_x u_y, J~_y u_y

  // The tile and its domain: by value for a launch over one domain (block b
  // runs on XCD b % 8; each XCD gets a contiguous run of the row-major
  // tiles, so neighbouring tiles share an L2), from the tables otherwise.
  int x0, y0, ncol, nrow;
  TileDom d;
  const NPL_CONST DomDesc *D = (const NPL_CONST DomDesc *)a.s.doms;
  if (a.ntx) {
    const uint32_t t = (blockIdx.x & 7) * a.per + (blockIdx.x >> 3);
    if (t >= a.ntile) return;
    const uint32_t r = __umulhi(t, a.div);
    d = a.d;
    x0 = (int)(t - r * a.ntx) * kTW;
    y0 = (int)r * TY;
    ncol = min(kTW, d.nx - x0);
    nrow = min(TY, d.ny - y0);
  } else {
    const NPL_CONST StripDesc *sp = (const NPL_CONST StripDesc *)a.s.strips + blockIdx.x;
    if (sp->dom < 0) return;
    D += sp->dom;
    if (a.s.substep >= D->steps_left) return;
    const int par = (a.s.substep + D->parity0) & 1;
    x0 = sp->x0;
    y0 = sp->y0;
    ncol = sp->x1 - x0;
    nrow = sp->y1 - y0;
    d.src[0] = D->h[par];
    d.src[1] = D->g[par];
    d.src[2] = D->prev[par];
    d.dst[0] = D->h[par ^ 1];
    d.dst[1] = D->g[par ^ 1];
    d.dst[2] = D->prev[par ^ 1];
    d.pb = (uint32_t)D->ps[0] * (uint32_t)sizeof(Real);
    for (int G = 0; G < 3; ++G) d.rb[G] = (uint32_t)D->rs[G] * (uint32_t)sizeof(Real);
    d.nx = D->nx;
    d.ny = D->ny;
    d.wall = D->wall;
  }
  const NPL_CONST Consts<Real> &K = *consts_of<Real>(D);
  const NPL_CONST Consts<double> &KD = *consts_of<double>(D);
  const int nx = d.nx, ny = d.ny;
  const bool wall = d.wall != 0;
  constexpr uint32_t SZ = sizeof(Real);
  const uint32_t pb = d.pb, rbh = d.rb[0], rbg = d.rb[1], rbp = d.rb[2];
  // one resource per group: the host picks this kernel only for domains
  // whose groups stay below 2^31 bytes
  const Rsrc rh = row_rsrc(d.src[0], rbh * (uint32_t)ny, 0),
             rg = row_rsrc(d.src[1], rbg * (uint32_t)ny, 0),
             rp = row_rsrc(d.src[2], rbp * (uint32_t)ny, 0);

  const int tid = threadIdx.x;
  // (uniform over a wave)
  const bool helper = kHelp && __builtin_amdgcn_readfirstlane(tid / kNT) != 0;
  const int ht = tid % kNT;
  const int lx = ht % kTW, ly = ht / kTW;
  // the thread's phases: ph0 + j, j < nph
  const int ph0 = helper ? kOwn : 0, nph = helper ? M - kOwn : kOwn;
  // Lattice node of tile position (px, py), px, py >= -kHalo: periodic in
  // x; periodic or mirrored at the walls in y.  Positions more than kHalo
  // beyond a ragged edge are never asked for.
  auto col_of = [&](int px) {
    int x = x0 + px;
    x = x < 0 ? x + nx : x;
    return x >= nx ? x - nx : x;
  };
  auto row_of = [&](int py) {
    int y = y0 + py;
    if (wall)
      y = y < 0 ? -1 - y : (y >= ny ? 2 * ny - 1 - y : y);
    else
      y = y < 0 ? y + ny : (y >= ny ? y - ny : y);
    return y;
  };
  // Byte offsets, direction plane included, of the populations arriving at
  // node (x, y) in a group with row block rb: from x - c_k, or the node's
  // own opposite direction when x - c_k lies beyond a wall.
  auto sources = [&](int x, int y, uint32_t rb, uint32_t (&o)[9]) {
    const uint32_t c0 = (uint32_t)x * SZ;
    const uint32_t cw = (uint32_t)(x == 0 ? nx - 1 : x - 1) * SZ;
    const uint32_t ce = (uint32_t)(x == nx - 1 ? 0 : x + 1) * SZ;
    const uint32_t r0 = (uint32_t)y * rb;
    const uint32_t rs = (uint32_t)(y == 0 ? ny - 1 : y - 1) * rb;
    const uint32_t rn = (uint32_t)(y == ny - 1 ? 0 : y + 1) * rb;
    const bool bs = wall && y == 0, bn = wall && y == ny - 1;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const int cx = cxk(k), cy = cyk(k);
      const uint32_t c = cx == 1 ? cw : (cx == -1 ? ce : c0);
      const uint32_t r = cy == 1 ? rs : (cy == -1 ? rn : r0);
      const bool b = (cy == 1 && bs) || (cy == -1 && bn);
      o[k] = b ? r0 + c0 + (uint32_t)oppk(k) * pb : r + c + (uint32_t)k * pb;
    }
  };

  // ---- stage A: all loads of the step ----
  // own node; threads up to kHalo beyond a ragged edge bring halo nodes, those
  // further right the last of these once more.  x and y are a node's for every
  // thread (rows further up are not pulled), which spares the branches of a
  // choice (128 x 96 N = 2 FP32 3.78 us a step against 3.84).
  const bool active = kSplit || !helper;  // has part in a node's collision
  const bool own = active && ly < nrow + kHalo;
  // Columns past a ragged right end are stored too: they fall into the
  // padding of the row pitch, which nothing reads, and whole lines store
  // faster than parts of one (100 x 96 N = 2 FP32: 5.5 us against 6.5 us).
  // They collide what they pulled on the last column's phi and C, so that
  // every value they store is a defined one (against lanes that pull nothing
  // there: 400 x 200 N = 3 FP64 10.04 -> 10.05 us a step, 128 x 96 N = 2 FP32 3.78
  // -> 3.78, N = 3 4.99 -> 4.89, 200 x 320 N = 5 mixed 11.82 -> 11.60; with zeros
  // selected at each store 10.12, 3.79, 5.00, 11.79).
  const bool storing = active && ly < nrow;
  const int lc0 = min(lx, ncol - 1);  // column of phi and C at the collision
  const int x = col_of(min(lx, ncol + kHalo - 1)), y = row_of(min(ly, nrow + kHalo - 1));
  Real h[kPh][9], hi[kPh], g[9], pu[2];
  if (own) {
    uint32_t o[9];
    sources(x, y, rbh, o);
#pragma unroll
    for (int j = 0; j < kPh; ++j)
      if (j < nph)
#pragma unroll
        for (int k = 0; k < 9; ++k) h[j][k] = bld<Real>(rh, o[k], (uint32_t)((ph0 + j) * 9) * pb);
    const uint32_t op = (uint32_t)y * rbp + (uint32_t)x * SZ;
#pragma unroll
    for (int j = 0; j < kPh; ++j)
      if (j < nph) hi[j] = bld<Real>(rp, op, (uint32_t)(ph0 + j) * pb);
  }
  // halo nodes: position q of the frame around the tile, one phase each
  constexpr int kHN = 2 * kHalo * (kPW + TY);         // nodes of the frame
  constexpr int kRounds = (kHN * M + kHT - 1) / kHT;  // items per thread
  auto load_item = [&](int r, Real (&v)[10]) {
    const int it = (kSplit ? tid : ht) + r * kHT;
    const int i = it / kHN;
    int px, py;
    frame_at<kHalo, TY>(it % kHN, px, py);
    px -= kHalo;
    py -= kHalo;
    if (i < M && px < ncol + kHalo && py < nrow + kHalo) {
      const int xn = col_of(px), yn = row_of(py);
      uint32_t o[9];
      sources(xn, yn, rbh, o);
      const uint32_t ip = (uint32_t)(i * 9) * pb;
#pragma unroll
      for (int k = 0; k < 9; ++k) v[k] = bld<Real>(rh, o[k] + ip, 0u);
      v[9] = bld<Real>(rp, (uint32_t)yn * rbp + (uint32_t)xn * SZ + (uint32_t)i * pb, 0u);
    }
  };
  auto store_item = [&](int r, const Real (&v)[10]) {
    const int it = (kSplit ? tid : ht) + r * kHT;
    const int i = it / kHN;
    int px, py;
    frame_at<kHalo, TY>(it % kHN, px, py);
    px -= kHalo;
    py -= kHalo;
    if (i < M && px < ncol + kHalo && py < nrow + kHalo) {
      Real lo = v[0];
#pragma unroll
      for (int k = 1; k < 9; ++k) lo += v[k];
      sphi[i][py + kHalo][px + kHalo] = v[9] + lo;
    }
  };
  auto store_own = [&]() {
    if (own)
#pragma unroll
      for (int j = 0; j < kPh; ++j)
        if (j < nph) sphi[ph0 + j][ly + kHalo][lx + kHalo] = hi[j] + lo_sum(h[j]);  // eq:N28
  };
  constexpr int kGroup = kGrouped ? 3 : kRounds;
  if constexpr (kGrouped) {
    store_own();
    __builtin_amdgcn_sched_barrier(0);
  }
  Real hv[kGroup][10];
  const bool halo = !kHelp || kSplit || helper;  // has part in bringing the halo
  if (halo)
#pragma unroll
    for (int r = 0; r < kGroup; ++r) load_item(r, hv[r]);
  if (storing) {
    if (!helper) {
      uint32_t o[9];
      sources(x, y, rbg, o);
#pragma unroll
      for (int k = 1; k < 9; ++k) g[k] = bld<Real>(rg, o[k] - pb, 0u);
    }
    const uint32_t op = (uint32_t)y * rbp + (uint32_t)x * SZ;
    pu[0] = bld<Real>(rp, op, (uint32_t)M * pb);
    pu[1] = bld<Real>(rp, op, (uint32_t)(M + 1) * pb);
  }
  // Read one word of every cache line of constants while the loads above are
  // in flight, so that the scalar loads of the later stages hit the scalar
  // cache (cold at the start of a launch) instead of waiting in turn.
  touch_consts<N>(K);
  if constexpr (sizeof(Real) == 4) touch_consts<N>(KD);
  if constexpr (!kGrouped) store_own();
  if (halo) {
#pragma unroll
    for (int r = 0; r < kGroup; ++r) store_item(r, hv[r]);
#pragma unroll
    for (int q = kGroup; q < kRounds; q += kGroup) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < kGroup; ++r)
        if (q + r < kRounds) load_item(q + r, hv[r]);
#pragma unroll
      for (int r = 0; r < kGroup; ++r)
        if (q + r < kRounds) store_item(q + r, hv[r]);
    }
  }
  __syncthreads();

  // ---- stage B: chemical potentials on the tile and kRing around it ----
  // (ghost positions beyond a wall are evaluated on the mirrored phi, which
  // gives the mirror of C bit for bit: the sums pair opposite neighbours)
  auto chem_at = [&](int cx, int cy) {
    if (cx < ncol + 2 * kRing && cy < nrow + 2 * kRing)
      chem_node<N, Real>(
          K, [&](int i, int dx, int dy) { return sphi[i][cy + 1 + dy][cx + 1 + dx]; },
          [&](int i, Real v) { sC[i][cy][cx] = v; });
  };
  if constexpr (kHelp) {
    for (int q = helper ? ht : 0; q < (helper ? 2 * kRing * (kCW + TY) : 1); q += kNT) {
      int cx = lx + kRing, cy = ly + kRing;
      if (helper) frame_at<kRing, TY>(q, cx, cy);
      chem_at(cx, cy);
    }
  } else {
    for (int q = tid; q < kCW * kCR; q += kNT) chem_at(q % kCW, q / kCW);
  }
  __syncthreads();

  // ---- stage J (Remark 1): J~ and the products J~_b u_a ----
  // J~ from the eq:N31a gradients of C on the tile and one node around it,
  // u the stored velocity of the previous step.  Rows beyond a wall are not
  // formed: stage C reads the row they mirror.
  if constexpr (kR1) {
    auto prod_at = [&](int qx, int qy) {
      const int r = y0 + qy - 1;
      if (qx < ncol + 2 && qy < nrow + 2 && !(wall && (r < 0 || r >= ny))) {
        Real Jx = Real(0), Jy = Real(0);
#pragma unroll
        for (int i = 0; i < M; ++i) {
          Real gx, gy;
          grad_central<Real>([&](int dx, int dy) { return sC[i][qy + 1 + dy][qx + 1 + dx]; }, gx,
                             gy);
          Jx += K.Jc[i] * gx;
          Jy += K.Jc[i] * gy;
        }
        const uint32_t op =
            (uint32_t)row_of(qy - 1) * rbp + (uint32_t)col_of(qx - 1) * SZ + (uint32_t)M * pb;
        const Real ux = bld<Real>(rp, op, 0u), uy = bld<Real>(rp, op + pb, 0u);
        sQ[0][qy][qx] = Jx * ux;
        sQ[1][qy][qx] = Jy * ux;
        sQ[2][qy][qx] = Jx * uy;
        sQ[3][qy][qx] = Jy * uy;
      }
    };
    if constexpr (kHelp) {
      for (int q = helper ? ht : 0; q < (helper ? 2 * (kQW + TY) : 1); q += kNT) {
        int qx = lx + 1, qy = ly + 1;
        if (helper) frame_at<1, TY>(q, qx, qy);
        prod_at(qx, qy);
      }
    } else {
      for (int q = tid; q < kQW * kQR; q += kNT) prod_at(q % kQW, q / kQW);
    }
    __syncthreads();
  }

  // ---- stage C: gradients and collisions ----
  if constexpr (!kSplit)
    if (!storing) return;
  // phi and C stay in registers from here where these suffice, and are read
  // again by each CH collision where they would spill (N = 8 FP64 on 250 x
  // 380: 29.6 against 40.7 us a step)
  constexpr bool kKeep = !kSplit && N * sizeof(Real) <= 32;
  Real phi[M], Cv[kKeep ? M : 1];
  GradSums<Real> G{};
  NodeFlow f;
  int lc = lc0;
  auto grad = [&](auto at, Real &gx, Real &gy) {
    if constexpr (kTwoHop)
      grad_two_hop<Real>(at, gx, gy);
    else
      grad_central<Real>(at, gx, gy);
  };
  // The next phase's LDS reads wait for this phase's sums (their index
  // passes through an empty asm that takes them).  Left alone the compiler
  // issues the reads of all phases first and holds them: 216 against 108
  // registers for FP32 mixed N = 5 (512^2: 29.9 against 25.0 us a step),
  // and spills for FP64 mixed N >= 7 (N = 8, 512^2: 288 against 111 us).
  auto in_turn = [&]() {
    asm("" : "+v"(lc) : "v"(G.grs), "v"(G.gys), "v"(G.Fxs), "v"(G.Fys), "v"(G.Jxs), "v"(G.Jys));
  };
  auto phi_grads = [&](int i, Real C) {
    Real gx, gy;
    grad([&](int dx, int dy) { return sphi[i][ly + kHalo + dy][lc + kHalo + dx]; }, gx, gy);
    G.grs += K.rA[i] * gx;
    G.gys += K.rA[i] * gy;
    G.Fxs += C * gx;
    G.Fys += C * gy;
  };
  auto c_grads = [&](int i) {
    Real gx, gy;
    grad([&](int dx, int dy) { return sC[i][ly + kRing + dy][lc + kRing + dx]; }, gx, gy);
    G.Jxs += K.Jc[i] * gx;
    G.Jys += K.Jc[i] * gy;
  };
  if (!kSplit || (!helper && storing)) {
#pragma unroll
    for (int i = 0; i < M; ++i) {
      phi[i] = sphi[i][ly + kHalo][lc0 + kHalo];
      const Real C = sC[i][ly + kRing][lc0 + kRing];
      if constexpr (kKeep) Cv[i] = C;
      in_turn();
      phi_grads(i, C);
      if constexpr (!kR1 && !kSplit) c_grads(i);
    }
    Acc divx = Acc(0), divy = Acc(0);
    if constexpr (kR1) {
      const int s0 = ly + 1;
      const int sN = wall && y0 + ly == ny - 1 ? s0 : s0 + 1,
                sS = wall && y0 + ly == 0 ? s0 : s0 - 1;
      auto q = [&](int c) {
        return [&, c](int dx, int dy) {
          return sQ[c][dy == 0 ? s0 : (dy > 0 ? sN : sS)][lc0 + 1 + dx];
        };
      };
      divx = ddx_central(q(0)) + ddy_central(q(1));
      divy = ddx_central(q(2)) + ddy_central(q(3));
    }
    f = flow_node<N, Real, kR1>(KD, phi, G, divx, divy, g);
  }
  if constexpr (kSplit) {
    if (helper) {
      if constexpr (!kR1) {
        if (storing) {
#pragma unroll
          for (int i = 0; i < M; ++i) {
            in_turn();
            c_grads(i);
          }
          sJ[0][ht] = G.Jxs;
          sJ[1][ht] = G.Jys;
        }
      }
    } else if (storing) {
      sU[0][ht] = f.ux;
      sU[1][ht] = f.uy;
    }
    __syncthreads();
    if (!storing) return;
    if (helper) {
      f.ux = sU[0][ht];
      f.uy = sU[1][ht];
    } else if constexpr (!kR1) {
      G.Jxs = sJ[0][ht];
      G.Jys = sJ[1][ht];
    }
  }
  const Rsrc wh = row_rsrc(d.dst[0], rbh * (uint32_t)ny, 0),
             wg = row_rsrc(d.dst[1], rbg * (uint32_t)ny, 0),
             wp = row_rsrc(d.dst[2], rbp * (uint32_t)ny, 0);
  const uint32_t oc = (uint32_t)(x0 + lx) * SZ, yr = (uint32_t)(y0 + ly);
  const uint32_t oh = yr * rbh + oc, og = yr * rbg + oc, op = yr * rbp + oc;
  // plain stores: the state is read back by the next launch from L2 or MALL
  auto sg = [&](int plane, Real v) { bst<Real, false>(wg, og, (uint32_t)plane * pb, v); };
  auto sh = [&](int plane, Real v) { bst<Real, false>(wh, oh, (uint32_t)plane * pb, v); };
  auto sp = [&](int plane, Real v) { bst<Real, false>(wp, op, (uint32_t)plane * pb, v); };
  if (!kSplit || !helper) {
    collide_ns<N, Real, kR1>(KD, phi, G, f, g, sg);
    sp(M, (Real)f.ux);
    sp(M + 1, (Real)f.uy);
  }
#pragma unroll
  for (int j = 0; j < kPh; ++j)
    if (j < nph) {
      Real pj, Cj;
      if constexpr (kKeep) {
        pj = phi[j];
        Cj = Cv[j];
      } else {
        pj = sphi[ph0 + j][ly + kHalo][lc0 + kHalo];
        Cj = sC[ph0 + j][ly + kRing][lc0 + kRing];
      }
      collide_ch<Real>(K, ph0 + j, pj, Cj, f.ux, f.uy, hi[j], pu, h[j], sh, sp);
    }
}

// The most 8-row tiles of a launch with two threads per node: while every
// workgroup is resident at once, one per compute unit, or two where the
// registers allow four waves per SIMD (FP32, N = 2 FP64).  A step with and
// without: 256 x 256 (256 tiles) FP32 N = 5 9.4 / 10.9 us; 385 x 257 (429
// tiles) FP32 N = 5 13.8 / 14.8, N = 6 16.4 / 17.3, N = 8 20.0 / 22.2, FP64
// N = 3 12.4 / 12.5, N = 5 24.0 / 19.3; 512 x 512 (1024 tiles) FP32 N = 5
// 25.5 / 23.5.  With the most phases one thread holds so many registers that
// two per node are faster at any count (620 x 620, 1560 tiles: FP32 N = 8
// 58.4 / 61.7, mixed 63.6 / 80.9; FP64 mixed N = 8 on 448 x 448 78 / 96).
template <int N, typename Real>
constexpr int help_limit() {
  constexpr bool f32 = sizeof(Real) == 4;
  constexpr bool big = f32 && N == 8 && NPL_GS == kSchemeRemark1;  // 129 registers
  if (f32 ? N >= 7 && !big : N == 8 && NPL_GS != kSchemeCentral) return INT_MAX;
  return kComputeUnits * ((f32 && !big) || N == 2 ? 2 : 1);
}

template <int N, typename Real, int TY, bool kHelp>
hipError_t launch_k(const TileArgs &a, int nblocks, hipStream_t st) {
  hipLaunchKernelGGL((k_tile<N, Real, TY, NPL_GS, kHelp>), dim3(nblocks),
                     dim3(kTW * TY * (kHelp ? 2 : 1)), 0, st, a);
  return hipGetLastError();
}

template <int N, typename Real>
hipError_t launch_ty(int ty, const TileArgs &a, int nblocks, hipStream_t st) {
  // 4 rows: two threads per node at any count (FP64 N = 3 on 512 x 512, 2048
  // tiles, 23.2 us a step against 25.0)
  if (ty == 4) return launch_k<N, Real, 4, true>(a, nblocks, st);
  if constexpr (tile12_built(N, (int)sizeof(Real)))
    if (ty == 12) return launch_k<N, Real, 12, true>(a, nblocks, st);
  if (ty != 8) return hipErrorInvalidValue;
  if constexpr (help_limit<N, Real>() < INT_MAX)
    if (nblocks > help_limit<N, Real>()) return launch_k<N, Real, 8, false>(a, nblocks, st);
  return launch_k<N, Real, 8, true>(a, nblocks, st);
}

template <int N>
hipError_t launch_n(int precision, int ty, const TileArgs &a, int nblocks, hipStream_t st) {
  return precision == 64 ? launch_ty<N, double>(ty, a, nblocks, st)
                         : launch_ty<N, float>(ty, a, nblocks, st);
}

}  // namespace

#if NPL_GS == 0
#define NPL_SCHEME_FN(name) name##_central
#elif NPL_GS == 1
#define NPL_SCHEME_FN(name) name##_mixed
#else
#define NPL_SCHEME_FN(name) name##_remark1
#endif

hipError_t NPL_SCHEME_FN(launch_tile)(int N, int precision, int ty, const TileArgs &a,
                                      int nblocks, hipStream_t st) {
  if (nblocks <= 0) return hipSuccess;
  switch (N) {
    case 2: return launch_n<2>(precision, ty, a, nblocks, st);
    case 3: return launch_n<3>(precision, ty, a, nblocks, st);
    case 4: return launch_n<4>(precision, ty, a, nblocks, st);
    case 5: return launch_n<5>(precision, ty, a, nblocks, st);
    case 6: return launch_n<6>(precision, ty, a, nblocks, st);
    case 7: return launch_n<7>(precision, ty, a, nblocks, st);
    case 8: return launch_n<8>(precision, ty, a, nblocks, st);
    default: return hipErrorInvalidValue;
  }
}

#if NPL_GS == 0
hipError_t launch_tile(int N, int precision, int scheme, int ty, const TileArgs &a, int nblocks,
                       hipStream_t st) {
  return scheme == kSchemeMixed     ? launch_tile_mixed(N, precision, ty, a, nblocks, st)
         : scheme == kSchemeRemark1 ? launch_tile_remark1(N, precision, ty, a, nblocks, st)
                                    : launch_tile_central(N, precision, ty, a, nblocks, st);
}

hipError_t launch_geom_step(int N, int precision, int scheme, const StepGeom &g, const StepArgs &a,
                            int nblocks, const DomDesc *one, hipStream_t st) {
  if (!g.ty) return launch_step(N, precision, scheme, g.bw, a, nblocks, st);
  TileArgs t{};
  t.s = a;
  if (one) {
    const int par = (a.substep + one->parity0) & 1;
    const uint32_t sz = (uint32_t)(precision / 8);
    t.d.src[0] = one->h[par];
    t.d.src[1] = one->g[par];
    t.d.src[2] = one->prev[par];
    t.d.dst[0] = one->h[par ^ 1];
    t.d.dst[1] = one->g[par ^ 1];
    t.d.dst[2] = one->prev[par ^ 1];
    t.d.pb = (uint32_t)one->ps[0] * sz;
    for (int G = 0; G < 3; ++G) t.d.rb[G] = (uint32_t)one->rs[G] * sz;
    t.d.nx = one->nx;
    t.d.ny = one->ny;
    t.d.wall = one->wall;
    tile_grid(one->nx, one->ny, g.ty, t);
    if (t.ntx) nblocks = (int)(t.per * 8);
  }
  return launch_tile(N, precision, scheme, g.ty, t, nblocks, st);
}
#endif

}  // namespace nplbm
