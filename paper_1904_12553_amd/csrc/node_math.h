// node_math.h -- the per-node arithmetic of the 2-D step (D2Q9), shared by
// the marching kernel (step_kernel.hip) and the tile kernel
// (tile_kernel.hip) so that a node's new state does not depend on which of
// the two advances it.
//
// Contraction: with the compiler's default, whether a product and a sum in
// two statements become one fused operation depends on the code around
// them, so two kernels that inline the same function can round differently.
// The pragma below restricts fusing to single expressions, where the choice
// is made from the source alone; both kernels include this header first and
// are compared bitwise in the tests.
#pragma once

#pragma clang fp contract(on)

#include "buffer_io.h"
#include "lattice.h"
#include "nplbm_internal.h"
#include "relaxation.h"

namespace nplbm {

// Address spaces: the descriptors and constants are read-only for the whole
// launch and uniform per workgroup, so they are read through constant
// (scalar-load) pointers.
#define NPL_CONST __attribute__((address_space(4)))

template <typename Real>
__device__ __forceinline__ const NPL_CONST Consts<Real> *consts_of(const NPL_CONST DomDesc *d);
template <>
__device__ __forceinline__ const NPL_CONST Consts<double> *consts_of<double>(
    const NPL_CONST DomDesc *d) {
  return &d->cd;
}
template <>
__device__ __forceinline__ const NPL_CONST Consts<float> *consts_of<float>(
    const NPL_CONST DomDesc *d) {
  return &d->cf;
}

// The NS part of the collision (density, u, p, g^eq, G and the g update)
// is evaluated in FP64 arithmetic in both modes; the FP32 mode still
// stores FP32 populations.  Evaluated in FP32, the rounding of g^eq
// and of the update leaves each node's momentum off by a fraction of an
// ulp, in the same direction wherever the flow state repeats (inside a
// moving droplet), so droplets gain momentum steadily and interfaces drift
// as t^2: FP32 vs FP64 on the 512^2 N = 4 droplet collision went from
// 2.6e-5 to 7e-8 in c after 2000 steps (2e-3 to 7e-7 after 50000), for
// 2.7% more kernel time, most of which the evaluation per pair of
// opposite directions below won back.
using Acc = double;

// c_k . (a, b); c_k has components 0 and +-1, so no product is formed
template <typename T>
__device__ __forceinline__ T cdot(int k, T a, T b) {
  const int cx = cxk(k), cy = cyk(k);
  if (cy == 0) return cx > 0 ? a : -a;
  if (cx == 0) return cy > 0 ? b : -b;
  return (cx > 0 ? a : -a) + (cy > 0 ? b : -b);
}

// lo part of phi_i: the stored deviation of h_0 plus the moving populations
template <typename Real>
__device__ __forceinline__ Real lo_sum(const Real (&h)[9]) {
  Real lo = h[0];
#pragma unroll
  for (int k = 1; k < 9; ++k) lo += h[k];
  return lo;
}

// Chemical potentials of one node from the phi around it (eq:N31b, eq:N18
// line 3 with eq:N17).  f(i, dx, dy) is phi_i at the offset; the sums are
// symmetric in y, so a march may name either neighbour row dy = +1.
// store(i, C_i) takes the results.
template <int N, typename Real, typename F, typename S>
__device__ __forceinline__ void chem_node(const NPL_CONST Consts<Real> &K, F f, S store) {
  constexpr int M = N - 1;
  Real phi[M], lap[M];
#pragma unroll
  for (int i = 0; i < M; ++i) {
    const Real c = f(i, 0, 0);
    const Real e = f(i, 1, 0), w = f(i, -1, 0);
    const Real n = f(i, 0, 1), s = f(i, 0, -1);
    const Real ne = f(i, 1, 1), nw = f(i, -1, 1);
    const Real se = f(i, 1, -1), sw = f(i, -1, -1);
    // eq:N31b on D2Q9: (4 sum_axis + sum_diag - 20 zeta) / 6
    lap[i] = (Real(4) * ((e + w) + (n + s)) + ((ne + nw) + (se + sw)) - Real(20) * c) *
             (Real(1) / Real(6));
    phi[i] = c;
  }
  Real wv[N];
#pragma unroll
  for (int k = 0; k < N; ++k) {
    Real ck = K.ca[k];
#pragma unroll
    for (int i = 0; i < M; ++i) ck += K.cA[k][i] * phi[i];
    wv[k] = ck * (Real(1) - ck) * (Real(1) - Real(2) * ck);
  }
#pragma unroll
  for (int i = 0; i < M; ++i) {
    Real Ci = Real(0);
#pragma unroll
    for (int j = 0; j < M; ++j) Ci -= K.lam[i][j] * lap[j];
#pragma unroll
    for (int k = 0; k < N; ++k) Ci += K.KH[k][i] * wv[k];
    store(i, Ci);
  }
}

// eq:N31a on D2Q9: d/dx = [4 (E - W) + (NE - NW + SE - SW)] / 12; f(dx, dy)
template <typename Real, typename F>
__device__ __forceinline__ void grad_central(F f, Real &gx, Real &gy) {
  const Real e = f(1, 0), w = f(-1, 0);
  const Real n = f(0, 1), s = f(0, -1);
  const Real ne = f(1, 1), nw = f(-1, 1);
  const Real se = f(1, -1), sw = f(-1, -1);
  gx = (Real(4) * (e - w) + ((ne - nw) + (se - sw))) * (Real(1) / Real(12));
  gy = (Real(4) * (n - s) + ((ne + nw) - (se + sw))) * (Real(1) / Real(12));
}

// eq:N40 summed over the D2Q9 directions.  Per direction c the
// difference is -z(x+2c) + 5 z(x+c) - 3 z(x) - z(x-c); with w_c, c_x
// and 1/(4 c_s^2) the z(x) terms cancel and opposite directions pair:
//   d/dx = [24 (E - W) - 4 (E2 - W2) + 6 (NE - NW + SE - SW)
//           - (NE2 - NW2 + SE2 - SW2)] / 48
// (E2 = z(x+2, y), NE2 = z(x+2, y+2), ...), and likewise d/dy.
template <typename Real, typename F>
__device__ __forceinline__ void grad_two_hop(F f, Real &gx, Real &gy) {
  const Real e = f(1, 0), w = f(-1, 0);
  const Real e2 = f(2, 0), w2 = f(-2, 0);
  const Real n = f(0, 1), s = f(0, -1);
  const Real n2 = f(0, 2), s2 = f(0, -2);
  const Real ne = f(1, 1), nw = f(-1, 1);
  const Real se = f(1, -1), sw = f(-1, -1);
  const Real ne2 = f(2, 2), nw2 = f(-2, 2);
  const Real se2 = f(2, -2), sw2 = f(-2, -2);
  gx = (Real(24) * (e - w) - Real(4) * (e2 - w2) + Real(6) * ((ne - nw) + (se - sw)) -
        ((ne2 - nw2) + (se2 - sw2))) *
       (Real(1) / Real(48));
  gy = (Real(24) * (n - s) - Real(4) * (n2 - s2) + Real(6) * ((ne + nw) - (se + sw)) -
        ((ne2 + nw2) - (se2 + sw2))) *
       (Real(1) / Real(48));
}

// Remark 1: the derivatives of one product J~_b u_a (eq:N31a, in FP64);
// f(dx, dy) is the product at the offset
template <typename F>
__device__ __forceinline__ Acc ddx_central(F f) {
  return (Acc(4) * (f(1, 0) - f(-1, 0)) + ((f(1, 1) - f(-1, 1)) + (f(1, -1) - f(-1, -1)))) *
         (Acc(1) / Acc(12));
}
template <typename F>
__device__ __forceinline__ Acc ddy_central(F f) {
  return (Acc(4) * (f(0, 1) - f(0, -1)) + ((f(1, 1) + f(-1, 1)) - (f(1, -1) + f(-1, -1)))) *
         (Acc(1) / Acc(12));
}

// Sums over the phases of the gradient terms (in the state type: measured,
// FP64 there changes nothing): grad rho, F_s and J~.
template <typename Real>
struct GradSums {
  Real grs, gys, Fxs, Fys, Jxs, Jys;
};

// Density, force and velocity of a node.
struct NodeFlow {
  Acc rho, irho, Fx, Fy, ux, uy;
};

// phi: order parameters; G: the sums above; divx, divy: -div(J~ u) of
// Remark 1 (0 otherwise); gin[1..8] the pulled NS populations.
template <int N, typename Real, bool kR1>
__device__ __forceinline__ NodeFlow flow_node(const NPL_CONST Consts<double> &KD,
                                              const Real (&phi)[N - 1], const GradSums<Real> &G,
                                              Acc divx, Acc divy, const Real (&gin)[9]) {
  NodeFlow f;
  f.rho = KD.ra;
#pragma unroll
  for (int i = 0; i < N - 1; ++i) f.rho += KD.rA[i] * phi[i];
  f.Fx = G.Fxs;
  f.Fy = G.Fys;
  f.Fx += f.rho * KD.gx;
  f.Fy += f.rho * KD.gy;
  if constexpr (kR1) {
    f.Fx -= divx;
    f.Fy -= divy;
  }
  f.irho = Acc(1) / f.rho;
  Acc g[9];
#pragma unroll
  for (int k = 1; k < 9; ++k) g[k] = gin[k];
  const Acc mx = (g[1] - g[3]) + (g[5] - g[6]) + (g[8] - g[7]);
  const Acc my = (g[2] - g[4]) + (g[5] + g[6]) - (g[7] + g[8]);
  f.ux = (mx + Acc(0.5) * f.Fx) * f.irho;  // eq:N22_1
  f.uy = (my + Acc(0.5) * f.Fy) * f.irho;
  return f;
}

// NS collision of a node; sg(plane, v) stores into the NS group.
template <int N, typename Real, bool kR1, typename SG>
__device__ __forceinline__ void collide_ns(const NPL_CONST Consts<double> &KD,
                                           const Real (&phi)[N - 1], const GradSums<Real> &G,
                                           const NodeFlow &f, const Real (&gin)[9], SG sg) {
  constexpr int M = N - 1;
  const Acc rho = f.rho, Fx = f.Fx, Fy = f.Fy, ux = f.ux, uy = f.uy;
  const Acc grx = G.grs, gry = G.gys, Jx = G.Jxs, Jy = G.Jys;
  Acc itau, srcg, theta;
  if (KD.const_tau) {
    itau = KD.itau_g;
    srcg = KD.src_g;
    theta = KD.theta_g;
  } else {
    Acc mu = KD.ma;
#pragma unroll
    for (int i = 0; i < M; ++i) mu += KD.mA[i] * phi[i];
    ns_relaxation(mu, rho, f.irho, itau, srcg, theta);
  }
  Acc g[9];
#pragma unroll
  for (int k = 1; k < 9; ++k) g[k] = gin[k];
  Acc sumg = g[1];
#pragma unroll
  for (int k = 2; k < 9; ++k) sumg += g[k];
  const Acc usq = ux * ux + uy * uy;
  const Acc udr = ux * grx + uy * gry;
  // eq:N23: p = c_s^2 / (1 - w_0) [sum_{k!=0} g_k + u.grad(rho)/2 + rho s_0(u)]
  const Acc p = Acc(0.6) * (sumg + Acc(0.5) * udr - Acc(2) / Acc(3) * rho * usq);
  const Acc uF = ux * Fx + uy * Fy;
  const Acc Ju = Jx * ux + Jy * uy;
  // isotropic part of eq:N20_1: u.grad(rho) - tr(T) / (2 c_s^2)
  const Acc gbase =
      udr - Acc(1.5) * (Acc(2) * uF + Acc(2) / Acc(3) * udr + (kR1 ? Acc(0) : theta * Ju));
  // g* = (1 - 1/tau) g + g^eq / tau + (1 - 1/(2 tau)) G (eq:24), with
  // g^eq (eq:25) and G (eq:N20_1) split into the parts even and odd in
  // c_k: opposite directions share the even part and negate the odd one,
  // so each pair is evaluated once
  const Acc keep = Acc(1) - itau;
  const Acc e0 = Acc(3) * p - Acc(1.5) * rho * usq;
#pragma unroll
  for (int k = 1; k < 9; ++k) {
    if (oppk(k) < k) continue;
    const int ko = oppk(k);
    const Acc w = wk<Acc>(k);
    const Acc cu = cdot(k, ux, uy), cF = cdot(k, Fx, Fy);
    const Acc cr = cdot(k, grx, gry), cJ = cdot(k, Jx, Jy);
    const Acc ev = w * (itau * (e0 + Acc(4.5) * rho * cu * cu) +
                        srcg * (gbase + Acc(4.5) * cu *
                                            (Acc(2) * cF + Acc(2) / Acc(3) * cr +
                                             (kR1 ? Acc(0) : theta * cJ))));
    const Acc od = w * Acc(3) * (itau * rho * cu + srcg * cF);
    sg(k - 1, (Real)(keep * g[k] + ev + od));
    sg(ko - 1, (Real)(keep * g[ko] + ev - od));
  }
}

// CH collision of one phase of a node: phi, C its order parameter and chemical
// potential, pp its previous order parameter, h its pulled populations
// (element 0 the stored deviation of h_0), ux, uy the velocity and pu the
// previous one.  sh(plane, v) stores into the CH group, sp(i, v) into the
// previous-step group.
template <typename Real, typename SH, typename SP>
__device__ __forceinline__ void collide_ch(const NPL_CONST Consts<Real> &K, int i, Real phi,
                                           Real C, Acc ux, Acc uy, Real pp, const Real (&pu)[2],
                                           const Real (&h)[9], SH sh, SP sp) {
  const Real psx = phi * ux, psy = phi * uy;
  const Real dx = psx - pp * pu[0], dy = psy - pp * pu[1];  // eq:N27
  const Real ec = K.eta_i[i] * C;
  const Real it = K.itau_i[i], sr = K.src_i[i];
  // h* = (1 - 1/tau_i) h + h^eq / tau_i + R_k with h^eq (eq:N25) and R_k
  // (eq:N26) split into the parts even and odd in c_k, per pair of
  // opposite directions
  const Real kp = Real(1) - it;
  Real hsum = Real(0);
#pragma unroll
  for (int k = 1; k < 9; ++k) {
    if (oppk(k) < k) continue;
    const int ko = oppk(k);
    const Real w = wk<Real>(k);
    const Real ev = it * w * ec;
    const Real od = w * Real(3) * (it * cdot(k, psx, psy) + sr * cdot(k, dx, dy));
    const Real hn = kp * h[k] + ev + od;
    const Real ho = kp * h[ko] + ev - od;
    hsum += hn + ho;
    sh(i * 9 + k, hn);
    sh(i * 9 + ko, ho);
  }
  // phi_i = pp + lo exactly; phi = fl(pp + lo) is stored as the new
  // previous phi and the k = 0 slot keeps (pp + lo - phi) - sum h_k
  // (error-free two-sum for the rounding part).
  const Real lo = lo_sum(h);
  const Real bb = phi - pp;
  const Real err = (pp - (phi - bb)) + (lo - bb);
  sh(i * 9, err - hsum);
  sp(i, phi);
}

// Both collisions of one node: hphase(i) names phase i's pulled CH
// populations, hi the previous phi.
template <int N, typename Real, bool kR1, typename HP, typename SG, typename SH, typename SP>
__device__ __forceinline__ void collide_node(
    const NPL_CONST Consts<Real> &K, const NPL_CONST Consts<double> &KD,
    const Real (&phi)[N - 1], const Real (&Cv)[N - 1], const GradSums<Real> &G, Acc divx,
    Acc divy, HP hphase, const Real (&hi)[N - 1], const Real (&gin)[9],
    const Real (&pu)[2], SG sg, SH sh, SP sp) {
  const NodeFlow f = flow_node<N, Real, kR1>(KD, phi, G, divx, divy, gin);
  collide_ns<N, Real, kR1>(KD, phi, G, f, gin, sg);
#pragma unroll
  for (int i = 0; i < N - 1; ++i)
    collide_ch<Real>(K, i, phi[i], Cv[i], f.ux, f.uy, hi[i], pu, hphase(i), sh, sp);
  sp(N - 1, (Real)f.ux);
  sp(N, (Real)f.uy);
}

}  // namespace nplbm
