// node_math3.h -- the per-node arithmetic of the D3Q15 step, shared by the
// marching kernel (step3d_kernel.hip) and the node kernels
// (step3n_kernel.hip) so that a node's new state does not depend on which
// of them advances it; contraction as in node_math.h.
//
// Stencils on D3Q15 (eq:N31 with the weights 1/9 and 1/72, c_s^2 = 1/3):
//   lap   = (8 sum_faces + sum_corners - 56 zeta) / 12
//   d/dx  = (8 (E - W) + sum_corners c_x zeta) / 24     (likewise y, z)
#pragma once

#include "node_math.h"

#include "lattice3.h"

namespace nplbm {

// c_k . v; c_k has components 0 and +-1, so no product is formed
template <typename T>
__device__ __forceinline__ T cdot3(int k, const T (&v)[3]) {
  const int c[3] = {ex3(k), ey3(k), ez3(k)};
  T s = T(0);
  bool first = true;
#pragma unroll
  for (int d = 0; d < 3; ++d)
    if (c[d]) {
      const T t = c[d] > 0 ? v[d] : -v[d];
      s = first ? t : s + t;
      first = false;
    }
  return s;
}

// eq:N31b on D3Q15; f(dx, dy, dz)
template <typename Real, typename F>
__device__ __forceinline__ Real lap_node3(F f) {
  const Real faces = (f(1, 0, 0) + f(-1, 0, 0)) + (f(0, 1, 0) + f(0, -1, 0)) +
                     (f(0, 0, 1) + f(0, 0, -1));
  const Real corners = ((f(1, 1, 1) + f(-1, 1, 1)) + (f(1, -1, 1) + f(-1, -1, 1))) +
                       ((f(1, 1, -1) + f(-1, 1, -1)) + (f(1, -1, -1) + f(-1, -1, -1)));
  return (Real(8) * faces + corners - Real(56) * f(0, 0, 0)) * (Real(1) / Real(12));
}

// Chemical potentials of one node (eq:N18 line 3 with eq:N17); f(i, dx, dy,
// dz) is phi_i at the offset, store(i, C_i) takes the results.
template <int N, typename Real, typename F, typename S>
__device__ __forceinline__ void chem_node3(const NPL_CONST Consts<Real> &K, F f, S store) {
  constexpr int M = N - 1;
  Real phi[M], lap[M];
#pragma unroll
  for (int i = 0; i < M; ++i) {
    phi[i] = f(i, 0, 0, 0);
    lap[i] = lap_node3<Real>([&](int dx, int dy, int dz) { return f(i, dx, dy, dz); });
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

// eq:N31a on D3Q15; f(dx, dy, dz)
template <typename Real, typename F>
__device__ __forceinline__ void grad_node3(F f, Real (&g)[3]) {
  const Real upp = f(1, 1, 1), upm = f(-1, 1, 1), ump = f(1, -1, 1), umm = f(-1, -1, 1);
  const Real dpp = f(1, 1, -1), dpm = f(-1, 1, -1), dmp = f(1, -1, -1), dmm = f(-1, -1, -1);
  const Real cx = ((upp - upm) + (ump - umm)) + ((dpp - dpm) + (dmp - dmm));
  const Real cy = ((upp + upm) - (ump + umm)) + ((dpp + dpm) - (dmp + dmm));
  const Real cz = ((upp + upm) + (ump + umm)) - ((dpp + dpm) + (dmp + dmm));
  g[0] = (Real(8) * (f(1, 0, 0) - f(-1, 0, 0)) + cx) * (Real(1) / Real(24));
  g[1] = (Real(8) * (f(0, 1, 0) - f(0, -1, 0)) + cy) * (Real(1) / Real(24));
  g[2] = (Real(8) * (f(0, 0, 1) - f(0, 0, -1)) + cz) * (Real(1) / Real(24));
}

// Sums over the phases of what the NS part needs: rho and mu (in FP64, see
// node_math.h), grad rho, F_s and J~ (in the state type).
template <typename Real>
struct Sums3 {
  Acc rho, mu;
  Real gr[3], F[3], J[3];
};
template <int N, typename Real>
__device__ __forceinline__ Sums3<Real> sums3_begin(const NPL_CONST Consts<double> &KD) {
  return {KD.ra, KD.ma, {Real(0), Real(0), Real(0)}, {Real(0), Real(0), Real(0)},
          {Real(0), Real(0), Real(0)}};
}
template <typename Real>
__device__ __forceinline__ void sums3_add(const NPL_CONST Consts<Real> &K,
                                          const NPL_CONST Consts<double> &KD, int i, Real phi,
                                          Real C, const Real (&gp)[3], const Real (&gc)[3],
                                          Sums3<Real> &S) {
  S.rho += KD.rA[i] * phi;
  S.mu += KD.mA[i] * phi;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    S.gr[d] += K.rA[i] * gp[d];
    S.F[d] += C * gp[d];
    S.J[d] += K.Jc[i] * gc[d];
  }
}

// Makes x, an index of the next phase's stencil reads, wait for the sums so
// far (an empty asm takes both), so that the compiler does not issue the
// reads of all phases first and hold them.
template <typename Real>
__device__ __forceinline__ void sums3_order(int &x, const Sums3<Real> &S) {
  asm("" : "+v"(x) : "v"(S.gr[0]), "v"(S.gr[1]), "v"(S.gr[2]), "v"(S.F[0]), "v"(S.F[1]),
      "v"(S.F[2]), "v"(S.J[0]), "v"(S.J[1]), "v"(S.J[2]));
}

// Both collisions of one node.  g[1..14] and pu: pulled NS populations and
// stored previous u.  phase(i, h, hi, phi, C) gives phase i's pulled CH
// populations (h[0] the stored deviation), stored previous phi, phi and C.
// sg, sh, sp (plane, v) store into the NS, CH and previous-step groups.
template <int N, typename Real, typename PH, typename SG, typename SH, typename SP>
__device__ __forceinline__ void collide_node3(const NPL_CONST Consts<Real> &K,
                                              const NPL_CONST Consts<double> &KD,
                                              const Sums3<Real> &S, const Real (&g)[15],
                                              const Real (&pu)[3], PH phase, SG sg, SH sh,
                                              SP sp) {
  constexpr int M = N - 1;
  const Acc rho = S.rho;
  const Acc gr[3] = {S.gr[0], S.gr[1], S.gr[2]}, J[3] = {S.J[0], S.J[1], S.J[2]};
  Acc F[3] = {S.F[0], S.F[1], S.F[2]};
  F[0] += rho * KD.gx;
  F[1] += rho * KD.gy;
  F[2] += rho * KD.gz;
  const Acc irho = Acc(1) / rho;
  Acc itau, srcg, theta;
  if (KD.const_tau) {
    itau = KD.itau_g;
    srcg = KD.src_g;
    theta = KD.theta_g;
  } else {
    ns_relaxation(S.mu, rho, irho, itau, srcg, theta);
  }
  Acc m[3] = {Acc(0), Acc(0), Acc(0)}, sumg = Acc(0);
#pragma unroll
  for (int k = 1; k < 15; ++k) {
    if (ex3(k)) m[0] += Acc(ex3(k)) * g[k];
    if (ey3(k)) m[1] += Acc(ey3(k)) * g[k];
    if (ez3(k)) m[2] += Acc(ez3(k)) * g[k];
    sumg += g[k];
  }
  Acc u[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) u[d] = (m[d] + Acc(0.5) * F[d]) * irho;  // eq:N22_1
  const Acc usq = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
  const Acc udr = u[0] * gr[0] + u[1] * gr[1] + u[2] * gr[2];
  // eq:N23 with w_0 = 2/9: c_s^2 / (1 - w_0) = 3/7, rho s_0 = -(1/3) rho |u|^2
  const Acc p = Acc(3) / Acc(7) * (sumg + Acc(0.5) * udr - Acc(1) / Acc(3) * rho * usq);
  const Acc uF = u[0] * F[0] + u[1] * F[1] + u[2] * F[2];
  const Acc Ju = J[0] * u[0] + J[1] * u[1] + J[2] * u[2];
  // isotropic part of eq:N20_1: u.grad(rho) - tr(T) / (2 c_s^2)
  const Acc gbase = udr - Acc(1.5) * (Acc(2) * uF + Acc(2) / Acc(3) * udr + theta * Ju);
  // eq:24 with g^eq and G split into the parts even and odd in c_k, each
  // pair of opposite directions evaluated once
  const Acc keep = Acc(1) - itau;
  const Acc e0 = Acc(3) * p - Acc(1.5) * rho * usq;
#pragma unroll
  for (int k = 1; k < 15; ++k) {
    if (opp3(k) < k) continue;
    const int ko = opp3(k);
    const Acc w = w3<Acc>(k);
    const Acc cu = cdot3(k, u), cF = cdot3(k, F), cr = cdot3(k, gr), cJ = cdot3(k, J);
    const Acc ev =
        w * (itau * (e0 + Acc(4.5) * rho * cu * cu) +
             srcg * (gbase + Acc(4.5) * cu * (Acc(2) * cF + Acc(2) / Acc(3) * cr + theta * cJ)));
    const Acc od = w * Acc(3) * (itau * rho * cu + srcg * cF);
    sg(k - 1, (Real)(keep * g[k] + ev + od));
    sg(ko - 1, (Real)(keep * g[ko] + ev - od));
  }
#pragma unroll
  for (int i = 0; i < M; ++i) {
    phase(i, [&](const Real(&h)[15], Real pp, Real phi, Real C) {
      Real ps[3], dd[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        ps[d] = phi * u[d];
        dd[d] = ps[d] - pp * pu[d];  // eq:N27
      }
      const Real ec = K.eta_i[i] * C;
      const Real it = K.itau_i[i], sr = K.src_i[i];
      // eq:N24 with h^eq (eq:N25) and R_k (eq:N26) split into the parts
      // even and odd in c_k, per pair of opposite directions
      const Real kp = Real(1) - it;
      Real hsum = Real(0);
#pragma unroll
      for (int k = 1; k < 15; ++k) {
        if (opp3(k) < k) continue;
        const int ko = opp3(k);
        const Real w = w3<Real>(k);
        const Real ev = it * w * ec;
        const Real od = w * Real(3) * (it * cdot3(k, ps) + sr * cdot3(k, dd));
        const Real hn = kp * h[k] + ev + od;
        const Real ho = kp * h[ko] + ev - od;
        hsum += hn + ho;
        sh(i * 15 + k, hn);
        sh(i * 15 + ko, ho);
      }
      // phi_i = pp + lo exactly; fl(phi_i) is stored as the new previous
      // phi and the k = 0 slot keeps (pp + lo - fl(phi_i)) - sum h_k
      Real lo = h[0];
#pragma unroll
      for (int k = 1; k < 15; ++k) lo += h[k];
      const Real bb = phi - pp;
      const Real err = (pp - (phi - bb)) + (lo - bb);
      sh(i * 15, err - hsum);
      sp(i, phi);
    });
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) sp(M + d, (Real)u[d]);
}

}  // namespace nplbm
