// dimp_calib.hpp -- the stages of the calibrated step: 2-D grids, two
// materials without a history slot, van Albada limiter, split integrator.
//
// The adjoint differentiates this step, and its gradients magnify a rounding
// of a state: in a solid at a pressure far below its moduli the differences of
// p that the limiter and the predictor see carry 1e-6 of relative rounding,
// and the gradient fields follow with 1e-10 to 1e-8 of their norm (a 512x512
// plate, 1 to 8 steps, with the states one rounding apart).  So the step that
// is differentiated keeps one fixed arithmetic, the same in the forward run,
// the replay and the adjoint's recomputation, and gradients are reproduced
// from one version of the library to the next: the forms below (1/rho closures,
// IEEE quotients where they stand) are not the cheaper ones of
// dimp_device.hpp and dimp_stencil.hpp, which every other run takes.
//
// On the grids that the adjoint takes (Params::calib, whether or not gradients are
// taken) these kernels follow it: the split sweeps with their fused plastic step
// and wave speed, the initial state from primitive fields, the boundary fluxes of
// a refined patch, and the adjoint's recomputation.  The general forms stay in the
// wave speed of a given state (the first dt of device CFL steps), the source step
// called by itself, the conversion to primitive fields, the state check, and the
// unsplit integrator's passes.  A run forward only pays for it: four steps of
// 2048^2, van Albada, 2820 us against 2265 with the general stages (700^2: 420, 350).
#pragma once
#include "dimp_stencil.hpp"

namespace dimp {
namespace calib {

constexpr int D = 2, N = 2, RX = 0;
using L = Lay<D, N, RX>;
constexpr int F = L::F;

// 1/b: the hardware reciprocal refined by two Newton steps
__device__ __forceinline__ double rcp2(double b) {
  double r = __builtin_amdgcn_rcp(b);
  double e = fma(-b, r, 1.0);
  r = fma(r, e, r);
  e = fma(-b, r, 1.0);
  return fma(r, e, r);
}

__device__ __forceinline__ double vget(const double* V, int i, int j) { return dimp::vget<D, N, RX>(V, i, j); }

// ----------------------------------------------------------- closures
struct EosV {
  double Gam, invGam, pref, eref, dpref, deref, G;
};

// Sec. 2.3 closures at phasic density rho (1/rho given) and strain invariant J2
__device__ __forceinline__ EosV eos_eval(const MatP& m, double rho, double irho, double J2) {
  EosV e;
  e.Gam = m.Gam;
  e.invGam = m.invGam;
  if (m.eos != EOS_ROMENSKII) {
    e.pref = m.pref0;
    e.eref = m.eref0;
    e.dpref = 0.0;
    e.deref = 0.0;
    e.G = 0.0;
    return e;
  }
  const double x = rho * m.inv_rho0;
  const double xa = m.abar_one ? x : pow(x, m.abar);
  const double ec = m.ec_coef * (xa - 1.0) * (xa - 1.0);
  const double pc = m.K0a * x * xa * (xa - 1.0);
  const double dpc = m.dpc_coef * ((2.0 * m.abar + 1.0) * xa * xa - (m.abar + 1.0) * xa);
  double G;
  if (m.bbar_three) {
    const double x2 = x * x;
    G = m.G0 * (x2 * x2);
  } else {
    G = m.G0 * pow(x, m.bbar + 1.0);
  }
  const double GJ = G * J2;
  e.pref = pc + m.bbar * GJ;
  e.eref = ec + GJ * irho;
  e.dpref = dpc + m.bbar * (m.bbar + 1.0) * GJ * irho;
  e.deref = e.pref * irho * irho;
  e.G = G;
  return e;
}

__device__ __forceinline__ double c2_mat(const EosV& e, double rho, double irho, double p) {
  return e.dpref - rho * e.Gam * e.deref + ((1.0 + e.Gam) * p - e.pref) * irho;
}

// Hencky strain dev H ~ dev((B - adj B)/4), B = V V^T (Sec. 3.2: Bazant
// approximation with the cofactor standing in for the inverse of the
// unimodular B), and J^2 = tr(H H^T).
__device__ __forceinline__ void strain(const double* V, double H[6], double& J2) {
  double B[6];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = i; j < 3; ++j) {
      double s = 0.0;
      bool first = true;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        if (L::vq(i, k) >= 0 && L::vq(j, k) >= 0) {
          const double t = vget(V, i, k) * vget(V, j, k);
          s = first ? t : s + t;
          first = false;
        }
      }
      B[hs(i, j)] = s;
    }
  double A[6];
  A[0] = B[3] * B[5];
  A[1] = -B[1] * B[5];
  A[3] = B[0] * B[5];
  A[5] = B[0] * B[3] - B[1] * B[1];
  A[2] = A[4] = 0.0;
  double K[6];
#pragma unroll
  for (int s = 0; s < 6; ++s) K[s] = 0.25 * (B[s] - A[s]);
  const double tr = (K[0] + K[3] + K[5]) * (1.0 / 3.0);
  H[0] = K[0] - tr;
  H[3] = K[3] - tr;
  H[5] = K[5] - tr;
  H[1] = K[1];
  H[2] = K[2];
  H[4] = K[4];
  J2 = H[0] * H[0] + H[3] * H[3] + H[5] * H[5];
  J2 += 2.0 * (H[1] * H[1]);
}

// phi_l, rho_l and 1/rho_l of every material.  For two materials one
// division serves both densities and one both inverses.
struct Phases {
  double phi[N], rho[N], irho[N];
};

__device__ __forceinline__ void phases_from_partial(const double* phi_st, const double* m, Phases& Q) {
  double sphi = 0.0;
#pragma unroll
  for (int l = 0; l < N - 1; ++l) {
    Q.phi[l] = phi_st[l];
    sphi += Q.phi[l];
  }
  Q.phi[N - 1] = 1.0 - sphi;
  const double ip = rcp2(Q.phi[0] * Q.phi[1]);
  const double im = rcp2(m[0] * m[1]);
  Q.rho[0] = m[0] * (Q.phi[1] * ip);
  Q.rho[1] = m[1] * (Q.phi[0] * ip);
  Q.irho[0] = Q.phi[0] * (m[1] * im);
  Q.irho[1] = Q.phi[1] * (m[0] * im);
}

__device__ __forceinline__ void phases_from_prim(const double* phi_st, const double* rho, Phases& Q) {
  double sphi = 0.0;
#pragma unroll
  for (int l = 0; l < N - 1; ++l) {
    Q.phi[l] = phi_st[l];
    sphi += Q.phi[l];
  }
  Q.phi[N - 1] = 1.0 - sphi;
#pragma unroll
  for (int l = 0; l < N; ++l) Q.rho[l] = rho[l];
  const double ir = rcp2(rho[0] * rho[1]);
  Q.irho[0] = rho[1] * ir;
  Q.irho[1] = rho[0] * ir;
}

struct Thermo {
  EosV e[N];
  double xi, ixi;  // sum phi_l / Gamma_l and its inverse
  double rho, irho;
  double p, rhoe;
  double Gmix, c2, cL2;
};

__device__ __forceinline__ void eos_all(const Params& P, const Phases& Q, double J2, Thermo& T) {
#pragma unroll
  for (int l = 0; l < N; ++l) {
    T.e[l] = eos_eval(P.mat[l], Q.rho[l], Q.irho[l], J2);
  }
}

// pressure from the conserved energy (Appendix B pressure function without
// reactive terms).  Leaves xi and 1/xi in T.
__device__ __forceinline__ void pressure_from_rhoe(const Params& P, const Phases& Q, Thermo& T) {
  double den = 0.0, num = T.rhoe;
#pragma unroll
  for (int l = 0; l < N; ++l) {
    den += Q.phi[l] * T.e[l].invGam;
    num += Q.phi[l] * (T.e[l].pref * T.e[l].invGam - Q.rho[l] * T.e[l].eref);
  }
  T.xi = den;
  T.ixi = rcp2(den);
  T.p = num * T.ixi;
}

// mixture modulus and sound speeds (Allaire form of the mixture rule; c_L^2 =
// c^2 + 4G/(3 rho)) once p, the split and (optionally) 1/xi are known
__device__ __forceinline__ void finish(const Params& P, const Phases& Q, Thermo& T,
                                       bool have_xi, bool have_rho = false) {
  if (!have_rho) {
    double r = 0.0;
#pragma unroll
    for (int l = 0; l < N; ++l) r += Q.phi[l] * Q.rho[l];
    T.rho = r;
    T.irho = rcp2(r);
  }
  double xi = 0.0, gnum = 0.0, cnum = 0.0;
#pragma unroll
  for (int l = 0; l < N; ++l) {
    double cl2, gl;
    gl = T.e[l].invGam;
    cl2 = c2_mat(T.e[l], Q.rho[l], Q.irho[l], T.p);
    gnum += Q.phi[l] * T.e[l].G * gl;
    xi += Q.phi[l] * gl;
    cnum += (Q.phi[l] * Q.rho[l] * T.irho) * cl2 * gl;
  }
  if (!have_xi) {
    T.xi = xi;
    T.ixi = rcp2(xi);
  }
  T.Gmix = gnum * T.ixi;
  T.c2 = cnum * T.ixi;
  T.cL2 = T.c2 + (4.0 / 3.0) * T.Gmix * T.irho;
}

// conserved -> primitive of one cell; W receives the primitive vector
__device__ __forceinline__ void cons_to_prim(const Params& P, const double* U, double* W, Thermo& T,
                                             double H[6], double& J2) {
  Phases Q;
  phases_from_partial(U, U + L::M0, Q);
  double r = 0.0;
#pragma unroll
  for (int l = 0; l < N; ++l) r += U[L::M0 + l];
  const double inv_r = rcp2(r);
  T.rho = r;
  T.irho = inv_r;
  double uu = 0.0;
#pragma unroll
  for (int k = 0; k < D; ++k) {
    W[L::MOM0 + k] = U[L::MOM0 + k] * inv_r;
    uu += W[L::MOM0 + k] * W[L::MOM0 + k];
  }
  strain(U + L::V0, H, J2);
  eos_all(P, Q, J2, T);
  T.rhoe = U[L::E] - 0.5 * r * uu;
  pressure_from_rhoe(P, Q, T);
  finish(P, Q, T, true, true);
#pragma unroll
  for (int l = 0; l < N - 1; ++l) W[l] = Q.phi[l];
#pragma unroll
  for (int l = 0; l < N; ++l) W[L::M0 + l] = Q.rho[l];
  W[L::E] = T.p;
#pragma unroll
  for (int q = 0; q < L::NV; ++q) W[L::V0 + q] = U[L::V0 + q];
}

// primitive -> thermodynamic state (energy from p)
__device__ __forceinline__ void prim_thermo(const Params& P, const double* W, Thermo& T, double H[6],
                                            double& J2, bool need_energy) {
  Phases Q;
  phases_from_prim(W, W + L::M0, Q);
  strain(W + L::V0, H, J2);
  eos_all(P, Q, J2, T);
  T.p = W[L::E];
  if (need_energy) {
    double e = 0.0;
#pragma unroll
    for (int l = 0; l < N; ++l) {
      e += Q.phi[l] * ((T.p - T.e[l].pref) * T.e[l].invGam + Q.rho[l] * T.e[l].eref);
    }
    T.rhoe = e;
  }
  finish(P, Q, T, false);
}

// Mixture shear modulus G = sum(phi_l G_l / Gamma_l) / xi and strain of a
// primitive state: all the stress needs besides p
__device__ __forceinline__ double prim_shear(const Params& P, const double* W, double H[6]) {
  double phi[N];
  double sphi = 0.0;
#pragma unroll
  for (int l = 0; l < N - 1; ++l) {
    phi[l] = W[l];
    sphi += phi[l];
  }
  phi[N - 1] = 1.0 - sphi;
  double xi = 0.0, gnum = 0.0;
#pragma unroll
  for (int l = 0; l < N; ++l) {
    const double gl = P.mat[l].invGam;
    xi += phi[l] * gl;
    gnum += phi[l] * shear_modulus(P.mat[l], W[L::M0 + l]) * gl;
  }
  double J2;
  strain(W + L::V0, H, J2);
  return gnum * rcp2(xi);
}

__device__ __forceinline__ double vanalbada(double a, double b, double e2) {
  return (a * (b * b + e2) + b * (a * a + e2)) / (a * a + b * b + 2.0 * e2);
}

__device__ __forceinline__ double slope(const Params& P, int f, double wm, double w0, double wp) {
  const double a = w0 - wm, b = wp - w0;
  return vanalbada(a, b, P.va_e2[L::kind(f)]);
}

// MUSCL edges (mL, mR) of phi and the THINC-or-MUSCL pair (tL, tR).  The
// interface normal (a sqrt and two divisions) and the three transcendentals
// are only evaluated in mixed cells (Appendix A criterion); cosh and tanh of
// beta come from one exponential.
template <class Youngs>
__device__ __forceinline__ Cand phi_candidates(const Params& P, double qm, double q0, double qp, Youngs&& nd_of) {
  Cand c;
  const double s = slope(P, 0, qm, q0, qp);
  c.mL = q0 - 0.5 * s;
  c.mR = q0 + 0.5 * s;
  c.tL = c.mL;
  c.tR = c.mR;
  if (!P.thinc) return c;
  const double qmin = fmin(qm, qp);
  const double qmax = fmax(qm, qp) - qmin;
  // mixed-cell test delta < C < 1 - delta with C = (q0 - qmin + eps)/(qmax + eps),
  // multiplied through by the non-negative denominator
  const double num = q0 - qmin + P.eps, den = qmax + P.eps;
  if (!((P.delta * den < num) && (num < (1.0 - P.delta) * den) && ((qp - q0) * (q0 - qm) > 0.0))) return c;
  const double C = num / den;
  const double beta = P.beta0 * nd_of() + 0.01;
  const double eb = exp(beta);
  const double ieb = 1.0 / eb;
  const double ch = 0.5 * (eb + ieb);
  const double tb = (eb - ieb) / (eb + ieb);
  const double Bv = exp(beta * (2.0 * C - 1.0));
  const double A = (Bv / ch - 1.0) / tb;
  const double lo = qmin + 0.5 * qmax * (1.0 + A);
  const double hi = qmin + 0.5 * qmax * (1.0 + (tb + A) / (1.0 + A * tb));
  // evaluated in the increasing orientation, swapped back for a decreasing stencil
  const bool dec = (qp - qm) < 0.0;
  c.tL = dec ? hi : lo;
  c.tR = dec ? lo : hi;
  return c;
}

// stress column sigma_{k,DIR} = 2 G dev H - p delta of a primitive state
template <int DIR>
__device__ __forceinline__ void stress_col(const Params& P, const double* W, double sig[3]) {
  if (!P.any_shear) {
#pragma unroll
    for (int k = 0; k < 3; ++k) sig[k] = (k == DIR) ? -W[L::E] : 0.0;
    return;
  }
  double H[6];
  const double G = prim_shear(P, W, H);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    if (hnz<D>(k, DIR))
      sig[k] = 2.0 * G * H[hs(k, DIR)] - ((k == DIR) ? W[L::E] : 0.0);
    else
      sig[k] = 0.0;
  }
}

__device__ __forceinline__ void edges_muscl(const Params& P, const double* Wm, const double* W0, const double* Wp,
                                            const Cand& cm, const Cand& c0, const Cand& cp, double* WL, double* WR) {
#pragma unroll
  for (int f = 0; f < F; ++f) {
    const double s = slope(P, f, Wm[f], W0[f], Wp[f]);
    WL[f] = W0[f] - 0.5 * s;
    WR[f] = W0[f] + 0.5 * s;
  }
  if (P.thinc) {
    const double tm = tbv(cm, cp, c0.mL, c0.mR);
    const double tt = tbv(cm, cp, c0.tL, c0.tR);
    const bool th = tt < tm;
    WL[0] = th ? c0.tL : c0.mL;
    WR[0] = th ? c0.tR : c0.mR;
  }
}

template <int DIR>
__device__ __forceinline__ void edges_predict(const Params& P, const double* Wm, const double* W0, const double* Wp,
                                              double irho0, double rc2, const Cand& cm, const Cand& c0, const Cand& cp,
                                              double nu, double* WL, double* WR) {
  edges_muscl(P, Wm, W0, Wp, cm, c0, cp, WL, WR);
  double sL[3], sR[3];
  stress_col<DIR>(P, WL, sL);
  stress_col<DIR>(P, WR, sR);
  double dW[F];
#pragma unroll
  for (int f = 0; f < F; ++f) dW[f] = WR[f] - WL[f];
  const double un = W0[L::MOM0 + DIR];
  const double dun = dW[L::MOM0 + DIR];
  double inc[F];
#pragma unroll
  for (int l = 0; l < N - 1; ++l) inc[l] = un * dW[l];
#pragma unroll
  for (int l = 0; l < N; ++l) inc[L::M0 + l] = un * dW[L::M0 + l] + W0[L::M0 + l] * dun;
#pragma unroll
  for (int k = 0; k < D; ++k) inc[L::MOM0 + k] = un * dW[L::MOM0 + k] - (sR[k] - sL[k]) * irho0;
  inc[L::E] = un * dW[L::E] + rc2 * dun;
#pragma unroll
  for (int q = 0; q < L::NV; ++q) {
    const int a = L::vi(q), b = L::vj(q);
    double v = un * dW[L::V0 + q];
    if (a < D && L::vq(DIR, b) >= 0) v -= vget(W0 + L::V0, DIR, b) * dW[L::MOM0 + (a < D ? a : 0)];
    v += (1.0 / 3.0) * W0[L::V0 + q] * dun;
    inc[L::V0 + q] = v;
  }
  const double h = 0.5 * nu;
#pragma unroll
  for (int f = 0; f < F; ++f) {
    WL[f] -= h * inc[f];
    WR[f] -= h * inc[f];
  }
#pragma unroll
  for (int l = 0; l < N - 1; ++l) {
    WL[l] = fmin(fmax(WL[l], 0.0), 1.0);
    WR[l] = fmin(fmax(WR[l], 0.0), 1.0);
  }
}

// ----------------------------------------------------------- face flux
using Side = dimp::Side<D, N, RX>;
using FaceV = dimp::FaceV<D, N, RX>;

template <int DIR>
__device__ __forceinline__ void side_state(const Params& P, const double* W, Side& S) {
  Thermo T;
  double H[6], J2;
  prim_thermo(P, W, T, H, J2, true);
  S.rho = T.rho;
  double uu = 0.0;
#pragma unroll
  for (int k = 0; k < D; ++k) {
    S.u[k] = W[L::MOM0 + k];
    uu += S.u[k] * S.u[k];
  }
  S.E = T.rhoe + 0.5 * T.rho * uu;
  S.cl = sqrt(T.cL2);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    if (hnz<D>(k, DIR))
      S.sig[k] = 2.0 * T.Gmix * H[hs(k, DIR)] - ((k == DIR) ? T.p : 0.0);
    else
      S.sig[k] = 0.0;
  }
}

// Flux of side K: the physical flux F_K plus S_K (U*_K - U_K), the HLLC-type
// star state with velocity (S*, u*_t) and traction continuous across the
// contact and Rankine-Hugoniot across S_K.  A supersonic face passes SK = 0
// with a = inv = 1, which returns F_K exactly.
template <int DIR>
__device__ __forceinline__ void star_flux(const Params& P, const double* W, const Side& S, double SK,
                                          double a, double inv, const double ust[D], double mK,
                                          FaceV& out) {
  const double un = S.u[DIR];
  const double r = a * inv;
  const double rm1 = r - 1.0;
  const double us_face = un + SK * rm1;
  double phiN = 1.0;
#pragma unroll
  for (int l = 0; l < N - 1; ++l) {
    phiN -= W[l];
    out.F[l] = W[l] * us_face;  // phi_K u*, the same u* as in the phi source
  }
#pragma unroll
  for (int l = 0; l < N; ++l) {
    const double m = (l < N - 1 ? W[l] : phiN) * W[L::M0 + l];
    out.F[L::M0 + l] = m * un + SK * (rm1 * m);
  }
  const double rs = r * S.rho;
  double usK = 0.0, usS = 0.0;
#pragma unroll
  for (int k = 0; k < D; ++k) {
    const double mom = S.rho * S.u[k];
    out.F[L::MOM0 + k] = mom * un - S.sig[k] + SK * (rs * ust[k] - mom);
    const double sst = S.sig[k] - mK * (ust[k] - S.u[k]);
    usK += S.u[k] * S.sig[k];
    usS += ust[k] * sst;
  }
  const double Es = (S.E * a + (usK - usS)) * inv;
  out.F[L::E] = S.E * un - usK + SK * (Es - S.E);
#pragma unroll
  for (int q = 0; q < L::NV; ++q) {
    const int i = L::vi(q), j = L::vj(q);
    const double V = W[L::V0 + q];
    const bool coupled = (i < D) && (L::vq(DIR, j) >= 0);
    const double Vn = coupled ? vget(W + L::V0, DIR, j) : 0.0;
    const int ii = i < D ? i : 0;
    double Fx = V * un;
    if (coupled) Fx -= Vn * S.u[ii];
    if (i == DIR) {
      out.F[L::V0 + q] = Fx;  // normal row continuous: U* = U
    } else {
      double Vs = a * V;
      if (coupled) Vs -= Vn * (ust[ii] - S.u[ii]);
      out.F[L::V0 + q] = Fx + SK * (Vs * inv - V);
    }
  }
  out.ustar = us_face;
#pragma unroll
  for (int j = 0; j < D; ++j) out.Vn[j] = vget(W + L::V0, DIR, j);
}

template <int DIR>
__device__ __forceinline__ void face_flux(const Params& P, const double* WL, const double* WR,
                                          FaceV& out, bool wall = false) {
  Side A, B;
  side_state<DIR>(P, WL, A);
  side_state<DIR>(P, WR, B);
  const double uL = A.u[DIR], uR = B.u[DIR];
  const double SL = fmin(uL - A.cl, uR - B.cl);
  const double SR = fmax(uL + A.cl, uR + B.cl);
  const double mL = A.rho * (SL - uL);
  const double mR = B.rho * (SR - uR);
  const double iden = rcp2(mL - mR);
  double ust[D];
#pragma unroll
  for (int k = 0; k < D; ++k) ust[k] = ((A.sig[k] - B.sig[k]) + (mL * A.u[k] - mR * B.u[k])) * iden;
  // a reflective wall between a cell and its mirror image has S* = 0 exactly
  // (computed so in exact arithmetic; the GPU's round-off is not mirror-exact)
  if (wall) ust[DIR] = 0.0;
  const double Sst = ust[DIR];
  const bool supL = SL >= 0.0, supR = SR <= 0.0;
  const bool sup = supL || supR;
  const bool left = supL || (!supR && Sst > 0.0);
  const bool tie = !sup && (Sst == 0.0);
  // select side K (one star evaluation per face)
  double WK[F];
#pragma unroll
  for (int f = 0; f < F; ++f) WK[f] = left ? WL[f] : WR[f];
  Side SK;
  SK.rho = left ? A.rho : B.rho;
  SK.E = left ? A.E : B.E;
  SK.cl = 0.0;
#pragma unroll
  for (int k = 0; k < D; ++k) SK.u[k] = left ? A.u[k] : B.u[k];
#pragma unroll
  for (int k = 0; k < 3; ++k) SK.sig[k] = left ? A.sig[k] : B.sig[k];
  const double S_K = left ? SL : SR;
  const double m_K = left ? mL : mR;
  const double a = sup ? 1.0 : S_K - SK.u[DIR];
  const double inv = sup ? 1.0 : rcp2(S_K - Sst);
  star_flux<DIR>(P, WK, SK, sup ? 0.0 : S_K, a, inv, ust, m_K, out);
  if (tie) {
    // S* exactly zero: the average of both star fluxes.  A tie is never
    // 'left', so out already holds the right one; only the left one is
    // added.  (Every face between cells of a fluid at rest is a tie.)
    FaceV o1;
    const double a1 = SL - A.u[DIR];
    star_flux<DIR>(P, WL, A, SL, a1, rcp2(SL), ust, mL, o1);
#pragma unroll
    for (int f = 0; f < F; ++f) out.F[f] = 0.5 * (o1.F[f] + out.F[f]);
    out.ustar = 0.5 * (o1.ustar + out.ustar);
#pragma unroll
    for (int j = 0; j < D; ++j) out.Vn[j] = 0.5 * (o1.Vn[j] + out.Vn[j]);
  }
}

// ---------------------------------------------------------------- update
// U^{new} = U - nu (F_b - F_a) with phi's source phi div u and Vbar's sources
// (2/3) Vbar div u - u_i beta_j taken with the face velocities u* and the
// upwinded normal rows Vbar*_{n j} (cell-centre coefficients).
template <int DIR>
__device__ __forceinline__ void update_cell(const double* U, double inv_rho, const FaceV& a,
                                            const FaceV& b, double nu, double* Un) {
  const double du = b.ustar - a.ustar;
#pragma unroll
  for (int l = 0; l < N - 1; ++l) Un[l] = U[l] - nu * ((b.F[l] - a.F[l]) - U[l] * du);
#pragma unroll
  for (int f = N - 1; f < L::V0; ++f) Un[f] = U[f] - nu * (b.F[f] - a.F[f]);
#pragma unroll
  for (int q = 0; q < L::NV; ++q) {
    const int i = L::vi(q), j = L::vj(q);
    double src = (2.0 / 3.0) * U[L::V0 + q] * du;
    if (i < D && j < D) src -= (U[L::MOM0 + (i < D ? i : 0)] * inv_rho) * (b.Vn[j < D ? j : 0] - a.Vn[j < D ? j : 0]);
    Un[L::V0 + q] = U[L::V0 + q] - nu * ((b.F[L::V0 + q] - a.F[L::V0 + q]) - src);
  }
}

// The last sweep's epilogue on the new conserved state: plastic relaxation,
// and the per-direction wave speed of the result.
__device__ __forceinline__ void epilogue_cell(const Params& P, double* U, double dt, double s[D]) {
  Phases Q;
  phases_from_partial(U, U + L::M0, Q);
  double r = 0.0;
#pragma unroll
  for (int l = 0; l < N; ++l) r += U[L::M0 + l];
  const double inv_r = rcp2(r);
  double u[D], uu = 0.0;
#pragma unroll
  for (int k = 0; k < D; ++k) {
    u[k] = U[L::MOM0 + k] * inv_r;
    uu += u[k] * u[k];
  }
  // plastic step (Sec. 3.2)
  double H[6], J2;
  strain(U + L::V0, H, J2);
  const double J = sqrt(J2);
  double xi = 0.0, num = 0.0;
#pragma unroll
  for (int l = 0; l < N; ++l) {
    const MatP& m = P.mat[l];
    const double wl = Q.phi[l] * m.invGam;
    xi += wl;
    if (!m.shear) continue;
    double Jl = J;
    if (m.plast == PLAST_PERFECT) Jl = fmin(J, m.yield_s6 * rcp2(shear_modulus(m, Q.rho[l])));
    num += wl * Jl;
  }
  const double fac = (J > 0.0) ? (num * rcp2(xi)) * rcp2(J) : 0.0;
  double Mm[6], Mp[6];
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    const double id = (q == 0 || q == 3 || q == 5) ? 1.0 : 0.0;
    const double hq = (J > 0.0) ? fac * H[q] : 0.0;
    Mm[q] = id - 0.5 * hq;
    Mp[q] = id + 0.5 * hq;
  }
  double A[6];
  A[0] = Mm[3] * Mm[5] - Mm[4] * Mm[4];
  A[1] = Mm[2] * Mm[4] - Mm[1] * Mm[5];
  A[2] = Mm[1] * Mm[4] - Mm[2] * Mm[3];
  A[3] = Mm[0] * Mm[5] - Mm[2] * Mm[2];
  A[4] = Mm[2] * Mm[1] - Mm[0] * Mm[4];
  A[5] = Mm[0] * Mm[3] - Mm[1] * Mm[1];
  const double inv_det = rcp2(Mm[0] * A[0] + Mm[1] * A[1] + Mm[2] * A[2]);
#pragma unroll
  for (int q = 0; q < L::NV; ++q) {
    const int i = L::vi(q), j = L::vj(q);
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (hnz<D>(i, k) && hnz<D>(k, j)) v += A[hs(i, k)] * Mp[hs(k, j)];
    U[L::V0 + q] = v * inv_det;
  }
  // wave speed of the relaxed state
  strain(U + L::V0, H, J2);
  Thermo T;
  T.rho = r;
  T.irho = inv_r;
  eos_all(P, Q, J2, T);
  T.rhoe = U[L::E] - 0.5 * r * uu;
  pressure_from_rhoe(P, Q, T);
  finish(P, Q, T, true, true);
  const double cl = sqrt(T.cL2);
#pragma unroll
  for (int k = 0; k < D; ++k) s[k] = fabs(u[k]) + cl;
}

// The stages of one sweep for a wave holding one cell per lane (as lane_face
// and lane_sweep of dimp_lane.hpp)
template <int DIR, class LoadU, class PhiAt>
__device__ __forceinline__ void lane_face(const Params& P, LoadU&& load_U, PhiAt&& phi_at, double nu,
                                          FaceV& fa, double& irho0, bool wall) {
  double W[F];
  double rc2;
  {
    double U[F];
    load_U(U);
    Thermo T;
    double H[6], J2;
    cons_to_prim(P, U, W, T, H, J2);
    irho0 = T.irho;  // 1 / sum of partial densities
    rc2 = T.rho * T.c2;
  }
  double Wm[F], Wp[F];
#pragma unroll
  for (int f = 0; f < F; ++f) {
    Wm[f] = from_left(W[f]);
    Wp[f] = from_right(W[f]);
  }
  // phi stencil along the sweep axis for the interface normal (all lanes
  // shuffle; the normal itself is only evaluated in mixed cells)
  double phi_t[3][3], sm[3][3], sp[3][3];
  if (P.thinc) {
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      phi_t[b][1] = (b == 1) ? W[0] : phi_at(b, 1);
      sm[b][1] = from_left(phi_t[b][1]);
      sp[b][1] = from_right(phi_t[b][1]);
    }
  }
  auto normal = [&]() -> double {
    // axes (x, y): the sweep axis DIR and the transverse offset b
    double st[3][3];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const double v0 = sm[b][1], v1 = phi_t[b][1], v2 = sp[b][1];
      if (DIR == 0) {
        st[0][b] = v0; st[1][b] = v1; st[2][b] = v2;
      } else {
        st[b][0] = v0; st[b][1] = v1; st[b][2] = v2;
      }
    }
    return youngs2(st, P.dx, DIR);
  };
  // the neighbours' right (left) edge candidates by shifts
  Cand cm, cp;
  const Cand c0 = phi_candidates(P, Wm[0], W[0], Wp[0], normal);
  cm.mR = from_left(c0.mR);
  cm.tR = from_left(c0.tR);
  cp.mL = from_right(c0.mL);
  cp.tL = from_right(c0.tL);
  double WL[F], WR[F];
  edges_predict<DIR>(P, Wm, W, Wp, irho0, rc2, cm, c0, cp, nu, WL, WR);
  // face on the left of this cell: right edge of the left neighbour | my left edge
  double WRm[F];
#pragma unroll
  for (int f = 0; f < F; ++f) WRm[f] = from_left(WR[f]);
  face_flux<DIR>(P, WRm, WL, fa, wall);
}

template <int DIR, bool FUSE, class LoadU, class PhiAt>
__device__ __forceinline__ void lane_sweep(const Params& P, LoadU&& load_U, PhiAt&& phi_at, double nu,
                                           double dt, bool writer, double* Un, double* s, bool wall = false) {
  FaceV fa, fb;
  double irho0;
  lane_face<DIR>(P, load_U, phi_at, nu, fa, irho0, wall);
#pragma unroll
  for (int f = 0; f < F; ++f) fb.F[f] = from_right(fa.F[f]);
  fb.ustar = from_right(fa.ustar);
#pragma unroll
  for (int j = 0; j < D; ++j) fb.Vn[j] = from_right(fa.Vn[j]);
  {
    double U[F];
    load_U(U);
    update_cell<DIR>(U, irho0, fa, fb, nu, Un);
  }
#pragma unroll
  for (int k = 0; k < D; ++k) s[k] = 0.0;
  if (FUSE && writer) epilogue_cell(P, Un, dt, s);
}

}  // namespace calib
}  // namespace dimp
