// Test library: the boundary fluxes that a refined patch records
// (launch_amr_flux) beside the sweep whose fluxes they stand for
// (launch_sweep), on one periodic 2-D grid of a gas and a solid.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>

#include "../include/dimp.h"
#include "dimp_amr.hpp"
#include "dimp_internal.hpp"

using namespace dimp;

namespace {

MatP pack(const dimp_material& m) {
  MatP q;
  std::memset(&q, 0, sizeof q);
  q.eos = m.eos;
  q.plast = m.plast;
  q.abar_one = q.bbar_three = 1;
  if (m.eos == DIMP_EOS_ROMENSKII) {
    q.Gam = m.Gamma0;
    q.inv_rho0 = 1.0 / m.rho0;
    q.abar = m.abar;
    q.bbar = m.bbar;
    q.K0a = m.K0 / m.abar;
    q.ec_coef = m.K0 / (2.0 * m.rho0 * m.abar * m.abar);
    q.dpc_coef = m.K0 / (m.abar * m.rho0);
    q.G0 = m.G0;
    q.abar_one = (m.abar == 1.0);
    q.bbar_three = (m.bbar == 3.0);
    q.shear = (m.G0 > 0.0);
    q.yield_s6 = m.yield / std::sqrt(6.0);
  } else {
    q.Gam = m.gamma - 1.0;
    q.pref0 = -m.gamma * m.pinf;
    q.eref0 = m.eref;
  }
  q.invGam = 1.0 / q.Gam;
  return q;
}

}  // namespace

extern "C" {

// One unfused split sweep along dir of the device state U (11 fields of n[0] x
// n[1]) into Un, and the fluxes through the left (flux[.][0]) and right faces
// (flux[.][1]) of the cells at index pos along dir, transverse cells t0 .. t0 +
// len - 1.  calib: the calibrated step's arithmetic.
int flux_unit(const dimp_material* mats, const dimp_options* o, const int64_t* n, const double* dx, int calib, int dir,
              double dt, int64_t pos, int64_t t0, int64_t len, const double* U, double* Un, double* flux) {
  Params P;
  std::memset(&P, 0, sizeof P);
  for (int d = 0; d < 3; ++d) {
    P.n[d] = d < 2 ? n[d] : 1;
    P.dx[d] = d < 2 ? dx[d] : 1.0;
    P.idx[d] = 1.0 / P.dx[d];
    P.idl[d] = std::fma(-P.idx[d], P.dx[d], 1.0) / P.dx[d];
    P.bc[d] = BC_PERIODIC;
  }
  P.ncell = n[0] * n[1];
  P.limiter = o->limiter;
  P.thinc = o->thinc;
  P.beta0 = o->beta0;
  P.delta = o->delta;
  P.eps = o->eps;
  for (int i = 0; i < 6; ++i) P.va_e2[i] = (1e-6 * o->va_scale[i]) * (1e-6 * o->va_scale[i]);
  P.nmat = 2;
  for (int l = 0; l < 2; ++l) {
    P.mat[l] = pack(mats[l]);
    if (P.mat[l].shear) P.any_shear = 1;
  }
  P.prof = PROF_GAS_SOLID;
  P.calib = calib;
  P.rx.mat = -1;
  if (launch_sweep(P, 2, 0, U, Un, dt, nullptr, dir, false, nullptr, nullptr) != hipSuccess) return 1;
  const FaceSet fs{{pos, pos + 1}, t0, len};
  if (launch_amr_flux(P, 0, dir, fs, U, dt, flux, nullptr) != hipSuccess) return 2;
  return hipDeviceSynchronize() != hipSuccess;
}

}  // extern "C"
