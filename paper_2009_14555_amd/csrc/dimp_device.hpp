// dimp_device.hpp -- device-side physics of the diffuse-interface step (gfx950).
//
// Pointwise pieces of the method of arXiv 2009.14555, written for registers:
//   Mie-Grueneisen closures and mixture rules ....... Sec. 2.2, 2.3
//   reactive mixture (equal p and T split) ........... Sec. 2.3.1, Appendix B
//   strain from the stretch tensor, Pade exp ........ Sec. 3.2
//   HLLC-type flux for the whole system ............. Sec. 3.1 (flux differences)
//   THINC edges, mixed-cell test, BVD ............... Appendix A
//   plastic relaxation, reaction RK4 ................ Sec. 3.2, 3.3
// Layout and arithmetic are specialised at compile time on the dimension D,
// the number of materials N and the presence of a reactive mixture RX, so
// structural zeros of the stretch tensor never reach the FP64 pipes.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace dimp {

// ------------------------------------------------------------ parameters
struct MatP {
  int eos, plast, shear, abar_one, bbar_three, pad;
  double Gam, invGam;   // Gruneisen coefficient and its inverse
  double pref0, eref0;  // constant reference curves of ideal / stiffened gases
  double inv_rho0, abar, bbar, K0a, ec_coef, dpc_coef, G0;
  double yield_s6;      // sigma_Y / sqrt(6)
  double cv;
  // Johnson-Cook (plast == 2): sigma_Y = (c1 + c2 eps^n)(1 - theta^m), rate
  // chi0 exp((s - 1)/c3), theta = (T - T0)/(Tmelt - T0) in [0, 1]
  double jc_c1, jc_c2, jc_inv_c3, jc_n, jc_m, jc_t0, jc_inv_dT, jc_chi0;
};

// The RX template argument of the layouts and kernels: 0 no history slot;
// 1 a history slot (a reactive mixture of gases, or a Johnson-Cook solid's
// plastic strain); 2 a reactive mixture with a JWL component (the general
// Appendix B split).
// The history slot of the RX layouts holds either the reactive mixture's
// phi_y rho_y lambda (kind RXK_MIX) or the plastic strain phi_y rho_y eps_p
// of a Johnson-Cook solid y (kind RXK_EPS); the slot is transported the same
// way, the closures and sources differ.
constexpr int RXK_MIX = 0, RXK_EPS = 1;
constexpr int LAW_POWER = 0, LAW_IG = 1;
struct RxP {
  int mat, n_is2;
  int kind, gen;  // gen: a component has density-dependent (JWL) reference curves
  int law, pad;   // LAW_POWER or LAW_IG
  int jwl[2];     // component c is JWL
  double invGa, pa, ea;  // reactant: 1/Gamma, constant p_ref, e_ref
  double invGb, pb, eb;  // product (e_ref already lowered by Q)
  double iGca, iGcb;     // 1 / (Gamma C_V)
  double k, n, inv_pref;          // LAW_POWER: -k lam (max(p,0)/pref)^n
  // JWL terms of component c: A, B, R1 rho0, R2 rho0 and 1/(R1 rho0), 1/(R2 rho0)
  double jA[2], jB[2], jR1[2], jR2[2], jiR1[2], jiR2[2];
  // LAW_IG (three-term ignition and growth of F = 1 - lam): I, G1, G2, the
  // exponents b, c, d, e, g, x, y, z, threshold a, switches F_ig, F_G1,
  // F_G2, the reference density and the pressure unit
  double igI, igG1, igG2, ig_a, ig_b, ig_c, ig_d, ig_e, ig_g, ig_x, ig_y, ig_z;
  double igFig, igFG1, igFG2;
  double ig_irho0[2], ig_ipunit[2];  // inverses of the reference density and the pressure unit, and what those lack
  int ign[8];  // b, c, d, e, g, x, y, z where they are small whole numbers, else 0
};

// materials the kernels are built for: two or three (the layouts are generic
// in N; the launchers instantiate N = 2 everywhere and N = 3 on 1-D and 2-D
// grids)
constexpr int MAXMAT = 3;

struct Params {
  int64_t n[3];
  int64_t ncell;
  double dx[3], idx[3], idl[3];  // cell widths, their inverses, and what those lack of 1/dx
  int bc[3];
  int limiter, thinc, any_shear, geom;  // geom 1: cylindrical (2-D, x = r, y = z)
  double r_lo;                           // cylindrical: radius of the grid's low x face
  double beta0, delta, eps;
  double va_e2[6];  // squared van Albada epsilon per field kind
  int nmat;
  int prof;        // material profile (PROF_*), by the materials' types
  int calib, pad;  // the step the adjoint differentiates (dimp_calib.hpp)
  MatP mat[MAXMAT];
  RxP rx;
};

constexpr int EOS_IDEAL = 0, EOS_STIFFENED = 1, EOS_ROMENSKII = 2;
constexpr int PLAST_PERFECT = 1, PLAST_JC = 2;

// the RX layout's history slot is the reactive mixture's (closures of
// Appendix B apply to material y)
template <int RX>
__device__ __forceinline__ bool rx_mix(const Params& P) {
  return RX && P.rx.kind == RXK_MIX;
}
constexpr int BC_PERIODIC = 1, BC_REFLECTIVE = 2, BC_AXIS = 3;

// Material profiles.  The kernels are compiled for any materials (PROF_ANY:
// every closure behind uniform branches on the material's type, with the
// general powers of the Romenskii curves) and for the combinations the
// workloads run, with the types stated at compile time:
//   PROF_GAS_SOLID  material 0 a gas or the reactive mixture, material 1 a
//                   Romenskii solid (perfect plasticity or elastic), and no
//                   Romenskii curve with exponents other than alpha-bar = 1,
//                   beta-bar = 3 (Table 1); a third material may be either;
//                   a mixture of two gases burns by the quadratic power law,
//                   one of two JWL components by ignition and growth;
//   PROF_GAS_JC     the same with a Johnson-Cook solid in the history slot;
//   PROF_GAS_GAS    two gases.
// The chosen instance computes the same expressions.  Without the branches a
// sweep is a few long blocks that the scheduler can fill: the 2-D sweeps of
// PROF_GAS_SOLID take 122-136 VGPRs against 149-151 and hardly spill scalar
// registers (10 lane moves against 100-190); 1024 x 900 with Johnson-Cook copper
// 528 -> 394 us a pass from the profiles alone, 256^3 22260 -> 18350.
//   PROF_CALIB      not a statement about the materials: the stages of
//                   dimp_calib.hpp (Params::calib, sweeps and the initial state)
constexpr int PROF_ANY = 0, PROF_GAS_SOLID = 1, PROF_GAS_JC = 2, PROF_GAS_GAS = 3, PROF_CALIB = 4;

template <int N, int RX, int PROF>
__device__ __forceinline__ void assume_profile(const Params& P) {
  if constexpr (PROF != PROF_ANY && PROF != PROF_CALIB) {
    __builtin_assume(P.mat[0].eos != EOS_ROMENSKII);
    __builtin_assume(P.mat[0].shear == 0);
    __builtin_assume(P.mat[1].abar_one != 0);
    __builtin_assume(P.mat[1].bbar_three != 0);
    if constexpr (N == 3) {
      __builtin_assume(P.mat[2].abar_one != 0);
      __builtin_assume(P.mat[2].bbar_three != 0);
    }
    if constexpr (PROF == PROF_GAS_GAS) {
      __builtin_assume(P.mat[1].eos != EOS_ROMENSKII);
      __builtin_assume(P.mat[1].shear == 0);
      __builtin_assume(P.any_shear == 0);
    } else {
      __builtin_assume(P.mat[1].eos == EOS_ROMENSKII);
      __builtin_assume(P.mat[1].shear != 0);
      __builtin_assume(P.any_shear != 0);
    }
    if constexpr (RX != 0) {
      __builtin_assume(P.rx.kind == (PROF == PROF_GAS_JC ? RXK_EPS : RXK_MIX));
      __builtin_assume(P.rx.mat == (PROF == PROF_GAS_JC ? 1 : 0));
      if constexpr (RX == 1 && PROF == PROF_GAS_SOLID) {
        __builtin_assume(P.rx.law == LAW_POWER);
        __builtin_assume(P.rx.n_is2 != 0);
      }
      if constexpr (RX == 2) {
        __builtin_assume(P.rx.law == LAW_IG);
        __builtin_assume(P.rx.jwl[0] != 0);
        __builtin_assume(P.rx.jwl[1] != 0);
      }
    }
  }
}

// The parameters, read anew from the kernel's arguments (PROF < 0: P itself).
// They must be the kernel's first: kernels whose stages call this are launched by
// launch_params, which takes no others.  The compiler reads what a kernel uses of them
// once, at its start, and parks what exceeds the 100 scalar registers in vector
// lanes: a fused sweep of a JWL mixture had 1640-3100 lane reads among its 11800
// instructions and a three-material one 1389-1761, and the parked values took
// 15-30 vector registers.  Read anew at each stage (half step, flux, sources)
// they come through the scalar cache: 530-760 and 33-51 lane reads left, 165
// vector registers instead of 180-193; 256^3 12160 -> 11880 us.
template <int N, int RX, int PROF>
__device__ __forceinline__ const Params& fresh(const Params& P) {
  if constexpr (PROF < 0) return P;
  auto* p = (const __attribute__((address_space(4))) Params*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  const Params& q = *(const Params*)p;
  assume_profile<N, RX, PROF>(q);
  return q;
}

// kernel(P, args...) for kernels whose first parameter is Params (see fresh)
template <class... A, class... B>
static inline void launch_params(void (*kernel)(Params, A...), dim3 grid, dim3 block, size_t lds, hipStream_t st,
                                 const Params& P, B... args) {
  static_assert(sizeof...(A) == sizeof...(B), "the kernel's other arguments");
  hipLaunchKernelGGL(kernel, grid, block, lds, st, P, static_cast<A>(args)...);
}

// f(std::integral_constant<int, PROF>) for the profile that P states, among
// the ones compiled for N materials and the RX layout
template <int N, int RX, class Fn>
static inline hipError_t by_profile(const Params& P, Fn&& f) {
  if (P.prof == PROF_GAS_SOLID) return f(std::integral_constant<int, PROF_GAS_SOLID>{});
  if constexpr (RX == 1)
    if (P.prof == PROF_GAS_JC) return f(std::integral_constant<int, PROF_GAS_JC>{});
  if constexpr (RX == 0 && N == 2)
    if (P.prof == PROF_GAS_GAS) return f(std::integral_constant<int, PROF_GAS_GAS>{});
  return f(std::integral_constant<int, PROF_ANY>{});
}

// ---------------------------------------------------------------- layout
template <int D, int N, int RX>
struct Lay {
  static constexpr int NPHI = N - 1;
  static constexpr int M0 = N - 1;
  static constexpr int LAM = 2 * N - 1;
  static constexpr int MOM0 = 2 * N - 1 + (RX ? 1 : 0);
  static constexpr int E = MOM0 + D;
  static constexpr int V0 = E + 1;
  static constexpr int NV = (D == 1) ? 3 : (D == 2) ? 5 : 9;
  static constexpr int F = V0 + NV;
  __host__ __device__ static constexpr int vi(int q) {
    return D == 1 ? q : D == 2 ? (q < 2 ? 0 : q < 4 ? 1 : 2) : q / 3;
  }
  __host__ __device__ static constexpr int vj(int q) {
    return D == 1 ? q : D == 2 ? (q == 0 ? 0 : q == 1 ? 1 : q == 2 ? 0 : q == 3 ? 1 : 2) : q % 3;
  }
  // slot of Vbar(i,j) among the stored entries, -1 for a structural zero
  __host__ __device__ static constexpr int vq(int i, int j) {
    return D == 1 ? (i == j ? i : -1)
           : D == 2 ? ((i < 2 && j < 2) ? 2 * i + j : (i == 2 && j == 2) ? 4 : -1)
                    : 3 * i + j;
  }
  // field kind for the van Albada scale: 0 phi, 1 rho, 2 lambda, 3 u, 4 p, 5 Vbar
  __host__ __device__ static constexpr int kind(int f) {
    return f < NPHI ? 0 : f < 2 * N - 1 ? 1 : (RX && f == LAM) ? 2 : f < E ? 3 : f == E ? 4 : 5;
  }
};

// field f changes sign in the mirror image across a wall normal to axis d:
// the normal momentum and the stretch-tensor entries with exactly one
// normal index (V -> M V M, M the reflection)
template <int D, int N, int RX>
__host__ __device__ constexpr bool mirror_odd(int f, int d) {
  using L = Lay<D, N, RX>;
  return f == L::MOM0 + d ||
         (f >= L::V0 && f < L::F && ((L::vi(f - L::V0) == d) != (L::vj(f - L::V0) == d)));
}

// symmetric 3x3 with structural zeros: slots 00,01,02,11,12,22
template <int D>
__host__ __device__ constexpr bool hnz(int i, int j) {
  return D == 3 ? true : D == 2 ? ((i < 2 && j < 2) || (i == 2 && j == 2)) : (i == j);
}
__host__ __device__ constexpr int hs(int i, int j) {
  // not recursive: a recursive form is turned into a runtime loop in some
  // inlined contexts, and the arrays it indexes then go to scratch memory
  const int a = (i < j) ? i : j, b = (i < j) ? j : i;
  return a == 0 ? b : a == 1 ? 2 + b : 5;
}

// Neighbour exchange within a wave: lane i receives the value of lane i - 1
// (from_left) or i + 1 (from_right); lane 0 (from_left) and lane 63
// (from_right), which have no such neighbour, receive 0.  Those are halo
// lanes of every kernel that shifts this way (their results reach no lane
// that is written), and taking 0 lets the move write a fresh register
// instead of first copying the value it would otherwise keep.  Wave-wide DPP
// shifts are plain vector moves, with none of the latency of a permute
// through the LDS crossbar.
__device__ __forceinline__ double from_left(double v) {
  return __builtin_amdgcn_mov_dpp(v, 0x138 /* wave_shr:1 */, 0xf, 0xf, true);
}
__device__ __forceinline__ double from_right(double v) {
  return __builtin_amdgcn_mov_dpp(v, 0x130 /* wave_shl:1 */, 0xf, 0xf, true);
}
// the same shifts with lanes 0 and 63 keeping their own value
__device__ __forceinline__ double from_left_keep(double v) {
  return __builtin_amdgcn_update_dpp(v, v, 0x138 /* wave_shr:1 */, 0xf, 0xf, false);
}
__device__ __forceinline__ double from_right_keep(double v) {
  return __builtin_amdgcn_update_dpp(v, v, 0x130 /* wave_shl:1 */, 0xf, 0xf, false);
}

// 1/b from the hardware reciprocal r (about 2^-23 relative) refined by the
// cubic step r (1 + e + e^2), e = 1 - b r: rounded as 1/b (max error 0.5000 ulp on
// the GPU), in one instruction fewer than two Newton steps and at well under
// half the cost of an IEEE division
__device__ __forceinline__ double frcp(double b) {
  const double r = __builtin_amdgcn_rcp(b);
  const double e = fma(-b, r, 1.0);
  return fma(r, fma(e, e, e), r);
}

// a/b: the product with frcp and one correction by its residual, which rounds as an
// IEEE quotient does (max error 0.5000 ulp on the GPU, the product alone 1.46) in
// half its instructions.  The densities, the progress and what is differenced or
// cancelled afterwards are formed this way
__device__ __forceinline__ double quot(double a, double b) {
  const double r = frcp(b), q = a * r;
  return fma(fma(-b, q, a), r, q);
}

// x/b, rounded as the quotient, from the inverse i of b and what i lacks of 1/b
__device__ __forceinline__ double times_inverse(double x, double i, double il) { return fma(x, i, x * il); }

// dt/dx of axis d
__device__ __forceinline__ double over_dx(const Params& P, int d, double dt) {
  return times_inverse(dt, P.idx[d], P.idl[d]);
}

// square root from the hardware reciprocal square root: one joint step for the
// root g and its half inverse h, then a correction by the residual x - g^2 (max
// error 0.5000 ulp on the GPU for x > 1e-290).  0 and infinity are their own roots;
// a negative x gives NaN.
__device__ __forceinline__ double fsqrt(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  const double r = fma(-g, h, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  g = fma(fma(-g, g, x), h, g);
  return __builtin_amdgcn_class(x, 0x260 /* -0, 0, +infinity */) ? x : g;
}

// e^x for the reference curves (x <= 0 there): x = n ln2 + r, |r| <= ln2/2, the
// Taylor series of e^r to the 13th power (truncation 4e-18), times 2^n.  20
// instructions where the library function takes 40 with its range checks; a
// JWL split evaluates four per trial.  Max error 0.86 ulp, as the GPU library's
// (4e6 points of -60..0).  It underflows to 0 (x above -1e30), overflows to
// infinity, and keeps NaN.
__device__ __forceinline__ double exp_curve(double x) {
  const double n = rint(x * 0x1.71547652b82fep0);  // 1/ln2
  double r = fma(n, -0x1.62e42fefa39efp-1, x);     // ln2
  r = fma(n, -0x1.abc9e3b39803fp-56, r);           // ln2 less its double
  double p = 1.0 / 6227020800.0;
  p = fma(p, r, 1.0 / 479001600.0);
  p = fma(p, r, 1.0 / 39916800.0);
  p = fma(p, r, 1.0 / 3628800.0);
  p = fma(p, r, 1.0 / 362880.0);
  p = fma(p, r, 1.0 / 40320.0);
  p = fma(p, r, 1.0 / 5040.0);
  p = fma(p, r, 1.0 / 720.0);
  p = fma(p, r, 1.0 / 120.0);
  p = fma(p, r, 1.0 / 24.0);
  p = fma(p, r, 1.0 / 6.0);
  p = fma(p, r, 0.5);
  p = fma(p, r, 1.0);
  p = fma(p, r, 1.0);
  return __builtin_amdgcn_ldexp(p, (int)fmin(fmax(n, -2000.0), 2000.0));
}

// x^e, by products where e is the whole number n (n = 0: any e)
__device__ __forceinline__ double pow_of(double x, double e, int n) {
  if (n == 0) return pow(x, e);
  double r = x;
  for (int k = 1; k < n; ++k) r *= x;
  return r;
}

// a[y] for a runtime index y < M, read with compile-time indices and selects
// so that a register array is never placed in private memory (the empty asm
// keeps the optimiser from folding the selects back into one indexed load)
template <int M>
__device__ __forceinline__ double pick(const double* a, int y) {
  double r = a[0];
#pragma unroll
  for (int l = 1; l < M; ++l) {
    double v = a[l];
    asm volatile("" : "+v"(v));
    r = (l == y) ? v : r;
  }
  return r;
}

template <int D, int N, int RX>
__device__ __forceinline__ double vget(const double* V, int i, int j) {
  using L = Lay<D, N, RX>;
  return L::vq(i, j) >= 0 ? V[L::vq(i, j) >= 0 ? L::vq(i, j) : 0] : 0.0;
}

// ----------------------------------------------------------- closures
// Sec. 2.3 closures at phasic density rho and strain invariant J2, in the
// volume-specific forms the mixture rules use, none of which needs 1/rho: with
// e_ref' = p_ref / rho^2 on a Romenskii curve,
//   rho c^2 = rho p_ref' - (1 + Gamma) p_ref + (1 + Gamma) p
// (a gas, with constant curves: (1 + Gamma) p - p_ref); rc is that less
// (1 + Gamma) p, re = rho e_ref.
struct Curve {
  double pref, re, G, rc;
};

__device__ __forceinline__ Curve curve_eval(const MatP& m, double rho, double J2) {
  Curve c;
  if (m.eos != EOS_ROMENSKII) {
    c.pref = m.pref0;
    c.re = rho * m.eref0;
    c.G = 0.0;
    c.rc = -m.pref0;
    return c;
  }
  const double x = rho * m.inv_rho0;
  const double xa = m.abar_one ? x : pow(x, m.abar);
  const double xm = xa - 1.0;
  const double kx = m.K0a * (x * xa);
  const double slope = m.abar_one ? fma(3.0, xm, 1.0) : (2.0 * m.abar + 1.0) * xa - (m.abar + 1.0);
  if (m.bbar_three) {
    const double x2 = x * x;
    c.G = m.G0 * (x2 * x2);
  } else {
    c.G = m.G0 * pow(x, m.bbar + 1.0);
  }
  const double GJ = c.G * J2;
  const double bG = m.bbar_three ? 3.0 * GJ : m.bbar * GJ;
  c.pref = fma(kx, xm, bG);
  c.re = fma(rho, m.ec_coef * (xm * xm), GJ);
  const double b1 = m.bbar_three ? 4.0 * bG : (m.bbar + 1.0) * bG;
  c.rc = fma(kx, slope, b1) - (1.0 + m.Gam) * c.pref;
  return c;
}

// shear modulus only (no reference curves)
__device__ __forceinline__ double shear_modulus(const MatP& m, double rho) {
  if (!m.shear) return 0.0;
  const double x = rho * m.inv_rho0;
  if (m.bbar_three) {
    const double x2 = x * x;
    return m.G0 * (x2 * x2);
  }
  return m.G0 * pow(x, m.bbar + 1.0);
}

// Hencky strain dev H ~ dev((B - adj B)/4), B = V V^T (Sec. 3.2: Bazant
// approximation with the cofactor standing in for the inverse of the
// unimodular B), and J^2 = tr(H H^T).  strain4 leaves 4 H: the quarter is
// folded into what multiplies it.
template <int D, int N, int RX>
__device__ __forceinline__ void strain4(const double* V, double H[6], double& J2) {
  double B[6];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = i; j < 3; ++j) {
      double s = 0.0;
      bool first = true;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        if (Lay<D, N, RX>::vq(i, k) >= 0 && Lay<D, N, RX>::vq(j, k) >= 0) {
          const double t = vget<D, N, RX>(V, i, k) * vget<D, N, RX>(V, j, k);
          s = first ? t : s + t;
          first = false;
        }
      }
      B[hs(i, j)] = s;
    }
  double A[6];
  if (D == 1) {
    A[0] = B[3] * B[5];
    A[3] = B[0] * B[5];
    A[5] = B[0] * B[3];
    A[1] = A[2] = A[4] = 0.0;
  } else if (D == 2) {
    A[0] = B[3] * B[5];
    A[1] = -B[1] * B[5];
    A[3] = B[0] * B[5];
    A[5] = B[0] * B[3] - B[1] * B[1];
    A[2] = A[4] = 0.0;
  } else {
    A[0] = B[3] * B[5] - B[4] * B[4];
    A[1] = B[2] * B[4] - B[1] * B[5];
    A[2] = B[1] * B[4] - B[2] * B[3];
    A[3] = B[0] * B[5] - B[2] * B[2];
    A[4] = B[2] * B[1] - B[0] * B[4];
    A[5] = B[0] * B[3] - B[1] * B[1];
  }
#pragma unroll
  for (int s = 0; s < 6; ++s) H[s] = B[s] - A[s];
  const double tr = (H[0] + H[3] + H[5]) * (1.0 / 3.0);
  H[0] = H[0] - tr;
  H[3] = H[3] - tr;
  H[5] = H[5] - tr;
  double j2 = H[0] * H[0] + H[3] * H[3] + H[5] * H[5];
  if (D >= 2) j2 += 2.0 * (H[1] * H[1]);
  if (D == 3) j2 += 2.0 * (H[2] * H[2] + H[4] * H[4]);
  J2 = 0.0625 * j2;
}

template <int D, int N, int RX>
__device__ __forceinline__ void strain(const double* V, double H[6], double& J2) {
  strain4<D, N, RX>(V, H, J2);
#pragma unroll
  for (int s = 0; s < 6; ++s) H[s] = 0.25 * H[s];
}

// ------------------------------------------------------ phase densities
// phi_l and rho_l of every material
template <int N>
struct Phases {
  double phi[N], rho[N];
};

template <int N>
__device__ __forceinline__ void phase_fractions(const double* phi_st, Phases<N>& Q) {
  double sphi = 0.0;
#pragma unroll
  for (int l = 0; l < N - 1; ++l) {
    Q.phi[l] = phi_st[l];
    sphi += Q.phi[l];
  }
  Q.phi[N - 1] = 1.0 - sphi;
}

// from partial densities; r is their sum and ir its inverse.  Each density is
// rounded once: a solid's pressure takes its modulus times the error (one
// reciprocal for all quotients of two materials left 2 ulp in them, and the
// momentum of a detonating stick after two steps 5.9e-16 of its norm from the
// exact step, now 3.7e-16, in the same time).
template <int N>
__device__ __forceinline__ void phases_from_partial(const double* phi_st, const double* m, Phases<N>& Q, double& r,
                                                    double& ir) {
  phase_fractions<N>(phi_st, Q);
  r = 0.0;
#pragma unroll
  for (int l = 0; l < N; ++l) {
    r += m[l];
    Q.rho[l] = quot(m[l], Q.phi[l]);
  }
  ir = frcp(r);
}

template <int N>
__device__ __forceinline__ void phases_from_prim(const double* phi_st, const double* rho, Phases<N>& Q) {
  phase_fractions<N>(phi_st, Q);
#pragma unroll
  for (int l = 0; l < N; ++l) Q.rho[l] = rho[l];
}

// ------------------------------------------------------ mixture state
// The reactive mixture's components at equal pressure and temperature: their
// volume shares s and s1 = 1 - s of the mixture, their reference curves, and
// what the density dependence of a JWL curve adds to rho c^2 per unit share
// (ka, kb: Gamma^-1 rho dp_ref/drho - (the JWL part of p_ref)).
struct Split {
  double s, s1;
  double pa, pb, ea, eb, ka, kb;
};

// The mixture of all materials at one state.  w_l = phi_l / Gamma_l; n0, d0:
// the sums of phi_l (p_ref / Gamma - rho e_ref) and of w_l over the
// non-reactive materials, so that rho e + n = p xi with the reactive terms
// added to both.
template <int N, int RX>
struct Thermo {
  Curve c[N];
  double w[N];
  double n0, d0;
  double xi, ixi;  // sum phi_l / Gamma_l (reactive: effective) and its inverse
  double rho, irho;
  double p, rhoe;
  double Gmix, rc2, c2, cL2;  // rc2 = rho c^2
  double yrc;                 // the reactive mixture's rc per unit of its volume
};

// Reference curves of reactive component C (0 reactant, 1 product) at
// density 1/irho: the constant part (a gas's p_ref and e_ref, the product's
// e_ref lowered by Q) plus, for a JWL component (Sec. 2.3),
// A exp(-R1 rho0/rho) + B exp(-R2 rho0/rho) and its energy
// A/(R1 rho0) exp(-R1 rho0/rho) + B/(R2 rho0) exp(-R2 rho0/rho).  j is the JWL
// part of p_ref and q = R1 rho0 A exp() + R2 rho0 B exp() its slope:
// dp_ref/drho = q / rho^2, de_ref/drho = j / rho^2.
struct RxRef {
  double p, e, j, q;
};

template <int C>
__device__ __forceinline__ RxRef rx_ref(const RxP& r, double irho) {
  RxRef o;
  o.p = C ? r.pb : r.pa;
  o.e = C ? r.eb : r.ea;
  o.j = 0.0;
  o.q = 0.0;
  if (r.jwl[C]) {
    const double xa = exp_curve(-r.jR1[C] * irho), xb = exp_curve(-r.jR2[C] * irho);
    const double pa = r.jA[C] * xa, pb = r.jB[C] * xb;
    o.j = pa + pb;
    o.p = o.j + o.p;
    o.e = (pa * r.jiR1[C] + pb * r.jiR2[C]) + o.e;
    o.q = r.jR1[C] * pa + r.jR2[C] * pb;
  }
  return o;
}

// the split of two components at densities 1/ira and 1/irb
__device__ __forceinline__ Split rx_split_of(const RxP& r, double s, double s1, double ira, double irb,
                                             const RxRef& A, const RxRef& B) {
  Split o;
  o.s = s;
  o.s1 = s1;
  o.pa = A.p;
  o.pb = B.p;
  o.ea = A.e;
  o.eb = B.e;
  o.ka = A.q * r.invGa * ira - A.j;
  o.kb = B.q * r.invGb * irb - B.j;
  return o;
}

// two components with constant curves
__device__ __forceinline__ Split rx_gas(const RxP& r, double s, double s1) {
  Split o;
  o.s = s;
  o.s1 = s1;
  o.pa = r.pa;
  o.pb = r.pb;
  o.ea = r.ea;
  o.eb = r.eb;
  o.ka = o.kb = 0.0;
  return o;
}

// Both components at the mixture's own density (a pure cell: no split; the
// shares are lam and 1 - lam).  A component whose weight is exactly zero keeps
// its constant part only: its terms vanish either way.
__device__ __forceinline__ Split rx_pure(const RxP& r, double lam, double ry) {
  const double iry = frcp(ry);
  RxRef A, B;
  A.p = r.pa;
  A.e = r.ea;
  B.p = r.pb;
  B.e = r.eb;
  A.j = A.q = B.j = B.q = 0.0;
  if (lam > 0.0) A = rx_ref<0>(r, iry);
  if (lam < 1.0) B = rx_ref<1>(r, iry);
  return rx_split_of(r, lam, 1.0 - lam, iry, iry, A, B);
}

// Appendix B with density-dependent reference curves: a root in (0, 1) of
// g(t) = rho_y (T_b - T_a) in t = rho_a / (rho_a + rho_b), a monotone
// function of the reactant density the paper bisects on; with D = lam (1-t)
// + (1-lam) t the specific-volume rule gives rho_a = rho_y D / (1-t), rho_b
// = rho_y D / t and the volume shares s = lam (1-t) / D, 1 - s = (1-lam) t /
// D.  Away from physical states (explosive traces in another material,
// low-density JWL reactant) g can change sign several times; the root taken
// is the first sign change met going outward from equal densities (t = 1/2,
// the split of the pure limits) towards the side g's sign points to (g < 0:
// above), on a fixed probe sequence: the ladder t = 3/4, 7/8, ... or
// t = 1/4, 1/8, ..., each probe halving the distance left to the end, until
// g changes sign; then RX_SUBSTEPS equal steps across that first bracket
// from its inner end until g changes sign again.  Inside the sub-bracket so
// found Newton steps from the secant point finish, halving whenever a step
// leaves it or is not finite; they end when a step is below the resolution
// the split needs, or when the steps, already below 1e-7 of the distance to
// the nearer end, stop halving: g is then its own rounding noise (strong
// cancellation in p(t)), and no further step moves t towards the root.
// Where g keeps its sign at every ladder probe
// the ends are taken: t = 1 (the pure state) once the probes reach 1 in
// double precision, t = 2^-65 after 64 probes down.  KNOWN_P: the pressure p
// is given (primitive branch); otherwise p(t) comes from the pressure
// function with its non-reactive part (num0, den0).
constexpr int RX_SUBSTEPS = 8;

template <bool KNOWN_P>
__device__ __forceinline__ Split rx_newton(const RxP& r, double lam, double py, double ry, double p, double num0,
                                           double den0) {
  const double l1 = 1.0 - lam;
  const double iry = frcp(ry), ila = frcp(lam), il1 = frcp(l1);
  const double ka = ila * r.iGca, kb = il1 * r.iGcb;
  const double la = lam * ry, lb = l1 * ry;
  // g and the state at t
  struct Eval {
    double g, pp, iden, iD, s, s1, ira, irb;
    RxRef A, B;
  };
  auto eval = [&](double t) {
    Eval e;
    const double t1 = 1.0 - t;
    e.iD = frcp(lam * t1 + l1 * t);
    const double ta = t1 * e.iD, tb = t * e.iD;
    e.s = lam * ta;
    e.s1 = l1 * tb;
    e.ira = ta * iry;
    e.irb = tb * iry;
    e.A = rx_ref<0>(r, e.ira);
    e.B = rx_ref<1>(r, e.irb);
    e.pp = p;
    e.iden = 1.0;
    if (!KNOWN_P) {
      const double num = num0 + py * (e.s * e.A.p * r.invGa - la * e.A.e) + py * (e.s1 * e.B.p * r.invGb - lb * e.B.e);
      e.iden = frcp(den0 + py * (e.s * r.invGa + e.s1 * r.invGb));
      e.pp = num * e.iden;
    }
    e.g = kb * (e.pp - e.B.p) * e.s1 - ka * (e.pp - e.A.p) * e.s;
    return e;
  };
  // Three loops, each with its own evaluation: the first two need g's sign
  // only, and a wave runs each for as long as its slowest lane (one loop with
  // the stage in a variable spent two thirds of its instructions on choosing:
  // the x sweep of a 400 x 1000 stick 111 -> 62 us, fused 396 -> 260).
  double ti = 0.5, gi = eval(0.5).g, to = 0.5, go = gi;  // the bracket's inner and outer end
  const bool up = gi < 0.0;
  bool found = false;
#pragma unroll 1
  for (int probes = 1; probes < 64; ++probes) {
    const double tn = up ? 0.5 * (ti + 1.0) : 0.5 * ti;
    if (up && !(tn < 1.0)) break;
    const double g = eval(tn).g;
    if ((g < 0.0) != up) {
      to = tn;
      go = g;
      found = true;
      break;
    }
    ti = tn;
    gi = g;
  }
  if (!found && up) return rx_pure(r, lam, ry);  // g < 0 at every probe below 1
  double lo = 0.0, hi = 1.0, t = 0.5 * ti;       // g >= 0 at every probe down to 2^-64: 2^-65
  if (found) {
    const double base = ti, w = (to - ti) / RX_SUBSTEPS;
#pragma unroll 1
    for (int k = 1; k < RX_SUBSTEPS; ++k) {
      const double tn = base + double(k) * w, g = eval(tn).g;
      if ((g < 0.0) != up) {
        to = tn;
        go = g;
        break;
      }
      ti = tn;
      gi = g;
    }
    lo = up ? ti : to;
    hi = up ? to : ti;
    t = ti - gi * (to - ti) * frcp(go - gi);
    if (!(t > lo && t < hi)) t = 0.5 * (lo + hi);
  }
  // d p_ref / ds of a component is its slope q times a constant: ds/s at
  // fixed masses is -drho/rho
  const double da = -(iry * ila), db = iry * il1;
  double last = 1.0;  // size of the previous Newton step
  Eval e;
#pragma unroll 1
  for (int it = 0; it < 100; ++it) {
    e = eval(t);
    if (!found || e.g == 0.0) break;
    if (e.g < 0.0)
      lo = t;
    else
      hi = t;
    // dg/dt = lam (1-lam) / D^2 df/ds
    const double dA = e.A.q * da, dB = e.B.q * db;
    double dp = 0.0;
    if (!KNOWN_P) {
      const double dnum =
          py * ((e.A.p + e.s * dA) * r.invGa + e.A.j + (e.s1 * dB - e.B.p) * r.invGb - e.B.j);
      dp = (dnum - e.pp * py * (r.invGa - r.invGb)) * e.iden;
    }
    const double df = ka * ((dp - dA) * e.s + (e.pp - e.A.p)) - kb * ((dp - dB) * e.s1 - (e.pp - e.B.p));
    // the current state is kept once the Newton step is below the
    // resolution the split needs (or below half an ulp of t)
    const double step = e.g * frcp(df * (lam * l1) * (e.iD * e.iD)), size = fabs(step), room = fmin(t, 1.0 - t);
    if (isfinite(step) && !(size > fmax(1e-14 * room, 0x1p-53 * t))) break;
    // the noise floor (a triple root, whose steps shrink by 2/3, lies
    // above it only where the root itself is known to 1e-5).  Without this
    // test about one split in 300 of a detonation front ran all 160
    // evaluations, and the waves that hold one set the kernels' time: two
    // steps of a 400 x 1000 rate stick took 5.5 ms, with it 1.43 ms (0.45 with
    // the steps after it)
    if (size > 0.5 * last && last <= 1e-7 * room) break;
    last = size;
    t = t - step;
    if (!(t > lo && t < hi)) t = 0.5 * (lo + hi);  // NaN steps land here too
  }
  return rx_split_of(r, e.s, e.s1, e.ira, e.irb, e.A, e.B);
}

// The split's root rule for two gas components (Appendix B, with the reading
// stated at rx_newton).  Here the residual changes sign at the roots of a
// polynomial of degree <= 2 in the reactant's volume share s (s = lam at
// equal densities t = 1/2; t = lam (1 - s) / (lam (1 - s) + (1 - lam) s)
// decreases with s).  The probe sequence of rx_newton changes sign between
// two probes where an odd number of roots lies between them, so its outcome
// follows from the roots alone: the root nearest t = 1/2 on the side g(1/2)
// points to (t >= 1/2 when g(1/2) < 0, else t <= 1/2), unless the other root
// lies in the same ladder bracket [1 - 2^-(k-1), 1 - 2^-k] (resp. [2^-k,
// 2^-(k-1)]): then both cancel and the ladder runs to its end, t = 1 (the
// pure state; brackets exist for k <= 53) or t = 2^-65 (after the probe
// 2^-64).  Sets s (true) or the end value t_end (false).
__device__ __forceinline__ int rx_bracket(double u) {
  int e;
  frexp(u, &e);  // u in [2^(e-1), 2^e)
  return (1 - e) < 2 ? 2 : 1 - e;
}

__device__ __forceinline__ bool rx_pick(const double* sr, int nr, bool up, double lam, double& s,
                                        double& t_end) {
  // t >= 1/2 exactly where s <= lam, and nearer 1/2 in t is nearer lam in s
  double sa = -1.0, sb = -1.0;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    if (i >= nr) break;
    const double si = sr[i];
    const bool side = up ? (si > 0.0 && si <= lam) : (si >= lam && si < 1.0);
    if (!side) continue;
    if (sa < 0.0 || fabs(si - lam) < fabs(sa - lam)) {
      sb = sa;
      sa = si;
    } else {
      sb = si;
    }
  }
  t_end = up ? 1.0 : 0x1p-65;
  if (sa < 0.0) return false;
  // the distance of the root's t from the end it points to: 1 - t (up) or t
  auto dist = [&](double x) {
    const double a = lam * (1.0 - x), b = (1.0 - lam) * x;
    return (up ? b : a) * frcp(a + b);
  };
  const int ka = rx_bracket(dist(sa));
  if (ka > (up ? 53 : 64)) return false;                         // beyond the last probe
  if (sb >= 0.0 && rx_bracket(dist(sb)) == ka) return false;     // a pair cancels
  s = sa;
  return true;
}

// the shares of a picked s, or of the end value t_end (pure at 1): s = lam
// (1 - t) / D, 1 - s = (1 - lam) t / D, D = lam (1 - t) + (1 - lam) t
__device__ __forceinline__ Split rx_from_pick(const RxP& r, bool picked, double s, double t_end, double lam) {
  if (picked) return rx_gas(r, s, 1.0 - s);
  if (!(t_end < 1.0)) return rx_gas(r, lam, 1.0 - lam);
  const double a = lam * (1.0 - t_end), b = (1.0 - lam) * t_end;
  const double iD = frcp(a + b);
  return rx_gas(r, a * iD, b * iD);
}

// Reactive split from a known pressure (Appendix B, primitive branch).  For
// two gas components temperature equality is linear in t: h(t) = (alpha +
// beta) t - alpha, alpha = (p - p_a)/(Gamma_a C_V,a), beta = (p - p_b)/(Gamma_b
// C_V,b).
template <bool GEN>
__device__ __forceinline__ Split rx_split_p(const RxP& r, double lam, double rho_y, double p) {
  const bool pure = lam >= 1.0 - 1e-12 || lam <= 1e-12;
  if constexpr (GEN) return pure ? rx_pure(r, lam, rho_y) : rx_newton<true>(r, lam, 0.0, rho_y, p, 0.0, 0.0);
  if (pure) return rx_gas(r, lam, 1.0 - lam);
  // in t the residual is linear, (alpha + beta) t - alpha with alpha = (p -
  // p_a)/(Gamma_a C_V,a), beta = (p - p_b)/(Gamma_b C_V,b): g(1/2) < 0 where
  // beta < alpha, and the root t = alpha/(alpha + beta) lies in (0, 1) on
  // that side exactly where alpha > 0 and beta > 0 (else the ladder runs to
  // its end); the share of the root is s = lam beta / (lam beta + (1 - lam)
  // alpha)
  const double alpha = (p - r.pa) * r.iGca, beta = (p - r.pb) * r.iGcb;
  const bool up = beta < alpha;
  const bool found = alpha > 0.0 && beta > 0.0 &&
                     (up ? beta >= 0x1p-53 * (alpha + beta) : alpha >= 0x1p-64 * (alpha + beta));
  const double a = found ? lam * beta : lam * (up ? 1.0 : 1.0 - 0x1p-65);
  const double b = found ? (1.0 - lam) * alpha : (1.0 - lam) * (up ? 1.0 : 0x1p-65);
  const double iD = frcp(a + b);
  return rx_gas(r, a * iD, b * iD);
}

// Reactive split from the conserved energy (Appendix B, conservative
// branch).  With the pressure function linear-fractional in the reactant's
// volume share s, p(s) = (A0 + A1 s)/(B0 + B1 s), and constant reference
// curves, temperature equality is Q(s) = Q2 s^2 + Q1 s + Q0 = 0, with g < 0
// where Q > 0; its roots (stable formula, one Newton polish each) go to the
// rule.
__device__ __forceinline__ Split rx_solve_gas(const RxP& r, double lam, double A0, double A1, double B0, double B1) {
  if (lam >= 1.0 - 1e-12 || lam <= 1e-12) return rx_gas(r, lam, 1.0 - lam);
  // (both weights times lam (1 - lam))
  const double ka = (1.0 - lam) * r.iGca;
  const double kb = lam * r.iGcb;
  const double a0 = A0 - r.pa * B0, a1 = A1 - r.pa * B1;
  const double b0 = A0 - r.pb * B0, b1 = A1 - r.pb * B1;
  const double Q2 = ka * a1 + kb * b1;
  const double Q1 = ka * a0 - kb * (b1 - b0);
  const double Q0 = -kb * b0;
  double sr[2];
  int nr = 0;
  if (Q2 == 0.0) {
    if (Q1 != 0.0) sr[nr++] = -Q0 * frcp(Q1);
  } else {
    const double disc = Q1 * Q1 - 4.0 * Q2 * Q0;
    if (disc >= 0.0) {
      const double q = -0.5 * (Q1 + copysign(fsqrt(disc), Q1));
      if (q != 0.0) {
        sr[nr++] = Q0 * frcp(q);
        sr[nr++] = q * frcp(Q2);
      } else {
        sr[nr++] = 0.0;
      }
    }
  }
  const bool up = (Q2 * lam + Q1) * lam + Q0 > 0.0;  // g(1/2) < 0
  double sp = 0.0, t_end = 1.0;
  const bool picked = rx_pick(sr, nr, up, lam, sp, t_end);
  if (picked) {
    // one Newton polish of the root taken, on Q's own factors: at a low pressure
    // b0 + b1 s and 1 - s are small differences (1e-5 and 1e-7 in unreacted
    // explosive at rest) that Q2 s^2 + Q1 s + Q0 loses to rounding
    const double qv = ka * sp * fma(a1, sp, a0) - kb * (1.0 - sp) * fma(b1, sp, b0), dq = 2.0 * Q2 * sp + Q1;
    if (dq != 0.0) sp = sp - qv * frcp(dq);
  }
  return rx_from_pick(r, picked, sp, t_end, lam);
}

// What the mixture rules take of a split, per unit of the mixture's volume:
// 1/Gamma, p_ref/Gamma - rho e_ref, and rc (rho c^2 / Gamma less (1 + 1/Gamma)
// p, as of a Curve times 1/Gamma)
struct MixY {
  double xi, num, rc;
};

template <bool GEN>
__device__ __forceinline__ MixY rx_mixture(const RxP& r, const Split& o, double lam, double ry) {
  MixY m;
  m.xi = o.s * r.invGa + o.s1 * r.invGb;
  const double pg = o.s * (o.pa * r.invGa) + o.s1 * (o.pb * r.invGb);
  m.num = pg - ry * (lam * o.ea + (1.0 - lam) * o.eb);
  m.rc = GEN ? (o.s * o.ka + o.s1 * o.kb) - pg : -pg;
  return m;
}

// the mixture of two primitive states (progress, density, pressure); with JWL
// components through one copy of the split (the instruction cache holds 64 KB:
// a fused sweep with a copy at every use was 120 KB)
template <int RX>
__device__ __forceinline__ void rx_mixture_pair(const RxP& r, const double lam[2], const double ry[2],
                                                const double p[2], MixY& a, MixY& b) {
  if constexpr (RX == 2) {
#pragma unroll 1
    for (int k = 0; k < 2; ++k) {
      const double l = k ? lam[1] : lam[0], d = k ? ry[1] : ry[0], q = k ? p[1] : p[0];
      const MixY m = rx_mixture<true>(r, rx_split_p<true>(r, l, d, q), l, d);
      if (k)
        b = m;
      else
        a = m;
    }
  } else {
    a = rx_mixture<false>(r, rx_split_p<false>(r, lam[0], ry[0], p[0]), lam[0], ry[0]);
    b = rx_mixture<false>(r, rx_split_p<false>(r, lam[1], ry[1], p[1]), lam[1], ry[1]);
  }
}

// the mixtures of two primitive states W
template <int D, int N, int RX>
__device__ __forceinline__ void mixtures_of(const Params& P, const double* Wa, const double* Wb, MixY& a, MixY& b) {
  using L = Lay<D, N, RX>;
  if (!rx_mix<RX>(P)) return;
  const int y = P.rx.mat;
  const double lam[2] = {fmin(fmax(Wa[L::LAM], 0.0), 1.0), fmin(fmax(Wb[L::LAM], 0.0), 1.0)};
  const double ry[2] = {pick<N>(Wa + L::M0, y), pick<N>(Wb + L::M0, y)};
  const double p[2] = {Wa[L::E], Wb[L::E]};
  rx_mixture_pair<RX>(P.rx, lam, ry, p, a, b);
}

// The reactive part of the pressure function (Appendix B, conservative
// branch) for a cell whose non-reactive part is (num0, den0): solves the
// split and leaves the full numerator and denominator (xi) of p; returns the
// mixture's rc.
template <bool GEN>
__device__ __forceinline__ double rx_cons(const RxP& r, double py, double ry, double lam, double num0, double den0,
                                          double& num, double& den) {
  Split o;
  if constexpr (GEN) {
    if (lam >= 1.0 - 1e-12 || lam <= 1e-12)
      o = rx_pure(r, lam, ry);
    else
      o = rx_newton<false>(r, lam, py, ry, 0.0, num0, den0);
  } else {
    const double A0 = num0 + py * (r.pb * r.invGb - ry * (lam * r.ea + (1.0 - lam) * r.eb));
    const double A1 = py * (r.pa * r.invGa - r.pb * r.invGb);
    const double B0 = den0 + py * r.invGb;
    const double B1 = py * (r.invGa - r.invGb);
    o = rx_solve_gas(r, lam, A0, A1, B0, B1);
  }
  const MixY m = rx_mixture<GEN>(r, o, lam, ry);
  den = den0 + py * m.xi;
  num = num0 + py * m.num;
  return m.rc;
}

// closures of the non-reactive materials and their sums w, n0, d0
template <int N, int RX>
__device__ __forceinline__ void curves_all(const Params& P, const Phases<N>& Q, double J2, Thermo<N, RX>& T) {
  T.n0 = 0.0;
  T.d0 = 0.0;
#pragma unroll
  for (int l = 0; l < N; ++l) {
    T.w[l] = 0.0;
    if (rx_mix<RX>(P) && l == P.rx.mat) continue;
    T.c[l] = curve_eval(P.mat[l], Q.rho[l], J2);
    T.w[l] = Q.phi[l] * P.mat[l].invGam;
    T.d0 += T.w[l];
    T.n0 += T.w[l] * T.c[l].pref - Q.phi[l] * T.c[l].re;
  }
}

// pressure from the conserved energy T.rhoe (Appendix B pressure function;
// without the reactive terms when RX is false).  Leaves xi and 1/xi in T.
template <int N, int RX>
__device__ __forceinline__ void pressure_from_rhoe(const Params& P, const Phases<N>& Q, double lam,
                                                   Thermo<N, RX>& T) {
  double den = T.d0, num = T.rhoe + T.n0;
  if (rx_mix<RX>(P)) {
    const int y = P.rx.mat;
    T.yrc = rx_cons<RX == 2>(P.rx, pick<N>(Q.phi, y), pick<N>(Q.rho, y), lam, T.rhoe + T.n0, T.d0, num, den);
  }
  T.xi = den;
  T.ixi = frcp(den);
  T.p = num * T.ixi;
}

// rho c^2 and the mixture's shear modulus, both times xi: sum of w_l rho_l
// c_l^2 = p (1 + xi) + sum w_l rc_l since w_l Gamma_l = phi_l and the
// fractions sum to 1 (Allaire form of the mixture rule)
template <int N, int RX>
__device__ __forceinline__ void sound_sums(const Params& P, const Phases<N>& Q, const Thermo<N, RX>& T, double& cnum,
                                           double& gnum) {
  cnum = fma(T.p, T.xi, T.p);
  gnum = 0.0;
#pragma unroll
  for (int l = 0; l < N; ++l) {
    // (values, not sums, chosen by the material: with the additions under the
    // branch the compiler chose between the sums' addresses, in scratch memory)
    const bool mix = rx_mix<RX>(P) && l == P.rx.mat;
    cnum += mix ? Q.phi[l] * T.yrc : T.w[l] * T.c[l].rc;
    gnum += mix ? 0.0 : T.w[l] * T.c[l].G;
  }
}

// sound speeds (c_L^2 = c^2 + 4G/(3 rho)) and shear modulus once p, the split,
// 1/xi and 1/rho are known
template <int N, int RX>
__device__ __forceinline__ void finish(const Params& P, const Phases<N>& Q, Thermo<N, RX>& T) {
  double cnum, gnum;
  sound_sums<N, RX>(P, Q, T, cnum, gnum);
  T.Gmix = gnum * T.ixi;
  T.rc2 = cnum * T.ixi;
  T.c2 = T.rc2 * T.irho;
  T.cL2 = T.c2 + (4.0 / 3.0) * T.Gmix * T.irho;
}

// conserved -> primitive of one cell; W receives the primitive vector.  FIN
// = false leaves out the mixture's sound speeds and shear modulus (T.c2,
// T.cL2, T.Gmix; the plastic step needs the closures and p only).
template <int D, int N, int RX, bool FIN = true>
__device__ __forceinline__ void cons_to_prim(const Params& P, const double* U, double* W, Thermo<N, RX>& T,
                                             double H[6], double& J2) {
  using L = Lay<D, N, RX>;
  Phases<N> Q;
  phases_from_partial<N>(U, U + L::M0, Q, T.rho, T.irho);
  double lam = 0.0, hist = 0.0;
  if (RX) {
    const double my = pick<N>(U + L::M0, P.rx.mat);
    hist = quot(U[L::LAM], my);
    if (P.rx.kind == RXK_MIX)
      lam = fmin(fmax(hist, 0.0), 1.0);
    else
      hist = (my > 0.0) ? hist : 0.0;  // plastic strain
  }
  double uu = 0.0;
#pragma unroll
  for (int k = 0; k < D; ++k) {
    W[L::MOM0 + k] = U[L::MOM0 + k] * T.irho;
    uu += W[L::MOM0 + k] * W[L::MOM0 + k];
  }
  strain<D, N, RX>(U + L::V0, H, J2);
  curves_all<N, RX>(P, Q, J2, T);
  T.rhoe = U[L::E] - 0.5 * T.rho * uu;
  pressure_from_rhoe<N, RX>(P, Q, lam, T);
  if (FIN) finish<N, RX>(P, Q, T);
#pragma unroll
  for (int l = 0; l < N - 1; ++l) W[l] = Q.phi[l];
#pragma unroll
  for (int l = 0; l < N; ++l) W[L::M0 + l] = Q.rho[l];
  if (RX) W[L::LAM] = (P.rx.kind == RXK_MIX) ? lam : hist;
  W[L::E] = T.p;
#pragma unroll
  for (int q = 0; q < L::NV; ++q) W[L::V0 + q] = U[L::V0 + q];
}

// primitive -> mixture state (energy from p; my: the reactive mixture, if any):
// the closures, xi, rho and rho e; H holds 4 H
template <int D, int N, int RX>
__device__ __forceinline__ void prim_mix(const Params& P, const double* W, const MixY& my, Phases<N>& Q,
                                         Thermo<N, RX>& T, double H[6], double& J2) {
  using L = Lay<D, N, RX>;
  phases_from_prim<N>(W, W + L::M0, Q);
  strain4<D, N, RX>(W + L::V0, H, J2);
  curves_all<N, RX>(P, Q, J2, T);
  T.p = W[L::E];
  T.xi = T.d0;
  double n = T.n0;
  if (rx_mix<RX>(P)) {
    const double py = pick<N>(Q.phi, P.rx.mat);
    T.xi = T.d0 + py * my.xi;
    n += py * my.num;
    T.yrc = my.rc;
  }
  T.rhoe = fma(T.p, T.xi, -n);
  T.rho = 0.0;
#pragma unroll
  for (int l = 0; l < N; ++l) T.rho += Q.phi[l] * Q.rho[l];
}

// Mixture shear modulus G = sum(phi_l G_l / Gamma_l) / xi and 4 H of a
// primitive state (xi_y: of the reactive mixture): all the stress needs besides p
template <int D, int N, int RX>
__device__ __forceinline__ double prim_shear(const Params& P, const double* W, double xi_y, double H[6]) {
  using L = Lay<D, N, RX>;
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
    if (rx_mix<RX>(P) && l == P.rx.mat) {
      xi += phi[l] * xi_y;
    } else {
      const double wl = phi[l] * P.mat[l].invGam;
      xi += wl;
      gnum += wl * shear_modulus(P.mat[l], W[L::M0 + l]);
    }
  }
  double J2;
  strain4<D, N, RX>(W + L::V0, H, J2);
  return gnum * frcp(xi);
}

// ------------------------------------------------ reconstruction pieces
// 0 for differences of opposite sign, else the smaller one: of the two terms
// one is 0 (five instructions, where the comparisons and selects of the
// definition take seven)
__device__ __forceinline__ double minmod(double a, double b) {
  return fmax(fmin(a, b), 0.0) + fmin(fmax(a, b), 0.0);
}

__device__ __forceinline__ double vanalbada(double a, double b, double e2) {
  return quot(a * (b * b + e2) + b * (a * a + e2), a * a + b * b + 2.0 * e2);
}

template <int D, int N, int RX>
__device__ __forceinline__ double slope(const Params& P, int f, double wm, double w0, double wp) {
  const double a = w0 - wm, b = wp - w0;
  if (P.limiter == 1) return vanalbada(a, b, P.va_e2[Lay<D, N, RX>::kind(f)]);
  return minmod(a, b);
}

// Youngs normal |n_d| from a 3x3 (2-D) stencil phi9[a][b] (a along x, b
// along y, offsets -1..1) or a 3x3x3 stencil phi27[a][b][c]; symmetric pairs
// are summed first.
__device__ __forceinline__ double youngs2(const double s[3][3], const double* dx, int d) {
  const double gx = ((s[2][0] - s[0][0]) + (s[2][2] - s[0][2])) + 2.0 * (s[2][1] - s[0][1]);
  const double gy = ((s[0][2] - s[0][0]) + (s[2][2] - s[2][0])) + 2.0 * (s[1][2] - s[1][0]);
  const double ax = gx / dx[0], ay = gy / dx[1];
  const double nn = sqrt(ax * ax + ay * ay);
  if (!(nn > 0.0)) return 1.0;
  return fabs(d == 0 ? ax : ay) / nn;
}

__device__ __forceinline__ double youngs3(const double s[3][3][3], const double* dx, int d) {
  double g[3];
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    // difference along e at transverse offsets (t1, t2) over the other two axes
    auto df = [&](int t1, int t2) {
      int p[3], m[3];
      const int o1 = (e == 0) ? 1 : 0, o2 = (e == 2) ? 1 : 2;
      p[e] = 2;
      m[e] = 0;
      p[o1] = m[o1] = 1 + t1;
      p[o2] = m[o2] = 1 + t2;
      return s[p[0]][p[1]][p[2]] - s[m[0]][m[1]][m[2]];
    };
    const double corners = (df(-1, -1) + df(1, 1)) + (df(-1, 1) + df(1, -1));
    const double edges = (df(-1, 0) + df(1, 0)) + (df(0, -1) + df(0, 1));
    g[e] = ((corners + 2.0 * edges) + 4.0 * df(0, 0)) / dx[e];
  }
  const double nn = sqrt(g[0] * g[0] + g[1] * g[1] + g[2] * g[2]);
  if (!(nn > 0.0)) return 1.0;
  return fabs(g[d]) / nn;
}

// candidates of the volume fraction edges of one cell: MUSCL (mL, mR) and
// THINC-or-MUSCL (tL, tR)
struct Cand {
  double mL, mR, tL, tR;
};

// the candidates of every stored volume fraction (N - 1 of them), and the
// one of fraction l of either form (a single Cand is fraction 0)
template <int N>
struct CandSet {
  Cand c[N > 1 ? N - 1 : 1];
};
__device__ __forceinline__ const Cand& cand_at(const Cand& c, int) { return c; }
template <int N>
__device__ __forceinline__ const Cand& cand_at(const CandSet<N>& c, int l) {
  return c.c[l];
}

// ------------------------------------------------------- face exchange
template <int D, int N, int RX>
struct FaceV {
  double F[Lay<D, N, RX>::F];  // phi slots carry phi_K u*
  double ustar;
  double Vn[D];                // Vbar*_{n j} for the structurally non-zero j of row n
};

}  // namespace dimp
