// Test library: the reverse stages of the adjoint against central differences
// of the forward stages they reverse, those of the calibrated step
// (dimp_calib.hpp), each in the general instance (GS false) and in the one for
// a gas and a solid with exponents 1 and 3 (GS true).
#include "adjoint_units.hip"
#include "dimp_calib.hpp"

namespace {

template <bool GS>
struct CalC2P {
  static constexpr int NI = F2, NO = F2 + 2;
  __device__ static void fwd(const Params& P, double, const double* x, double* y) {
    calib::Thermo T;
    double H[6], J2;
    calib::cons_to_prim(P, x, y, T, H, J2);
    y[F2] = T.irho;
    y[F2 + 1] = T.rho * T.c2;
  }
  __device__ static void bwd(const Params& P, double, const double* x, const double* yb, double* xb) {
    adj::PBar pb;
    adj::pbar_zero(pb);
    adj::c2p_bwd<GS>(P, x, yb, yb[F2], yb[F2 + 1], xb, pb, true);
  }
};

template <int DIR, bool GS>
struct CalSide {
  static constexpr int NI = F2, NO = 8;
  __device__ static void fwd(const Params& P, double, const double* x, double* y) {
    calib::Side S;
    calib::side_state<DIR>(P, x, S);
    y[0] = S.rho; y[1] = S.E; y[2] = S.cl; y[3] = S.u[0]; y[4] = S.u[1];
    y[5] = S.sig[0]; y[6] = S.sig[1]; y[7] = S.sig[2];
  }
  __device__ static void bwd(const Params& P, double, const double* x, const double* yb, double* xb) {
    adj::PBar pb;
    adj::pbar_zero(pb);
    adj::SideB b;
    b.rho = yb[0]; b.E = yb[1]; b.cl = yb[2]; b.u[0] = yb[3]; b.u[1] = yb[4];
    b.sig[0] = yb[5]; b.sig[1] = yb[6]; b.sig[2] = yb[7];
    adj::side_bwd<DIR, GS>(P, x, b, xb, pb, true);
  }
};

template <int DIR, bool GS>
struct CalStress {
  static constexpr int NI = F2, NO = 3;
  __device__ static void fwd(const Params& P, double, const double* x, double* y) {
    calib::stress_col<DIR>(P, x, y);
  }
  __device__ static void bwd(const Params& P, double, const double* x, const double* yb, double* xb) {
    adj::PBar pb;
    adj::pbar_zero(pb);
    adj::stress_bwd<DIR, GS>(P, x, yb, xb, pb, true);
  }
};

template <int DIR, bool GS>
struct CalFace {
  static constexpr int NI = 2 * F2, NO = F2 + 3;
  __device__ static void fwd(const Params& P, double, const double* x, double* y) {
    calib::FaceV f;
    calib::face_flux<DIR>(P, x, x + F2, f);
    FaceIO::put(f, y);
  }
  __device__ static void bwd(const Params& P, double, const double* x, const double* yb, double* xb) {
    adj::PBar pb;
    adj::pbar_zero(pb);
    adj::face_bwd<DIR, GS>(P, x, x + F2, FaceIO::bar(yb), xb, xb + F2, pb, true);
  }
};

// (star_bwd has one instance)
template <int DIR>
struct CalStar : StStar<DIR> {
  __device__ static void fwd(const Params& P, double, const double* x, double* y) {
    calib::Side S;
    StStar<DIR>::side(x, S);
    const double* r = x + F2 + 8;
    const double ust[2] = {r[3], r[4]};
    calib::FaceV f;
    calib::star_flux<DIR>(P, x, S, r[0], r[1], r[2], ust, r[5], f);
    FaceIO::put(f, y);
  }
};

template <int DIR, bool GS>
struct CalEdges {
  static constexpr int NI = 3 * F2 + 2, NO = 2 * F2;
  __device__ static Cand cand(const Params& P, const double* x) {
    auto nd = []() { return 1.0; };
    return calib::phi_candidates(P, x[0], x[F2], x[2 * F2], nd);
  }
  __device__ static void fwd(const Params& P, double nu, const double* x, double* y) {
    const Cand c0 = cand(P, x);
    calib::edges_predict<DIR>(P, x, x + F2, x + 2 * F2, x[3 * F2], x[3 * F2 + 1], c0, c0, c0, nu, y, y + F2);
  }
  __device__ static void bwd(const Params& P, double nu, const double* x, const double* yb, double* xb) {
    const Cand c0 = cand(P, x);
    adj::PBar pb;
    adj::pbar_zero(pb);
    double cb[4];
    adj::edges_bwd<DIR, GS>(P, x, x + F2, x + 2 * F2, x[3 * F2], x[3 * F2 + 1], c0, c0, c0, nu, yb, yb + F2, xb,
                            xb + F2, xb + 2 * F2, xb[3 * F2], xb[3 * F2 + 1], cb, pb, true);
    double st[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}}, stb[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
    adj::cand_bwd<DIR>(P, x[0], x[F2], x[2 * F2], st, cb, xb[0], xb[F2], xb[2 * F2], stb);
  }
};

// (update_bwd and plastic_bwd have one instance)
template <int DIR>
struct CalUpdate : StUpdate<DIR> {
  __device__ static void fwd(const Params& P, double nu, const double* x, double* y) {
    calib::FaceV a, b;
    FaceIO::get(x + F2 + 1, a);
    FaceIO::get(x + F2 + 1 + F2 + 3, b);
    calib::update_cell<DIR>(x, x[F2], a, b, nu, y);
  }
};

struct CalPlastic : StPlastic {
  __device__ static void fwd(const Params& P, double, const double* x, double* y) {
    for (int k = 0; k < F2; ++k) y[k] = x[k];
    double s[2];
    calib::epilogue_cell(P, y, 0.0, s);
  }
};

template <bool GS>
int stage_run_t(int stage, int dir, const Params& P, double nu, int n, const double* X, const double* V,
                const double* WY, double eps, double* out) {
  auto go = [&](auto along_x, auto along_y) {
    return dir == 0 ? run<decltype(along_x)>(P, nu, n, X, V, WY, eps, out)
                    : run<decltype(along_y)>(P, nu, n, X, V, WY, eps, out);
  };
  switch (stage) {
    case 0: return go(CalC2P<GS>{}, CalC2P<GS>{});
    case 1: return go(CalSide<0, GS>{}, CalSide<1, GS>{});
    case 2: return go(CalStress<0, GS>{}, CalStress<1, GS>{});
    case 3: return go(CalFace<0, GS>{}, CalFace<1, GS>{});
    case 4: return go(CalStar<0>{}, CalStar<1>{});
    case 5: return go(CalEdges<0, GS>{}, CalEdges<1, GS>{});
    case 6: return go(CalUpdate<0>{}, CalUpdate<1>{});
    case 7: return go(CalPlastic{}, CalPlastic{});
  }
  return -1;
}

}  // namespace

extern "C" {

// as unit_run, on the calibrated step's stages; gs: the reverse stages' instance
int stage_run(int gs, int stage, int dir, const dimp_material* mats, const dimp_options* opt, const double* dx,
              double nu, int n, const double* X, const double* V, const double* WY, double eps, double* out) {
  const Params P = make_params(mats, opt, dx);
  return gs ? stage_run_t<true>(stage, dir, P, nu, n, X, V, WY, eps, out)
            : stage_run_t<false>(stage, dir, P, nu, n, X, V, WY, eps, out);
}

}  // extern "C"
