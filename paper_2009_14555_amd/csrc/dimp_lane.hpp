// dimp_lane.hpp -- the stages of one sweep for a wave holding one cell per lane.
#pragma once
#include "dimp_stencil.hpp"

namespace dimp {

// The block that runs as the grid's b-th of nb.  The hardware deals blocks
// round-robin to the 8 XCDs, each with its own L2; here runs of consecutive
// blocks are dealt instead, so that neighbours share an L2, and many runs to
// each XCD, so that a costly region (the reaction zone above all) is spread over
// all of them.  One run for each XCD left a 400 x 1000 detonating stick at 691 us
// for two steps, where runs of 16 blocks take 445 (4: 458, 64: 538); 256^3, with
// 10 times the blocks, 13310 us, where runs of 64 take 12070 (16: 12140, 4:
// 12480); 2048^2 1935, 1852 (16: 1885, 4: 1978).  So runs of 4 and 16 start where
// they leave each XCD eight runs, and runs of 64 at 32 each: with 4096 to 16384
// blocks they would leave eight to 32, and the reaction zone of a 500 x 2000 stick
// (4500 blocks) takes 775 us for two steps against 640 in runs of 16, of an 800 x
// 2000 one (7000) 1005 against 855, while discs of 1000^2 to 1900^2, three materials
// at 1000^2 and slabs of 110^3 and 150^3 take the same in both.
__device__ __forceinline__ int64_t xcd_block(uint32_t b, uint32_t nb) {
  const int sh = nb >= 16384 ? 6 : nb >= 1024 ? 4 : nb >= 256 ? 2 : 0;  // log2 of the run
  const uint32_t group = 8u << sh;
  if (b >= nb - (nb & (group - 1))) return b;  // the last, incomplete deal
  return (b & ~(group - 1)) + ((b & 7) << sh) + ((b >> 3) & ((1u << sh) - 1));
}

// A [F][64][CW] tile of doubles in LDS, rows along the sweep axis, columns x
template <int CW>
struct TileGeom {
  // element (f, r, c) of a [F][64][CW] tile: the column index is XOR-swizzled
  // by the row so that both access patterns are free of LDS bank conflicts:
  // the coalesced copies (16 lanes = 16/CW rows x CW columns) and the
  // per-wave column reads (16 lanes = 16 rows of one column)
  static constexpr int RS = 16 / CW;
  __device__ static constexpr int at(int f, int r, int c) { return (f * 64 + r) * CW + (c ^ ((r / RS) & (CW - 1))); }
};

// THINC candidates of every stored volume fraction of the lane's cell, all
// with the normal of the first, and the BVD choice on them.
template <int D, int N, int RX, int DIR, class PhiAt>
__device__ __forceinline__ void lane_bvd(const Params& P, const double* Wm, const double* W, const double* Wp,
                                         PhiAt&& phi_at, double* WL, double* WR, double* jump) {
  // phi_1 around the lane's cell for the interface normal (all lanes load and
  // shuffle; the normal itself is only evaluated in mixed cells)
  double phi_t[3][3], sm[3][3], sp[3][3];
  if (D >= 2) {
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        if (D == 2 && c != 1) continue;
        phi_t[b][c] = (b == 1 && c == 1) ? W[0] : phi_at(b, c);
      }
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        if (D == 2 && c != 1) continue;
        sm[b][c] = from_left(phi_t[b][c]);
        sp[b][c] = from_right(phi_t[b][c]);
      }
  }
  auto normal = [&]() -> double {
    if (D == 1) return 1.0;
    if (D == 2) {
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
    }
    // 3-D: transverse offsets (b, c) run over the two other axes in order
    double st[3][3][3];
    constexpr int o1 = (DIR == 0) ? 1 : 0, o2 = (DIR == 2) ? 1 : 2;
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const double v[3] = {sm[b][c], phi_t[b][c], sp[b][c]};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          int idx[3];
          idx[DIR] = a;
          idx[o1] = b;
          idx[o2] = c;
          st[idx[0]][idx[1]][idx[2]] = v[a];
        }
      }
    return youngs3(st, P.dx, DIR);
  };
  // the neighbours' right (left) edge candidates by shifts
  CandSet<N> c0, cm, cp;
#pragma unroll
  for (int l = 0; l < N - 1; ++l) {
    c0.c[l] = phi_candidates<D, N, RX>(P, Wm[l], W[l], Wp[l], normal);
    cm.c[l].mR = from_left(c0.c[l].mR);
    cm.c[l].tR = from_left(c0.c[l].tR);
    cp.c[l].mL = from_right(c0.c[l].mL);
    cp.c[l].tL = from_right(c0.c[l].tL);
  }
  edges_bvd<N>(cm, c0, cp, WL, WR, jump);
}

// ------------------------------------------------- lane-per-cell sweep
// The stages of one sweep for a wave whose 64 lanes hold 64 consecutive cells
// along the sweep axis (3 halo cells on each side, lanes 3..60 are written).
// U: the lane's conserved state; phi_at(b, c): phi_1 of the lane's cell at
// transverse offsets (b - 1, c - 1) in {-1,0,1}^2 (2-D uses c = 1 only),
// called in waves that hold a mixed cell, with the offset along the sweep axis
// supplied by shuffles.
// U is read twice through load_U (for the primitive state and for the
// update) rather than kept in registers across the face computation.
// RK = false: the split MUSCL-Hancock sweep, Un = the updated state (and, with
// FUSE, the source steps and the wave speed s of the result).  RK = true: the
// direction's part of the unsplit operator of Sec. 3.1, Un = D_dir(q) with
// nu = 1/dx (edges without the predictor; FUSE is left to the caller).
//
// lane_face: the stages up to the flux through the face on the left of the
// lane's cell (fa; wall: that face is a reflective wall), and the cell's
// 1 / (sum of partial densities); it depends on the cells 3 to the left and
// 2 to the right.  lane_sweep adds the update.
template <int D, int N, int RX, int DIR, bool RK, int PROF = -1, class LoadU, class PhiAt>
__device__ __forceinline__ void lane_face(const Params& P, LoadU&& load_U, PhiAt&& phi_at, double nu,
                                          FaceV<D, N, RX>& fa, double& irho0, bool wall) {
  using L = Lay<D, N, RX>;
  constexpr int F = L::F;
  double W[F];
  double rc2;
  {
    double U[F];
    load_U(U);
    Thermo<N, RX> T;
    double H[6], J2;
    cons_to_prim<D, N, RX>(P, U, W, T, H, J2);
    irho0 = T.irho;  // 1 / sum of partial densities
    rc2 = T.rc2;
  }
  double Wm[F], Wp[F];
#pragma unroll
  for (int f = 0; f < F; ++f) {
    Wm[f] = from_left(W[f]);
    Wp[f] = from_right(W[f]);
  }
  double WL[F], WR[F], jump[F];
  edges_limited<D, N, RX>(P, Wm, W, Wp, WL, WR, jump);
  if (P.thinc) {
    // THINC and the BVD choice where a lane of the wave holds a mixed cell
    // (elsewhere both candidates of every fraction are the MUSCL edges)
    bool mixed = false;
#pragma unroll
    for (int l = 0; l < N - 1; ++l) {
      double num, den;
      mixed = mixed || thinc_mixed(P, Wm[l], W[l], Wp[l], num, den);
    }
    if (__builtin_amdgcn_ballot_w64(mixed) != 0) lane_bvd<D, N, RX, DIR>(P, Wm, W, Wp, phi_at, WL, WR, jump);
  }
  if (!RK) edges_half_step<D, N, RX, DIR>(fresh<N, RX, PROF>(P), W, jump, irho0, rc2, nu, WL, WR);
  // face on the left of this cell: right edge of the left neighbour | my left edge
  double WRm[F];
#pragma unroll
  for (int f = 0; f < F; ++f) WRm[f] = from_left(WR[f]);
  face_flux<D, N, RX, DIR>(fresh<N, RX, PROF>(P), WRm, WL, fa, wall);
}

template <int D, int N, int RX, int DIR, bool FUSE, bool RK = false, int PROF = -1, class LoadU, class PhiAt>
__device__ __forceinline__ void lane_sweep(const Params& P, LoadU&& load_U, PhiAt&& phi_at, double nu,
                                           double dt, bool writer, double* Un, double* s, bool wall = false) {
  constexpr int F = Lay<D, N, RX>::F;
  FaceV<D, N, RX> fa, fb;
  double irho0;
  lane_face<D, N, RX, DIR, RK, PROF>(P, load_U, phi_at, nu, fa, irho0, wall);
#pragma unroll
  for (int f = 0; f < F; ++f) fb.F[f] = from_right(fa.F[f]);
  fb.ustar = from_right(fa.ustar);
#pragma unroll
  for (int j = 0; j < D; ++j) fb.Vn[j] = from_right(fa.Vn[j]);
  {
    double U[F];
    load_U(U);
    if (RK)
      div_cell<D, N, RX, DIR>(U, irho0, fa, fb, nu, Un);
    else
      update_cell<D, N, RX, DIR>(U, irho0, fa, fb, nu, Un);
  }
#pragma unroll
  for (int k = 0; k < D; ++k) s[k] = 0.0;
  if (FUSE && !RK && writer) epilogue_cell<D, N, RX, PROF>(fresh<N, RX, PROF>(P), Un, dt, s);
}

}  // namespace dimp
