// dimp_sweeps.hpp -- the sweep kernels (row and tile) and their launch templates.
//
//  * sweep_row: sweep along x, the contiguous axis.  One cell per lane: a
//    wave covers 64 consecutive cells of a row, 3 on each side being halo,
//    so 58 cells are written per wave.  Stencil neighbours along x come from
//    cross-lane shuffles; no LDS, no barriers.  Loads and stores are
//    coalesced 512-byte rows per field.
//  * sweep_tile: sweep along y or z.  The same one-cell-per-lane stages on a
//    tile of 4 or 8 x columns by 64 cells, staged through LDS so that HBM sees
//    contiguous row segments.
// Both deal their blocks to the XCDs in short runs (xcd_block).
// The last sweep of a step can fuse the plastic and reactive fractional steps
// and the wave-speed reduction into its epilogue (FUSE), so a 2-D step reads
// and writes the state exactly twice.  Included by the translation units that
// instantiate the sweeps: dimp_kernels.hip (1-D and 2-D grids) and
// dimp_sweeps3.hip (3-D grids), compiled in parallel.
#pragma once
#include <hip/hip_runtime.h>

#include "dimp_calib.hpp"
#include "dimp_internal.hpp"
#include "dimp_lane.hpp"

namespace dimp {

// A tile sweep's block has four waves (eight in the wide 2-D tile below) and 4 or
// 8 columns (a wave takes its columns one after the other).  Eight columns read and write 64 contiguous
// bytes of a row instead of 32: 256^3, y 1757 -> 1549 us, z 2419 -> 2241 (with
// eight waves, and with 16 columns, slower by a third and more: the LDS of 17
// fields holds one such block a CU).  With the sources fused (z 3032, 3039) and
// on 2-D grids (2048^2: y 232, 249; fused 257, 260) the second column costs what
// the wider rows gain or more.
constexpr int TILE_WAVES = 4;
constexpr int tile_columns(int D, bool fuse) { return (D == 3 && !fuse) ? 8 : 4; }
// Two-dimensional y sweeps that run four waves a SIMD take eight columns with
// eight waves where the state read and the state written exceed the 256 MB
// cache in front of the memory, which takes the short rows' partial lines:
// y alone, four columns and eight: 777 x 1031 39 and 41 us, 1024^2 42 and 46,
// 1448^2 113 and 106, 2048^2 220 and 199, 4096^2 860 and 742.  (With the sources
// fused 2048^2 took 234 and 253.)
constexpr int64_t WIDE_TILE_BYTES = int64_t(256) << 20;

// waves per SIMD the sweep kernels are built for (launch bound): four where
// the state fits 128 VGPRs, the 1-D and 2-D instances of a two-material profile
// without a history slot (122-126; at five waves they spill 120 bytes a lane);
// three (168) with a history slot, for three materials and for the general and
// calibrated instances (134-167); the 3-D sweeps (nine stretch entries, up to
// 17 fields) need 176-182 VGPRs and run two without spilling, and so do the
// fused sweeps of a JWL mixture (207) and of three reacting materials; the fused
// x sweep of a gas mixture spills 60 bytes at three waves and is the faster for
// it (256^3: 2225 -> 2085 us; z fused 2430 -> 2920, x 1231 -> 1456)
template <int D, int N, int RX, int PROF, bool FUSE, bool TILE>
constexpr int sweep_waves() {
  if (D == 3) return (FUSE && !TILE && RX == 1 && PROF != PROF_ANY) ? 3 : 2;
  if (FUSE && (RX == 2 || (RX && N > 2))) return 2;
  return (N == 2 && RX == 0 && PROF != PROF_ANY && PROF != PROF_CALIB) ? 4 : 3;
}

// Output modes of the sweep kernels.  M_SPLIT: the split sweep, out = the
// updated state.  The unsplit SSP-RK3 of Sec. 3.1 evaluates D(q) direction
// by direction, y (and z) first through the tile kernel, x last through the
// row kernel, and builds the stage as it goes.  A stage is
//   a qn + b (q - dt D(q)),  (a, b) = (0, 1), (3/4, 1/4), (1/3, 2/3)
// for stages 1, 2, 3 (eq. (rk) with q^(2) and q^(4) folded in): M_RK_FIRST
// writes a qn + b (q - dt D_dir); M_RK_MID and M_RK_LAST write
// Rin - b dt D_dir (in 1-D the x pass is the first); the last pass of stage 3
// fuses the sources and the wave speed (FUSE).  The partial results differ
// from summing D first only by rounding.
enum { M_SPLIT = 0, M_RK_FIRST = 1, M_RK_MID = 2, M_RK_LAST = 3 };

__device__ __forceinline__ double rk_a(int stage) { return stage == 1 ? 0.0 : stage == 2 ? 0.75 : 1.0 / 3.0; }
__device__ __forceinline__ double rk_b(int stage) { return stage == 1 ? 1.0 : stage == 2 ? 0.25 : 2.0 / 3.0; }

// ----------------------------------------------------------- row sweep
// Sweep along x.  Each wave: one 64-cell segment of one row, loaded and
// stored straight from HBM (512-byte rows per field).
template <int D, int N, int RX, int PROF, bool FUSE, int MODE = M_SPLIT, bool WALL = false>
__global__ __launch_bounds__(256, (sweep_waves<D, N, RX, PROF, FUSE, false>())) void sweep_row(Params P, const double* __restrict__ in, double* __restrict__ out,
                                                  double dt_arg, const double* __restrict__ dtp,
                                                  double* __restrict__ part, const double* __restrict__ Rin,
                                                  const double* qn, int stage) {
  using L = Lay<D, N, RX>;
  constexpr int F = L::F;
  assume_profile<N, RX, PROF>(P);
  const double dt = dtp ? dtp[0] : dt_arg;
  const int lane = threadIdx.x & 63;
  const int64_t nx = P.n[0], ny = P.n[1], nz = P.n[2];
  const int64_t nseg = (nx + 57) / 58;
  // the blocks of a run are the same and the neighbouring rows, whose volume
  // fractions the THINC normals read
  const int64_t lb = xcd_block(blockIdx.x, gridDim.x);
  // one value per wave, told to the compiler so that the index arithmetic (its
  // divisions above all) runs on the scalar unit
  const int64_t wave = lb * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t row = wave / nseg;
  if (row >= ny * nz) return;  // uniform per wave
  const int64_t seg = wave - row * nseg;
  const int64_t x = seg * 58 + lane - 3;
  // WALL instances: reflective ends along x (mirror images, the wall's tie)
  const bool xflip = WALL && bc_mirrored(x, nx, P.bc[0]);
  const int64_t xm = WALL ? bc_map_wall(x, nx, P.bc[0]) : bc_map(x, nx, P.bc[0]);
  const int64_t yj = row % ny, zk = row / ny;
  const int64_t nc = P.ncell;
  const int64_t cell = row * nx + xm;
  // the conserved state is read from HBM once and parked in LDS (each lane
  // only touches its own slots) until the update needs it again
  __shared__ double stash[F * 256];
  bool first = true;
  auto load_U = [&](double* U) {
    if (first) {
#pragma unroll
      for (int f = 0; f < F; ++f) {
        U[f] = in[f * nc + cell];
        if (WALL && mirror_odd<D, N, RX>(f, 0) && xflip) U[f] = -U[f];  // a wall's mirror image
        stash[f * 256 + threadIdx.x] = U[f];
      }
      first = false;
    } else {
      asm volatile("" ::: "memory");  // re-read LDS rather than keep U live in registers
#pragma unroll
      for (int f = 0; f < F; ++f) U[f] = stash[f * 256 + threadIdx.x];
    }
  };
  auto phi_at = [&](int b, int c) -> double {
    const int64_t yy = bc_map(yj + b - 1, ny, P.bc[1]);
    const int64_t zz = (D == 3) ? bc_map(zk + c - 1, nz, P.bc[2]) : 0;
    return in[(zz * ny + yy) * nx + xm];
  };
  const bool writer = (lane >= 3) && (lane < 61) && (x < nx);
  // the face on this lane's left is a reflective wall
  const bool wall = WALL && ((x == 0 && (P.bc[0] == BC_REFLECTIVE || P.bc[0] == BC_AXIS)) ||
                             (x == nx && P.bc[0] == BC_REFLECTIVE));
  double Un[F], s[D];
  if constexpr (PROF == PROF_CALIB) {
    calib::lane_sweep<0, FUSE>(P, load_U, phi_at, dt / P.dx[0], dt, writer, Un, s, wall);
  } else if (MODE == M_SPLIT) {
    lane_sweep<D, N, RX, 0, FUSE, false, PROF>(P, load_U, phi_at, over_dx(P, 0, dt), dt, writer, Un, s, wall);
  } else {
    lane_sweep<D, N, RX, 0, false, true, PROF>(P, load_U, phi_at, P.idx[0], dt, writer, Un, s, wall);
    if (writer) {
      const double b = rk_b(stage);
      if (D > 1) {
        // the y (and z) passes have formed a qn + b (q - dt D_y ...)
#pragma unroll
        for (int f = 0; f < F; ++f) Un[f] = Rin[f * nc + cell] - (b * dt) * Un[f];
      } else {
        double U[F];
        load_U(U);
        const double a = rk_a(stage);
#pragma unroll
        for (int f = 0; f < F; ++f) {
          const double q = U[f] - dt * Un[f];
          Un[f] = (stage == 1) ? q : a * qn[f * nc + cell] + b * q;
        }
      }
      if (FUSE) epilogue_cell<D, N, RX>(P, Un, dt, s);
    }
  }
  if (writer) {
#pragma unroll
    for (int f = 0; f < F; ++f) out[f * nc + cell] = Un[f];
  }
  if (FUSE) {
#pragma unroll
    for (int k = 0; k < D; ++k) wave_max_store(s[k], part + wave * 3 + k);
  }
}

// ---------------------------------------------------------- tile sweep
// Sweep along y or z.  A block of NW waves covers CW consecutive x columns
// and 64 cells along the sweep axis; the tile is staged through LDS so that
// HBM sees rows of CW doubles, while each wave takes the columns w, w + NW, ...,
// one at a time with one cell per lane, through the same stages as the row
// sweep.  The blocks of a run (xcd_block) are neighbouring x chunks, which share L2 lines.
template <int D, int N, int RX, int PROF, int DIR, bool FUSE, int CW, int MODE = M_SPLIT, bool WALL = false,
          int NW = TILE_WAVES>
__global__ __launch_bounds__(64 * NW, (sweep_waves<D, N, RX, PROF, FUSE, true>())) void sweep_tile(Params P, const double* __restrict__ in,
                                                       double* __restrict__ out, double dt_arg,
                                                       const double* __restrict__ dtp,
                                                       double* __restrict__ part,
                                                       const double* __restrict__ Rin, const double* qn,
                                                       int stage) {
  using L = Lay<D, N, RX>;
  using G = TileGeom<CW>;
  constexpr int F = L::F;
  assume_profile<N, RX, PROF>(P);
  extern __shared__ double lds[];
  double* tileU = lds;  // [F][64][CW]: the input state, then the results in place
  const double dt = dtp ? dtp[0] : dt_arg;

  const int64_t lb = xcd_block(blockIdx.x, gridDim.x);
  const int64_t nx = P.n[0], ny = P.n[1], nz = P.n[2];
  const int64_t nm = P.n[DIR];
  const int oa = (DIR == 1) ? 2 : 1;  // the other transverse axis (3-D)
  const int64_t no = (D == 3) ? P.n[oa] : 1;
  const int64_t nxc = (nx + CW - 1) / CW;
  const int64_t xc = lb % nxc;
  int64_t rest = lb / nxc;
  const int64_t o = rest % no;
  const int64_t seg = rest / no;
  const int64_t x0 = xc * CW;
  const int64_t j0 = seg * 58 - 3;
  const int64_t sx = 1, sm = (DIR == 1) ? nx : nx * ny, so = (oa == 1) ? nx : nx * ny;
  const int64_t nc = P.ncell;
  const int tid = threadIdx.x;

  // load the tile: thread t -> row r (sweep axis), column c (x)
  for (int t = tid; t < 64 * CW; t += 64 * NW) {
    const int r = t / CW, c = t % CW;
    const int64_t xx = bc_map(x0 + c, nx, P.bc[0]);
    const int64_t jj = WALL ? bc_map_wall(j0 + r, nm, P.bc[DIR]) : bc_map(j0 + r, nm, P.bc[DIR]);
    const int64_t cell = xx * sx + jj * sm + o * so;
#pragma unroll
    for (int f = 0; f < F; ++f) tileU[G::at(f, r, c)] = in[f * nc + cell];
    // WALL instances: a wall's mirror image
    if (WALL && bc_mirrored(j0 + r, nm, P.bc[DIR])) {
#pragma unroll
      for (int f = 0; f < F; ++f)
        if (mirror_odd<D, N, RX>(f, DIR)) tileU[G::at(f, r, c)] = -tileU[G::at(f, r, c)];
    }
  }
  __syncthreads();
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  double smax[D];
#pragma unroll
  for (int k = 0; k < D; ++k) smax[k] = 0.0;
#pragma unroll 1
  for (int col = w; col < CW && x0 + col < nx; col += NW) {
    // every lane reads and writes its own slots of the wave's column only
    auto load_U = [&](double* U) {
      asm volatile("" ::: "memory");  // re-read LDS rather than keep U live in registers
#pragma unroll
      for (int f = 0; f < F; ++f) U[f] = tileU[G::at(f, lane, col)];
    };
    // transverse phi offsets: b along x, c along the other axis (3-D)
    auto phi_at = [&](int b, int c) -> double {
      const int64_t xx = bc_map(x0 + col + b - 1, nx, P.bc[0]);
      const int64_t jj = bc_map(j0 + lane, nm, P.bc[DIR]);
      const int64_t oo = (D == 3) ? bc_map(o + c - 1, no, P.bc[oa]) : 0;
      return in[xx * sx + jj * sm + oo * so];
    };
    // lane_sweep orders the transverse offsets over the other two axes in
    // increasing axis order: for DIR = 1 that is (x, z), for DIR = 2 (x, y)
    const bool writer = (lane >= 3) && (lane < 61) && (j0 + lane < nm);
    const int64_t jl = j0 + lane;
    const bool wall = WALL && ((jl == 0 && (P.bc[DIR] == BC_REFLECTIVE || P.bc[DIR] == BC_AXIS)) ||
                               (jl == nm && P.bc[DIR] == BC_REFLECTIVE));
    double Un[F], s[D];
    if constexpr (PROF == PROF_CALIB)
      calib::lane_sweep<DIR, FUSE>(P, load_U, phi_at, dt / P.dx[DIR], dt, writer, Un, s, wall);
    else if (MODE == M_SPLIT)
      lane_sweep<D, N, RX, DIR, FUSE, false, PROF>(P, load_U, phi_at, over_dx(P, DIR, dt), dt, writer, Un, s, wall);
    else
      lane_sweep<D, N, RX, DIR, false, true, PROF>(P, load_U, phi_at, P.idx[DIR], dt, writer, Un, s, wall);
    if (MODE == M_RK_FIRST && writer) {
      // q - dt D_y(q) (the input tile still holds q)
      double U[F];
      load_U(U);
#pragma unroll
      for (int f = 0; f < F; ++f) Un[f] = U[f] - dt * Un[f];
    }
    if (writer) {
#pragma unroll
      for (int f = 0; f < F; ++f) tileU[G::at(f, lane, col)] = Un[f];
    }
#pragma unroll
    for (int k = 0; k < D; ++k) smax[k] = (s[k] > smax[k] || s[k] != s[k]) ? s[k] : smax[k];
  }
  __syncthreads();
  for (int t = tid; t < 64 * CW; t += 64 * NW) {
    const int r = t / CW, c = t % CW;
    const int64_t xx = x0 + c, jj = j0 + r;
    if (r >= 3 && r < 61 && xx < nx && jj < nm) {
      const int64_t cell = xx * sx + jj * sm + o * so;
      if (MODE == M_SPLIT) {
#pragma unroll
        for (int f = 0; f < F; ++f) out[f * nc + cell] = tileU[G::at(f, r, c)];
      } else {
        // the stage's partial result: the tile holds D_z (mid) or
        // q - dt D_y (first)
        const double a = rk_a(stage), b = rk_b(stage);
#pragma unroll
        for (int f = 0; f < F; ++f) {
          const double d = tileU[G::at(f, r, c)];
          double v;
          if (MODE == M_RK_MID)
            v = Rin[f * nc + cell] - (b * dt) * d;
          else
            v = (stage == 1) ? d : a * qn[f * nc + cell] + b * d;
          out[f * nc + cell] = v;
        }
      }
    }
  }
  if (FUSE && MODE == M_SPLIT) {
    const int64_t slot = lb * NW + w;
#pragma unroll
    for (int k = 0; k < D; ++k) wave_max_store(smax[k], part + slot * 3 + k);
  }
}

// ---------------------------------------------------------------- launch
static inline int grid_for(int64_t work, int block) {
  int64_t g = (work + block - 1) / block;
  if (g > 65535LL * 64) g = 65535LL * 64;
  return (int)(g < 1 ? 1 : g);
}

template <int D, int N, int RX, int PROF, int DIR, bool FUSE, int MODE = M_SPLIT>
static void launch_tile(const Params& P, const double* in, double* out, double dt, const double* dtp,
                        double* part, hipStream_t st, const double* Rin = nullptr, const double* qn = nullptr,
                        int stage = 0) {
  using L = Lay<D, N, RX>;
  const int oa = (DIR == 1) ? 2 : 1;
  const int64_t no = (D == 3) ? P.n[oa] : 1;
  const int64_t segs = no * ((P.n[DIR] + 57) / 58);
  auto launch = [&](auto kernel, int cw, int waves) {
    launch_params(kernel, dim3((unsigned)(((P.n[0] + cw - 1) / cw) * segs)), dim3(64 * waves),
                       sizeof(double) * L::F * 64 * cw, st, P, in, out, dt, dtp, part, Rin, qn, stage);
  };
  constexpr int CW = tile_columns(D, FUSE);
  if constexpr (PROF != PROF_CALIB) {  // (those grids have no walls)
    if (P.bc[DIR] >= BC_REFLECTIVE)
      return launch(sweep_tile<D, N, RX, PROF, DIR, FUSE, CW, MODE, true>, CW, TILE_WAVES);
  }
  if constexpr (D == 2 && !FUSE && sweep_waves<D, N, RX, PROF, FUSE, true>() == 4) {
    if (2 * int64_t(sizeof(double)) * L::F * P.ncell > WIDE_TILE_BYTES)
      return launch(sweep_tile<D, N, RX, PROF, DIR, FUSE, 8, MODE, false, 8>, 8, 8);
  }
  launch(sweep_tile<D, N, RX, PROF, DIR, FUSE, CW, MODE>, CW, TILE_WAVES);
}

static inline int row_grid(const Params& P) {
  const int64_t nseg = (P.n[0] + 57) / 58;
  const int64_t waves = nseg * P.n[1] * P.n[2];
  return (int)((waves + 3) / 4);  // four waves a block
}

template <int D, int N, int RX, int PROF>
static hipError_t launch_rk_p(const Params& P, int dir, int mode, int stage, bool fuse, const double* in,
                              double* out, const double* Rin, const double* qn, double dt, const double* dtp,
                              double* part, hipStream_t st) {
  if (dir == 0) {
    if (mode != M_RK_LAST) return hipErrorInvalidValue;
    if (P.bc[0] >= BC_REFLECTIVE) {
      if (fuse)
        launch_params((sweep_row<D, N, RX, PROF, true, M_RK_LAST, true>), dim3(row_grid(P)), dim3(256), 0, st, P, in,
                           out, dt, dtp, part, Rin, qn, stage);
      else
        launch_params((sweep_row<D, N, RX, PROF, false, M_RK_LAST, true>), dim3(row_grid(P)), dim3(256), 0, st, P,
                           in, out, dt, dtp, part, Rin, qn, stage);
      return hipGetLastError();
    }
    if (fuse)
      launch_params((sweep_row<D, N, RX, PROF, true, M_RK_LAST>), dim3(row_grid(P)), dim3(256), 0, st, P, in, out, dt,
                         dtp, part, Rin, qn, stage);
    else
      launch_params((sweep_row<D, N, RX, PROF, false, M_RK_LAST>), dim3(row_grid(P)), dim3(256), 0, st, P, in, out,
                         dt, dtp, part, Rin, qn, stage);
    return hipGetLastError();
  }
  if constexpr (D >= 2) {
    if (dir == 1 && mode == M_RK_FIRST) {
      launch_tile<D, N, RX, PROF, 1, false, M_RK_FIRST>(P, in, out, dt, dtp, part, st, nullptr, qn, stage);
      return hipGetLastError();
    }
    if constexpr (D == 3) {
      if (dir == 2 && mode == M_RK_MID) {
        launch_tile<D, N, RX, PROF, 2, false, M_RK_MID>(P, in, out, dt, dtp, part, st, Rin, qn, stage);
        return hipGetLastError();
      }
    }
  }
  return hipErrorInvalidValue;
}

template <int D, int N, int RX, int PROF>
static hipError_t launch_sweep_p(const Params& P, const double* in, double* out, double dt, const double* dtp,
                                 int dir, bool fuse, double* part, hipStream_t st) {
  const int block = 256;
  if (dir == 0) {
    const int grid = row_grid(P);
    if constexpr (PROF != PROF_CALIB) {  // (those grids have no walls)
      if (P.bc[0] >= BC_REFLECTIVE) {
        if (fuse)
          launch_params((sweep_row<D, N, RX, PROF, true, M_SPLIT, true>), dim3(grid), dim3(block), 0, st, P, in,
                             out, dt, dtp, part, nullptr, nullptr, 0);
        else
          launch_params((sweep_row<D, N, RX, PROF, false, M_SPLIT, true>), dim3(grid), dim3(block), 0, st, P, in,
                             out, dt, dtp, part, nullptr, nullptr, 0);
        return hipGetLastError();
      }
    }
    if (fuse)
      launch_params((sweep_row<D, N, RX, PROF, true>), dim3(grid), dim3(block), 0, st, P, in, out, dt, dtp, part,
                         nullptr, nullptr, 0);
    else
      launch_params((sweep_row<D, N, RX, PROF, false>), dim3(grid), dim3(block), 0, st, P, in, out, dt, dtp, part,
                         nullptr, nullptr, 0);
    return hipGetLastError();
  }
  if constexpr (D >= 2) {
    if (dir == 1) {
      if (fuse) launch_tile<D, N, RX, PROF, 1, true>(P, in, out, dt, dtp, part, st);
      else launch_tile<D, N, RX, PROF, 1, false>(P, in, out, dt, dtp, part, st);
      return hipGetLastError();
    }
    if constexpr (D == 3) {
      if (fuse) launch_tile<D, N, RX, PROF, 2, true>(P, in, out, dt, dtp, part, st);
      else launch_tile<D, N, RX, PROF, 2, false>(P, in, out, dt, dtp, part, st);
      return hipGetLastError();
    }
  }
  return hipErrorInvalidValue;
}

// the instance of the materials' profile
template <int D, int N, int RX>
static hipError_t launch_sweep_t(const Params& P, const double* in, double* out, double dt, const double* dtp,
                                 int dir, bool fuse, double* part, hipStream_t st) {
  return by_profile<N, RX>(P, [&](auto prof) {
    return launch_sweep_p<D, N, RX, decltype(prof)::value>(P, in, out, dt, dtp, dir, fuse, part, st);
  });
}

template <int D, int N, int RX>
static hipError_t launch_rk_t(const Params& P, int dir, int mode, int stage, bool fuse, const double* in,
                              double* out, const double* Rin, const double* qn, double dt, const double* dtp,
                              double* part, hipStream_t st) {
  return by_profile<N, RX>(P, [&](auto prof) {
    return launch_rk_p<D, N, RX, decltype(prof)::value>(P, dir, mode, stage, fuse, in, out, Rin, qn, dt, dtp, part,
                                                        st);
  });
}

}  // namespace dimp
