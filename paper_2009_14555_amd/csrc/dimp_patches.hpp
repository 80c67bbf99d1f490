// dimp_patches.hpp -- split sweeps over a set of independent 2-D patches.
//
// AMR-style patch sets (the paper's AMR platform applies the single-grid
// update to every patch of a level in turn, Sec. 3): many small rectangular
// patches of different sizes, each stored with two ghost layers, all advanced
// with one global dt.  Instead of one launch per patch and sweep, one launch
// per sweep covers a precomputed task list of the whole set:
//  * psweep_row: a work item is one wave (one cell per lane, as in
//    sweep_row) holding segments of interior rows;
//  * psweep_tile: a work item is a CW-column x 64-row tile staged through LDS
//    (as in sweep_tile) holding segments of column chunks.
// Segments carry their own 3-lane halos, so short lines of different patches
// share a wave: a writer lane reads lanes within 3 of itself only, all inside
// its own segment, and the packing cannot change any result bit.
// Each wave/block takes one work item (a grid-stride persistent loop was
// measured first: its carried state pushed the sweep body into VGPR spills).
// Boundaries are transmissive per patch: halo reads are clamped into the
// patch interior, and every sweep also writes the ghost copies of the
// boundary cells it updates, so the stored ghost layers always hold the
// boundary images.  Per-patch launches run the same kernels on the task
// range of one patch, so both modes produce identical bits.
#pragma once
#include <hip/hip_runtime.h>

#include "dimp_internal.hpp"
#include "dimp_lane.hpp"

namespace dimp {

constexpr int PD = 2;
// waves per SIMD of the patch sweeps: 2 with a JWL mixture (its split holds
// more live state) or three materials, 4 where the state fits 128 VGPRs (a
// material profile without a history slot), else 3 (with the ghost positions in
// LDS and the tiles in place: 2048 patches of 16..128 cells a side, two steps,
// 1924 -> 1810 us)
template <int N, int RX, int PROF>
constexpr int patch_waves() {
  if (RX == 2 || N > 2) return 2;
  return (RX == 0 && PROF != PROF_ANY) ? 4 : 3;
}

// where a thread writes its cell: {element (low, high word), row pitch, sides
// of the patch it borders: 1 x low, 2 x high, 4 y low, 8 y high; -1 nothing to
// write}; parked in LDS while the sweep runs (in registers it pushed them past
// 128: 48 spilled bytes a lane)
__device__ __forceinline__ int4 patch_pos(const PatchGeo& g, int i, int j, bool live) {
  const int pitch = g.nx + 2 * PATCH_GHOST;
  const int64_t o = g.off + (int64_t)(j + PATCH_GHOST) * pitch + PATCH_GHOST + i;
  const int edge = (i == 0 ? 1 : 0) | (i == g.nx - 1 ? 2 : 0) | (j == 0 ? 4 : 0) | (j == g.ny - 1 ? 8 : 0);
  return make_int4((int)(uint32_t)o, (int)(o >> 32), pitch, live ? edge : -1);
}

// write the cell at pos, v(f) its fields, and, on a side, its ghost images; the
// conditions are taken once for all fields
template <int F, class V>
__device__ __forceinline__ void write_with_ghosts(const int4& pos, double* out, int64_t E, V&& v) {
  const int edge = pos.w;
  if (edge < 0) return;
  double* o = out + (((int64_t)pos.y << 32) | (uint32_t)pos.x);
#pragma unroll
  for (int f = 0; f < F; ++f) o[f * E] = v(f);
  if (edge == 0) return;
  const int di0 = (edge & 1) ? -PATCH_GHOST : 0, di1 = (edge & 2) ? PATCH_GHOST : 0;
  const int dj0 = (edge & 4) ? -PATCH_GHOST : 0, dj1 = (edge & 8) ? PATCH_GHOST : 0;
#pragma unroll 1
  for (int dj = dj0; dj <= dj1; ++dj)
#pragma unroll 1
    for (int di = di0; di <= di1; ++di) {
      if (di == 0 && dj == 0) continue;
      double* q = o + (int64_t)dj * pos.z + di;
#pragma unroll
      for (int f = 0; f < F; ++f) q[f * E] = v(f);
    }
}

// segment of lane (or tile row) r among segments [sb, se): the last one
// whose first lane is <= r
__device__ __forceinline__ int4 segment_of(const int4* __restrict__ seg, int sb, int se, int r) {
  int4 sg = seg[sb];
  for (int k = sb + 1; k < se; ++k) {
    const int4 c = seg[k];
    if (r >= (c.w & 255)) sg = c;
  }
  return sg;
}

template <int N, int RX, int PROF, bool FUSE, int WPB>
__global__ __launch_bounds__(64 * WPB, (patch_waves<N, RX, PROF>())) void psweep_row(
    Params P, const PatchGeo* __restrict__ geo, WorkList wl, int64_t w0, int64_t nwork, const double* __restrict__ in,
    double* __restrict__ out, double dt_arg, const double* __restrict__ dtp, double* __restrict__ part) {
  constexpr int F = Lay<PD, N, RX>::F;
  assume_profile<N, RX, PROF>(P);
  const int lane = threadIdx.x & 63;
  const int64_t wv = xcd_block(blockIdx.x, gridDim.x) * WPB + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (wv >= nwork) return;  // whole waves only: a work item is one wave
  const double dt = dtp ? dtp[0] : dt_arg;
  const double nu = over_dx(P, 0, dt);
  const int64_t E = P.ncell;
  __shared__ double stash[F * 64 * WPB];
  const int sb = wl.beg[w0 + wv], se = wl.beg[w0 + wv + 1];
  const int4 sg = segment_of(wl.seg, sb, se, lane);  // {patch, row, first x, lane0 | n << 8}
  const PatchGeo g = geo[sg.x];
  const int j = sg.y;
  const int q = lane - (sg.w & 255), ncl = sg.w >> 8;
  const int x = sg.z + q - SEG_HALO;
  const int xm = x < 0 ? 0 : (x > g.nx - 1 ? g.nx - 1 : x);
  const int64_t pitch = g.nx + 2 * PATCH_GHOST;
  const int64_t cell = g.off + (int64_t)(j + PATCH_GHOST) * pitch + PATCH_GHOST + xm;
  bool first = true;
  auto load_U = [&](double* U) {
    if (first) {
#pragma unroll
      for (int f = 0; f < F; ++f) {
        U[f] = in[f * E + cell];
        stash[f * 64 * WPB + threadIdx.x] = U[f];
      }
      first = false;
    } else {
      asm volatile("" ::: "memory");
#pragma unroll
      for (int f = 0; f < F; ++f) U[f] = stash[f * 64 * WPB + threadIdx.x];
    }
  };
  // rows j-1, j+1 clamped into the patch (stored ghost values are never read)
  auto phi_at = [&](int b, int) -> double {
    return in[b == 0 ? (j > 0 ? cell - pitch : cell) : (j < g.ny - 1 ? cell + pitch : cell)];
  };
  const bool writer = (q >= SEG_HALO) && (q < ncl + SEG_HALO);
  __shared__ int4 pos[64 * WPB];
  pos[threadIdx.x] = patch_pos(g, x, j, writer);
  double Un[F], s[PD];
  lane_sweep<PD, N, RX, 0, FUSE, false, PROF>(P, load_U, phi_at, nu, dt, writer, Un, s);
  asm volatile("" ::: "memory");
  write_with_ghosts<F>(pos[threadIdx.x], out, E, [&](int f) { return Un[f]; });
  if (FUSE) {
#pragma unroll
    for (int k = 0; k < PD; ++k) wave_max_store(s[k], part + (w0 + wv) * 3 + k);
  }
}

template <int N, int RX, int PROF, bool FUSE, int CW>
__global__ __launch_bounds__(64 * CW, (patch_waves<N, RX, PROF>())) void psweep_tile(
    Params P, const PatchGeo* __restrict__ geo, WorkList wl, int64_t w0, int64_t nwork, const double* __restrict__ in,
    double* __restrict__ out, double dt_arg, const double* __restrict__ dtp, double* __restrict__ part) {
  constexpr int F = Lay<PD, N, RX>::F;
  assume_profile<N, RX, PROF>(P);
  using G = TileGeom<CW>;
  extern __shared__ double tileU[];  // the input state, then the results in place
  const int64_t t = xcd_block(blockIdx.x, gridDim.x);
  if (t >= nwork) return;  // whole block: a work item is one tile
  const double dt = dtp ? dtp[0] : dt_arg;
  const double nu = over_dx(P, 1, dt);
  const int64_t E = P.ncell;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int sb = wl.beg[w0 + t], se = wl.beg[w0 + t + 1];
  // this thread's tile element (row r, column c) for the load and the store
  const int r = tid / CW, c = tid % CW;
  const int4 sr = segment_of(wl.seg, sb, se, r);  // {patch, x0, first y, lane0 | n << 8}
  const PatchGeo gr = geo[sr.x];
  const int64_t pr = gr.nx + 2 * PATCH_GHOST;
  const int qr = r - (sr.w & 255);
  const int xr = sr.y + c, jr = sr.z + qr - SEG_HALO;
  {
    const int xc = xr > gr.nx - 1 ? gr.nx - 1 : xr;
    const int jc = jr < 0 ? 0 : (jr > gr.ny - 1 ? gr.ny - 1 : jr);
    const int64_t cell = gr.off + (jc + PATCH_GHOST) * pr + PATCH_GHOST + xc;
#pragma unroll
    for (int f = 0; f < F; ++f) tileU[G::at(f, r, c)] = in[f * E + cell];
  }
  __shared__ int4 pos[64 * CW];
  pos[tid] = patch_pos(gr, xr, jr, qr >= SEG_HALO && qr < (sr.w >> 8) + SEG_HALO && xr < gr.nx);
  __syncthreads();
  auto load_U = [&](double* U) {
    asm volatile("" ::: "memory");
#pragma unroll
    for (int f = 0; f < F; ++f) U[f] = tileU[G::at(f, lane, w)];  // (the lane's own slots)
  };
  const int4 sl = segment_of(wl.seg, sb, se, lane);
  const PatchGeo gl = geo[sl.x];
  const int ql = lane - (sl.w & 255);
  const bool writer = (ql >= SEG_HALO) && (ql < (sl.w >> 8) + SEG_HALO) && (sl.y + w < gl.nx);
  // columns x-1, x+1 clamped into the patch
  auto phi_at = [&](int b, int) -> double {
    const int xx = sl.y + w + b - 1, jj = sl.z + ql - SEG_HALO;
    const int xc = xx < 0 ? 0 : (xx > gl.nx - 1 ? gl.nx - 1 : xx);
    const int jc = jj < 0 ? 0 : (jj > gl.ny - 1 ? gl.ny - 1 : jj);
    return in[gl.off + (jc + PATCH_GHOST) * (int64_t)(gl.nx + 2 * PATCH_GHOST) + PATCH_GHOST + xc];
  };
  double Un[F], s[PD];
  lane_sweep<PD, N, RX, 1, FUSE, false, PROF>(P, load_U, phi_at, nu, dt, writer, Un, s);
  if (writer) {
#pragma unroll
    for (int f = 0; f < F; ++f) tileU[G::at(f, lane, w)] = Un[f];
  }
  __syncthreads();
  write_with_ghosts<F>(pos[tid], out, E, [&](int f) { return tileU[G::at(f, tid / CW, tid % CW)]; });
  if (FUSE) {
#pragma unroll
    for (int k = 0; k < PD; ++k) wave_max_store(s[k], part + ((w0 + t) * CW + w) * 3 + k);
  }
}

template <int N, int RX, int CW>
size_t tile_lds_bytes() {
  return sizeof(double) * Lay<PD, N, RX>::F * 64 * CW;
}

// one sweep of a patch set with N materials and the RX layout (the
// launch_patch_sweep contract)
template <int N, int RX, int PROF>
hipError_t launch_patch_p(const Params& P, const PatchGeo* geo, WorkList wl, int64_t w0, int64_t nwork,
                          const double* in, double* out, double dt, const double* dtp, int dir, bool fuse,
                          double* part, int row_wpb, int cw, hipStream_t st) {
  if (nwork <= 0) return hipSuccess;
  if (dir == 0) {
    const dim3 grid((unsigned)((nwork + row_wpb - 1) / row_wpb));
    const dim3 block(64 * row_wpb);
#define DIMP_ROW(W)                                                                                              \
  if (fuse)                                                                                                     \
    launch_params((psweep_row<N, RX, PROF, true, W>), grid, block, 0, st, P, geo, wl, w0, nwork, in, out, dt, dtp,  \
                       part);                                                                                   \
  else                                                                                                          \
    launch_params((psweep_row<N, RX, PROF, false, W>), grid, block, 0, st, P, geo, wl, w0, nwork, in, out, dt, dtp, \
                       part);
    if (row_wpb == 1) {
      DIMP_ROW(1)
    } else if (row_wpb == 2) {
      DIMP_ROW(2)
    } else {
      DIMP_ROW(4)
    }
#undef DIMP_ROW
    return hipGetLastError();
  }
  const dim3 grid((unsigned)nwork);
  if (cw == 8) {
    const size_t lds = tile_lds_bytes<N, RX, 8>();
    if (fuse)
      launch_params((psweep_tile<N, RX, PROF, true, 8>), grid, dim3(512), lds, st, P, geo, wl, w0, nwork, in, out, dt,
                         dtp, part);
    else
      launch_params((psweep_tile<N, RX, PROF, false, 8>), grid, dim3(512), lds, st, P, geo, wl, w0, nwork, in, out, dt,
                         dtp, part);
  } else {
    const size_t lds = tile_lds_bytes<N, RX, 4>();
    if (fuse)
      launch_params((psweep_tile<N, RX, PROF, true, 4>), grid, dim3(256), lds, st, P, geo, wl, w0, nwork, in, out, dt,
                         dtp, part);
    else
      launch_params((psweep_tile<N, RX, PROF, false, 4>), grid, dim3(256), lds, st, P, geo, wl, w0, nwork, in, out, dt,
                         dtp, part);
  }
  return hipGetLastError();
}

// the instance of the materials' profile
template <int N, int RX>
hipError_t launch_patch_t(const Params& P, const PatchGeo* geo, WorkList wl, int64_t w0, int64_t nwork,
                          const double* in, double* out, double dt, const double* dtp, int dir, bool fuse,
                          double* part, int row_wpb, int cw, hipStream_t st) {
  return by_profile<N, RX>(P, [&](auto prof) {
    return launch_patch_p<N, RX, decltype(prof)::value>(P, geo, wl, w0, nwork, in, out, dt, dtp, dir, fuse, part,
                                                        row_wpb, cw, st);
  });
}

}  // namespace dimp
