// Launchers of the reverse-mode (adjoint) kernels of one timestep; internal to the library.
// Planes are dense [ny][nx]; the state planes phi^n, c^n are read from the field pool (row pitch `pitch`).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lbm_internal.h"

namespace lbm {

// Forward intermediates of step n, as exported by the stage-export kernels (doubles, dense planes).
struct AdjFwd {
  const double *mu, *X, *Fx, *Fy, *n, *ux, *uy, *ph, *ch, *Xh;
};

// Every plane an adjoint step reads or writes (T = arithmetic type, dense planes of nx * ny).
template <typename T>
struct AdjPlanes {
  const T *phi, *c;  // state at n (pitched rows)
  int pitch;
  const T *fb1, *pb1, *cb1;  // adjoint of f (9 planes), phi, c at n + 1
  T *fb, *pb, *cb;           // adjoint at n (outputs)
  // intermediate adjoints: of phi^{n+1/2}, c^{n+1/2} (K12 -> K3) and of the force (K3 -> K45)
  T *phb, *chb, *Fxb, *Fyb;
};

struct AdjModel {
  int nx, ny;
  int walls;  // LBM_WALLS_NONE or LBM_WALLS_Y
  double a, b, B0, B1, D, Gamma, gamma, omega, coef, ramp;  // ramp = min(n, t*): dA(n)/dA0
  double yper;
};

// The droplets as of one step: parameters from the table, centre k at cen[k * stride].
struct AdjDrops {
  const DropDev* table;
  const double* cen;
  int stride, n;
};

// One backward step: the adjoint at n + 1 -> the adjoint at n.  Each block adds its partial sum of
// sum_r cb1(r) * ramp * count_n(r) over its tile (the step's contribution to d/dA0) to part[tile]; part holds
// adj_parts(nx, ny) running totals, zeroed before the first step.
template <typename T>
hipError_t launch_adjoint_step(hipStream_t s, const AdjModel& m, const AdjFwd& f, const AdjPlanes<T>& p,
                               const AdjDrops& drops_n, double* part);

// Seed of the loss x_CM^N of droplet `drop`, whose table at N is drops_end: the sum sw of phi over the droplet's nodes
// (phi^N >= 0, nearest centre of step N - 1), then pb = (dx - delta) / sw on those nodes and 0 elsewhere (delta: the
// centre's last move), fb and cb cleared, and part (adj_parts values) zeroed.
template <typename T>
hipError_t launch_adjoint_seed(hipStream_t s, const AdjModel& m, const T* phi, int pitch, const AdjDrops& prev,
                               const DropDev* drops_end, int drop, T* fb, T* pb, T* cb, double* part, double* sw);

// *out = the sum of part[0 .. n), in twice the working precision.
hipError_t launch_adjoint_total(hipStream_t s, const double* part, int n, double* out);

// out[i] = src[i] for i < n, as doubles, to page-locked host memory.
template <typename T>
hipError_t launch_widen(hipStream_t s, const T* src, int64_t n, double* out);

// The step's kernels: one launch over tiles of ADJ_OX x ADJ_OY nodes that keep every intermediate in LDS (adj_tiled),
// or three launches over tiles of ADJ_TILE_X x ADJ_TILE_Y nodes (adj_blocks: one block per tile, at least one per 256
// nodes, which the seed kernel's one-dimensional blocks need).
constexpr int ADJ_TILE_X = 64, ADJ_TILE_Y = 4;
inline int adj_blocks(int nx, int ny) {
  return ((nx + ADJ_TILE_X - 1) / ADJ_TILE_X) * ((ny + ADJ_TILE_Y - 1) / ADJ_TILE_Y);
}
constexpr int ADJ_OX = 16, ADJ_OY = 16, ADJ_NT = 512;
constexpr int ADJ_RINGS = 5;  // a lattice is at least a tile and its rings on one side wide and high
inline int adj_tiles(int nx, int ny) { return ((nx + ADJ_OX - 1) / ADJ_OX) * ((ny + ADJ_OY - 1) / ADJ_OY); }
// One workgroup per compute unit at most: beyond, the rings' arithmetic costs more than the launches and planes saved.
// A backward step with its recomputed step, us, tiles / three launches: 200 x 200 FP64 24.4 / 35.3, 256 x 256 25.7 / 32.1
// (FP32 22.5 / 28.6); beyond, 300 x 300 40.0 / 40.2, 400 x 400 61.5 / 55.7, 512 x 512 82.7 / 70.2 (FP32 52.5 / 53.1),
// 1024 x 1024 311 / 238.
inline bool adj_tiled(int nx, int ny) {
  return nx >= ADJ_OX + ADJ_RINGS && ny >= ADJ_OY + ADJ_RINGS && adj_tiles(nx, ny) <= 256;
}
inline int adj_parts(int nx, int ny) { return adj_tiled(nx, ny) ? adj_tiles(nx, ny) : adj_blocks(nx, ny); }

}  // namespace lbm
