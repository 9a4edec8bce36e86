// Elastodynamics kernels (Eq. 7, 8): strain, stress with traction rows,
// divergence, magnetoelastic force, and the (u, v) Runge-Kutta stages.
#pragma once

#include <type_traits>

#include "common.h"
#include "prof.h"

namespace mmp {

// Blocks of the strain and force kernels over nz planes of nbx x nby tiles of
// 64x4 cells: the tiles, whose rows share their y neighbours, or 256
// consecutive cells each where more than a tenth of the tiles' lanes would lie
// past the grid.  Steps in tiles / linear (FP64): 16x8192 514 / 340 us, 1x65536
// 3525 / 1570, 65x4096 571 / 452, 160x1600 369 / 359, 300x200x4 382 / 395,
// 128x2048 334 / 337.  While every tile has a CU to itself idle lanes cost
// nothing (2048x1: 66 / 71).
// (The kernels are built for each: with a branch on it steps of 2048x64 FP32
// in tiles took 138 us instead of 137, linear ones of 16x8192 208 instead of 180.)
inline bool elastic_linear(long N, int nbx, int nby, int nz) {
  const long tiles = (long)nbx * nby * nz, lines = (N + 255) / 256;
  return tiles > 256 && 10 * tiles > 11 * lines;
}
inline int elastic_blocks(long N, int nbx, int nby, int nz) {
  return (int)(nbx == 0 || elastic_linear(N, nbx, nby, nz) ? (N + 255) / 256
                                                           : (long)nbx * nby * nz);
}

template <typename T>
struct ElasticArgs {
  int nx, ny, nz, nsub;
  long N;
  int nbx, nby;                  // 64x4 tiles; nbx 0: 256 consecutive cells a block
  T dx, dy, dz;
  T C11, C12, C44, eta, inv_rho;
  double trac_amp, trac_omega;   // sigma_xz(t) = amp sin(omega t) on x = 0
  T B1[2], B2[2];
  int mel[2];                    // sublattice contributes a force
  const Table<T>* tbl;
  Ctrl* ctrl;
  int rk;                        // the pair (RK::t), host side
  int stage;                     // 1..7, or 0 = evaluate at (un, vn)
  int fuse2;
  T* eps;                        // [6][N] strain of the stage input
  T beta;                        // Rayleigh stiffness coefficient, s
  T* sig;                        // [6][N] stress with traction rows
  double* epart;                 // [blocks] elastic energy partials (eval)
  double V;
  double rho;
};

// The instance of an elastic kernel: f(LIN, ONE) with 256 consecutive cells a
// block or tiles, and with an axis along x or y that may have one cell.  (The
// masks of such an axis, in every kernel, would cost 0.8 % of a step.)
template <typename T, typename F>
void elastic_variant(const ElasticArgs<T>& a, F f) {
  auto pick = [&](auto lin) {
    if (a.nx == 1 || a.ny == 1) f(lin, std::true_type{});
    else f(lin, std::false_type{});
  };
  if (a.nbx == 0) pick(std::true_type{});
  else pick(std::false_type{});
}

// strain of the stage-s displacement into eps (consumed by the field
// kernel's magnetoelastic term) and the stress with its traction rows into
// sig; eval: the elastic energy as well
template <typename T>
void launch_strain(const ElasticArgs<T>& a, bool eval, hipStream_t st, Prof* prof);
// divergence, forces, k_u/k_v and the next stage's u, v inputs
template <typename T>
void launch_force(const ElasticArgs<T>& a, hipStream_t st, Prof* prof);
template <typename T>
void launch_elastic_combine2(const Table<T>* tbl, const Ctrl* ctrl, long N, hipStream_t st,
                             Prof* prof);

}  // namespace mmp
