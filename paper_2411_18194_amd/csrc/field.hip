// Fused effective field + torque + Runge-Kutta stage kernel.
//
// One thread owns zc cells of an (x, y) column and marches along z with the
// z neighbours kept in registers; x/y neighbours come from global memory
// through L1/L2 (a 64x4 tile per block, blocks remapped so neighbouring
// tiles share an XCD's L2).  Shorter marches (small zc) give more waves to
// hide the latency of the dependent loads; longer ones re-read fewer
// z neighbours.  Per cell and sublattice it forms
//   B = B_demag + exchange (Eq. 3: 2A11/Ms lap m, A12/Ms lap m', 4A0/(Ms a^2) m')
//     + interfacial DMI (one sublattice) or homogeneous DMI d.(m1 x m2) (two)
//     + uniaxial/cubic anisotropy + Zeeman + B_mel (Eq. 9)
// and the torque tau = LLG (Eq. 2) + Zhang-Li, then, in a Runge-Kutta
// stage, writes k_s and immediately the next stage input
// y_{s+1} = normalise(y_n + h sum_j a_{s+1,j} k_j) (all point-wise), or at
// the last stage the FP64 error norm |sum_j e_j k_j| of the embedded pair in
// use (Table 2).
//
// Boundaries: a missing neighbour is the cell itself (Neumann), except in a
// layer with interfacial DMI, where the ghost is m -/+ d (dm/dn) with the
// natural boundary condition 2A dn m = -D (z x n) x m (Eq. 5 for one
// sublattice).  Zhang-Li uses clamped central differences.  Along a
// periodic axis (x or y) the neighbour of a boundary cell is the cell at the
// opposite end, for every stencil, and no boundary condition applies.
#include "field.h"
#include "elastic_dev.h"

namespace mmp {

template <typename T>
__device__ __forceinline__ void cross3(const T* a, const T* b, T* o) {
  o[0] = a[1] * b[2] - a[2] * b[1];
  o[1] = a[2] * b[0] - a[0] * b[2];
  o[2] = a[0] * b[1] - a[1] * b[0];
}

// a*b - c*d with one rounding error (Kahan's difference of products)
template <typename T>
__device__ __forceinline__ T dop(T a, T b, T c, T d) {
  const T w = c * d;
  const T e = fma(-c, d, w);
  const T f = fma(a, b, -w);
  return f + e;
}

// m x m' accurate to a few ulp of the result even when m' ~ -m
template <typename T>
__device__ __forceinline__ void cross3_acc(const T* a, const T* b, T* o) {
  o[0] = dop(a[1], b[2], a[2], b[1]);
  o[1] = dop(a[2], b[0], a[0], b[2]);
  o[2] = dop(a[0], b[1], a[1], b[0]);
}

// 1/|v|, with the roundings spelled out: the stage-2 input of a step is formed
// by different kernels (a stage's own, or the one that continues a run), and
// has to be the same bits from each
template <typename T>
__device__ __forceinline__ T inv_norm(const T* v) {
  return T(1) / sqrt(fma(v[2], v[2], fma(v[1], v[1], v[0] * v[0])));
}

template <typename T>
__device__ __forceinline__ double dot3d(const T* a, const T* b) {
  return (double)a[0] * b[0] + (double)a[1] * b[1] + (double)a[2] * b[2];
}

// Ghosts beyond one face (axis ax, outward side +-1, cell size h) of every
// sublattice from the Neumann condition of Eq. 6:
//   2 A11^(s) g_s = A12 (g_s' x m_s) x m_s + m_s x w_s,  w_s = side W^(s)_ax,
// with (g x m) x m = -Q g, Q = I - m m^T; for two sublattices g2 solves
// (2 A2 I - A12^2/(2 A1) Q2 Q1) g2 = b2 - A12/(2 A1) Q2 b1 (Cramer's rule),
// then g1 = (b1 - A12 Q1 g2)/(2 A1).  A sublattice with A11 = 0 keeps a
// plain copy.  ghost = m + h g.
template <typename T, int NSUB>
__device__ void eq6_ghost(const FieldArgs<T>& a, const T (*m)[3], int ax, T side, T h,
                          T (*out)[3]) {
  T b[NSUB][3], g[NSUB][3];
#pragma unroll
  for (int s = 0; s < NSUB; ++s) {
    T w[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) w[c] = side * a.eW[s][ax][c];
    cross3(m[s], w, b[s]);
#pragma unroll
    for (int c = 0; c < 3; ++c) g[s][c] = T(0);
  }
  if constexpr (NSUB == 1) {
    if (a.eA[0] != T(0))
#pragma unroll
      for (int c = 0; c < 3; ++c) g[0][c] = b[0][c] / (T(2) * a.eA[0]);
  } else {
    const T A1 = a.eA[0], A2 = a.eA[1], A12 = a.eA12;
    if (A1 != T(0) && A2 != T(0)) {
      T Q1[3][3], Q2[3][3], M[3][3], r[3];
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          Q1[i][j] = (i == j ? T(1) : T(0)) - m[0][i] * m[0][j];
          Q2[i][j] = (i == j ? T(1) : T(0)) - m[1][i] * m[1][j];
        }
      const T c = A12 * A12 / (T(2) * A1), e = A12 / (T(2) * A1);
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        T q2b1 = T(0);
#pragma unroll
        for (int k = 0; k < 3; ++k) q2b1 += Q2[i][k] * b[0][k];
        r[i] = b[1][i] - e * q2b1;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          T qq = T(0);
#pragma unroll
          for (int k = 0; k < 3; ++k) qq += Q2[i][k] * Q1[k][j];
          M[i][j] = (i == j ? T(2) * A2 : T(0)) - c * qq;
        }
      }
      const T det = M[0][0] * (M[1][1] * M[2][2] - M[1][2] * M[2][1]) -
                    M[0][1] * (M[1][0] * M[2][2] - M[1][2] * M[2][0]) +
                    M[0][2] * (M[1][0] * M[2][1] - M[1][1] * M[2][0]);
      const T id = T(1) / det;
      g[1][0] = id * (r[0] * (M[1][1] * M[2][2] - M[1][2] * M[2][1]) -
                      M[0][1] * (r[1] * M[2][2] - M[1][2] * r[2]) +
                      M[0][2] * (r[1] * M[2][1] - M[1][1] * r[2]));
      g[1][1] = id * (M[0][0] * (r[1] * M[2][2] - M[1][2] * r[2]) -
                      r[0] * (M[1][0] * M[2][2] - M[1][2] * M[2][0]) +
                      M[0][2] * (M[1][0] * r[2] - r[1] * M[2][0]));
      g[1][2] = id * (M[0][0] * (M[1][1] * r[2] - r[1] * M[2][1]) -
                      M[0][1] * (M[1][0] * r[2] - r[1] * M[2][0]) +
                      r[0] * (M[1][0] * M[2][1] - M[1][1] * M[2][0]));
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        T q1g2 = T(0);
#pragma unroll
        for (int k = 0; k < 3; ++k) q1g2 += Q1[i][k] * g[1][k];
        g[0][i] = (b[0][i] - A12 * q1g2) / (T(2) * A1);
      }
    } else if (A1 != T(0)) {
#pragma unroll
      for (int c = 0; c < 3; ++c) g[0][c] = b[0][c] / (T(2) * A1);
    } else if (A2 != T(0)) {
#pragma unroll
      for (int c = 0; c < 3; ++c) g[1][c] = b[1][c] / (T(2) * A2);
    }
  }
#pragma unroll
  for (int s = 0; s < NSUB; ++s)
#pragma unroll
    for (int c = 0; c < 3; ++c) out[s][c] = m[s][c] + h * g[s][c];
}

// Accesses of the field kernel: a wave-uniform base and a 32-bit byte offset
// per lane (grids have at most 2^28 cells, so an array's bytes per component
// stay below 2^32), which the hardware adds.  64-bit addresses per lane and
// array took two registers and an addition for every one of the up to 50
// loads of a cell: FP32 one sublattice 204 -> 97 registers (two -> four
// waves per SIMD), FP64 298 -> 172 (one -> two); 512x512x16 FP32 90 -> 87 us
// a stage (4.3 TB/s), FP64 204 -> 174 (4.2 TB/s; held to the 168 registers of
// three waves 176).
template <typename T>
__device__ __forceinline__ T ldo(gcptr<T> base, uint32_t o) {
  return *(gcptr<T>)((gcptr<char>)base + o);
}
template <typename T>
__device__ __forceinline__ T ldo_nt(gcptr<T> base, uint32_t o) {
  return __builtin_nontemporal_load((gcptr<T>)((gcptr<char>)base + o));
}
template <typename T>
__device__ __forceinline__ void sto(gptr<T> base, uint32_t o, T v) {
  *(gptr<T>)((gptr<char>)base + o) = v;
}

// Block w (tile-major over z chunks) of one grid; stage and fuse2 come from
// the launch so that one argument block serves every stage.
// GDMI: general DMI tensors with the Eq. 6 ghosts on every stencil.
// GBX: exchange links between different grains scaled by gbx_scale.
// NK: slopes a cell's sum may hold (the pair's stages less one); 6 serves every
// pair, the pairs of two and three run their own with several sublattices.
template <typename T, int NSUB, bool EVAL, bool GDMI = false, bool GBX = false, int NK = 6>
__device__ __forceinline__ void field_block(const FieldArgs<T>& a, const RKStage& rk, const int zero, const int w,
                                            const int stage, const int fuse2) {
  const int ntile = a.nbx * a.nby;
  if (w >= ntile * a.nzc) return;
  const int tile = w % ntile;
  const int z0 = (w / ntile) * a.zc;
  const int z1 = min(a.nz, z0 + a.zc);
  const int x = (tile % a.nbx) * kTileX + (int)(threadIdx.x % kTileX);
  const int y = (tile / a.nbx) * kTileY + (int)(threadIdx.x / kTileX);
  const bool in = x < a.nx && y < a.ny;
  const long N0 = a.N;
  // every pointer and the step size first: their loads and the controller's
  // flags make one trip, the data the second
  const gcptr<T> m = (gcptr<T>)table_slot<T>(a.tbl, rk.in + zero);
  double h = 0.0;
  const int ns = rk.ns;
  T ca[6] = {0, 0, 0, 0, 0, 0};
  gcptr<T> kin[6] = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
  gptr<T> kout = nullptr;
  gptr<T> ynext = nullptr;
  gcptr<T> yn = nullptr;
  if (!EVAL) {
    h = a.ctrl->h;
    kout = uni_ptr((gptr<T>)a.tbl->k[stage - 1]);
    yn = uni_ptr((gcptr<T>)a.tbl->yn);
#pragma unroll
    for (int j = 0; j < 6; ++j)
      if (j < stage - 1) kin[j] = uni_ptr((gcptr<T>)a.tbl->k[j]);
    ynext = (gptr<T>)table_slot<T>(a.tbl, rk.out + zero);
  }
  if (ctrl_stopped(a.ctrl, zero)) return;
  if (!EVAL) {
#pragma unroll
    for (int j = 0; j < 6; ++j) ca[j] = (T)((stage < ns ? rk.a[j] : (j == 0 ? rk.a10 : 0.0)) * h);
  }
  const double* ew = rk.e;
  // slopes the one-sublattice march loads up front (see below): the ones
  // this stage sums, and in the other slots a buffer read anyway (k_1, or
  // y_n at stage 1, which has no earlier slope; never a null table entry)
  const gcptr<T> spare = stage >= 2 ? kin[0] : yn;
  gcptr<T> kslot[6];
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    const bool used = !EVAL && (stage < ns ? j < stage - 1 : (j < ns - 1 && ew[j] != 0.0));
    kslot[j] = used ? kin[j] : spare;
  }
  const gcptr<T> yslot = stage < ns ? yn : spare;

  double eacc[kNE];
  for (int t = 0; t < kNE; ++t) eacc[t] = 0.0;
  double emax = 0.0;

  if (in) {
    T cur[NSUB][3], zm[NSUB][3], zp[NSUB][3];
    const long N = N0, N3 = 3 * N0;
    constexpr uint32_t S = sizeof(T);
    const uint32_t col = (uint32_t)(y * a.nx + x);
    const uint32_t plane = (uint32_t)(a.nx * a.ny);
    // A missing neighbour is the cell itself, so every neighbour load is an
    // unconditional load from a clamped offset: no branches between the
    // loads, which then all go out before the first wait.
    // (on a periodic axis the cell at the opposite end)
    const int dxm = x > 0 ? -1 : (a.per_x ? a.nx - 1 : 0);
    const int dxp = x + 1 < a.nx ? 1 : (a.per_x ? 1 - a.nx : 0);
    const int dym = y > 0 ? -a.nx : (a.per_y ? (a.ny - 1) * a.nx : 0);
    const int dyp = y + 1 < a.ny ? a.nx : (a.per_y ? -(a.ny - 1) * a.nx : 0);
    const bool layers = a.nz > 1;   // a single layer is its own z neighbour
    {
      const uint32_t o0 = ((uint32_t)z0 * plane + col) * S;
      const uint32_t om = z0 > 0 ? o0 - plane * S : o0;
#pragma unroll
      for (int s = 0; s < NSUB; ++s)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          cur[s][c] = ldo<T>(m + s * N3 + c * N, o0);
          zm[s][c] = layers ? ldo<T>(m + s * N3 + c * N, om) : cur[s][c];
        }
    }
    for (int z = z0; z < z1; ++z) {
      // The component stride of the short pairs is hidden too: the bases of
      // every array and component, kept from one iteration to the next, are
      // more than the scalar registers hold, and to fetch them back from
      // vector lanes takes longer than to add the stride anew.
      long N = N0;
      if constexpr (NSUB > 1 && NK < 6) asm volatile("" : "+s"(N));
      const long N3 = 3 * N;
      const uint32_t i = (uint32_t)z * plane + col, o = i * S;
      const int dzp = z + 1 < a.nz ? (int)plane : 0;
      const uint32_t oxm = o + (uint32_t)dxm * S, oxp = o + (uint32_t)dxp * S,
                     oym = o + (uint32_t)dym * S, oyp = o + (uint32_t)dyp * S,
                     ozp = o + (uint32_t)dzp * S;
      // What a stage does beside its slope is hidden from the compiler within
      // the iteration: it would make a copy of the loop for every answer, and
      // contract products and sums into fma differently from copy to copy.
      // The slope at a state has to be the same bits in every stage (a run
      // resumed from a saved state evaluates it as k_1, the run it continues
      // as the last slope).
      // (has_slots: whether there are slots to load, with short pairs how many)
      int has_slots = uni(NK == 6 ? !EVAL && (stage < ns || !fuse2)
                              : stage < ns ? max(stage - 1, 1)
                              : fuse2      ? 0
                                           : ns - 1),
          has_next = uni(stage < ns || fuse2),
          is_last = uni(stage >= ns);
      asm volatile("" : "+s"(has_slots), "+s"(has_next), "+s"(is_last));
      // the grain's axis is two loads one behind the other: first
      T uax[3];
      if (a.has_anis_u && a.grain) {
        const int g = a.grain[i];
        uax[0] = a.gaxes[3 * g];
        uax[1] = a.gaxes[3 * g + 1];
        uax[2] = a.gaxes[3 * g + 2];
      }
      // one sublattice: the stage slopes and y_n of this cell are requested
      // with the stencil loads (they do not depend on the field, and loaded
      // after the k_s stores below they would wait for a second round trip)
      // Every slot is loaded (a slot this stage does not use reads k_1
      // again, a cache hit): no branch between the loads, which then all go
      // out before the first wait.
      T kv1[NK][3], yv1[3];
      if constexpr (NSUB == 1 && !EVAL) {
        if (has_slots) {
#pragma unroll
          for (int j = 0; j < NK; ++j)
#pragma unroll
            for (int c = 0; c < 3; ++c) kv1[j][c] = ldo<T>(kslot[j] + c * N, o);
#pragma unroll
          for (int c = 0; c < 3; ++c) yv1[c] = ldo<T>(yslot + c * N, o);
        }
      }
#pragma unroll
      for (int s = 0; s < NSUB; ++s)
#pragma unroll
        for (int c = 0; c < 3; ++c)
          zp[s][c] = layers ? ldo<T>(m + s * N3 + c * N, ozp) : cur[s][c];
      T xm[NSUB][3], xp[NSUB][3], ym[NSUB][3], yp[NSUB][3];
#pragma unroll
      for (int s = 0; s < NSUB; ++s)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const gcptr<T> mc = m + s * N3 + c * N;
          xm[s][c] = ldo<T>(mc, oxm);
          xp[s][c] = ldo<T>(mc, oxp);
          ym[s][c] = ldo<T>(mc, oym);
          yp[s][c] = ldo<T>(mc, oyp);
        }
      T Bd[3] = {0, 0, 0};
      if (a.has_demag) {
#pragma unroll
        for (int c = 0; c < 3; ++c) Bd[c] = ldo_nt<T>((gcptr<T>)a.Bd + c * N, o);
      }
      T ep[6] = {0, 0, 0, 0, 0, 0};
      if (a.has_mel) {
#pragma unroll
        for (int c = 0; c < 6; ++c) ep[c] = ldo<T>((gcptr<T>)a.eps + c * N, o);
      }
      // link weights x-, x+, y-, y+, z-, z+ of the A11 and A12 stencils: the
      // scale across a grain boundary, 1 inside a grain and towards a
      // missing neighbour (its offset is 0, the cell's own grain)
      T wl[6];
      if constexpr (GBX) {
        const uint16_t* gr = a.grain + i;
        const int g0 = gr[0];
        const T f = a.gbx_scale;
        wl[0] = gr[dxm] == g0 ? T(1) : f;
        wl[1] = gr[dxp] == g0 ? T(1) : f;
        wl[2] = gr[dym] == g0 ? T(1) : f;
        wl[3] = gr[dyp] == g0 ? T(1) : f;
        wl[4] = gr[z > 0 ? -(int)plane : 0] == g0 ? T(1) : f;
        wl[5] = gr[dzp] == g0 ? T(1) : f;
      }
      auto lk = [&](int k, T v) -> T {
        if constexpr (GBX) return wl[k] * v;
        else return v;
      };
      const bool dmil = NSUB == 1 && a.has_dmi && (a.dmi_layer < 0 || z == a.dmi_layer);
      // neighbours seen by the exchange and DMI stencils: the loaded ones, or
      // the Eq. 6 ghosts on the faces of the open axes (z neighbours are
      // copied: the rotating z registers must keep the cells themselves)
      T sxm[NSUB][3], sxp[NSUB][3], sym[NSUB][3], syp[NSUB][3], szm[NSUB][3], szp[NSUB][3];
#pragma unroll
      for (int s = 0; s < NSUB; ++s)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          sxm[s][c] = xm[s][c]; sxp[s][c] = xp[s][c]; sym[s][c] = ym[s][c];
          syp[s][c] = yp[s][c]; szm[s][c] = zm[s][c]; szp[s][c] = zp[s][c];
        }
      if constexpr (GDMI) {
        if (x == 0 && !a.per_x) eq6_ghost<T, NSUB>(a, cur, 0, T(-1), a.dx, sxm);
        if (x + 1 == a.nx && !a.per_x) eq6_ghost<T, NSUB>(a, cur, 0, T(1), a.dx, sxp);
        if (y == 0 && !a.per_y) eq6_ghost<T, NSUB>(a, cur, 1, T(-1), a.dy, sym);
        if (y + 1 == a.ny && !a.per_y) eq6_ghost<T, NSUB>(a, cur, 1, T(1), a.dy, syp);
        if (z == 0) eq6_ghost<T, NSUB>(a, cur, 2, T(-1), a.dz, szm);
        if (z + 1 == a.nz) eq6_ghost<T, NSUB>(a, cur, 2, T(1), a.dz, szp);
      }

#pragma unroll
      for (int s = 0; s < NSUB; ++s) {
        const SubC<T>& C = a.sc[s];
        const T* mm = cur[s];
        // several sublattices: the slopes of one sublattice at a time, asked
        // for before its field is computed (both at once, with the stencil,
        // would cost more waves than it hides).  The short pairs ask for the
        // ones a stage sums and no more: with six slots per stage, as one load
        // without branches, Heun and Bogacki-Shampine steps of 512x512x2 FP64
        // took 88 and 132 us with two sublattices, 172 and 262 with three, and
        // take 79 and 119, 103 and 164.  (Dormand-Prince steps, 278 and 564,
        // are as fast with all six.)
        T kvs[NK][3], yvs[3];
        if constexpr (NSUB > 1 && !EVAL) {
          if (has_slots) {
#pragma unroll
            for (int j = 0; j < NK; ++j) {
              if (NK == 6 || j == 0 || has_slots > j) {
#pragma unroll
                for (int c = 0; c < 3; ++c) kvs[j][c] = ldo<T>(kslot[j] + s * N3 + c * N, o);
              } else {
                kvs[j][0] = kvs[j][1] = kvs[j][2] = T(0);
              }
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) yvs[c] = ldo<T>(yslot + s * N3 + c * N, o);
          }
        }
        // ghosted in-plane neighbours for exchange/DMI
        T gxm[3], gxp[3], gym[3], gyp[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          gxm[c] = sxm[s][c]; gxp[c] = sxp[s][c]; gym[c] = sym[s][c]; gyp[c] = syp[s][c];
        }
        if (dmil) {
          // boundary condition of Eq. 5 on the faces of the open axes
          const T k = C.kdmi;
          if (x == 0 && !a.per_x) {
            gxm[0] = mm[0] - a.dx * k * mm[2]; gxm[1] = mm[1]; gxm[2] = mm[2] + a.dx * k * mm[0];
          }
          if (x + 1 == a.nx && !a.per_x) {
            gxp[0] = mm[0] + a.dx * k * mm[2]; gxp[1] = mm[1]; gxp[2] = mm[2] - a.dx * k * mm[0];
          }
          if (y == 0 && !a.per_y) {
            gym[0] = mm[0]; gym[1] = mm[1] - a.dy * k * mm[2]; gym[2] = mm[2] + a.dy * k * mm[1];
          }
          if (y + 1 == a.ny && !a.per_y) {
            gyp[0] = mm[0]; gyp[1] = mm[1] + a.dy * k * mm[2]; gyp[2] = mm[2] - a.dy * k * mm[1];
          }
        }
        T B[3] = {0, 0, 0};     // field driving the torque (all but A0)
        T Bout[3] = {0, 0, 0};  // extra output-only part (A0, eval mode)
        bool a0_on = false;
        T bt[3];
        auto add = [&](int term, const T* b) {
          if (!EVAL || (a.mask & (1u << term))) {
            B[0] += b[0]; B[1] += b[1]; B[2] += b[2];
          }
        };
        // exchange
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const T l = (lk(0, gxm[c] - mm[c]) + lk(1, gxp[c] - mm[c])) * a.idx2 +
                      (lk(2, gym[c] - mm[c]) + lk(3, gyp[c] - mm[c])) * a.idy2 +
                      (lk(4, szm[s][c] - mm[c]) + lk(5, szp[s][c] - mm[c])) * a.idz2;
          bt[c] = C.cex * l;
        }
        add(1, bt);
        if (EVAL) eacc[1] += -0.5 * C.Ms_d * dot3d(mm, bt);
        // interfacial DMI
        if (dmil) {
          bt[0] = C.cdmi * ((gxp[2] - gxm[2]) * a.i2dx);
          bt[1] = C.cdmi * ((gyp[2] - gym[2]) * a.i2dy);
          bt[2] = -C.cdmi * ((gxp[0] - gxm[0]) * a.i2dx + (gyp[1] - gym[1]) * a.i2dy);
          add(4, bt);
          if (EVAL) eacc[4] += -0.5 * C.Ms_d * dot3d(mm, bt);
        }
        // DMI tensors (Eq. 4): B = sum_i d_i m x cW_i + d_i m' x cW'_i,
        // cW = -2 W/Ms, central differences over the Eq. 6 ghosts
        if constexpr (GDMI) {
          T dm[3][3], dmo[3][3];
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            dm[0][c] = (sxp[s][c] - sxm[s][c]) * a.i2dx;
            dm[1][c] = (syp[s][c] - sym[s][c]) * a.i2dy;
            dm[2][c] = (szp[s][c] - szm[s][c]) * a.i2dz;
            if (NSUB == 2) {
              const int o = 1 - s;
              dmo[0][c] = (sxp[o][c] - sxm[o][c]) * a.i2dx;
              dmo[1][c] = (syp[o][c] - sym[o][c]) * a.i2dy;
              dmo[2][c] = (szp[o][c] - szm[o][c]) * a.i2dz;
            }
          }
          T acc[3] = {0, 0, 0}, tmp[3];
#pragma unroll
          for (int i = 0; i < 3; ++i) {
            cross3(dm[i], a.cW[s][i], tmp);
            acc[0] += tmp[0]; acc[1] += tmp[1]; acc[2] += tmp[2];
            if (NSUB == 2) {
              cross3(dmo[i], a.cW12[s][i], tmp);
              acc[0] += tmp[0]; acc[1] += tmp[1]; acc[2] += tmp[2];
            }
          }
          add(4, acc);
          if (EVAL) eacc[4] += -0.5 * C.Ms_d * dot3d(mm, acc);
        }
        // inter-sublattice exchange (Eq. 3) with every other sublattice:
        // A12/Ms lap m' (inhomogeneous) and 4 A0/(Ms a^2) m' (homogeneous)
        if (NSUB >= 2) {
#pragma unroll
          for (int c = 0; c < 3; ++c) bt[c] = T(0);
#pragma unroll
          for (int o = 0; o < NSUB; ++o) {
            if (o == s) continue;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
              const T mo = cur[o][c];
              const T l = (lk(0, sxm[o][c] - mo) + lk(1, sxp[o][c] - mo)) * a.idx2 +
                          (lk(2, sym[o][c] - mo) + lk(3, syp[o][c] - mo)) * a.idy2 +
                          (lk(4, szm[o][c] - mo) + lk(5, szp[o][c] - mo)) * a.idz2;
              bt[c] += C.cnn * l;
            }
          }
          add(2, bt);
          if (EVAL) eacc[2] += -0.5 * C.Ms_d * dot3d(mm, bt);
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            T so = T(0);
#pragma unroll
            for (int o = 0; o < NSUB; ++o)
              if (o != s) so += cur[o][c];
            bt[c] = C.ccell * so;
          }
          // The homogeneous inter-sublattice field is ~1000x larger than the
          // torque it leaves when m' ~ -m, so its torque is formed from an
          // accurate m x m' (tau is linear in B) instead of from B.
          if (!EVAL || (a.mask & (1u << 3))) {
            a0_on = true;
            if (EVAL) {
              Bout[0] += bt[0]; Bout[1] += bt[1]; Bout[2] += bt[2];
            }
          }
          if (EVAL) eacc[3] += -0.5 * C.Ms_d * dot3d(mm, bt);
          // homogeneous DMI d.(m1 x m2): B = m' x dh, dh = -/+ d/Ms
          if (NSUB == 2 && a.has_dmih) {
            cross3(cur[1 - s], C.dh, bt);
            add(4, bt);
            if (EVAL) eacc[4] += -0.5 * C.Ms_d * dot3d(mm, bt);
          }
        }
        // demag
        if (a.has_demag && C.nonzero) {
          add(0, Bd);
          if (EVAL) eacc[0] += -0.5 * C.Ms_d * dot3d(mm, Bd);
        }
        // uniaxial anisotropy
        if (a.has_anis_u) {
          const T* u = a.grain ? uax : C.u;
          const T um = u[0] * mm[0] + u[1] * mm[1] + u[2] * mm[2];
          const T f = C.cku1 * um + C.cku2 * um * um * um;
          bt[0] = f * u[0]; bt[1] = f * u[1]; bt[2] = f * u[2];
          add(5, bt);
          if (EVAL && C.nonzero) {
            const double umd = (double)um;
            eacc[5] += -C.Ku1_d * umd * umd - C.Ku2_d * umd * umd * umd * umd;
          }
        }
        // cubic anisotropy
        if (a.has_anis_c) {
          const T a1 = C.c1[0] * mm[0] + C.c1[1] * mm[1] + C.c1[2] * mm[2];
          const T a2 = C.c2[0] * mm[0] + C.c2[1] * mm[1] + C.c2[2] * mm[2];
          const T a3 = C.c3[0] * mm[0] + C.c3[1] * mm[1] + C.c3[2] * mm[2];
          const T f1 = -C.ckc * a1 * (a2 * a2 + a3 * a3);
          const T f2 = -C.ckc * a2 * (a1 * a1 + a3 * a3);
          const T f3 = -C.ckc * a3 * (a1 * a1 + a2 * a2);
#pragma unroll
          for (int c = 0; c < 3; ++c) bt[c] = f1 * C.c1[c] + f2 * C.c2[c] + f3 * C.c3[c];
          add(6, bt);
          if (EVAL && C.nonzero) {
            const double d1 = a1, d2 = a2, d3 = a3;
            eacc[6] += C.Kc1_d * (d1 * d1 * d2 * d2 + d2 * d2 * d3 * d3 + d3 * d3 * d1 * d1);
          }
        }
        // Zeeman
        add(7, a.bext);
        if (EVAL) eacc[7] += -C.Ms_d * dot3d(mm, a.bext);
        // magnetoelastic field
        if (a.has_mel) {
          bt[0] = -(C.cmel1 * ep[0] * mm[0] + C.cmel2 * (ep[3] * mm[1] + ep[4] * mm[2]));
          bt[1] = -(C.cmel1 * ep[1] * mm[1] + C.cmel2 * (ep[3] * mm[0] + ep[5] * mm[2]));
          bt[2] = -(C.cmel1 * ep[2] * mm[2] + C.cmel2 * (ep[4] * mm[0] + ep[5] * mm[1]));
          add(8, bt);
          if (EVAL && C.nonzero) {
            const double m0 = mm[0], m1 = mm[1], m2 = mm[2];
            eacc[8] += C.B1_d * ((double)ep[0] * m0 * m0 + (double)ep[1] * m1 * m1 +
                                 (double)ep[2] * m2 * m2) +
                       2.0 * C.B2_d * ((double)ep[3] * m0 * m1 + (double)ep[4] * m0 * m2 +
                                       (double)ep[5] * m1 * m2);
          }
        }
        // torque
        T mxB[3], mxmxB[3], tau[3];
        cross3(mm, B, mxB);
        cross3(mm, mxB, mxmxB);
#pragma unroll
        for (int c = 0; c < 3; ++c) tau[c] = -C.gl * (mxB[c] + C.alpha * mxmxB[c]);
        if (NSUB >= 2 && a0_on) {
          T w[3] = {0, 0, 0}, mxw[3];
#pragma unroll
          for (int o = 0; o < NSUB; ++o) {
            if (o == s) continue;
            T wo[3];
            cross3_acc(mm, cur[o], wo);
            w[0] += wo[0]; w[1] += wo[1]; w[2] += wo[2];
          }
          cross3(mm, w, mxw);
#pragma unroll
          for (int c = 0; c < 3; ++c) tau[c] -= C.gl * C.ccell * (w[c] + C.alpha * mxw[c]);
        }
        const bool zl = EVAL ? (a.add_zl && C.has_zl) : C.has_zl;
        if (zl) {
          T dm[3], mxdm[3], mxmxdm[3];
#pragma unroll
          for (int c = 0; c < 3; ++c)
            dm[c] = C.zu[0] * (xp[s][c] - xm[s][c]) * a.i2dx +
                    C.zu[1] * (yp[s][c] - ym[s][c]) * a.i2dy +
                    C.zu[2] * (zp[s][c] - zm[s][c]) * a.i2dz;
          cross3(mm, dm, mxdm);
          cross3(mm, mxdm, mxmxdm);
#pragma unroll
          for (int c = 0; c < 3; ++c) tau[c] -= C.zla * mxmxdm[c] + C.zlb * mxdm[c];
        }
        if (EVAL) {
          if (a.bout) {
            const gptr<T> bo = (gptr<T>)a.bout + s * N3;
#pragma unroll
            for (int c = 0; c < 3; ++c)
              sto<T>(bo + c * N, o, a.out_torque ? tau[c] : B[c] + Bout[c]);
          }
        } else {
          if (!(isfinite(tau[0]) && isfinite(tau[1]) && isfinite(tau[2])))
            atomicOr(&a.ctrl->nonfinite, 1);
#pragma unroll
          for (int c = 0; c < 3; ++c) sto<T>(kout + s * N3 + c * N, o, tau[c]);
          // the slopes of this sublattice, loaded above
          const T(*kv)[3] = NSUB == 1 ? kv1 : kvs;
          const T* yv = NSUB == 1 ? yv1 : yvs;
          if (has_next) {
            T v[3];
            if (!is_last) {
#pragma unroll
              for (int c = 0; c < 3; ++c) {
                T acc = yv[c];
#pragma unroll
                for (int j = 0; j < (NK < 5 ? NK : 5); ++j)
                  if (j < stage - 1) acc = fma(ca[j], kv[j][c], acc);
                v[c] = fma(ca[stage - 1], tau[c], acc);
              }
            } else {
#pragma unroll
              for (int c = 0; c < 3; ++c) v[c] = fma(ca[0], tau[c], mm[c]);
            }
            const T inv = inv_norm(v);
#pragma unroll
            for (int c = 0; c < 3; ++c) sto<T>(ynext + s * N3 + c * N, o, v[c] * inv);
          } else {
            // error weights: e_j of the earlier slopes, then e_ns of this
            // stage's own slope
            double ev[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
              double acc = 0.0;
#pragma unroll
              for (int j = 0; j < NK; ++j)
                if (j < ns - 1 && ew[j] != 0.0) acc += ew[j] * (double)kv[j][c];
              ev[c] = acc + ew[ns - 1] * (double)tau[c];
            }
            const double nrm = sqrt(ev[0] * ev[0] + ev[1] * ev[1] + ev[2] * ev[2]);
            emax = nrm > emax ? nrm : emax;
          }
        }
      }
#pragma unroll
      for (int s = 0; s < NSUB; ++s)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          zm[s][c] = cur[s][c];
          cur[s][c] = zp[s][c];
        }
    }
  }

  if (EVAL) {
    if (a.epart) {
      __shared__ double red[kNE][256];
      for (int t = 0; t < kNE; ++t) red[t][threadIdx.x] = eacc[t] * a.V;
      __syncthreads();
      for (int st = 128; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st)
          for (int t = 0; t < kNE; ++t) red[t][threadIdx.x] += red[t][threadIdx.x + st];
        __syncthreads();
      }
      if (threadIdx.x < kNE) a.epart[(long)w * kNE + threadIdx.x] = red[threadIdx.x][0];
    }
  } else if (stage == ns && !fuse2) {
    __shared__ double red[256];
    red[threadIdx.x] = emax;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
      if ((int)threadIdx.x < st) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + st]);
      __syncthreads();
    }
    if (threadIdx.x == 0) a.errpart[w] = red[0];
  }
}

template <typename T, int NSUB, bool EVAL, bool GDMI = false, bool GBX = false, int NK = 6>
__global__ __launch_bounds__(256) void k_field(const FieldArgs<T> a, const RKStage rk) {
  const int zero = warm_args<FieldArgs<T>>();
  field_block<T, NSUB, EVAL, GDMI, GBX, NK>(a, rk, zero, xcd_remap(blockIdx.x, a.nb_pad), a.stage, a.fuse2);
}

// The field and the elastic force of one stage in one launch: both read the
// stage input, strain and stress and write different things, and each alone
// is a few microseconds of latency on a grid that leaves the chip half
// empty.  The force's blocks come first (they take longer).
template <typename T, int NSUB, bool LIN, bool ONE>
__global__ __launch_bounds__(256) void k_field_force(const FieldArgs<T> a, const RKStage rk,
                                                     const ElasticArgs<T> e, int nforce) {
  const int b = (int)blockIdx.x;
  const int zero = warm_args<FieldArgs<T>>();
  if (b < nforce) force_block<T, LIN, ONE>(e, rk, b);
  else field_block<T, NSUB, false>(a, rk, zero, xcd_remap(b - nforce, a.nb_pad), a.stage, a.fuse2);
}

// Many grids in one launch: block b runs block work[b].y of grid work[b].x
// (the argument blocks live in device memory); a grid whose run is over
// skips its blocks.
template <typename T, int NSUB>
__global__ __launch_bounds__(256) void k_field_multi(const FieldArgs<T>* __restrict__ args,
                                                     const int2* __restrict__ work, int nwork,
                                                     int nb_pad, int stage, int fuse2,
                                                     const RKStage rk) {
  const int b = xcd_remap(blockIdx.x, nb_pad);
  if (b >= nwork) return;
  const int2 wk = work[b];
  const FieldArgs<T>& a = args[wk.x];
  const int zero = warm_lines((const uint32_t*)&a, (int)sizeof(FieldArgs<T>));
  field_block<T, NSUB, false>(a, rk, zero, wk.y, stage, fuse2);
}

template <typename T>
void launch_field_multi(const FieldArgs<T>* args, const int2* work, int nwork, int nsub, int stage,
                        int fuse2, hipStream_t st) {
  const int nb_pad = round_up(nwork, 8);
  // a batch steps the Dormand-Prince pair
  const RKStage rk = rk_stage(RK::t[RK_DP45], stage);
  if (nsub == 1)
    hipLaunchKernelGGL((k_field_multi<T, 1>), dim3(nb_pad), dim3(256), 0, st, args, work, nwork,
                       nb_pad, stage, fuse2, rk);
  else
    hipLaunchKernelGGL((k_field_multi<T, 2>), dim3(nb_pad), dim3(256), 0, st, args, work, nwork,
                       nb_pad, stage, fuse2, rk);
}

// The Eq. 6 ghosts (GDMI) exist for one and two sublattices only.
template <typename T, bool EVAL, bool GDMI, bool GBX>
void launch_field_nsub(const FieldArgs<T>& a, hipStream_t st) {
  const dim3 g(a.nb_pad), b(256);
  const RKStage rk = rk_stage(RK::t[a.rk], a.stage);
  auto go = [&](auto nk) {
    constexpr int NK = decltype(nk)::value;
    if (a.nsub == 2) {
      hipLaunchKernelGGL((k_field<T, 2, EVAL, GDMI, GBX, NK>), g, b, 0, st, a, rk);
    } else if constexpr (!GDMI) {
      hipLaunchKernelGGL((k_field<T, 3, EVAL, GDMI, GBX, NK>), g, b, 0, st, a, rk);
    }
  };
  if (a.nsub == 1) {
    hipLaunchKernelGGL((k_field<T, 1, EVAL, GDMI, GBX>), g, b, 0, st, a, rk);
  } else if constexpr (EVAL) {
    go(std::integral_constant<int, 6>{});
  } else {
    if (rk.ns == 3) go(std::integral_constant<int, 2>{});
    else if (rk.ns == 4) go(std::integral_constant<int, 3>{});
    else go(std::integral_constant<int, 6>{});
  }
}

template <typename T, bool EVAL>
void launch_field_var(const FieldArgs<T>& a, hipStream_t st) {
  if (a.gdmi) {
    if (a.gbx) launch_field_nsub<T, EVAL, true, true>(a, st);
    else launch_field_nsub<T, EVAL, true, false>(a, st);
  } else {
    if (a.gbx) launch_field_nsub<T, EVAL, false, true>(a, st);
    else launch_field_nsub<T, EVAL, false, false>(a, st);
  }
}

template <typename T>
void launch_field(const FieldArgs<T>& a, bool eval, hipStream_t st, Prof* prof) {
  ProfScope ps(prof, P_FIELD, st);
  if (eval) launch_field_var<T, true>(a, st);
  else launch_field_var<T, false>(a, st);
}

template <typename T>
void launch_field_force(const FieldArgs<T>& a, const ElasticArgs<T>& e, hipStream_t st,
                        Prof* prof) {
  if (a.gdmi || a.gbx || a.nsub > 2) {
    launch_field<T>(a, false, st, prof);
    launch_force<T>(e, st, prof);
    return;
  }
  ProfScope ps(prof, P_FIELD, st);
  const int nforce = elastic_blocks(e.N, e.nbx, e.nby, e.nz);
  const dim3 g(a.nb_pad + nforce), b(256);
  const RKStage rk = rk_stage(RK::t[a.rk], a.stage);
  elastic_variant(e, [&](auto lin, auto one) {
    constexpr bool LIN = lin.value, ONE = one.value;
    if (a.nsub == 1)
      hipLaunchKernelGGL((k_field_force<T, 1, LIN, ONE>), g, b, 0, st, a, rk, e, nforce);
    else
      hipLaunchKernelGGL((k_field_force<T, 2, LIN, ONE>), g, b, 0, st, a, rk, e, nforce);
  });
}

// --------------------------------------------------------- combine2 ----
// Stage-2 input for a new attempt: normalise(y_n + h a21 k1).
template <typename T>
__device__ __forceinline__ void combine2_cell(const Table<T>* tbl, const Ctrl* ctrl, double a10,
                                              long Ncell, long i) {
  const long s = i / Ncell, cell = i - s * Ncell;
  const long base = s * 3 * Ncell + cell;
  const T c = (T)(a10 * ctrl->h);
  const gcptr<T> yn = (gcptr<T>)tbl->yn;
  const gcptr<T> k1 = (gcptr<T>)tbl->k[0];
  T v[3];
  for (int q = 0; q < 3; ++q) v[q] = fma(c, k1[base + q * Ncell], yn[base + q * Ncell]);
  const T inv = inv_norm(v);
  const gptr<T> o = (gptr<T>)tbl->sa;
  for (int q = 0; q < 3; ++q) o[base + q * Ncell] = v[q] * inv;
}

template <typename T>
__global__ void k_combine2_cells(const Table<T>* tbl, const Ctrl* ctrl, double a10, long Ncell,
                                 int nsub) {
  if (ctrl_stopped(ctrl)) return;
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= Ncell * nsub) return;
  combine2_cell<T>(tbl, ctrl, a10, Ncell, i);
}

template <typename T>
void launch_combine2(const Table<T>* tbl, const Ctrl* ctrl, int rk, long Ncell, int nsub,
                     hipStream_t st, Prof* prof) {
  ProfScope ps(prof, P_COMBINE, st);
  const long n = Ncell * nsub;
  hipLaunchKernelGGL((k_combine2_cells<T>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                     tbl, ctrl, RK::t[rk].a[1][0], Ncell, nsub);
}

// ---------------------------------------------------------- control ----
template <typename T>
__device__ __forceinline__ void control_block(Ctrl* c, Table<T>* tbl, const double* errpart,
                                              int nerr, int elastic) {
  if (c->done || c->status) return;
  __shared__ double red[256];
  double e = 0.0;
  if (!c->fixed)
    for (int i = threadIdx.x; i < nerr; i += blockDim.x) e = fmax(e, errpart[i]);
  red[threadIdx.x] = e;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  if (c->nonfinite) {
    c->status = MMP_E_NONFINITE;
    c->done = 1;
    return;
  }
  const double h = c->h;
  const double err = c->fixed ? 0.0 : h * red[0];
  c->err = err;
  const bool acc = c->fixed || err <= c->tol;
  c->accepted = acc ? 1 : 0;
  if (acc) {
    T* t;
    t = tbl->yn; tbl->yn = tbl->ynew; tbl->ynew = t;
    // the last stage's slope (at y_{n+1}) is the next step's k_1
    const int l = tbl->ns - 1;
    t = tbl->k[0]; tbl->k[0] = tbl->k[l]; tbl->k[l] = t;
    if (elastic) {
      t = tbl->un; tbl->un = tbl->unew; tbl->unew = t;
      t = tbl->vn; tbl->vn = tbl->vnew; tbl->vnew = t;
      t = tbl->ku[0]; tbl->ku[0] = tbl->ku[l]; tbl->ku[l] = t;
      t = tbl->kv[0]; tbl->kv[0] = tbl->kv[l]; tbl->kv[l] = t;
    }
    c->steps += 1;
    if (c->fixed) {
      c->sample_k += 1;  // counts steps of this segment
      c->t = c->t0 + (double)c->sample_k * h;
      if (c->max_attempts > 0 && c->sample_k >= c->max_attempts) c->done = 1;
    } else {
      c->t = c->land ? fmin(c->t_next, c->t_end) : c->t + h;
      if (c->land && c->sample_every > 0.0 && c->t == c->t_next) {
        c->sample_pending = 1;
        c->sample_k += 1;
        c->t_next = c->t0 + (double)c->sample_k * c->sample_every;
        // an output time a few ulp short of t_end is t_end itself
        if (c->t_next >= c->t_end - 1e-9 * (c->t_end - c->t0)) c->t_next = c->t_end;
      }
      if (c->t >= c->t_end) c->done = 1;
    }
  } else {
    c->rejects += 1;
  }
  if (!c->fixed) {
    double fac = c->fac_max;
    if (err > 0.0) fac = c->safety * pow(c->tol / err, 1.0 / (RK::t[tbl->rk].q + 1));
    fac = fmin(c->fac_max, fmax(c->fac_min, fac));
    c->dt = h * fac;
    if (c->dt_max > 0.0) c->dt = fmin(c->dt, c->dt_max);
    if (c->dt < c->dt_min) {
      c->status = MMP_E_DT_UNDERFLOW;
      c->done = 1;
    }
    if (c->max_attempts > 0 && c->steps + c->rejects >= c->max_attempts) c->done = 1;
    const double target = fmin(c->t_next, c->t_end);
    const double rem = target - c->t;
    c->land = c->dt >= rem ? 1 : 0;
    c->h = c->land ? rem : c->dt;
  }
}

template <typename T>
__global__ void k_control(Ctrl* c, Table<T>* tbl, const double* errpart, int nerr, int elastic) {
  control_block<T>(c, tbl, errpart, nerr, elastic);
}

// one block per grid of a batch
template <typename T>
__global__ void k_control_multi(const StepWork<T>* __restrict__ w) {
  const StepWork<T> g = w[blockIdx.x];
  control_block<T>(g.ctrl, g.tbl, g.errpart, g.nerr, 0);
}

template <typename T>
__global__ void k_combine2_multi(const StepWork<T>* __restrict__ w) {
  const StepWork<T> g = w[blockIdx.y];
  if (ctrl_stopped(g.ctrl)) return;
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= g.N * g.nsub) return;
  combine2_cell<T>(g.tbl, g.ctrl, RK::t[RK_DP45].a[1][0], g.N, i);
}

template <typename T>
void launch_step_multi(const StepWork<T>* w, int ngrids, long max_cells, hipStream_t st) {
  hipLaunchKernelGGL((k_control_multi<T>), dim3(ngrids), dim3(256), 0, st, w);
  hipLaunchKernelGGL((k_combine2_multi<T>), dim3((unsigned)((max_cells + 255) / 256), ngrids),
                     dim3(256), 0, st, w);
}

template <typename T>
void launch_control(Ctrl* ctrl, Table<T>* tbl, const double* errpart, int nerr, int elastic,
                    hipStream_t st, Prof* prof) {
  ProfScope ps(prof, P_CONTROL, st);
  hipLaunchKernelGGL((k_control<T>), dim3(1), dim3(256), 0, st, ctrl, tbl, errpart, nerr, elastic);
}

// ----------------------------------------------------------- sampling --
template <typename T>
__global__ void k_sample_part(const Ctrl* c, const Table<T>* tbl, int nsub, long N, double* part) {
  if (!c->sample_pending) return;
  __shared__ double red[9][256];
  double acc[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  const T* y = tbl->yn;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (long)gridDim.x * blockDim.x)
    for (int s = 0; s < nsub; ++s)
      for (int q = 0; q < 3; ++q) acc[s * 3 + q] += (double)y[(s * 3 + q) * N + i];
  for (int q = 0; q < 9; ++q) red[q][threadIdx.x] = acc[q];
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st)
      for (int q = 0; q < 9; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x < 9) part[blockIdx.x * 9 + threadIdx.x] = red[threadIdx.x][0];
}

// sum of up to any number of partial sums by one 256-thread block, to thread 0
__device__ __forceinline__ double block_sum(const double* part, int n, int stride, double* red) {
  double acc = 0.0;
  for (int b = threadIdx.x; b < n; b += 256) acc += part[(long)b * stride];
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

// One block: the averages of one output time.  (One thread walking the
// partial sums took 84 us for 240 of them, a block under 4.)
__global__ __launch_bounds__(256) void k_sample_final(Ctrl* c, const double* part, int nblk,
                                                      long N, int nsub, double* sample_t,
                                                      double* sample_m, int cap) {
  if (!c->sample_pending) return;
  __shared__ double red[4];
  const int k = c->nsamples;
  for (int q = 0; q < 3 * nsub; ++q) {
    const double acc = block_sum(part + q, nblk, 9, red);
    if (threadIdx.x == 0 && k < cap) sample_m[k * 3 * nsub + q] = acc / (double)N;
  }
  __syncthreads();   // every thread has read the controller
  if (threadIdx.x != 0) return;
  if (k < cap) sample_t[k] = c->t;
  c->nsamples = k + 1;
  c->sample_pending = 0;
}

template <typename T>
void launch_sample(Ctrl* ctrl, const Table<T>* tbl, int nsub, long N, double* part, int nblk,
                   double* sample_t, double* sample_m, int cap, hipStream_t st, Prof* prof) {
  ProfScope ps(prof, P_REDUCE, st);
  hipLaunchKernelGGL((k_sample_part<T>), dim3(nblk), dim3(256), 0, st, ctrl, tbl, nsub, N, part);
  hipLaunchKernelGGL(k_sample_final, dim3(1), dim3(256), 0, st, ctrl, part, nblk, N, nsub, sample_t,
                     sample_m, cap);
}

// one block per energy term
__global__ __launch_bounds__(256) void k_energy_final(const double* epart, int nblk, double* out) {
  __shared__ double red[4];
  const double acc = block_sum(epart + blockIdx.x, nblk, kNE, red);
  if (threadIdx.x == 0) out[blockIdx.x] = acc;
}

void launch_energy_final(const double* epart, int nblk, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_energy_final, dim3(kNE), dim3(256), 0, st, epart, nblk, out);
}

#define INST(T)                                                                              \
  template void launch_field<T>(const FieldArgs<T>&, bool, hipStream_t, Prof*);             \
  template void launch_field_force<T>(const FieldArgs<T>&, const ElasticArgs<T>&,           \
                                      hipStream_t, Prof*);                                  \
  template void launch_combine2<T>(const Table<T>*, const Ctrl*, int, long, int,            \
                                   hipStream_t, Prof*);                                                   \
  template void launch_control<T>(Ctrl*, Table<T>*, const double*, int, int, hipStream_t,   \
                                  Prof*);                                                    \
  template void launch_sample<T>(Ctrl*, const Table<T>*, int, long, double*, int, double*,  \
                                 double*, int, hipStream_t, Prof*);                          \
  template void launch_field_multi<T>(const FieldArgs<T>*, const int2*, int, int, int, int,   \
                                      hipStream_t);                                          \
  template void launch_step_multi<T>(const StepWork<T>*, int, long, hipStream_t);
INST(float)
INST(double)

}  // namespace mmp
