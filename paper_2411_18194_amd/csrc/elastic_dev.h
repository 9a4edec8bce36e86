// Device side of the elastic stages shared by the elastic kernels and the
// field kernel that carries the force (paper, Methods "Elasticity" and
// "Magnetoelasticity").
//
// Derivatives: 4th-order central (-f2 + 8 f1 - 8 f-1 + f-2)/(12 d) in the
// bulk, 2nd-order central one cell in from a face, 1st-order one-sided on a
// face cell (the paper uses lower-order schemes near and at boundaries); an
// axis with one cell has no derivative.
#pragma once

#include "elastic.h"

namespace mmp {

// The scheme of one cell along one axis: df = w1 (f[p1] - f[m1]) + w2 (f[p2] -
// f[m2]) at offsets clamped to the axis, so that the same two differences
// serve every position: (8, -1)/12d in the bulk, (1, 0)/2d one cell in, and
// on a face, where the clamped neighbour is the cell itself, (1, 0)/d.  The
// weights are formed once per cell and axis; a division per derivative and
// scheme (108 divisions per cell of the force) was most of that kernel.
// A zero weight would not leave out a value that is not finite: where the
// second difference does not count, its two points are both the first's p1,
// and where an axis may have one cell (ONE) its result is masked.  Eight steps
// of 2048x64x1 FP32: 695 us with selects of the sums, 617 this way.
template <typename T, bool ONE>
struct Diff {
  int m2, m1, p1, p2;
  int mask;   // ONE: 0 on an axis with one cell, else all bits
  T w1, w2;
};
template <typename T, bool ONE>
__device__ __forceinline__ Diff<T, ONE> diff_at(int i, int n, int stride, T h) {
  Diff<T, ONE> d;
  const bool face = i == 0 || i == n - 1, in1 = i == 1 || i == n - 2, near = face || in1;
  d.m1 = (max(i - 1, 0) - i) * stride;
  d.p1 = (min(i + 1, n - 1) - i) * stride;
  d.m2 = near ? d.p1 : -2 * stride;
  d.p2 = near ? d.p1 : 2 * stride;
  if constexpr (ONE) {
    // (hidden: a select on it would take the loads into a branch)
    d.mask = uni(n > 1 ? -1 : 0);
    asm volatile("" : "+s"(d.mask));
  }
  const T r = T(1) / h;
  d.w1 = face ? r : (in1 ? T(0.5) * r : T(2.0 / 3.0) * r);
  d.w2 = -r * T(1.0 / 12.0);
  return d;
}
template <typename T, bool ONE>
__device__ __forceinline__ T deriv(gcptr<T> f, const Diff<T, ONE>& d) {
  const T r = d.w1 * (f[d.p1] - f[d.m1]) + d.w2 * (f[d.p2] - f[d.m2]);
  if constexpr (!ONE)
    return r;
  else if constexpr (sizeof(T) == 4)
    return __int_as_float(__float_as_int(r) & d.mask);
  else
    return __hiloint2double(__double2hiint(r) & d.mask, __double2loint(r) & d.mask);
}

// input of stage s (0 or 1: the accepted state) among four buffers of u or v
template <typename T>
__device__ __forceinline__ gcptr<T> stage_pick(T* n, T* nw, T* a, T* b, int s, int ns) {
  return uni_ptr((gcptr<T>)(s <= 1 ? n : s == ns ? nw : (s & 1) ? b : a));
}
template <typename T>
__device__ __forceinline__ gcptr<T> u_in(const Table<T>* t, int s, int ns) {
  return stage_pick<T>(t->un, t->unew, t->usa, t->usb, s, ns);
}
template <typename T>
__device__ __forceinline__ gcptr<T> v_in(const Table<T>* t, int s, int ns) {
  return stage_pick<T>(t->vn, t->vnew, t->vsa, t->vsb, s, ns);
}

// cell of this thread in block w: 64x4 tile w of the plane-major tiles, or
// (LIN, see elastic_linear) the w-th 256 cells
template <typename T, bool LIN>
__device__ __forceinline__ bool tile_cell(const ElasticArgs<T>& a, int w, int* x, int* y, int* z) {
  if constexpr (LIN) {
    const int i = w * 256 + (int)threadIdx.x, r = i / a.nx;
    *x = i - r * a.nx;
    *y = r % a.ny;
    *z = r / a.ny;
    return i < a.N;
  } else {
    const int tx = w % a.nbx, r = w / a.nbx;
    *x = tx * 64 + (int)(threadIdx.x & 63);
    *y = (r % a.nby) * 4 + (int)(threadIdx.x >> 6);
    *z = r / a.nby;
    return *x < a.nx && *y < a.ny;
  }
}

// y_n + sum_{j<NJ} c_j k_j at one cell, every load issued before the first sum
template <typename T, int NJ>
__device__ __forceinline__ void stage_sum(const gcptr<T> yn, const gcptr<T>* k, const T* c, long i,
                                          long N, T* acc) {
  T kv[NJ > 0 ? NJ : 1][3];
#pragma unroll
  for (int q = 0; q < 3; ++q) acc[q] = yn[i + q * N];
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int q = 0; q < 3; ++q) kv[j][q] = k[j][i + q * N];
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int q = 0; q < 3; ++q) acc[q] += c[j] * kv[j][q];
}
template <typename T>
__device__ __forceinline__ void stage_sum_n(int nj, const gcptr<T> yn, const gcptr<T>* k,
                                            const T* c, long i, long N, T* acc) {
  switch (nj) {
    case 0: stage_sum<T, 0>(yn, k, c, i, N, acc); break;
    case 1: stage_sum<T, 1>(yn, k, c, i, N, acc); break;
    case 2: stage_sum<T, 2>(yn, k, c, i, N, acc); break;
    case 3: stage_sum<T, 3>(yn, k, c, i, N, acc); break;
    case 4: stage_sum<T, 4>(yn, k, c, i, N, acc); break;
    default: stage_sum<T, 5>(yn, k, c, i, N, acc); break;
  }
}

// Tile w of the force: divergence of the stress, magnetoelastic force of Eq.
// 8 per sublattice, k_u and k_v, and the next stage's u and v.
template <typename T, bool LIN, bool ONE>
__device__ __forceinline__ void force_block(const ElasticArgs<T>& a, const RKStage& rk, int w) {
  const int stage = a.stage, ns = rk.ns, nj = stage - 1;
  // pointers and step size first, in one trip with the controller's flags
  const gcptr<T> m0 = (gcptr<T>)table_slot<T>(a.tbl, rk.in), u0 = u_in<T>(a.tbl, stage, ns),
                 v0 = v_in<T>(a.tbl, stage, ns);
  const gptr<T> KU0 = uni_ptr((gptr<T>)a.tbl->ku[nj]), KV0 = uni_ptr((gptr<T>)a.tbl->kv[nj]);
  const gcptr<T> un = uni_ptr((gcptr<T>)a.tbl->un), vn = uni_ptr((gcptr<T>)a.tbl->vn);
  gcptr<T> pu[5], pv[5];
#pragma unroll
  for (int j = 0; j < 5; ++j) {
    pu[j] = pv[j] = nullptr;
    if (j < nj) {
      pu[j] = uni_ptr((gcptr<T>)a.tbl->ku[j]);
      pv[j] = uni_ptr((gcptr<T>)a.tbl->kv[j]);
    }
  }
  // the next stage's input (the last stage of a fixed step: stage 2's)
  const bool nxt = stage < ns && stage + 1 == ns;
  const bool tosa = stage >= ns || (stage & 1) != 0;
  const gptr<T> uo0 = uni_ptr((gptr<T>)(nxt ? a.tbl->unew : tosa ? a.tbl->usa : a.tbl->usb));
  const gptr<T> vo0 = uni_ptr((gptr<T>)(nxt ? a.tbl->vnew : tosa ? a.tbl->vsa : a.tbl->vsb));
  const double h = a.ctrl->h;
  if (ctrl_stopped(a.ctrl)) return;
  int x, y, z;
  if (!tile_cell<T, LIN>(a, w, &x, &y, &z)) return;
  const long N = a.N;
  const long i = ((long)z * a.ny + y) * a.nx + x;
  const auto dx = diff_at<T, ONE>(x, a.nx, 1, a.dx), dy = diff_at<T, ONE>(y, a.ny, a.nx, a.dy);
  const auto dz = diff_at<T, false>(z, a.nz, a.nx * a.ny, a.dz);
  const bool flat = a.nz == 1;   // no derivative along z
  const gcptr<T> sg = (gcptr<T>)a.sig + i;
  T f[3];
  f[0] = deriv(sg, dx) + deriv(sg + 3 * N, dy);
  f[1] = deriv(sg + 3 * N, dx) + deriv(sg + N, dy);
  f[2] = deriv(sg + 4 * N, dx) + deriv(sg + 5 * N, dy);
  if (!flat) {
    f[0] += deriv(sg + 4 * N, dz);
    f[1] += deriv(sg + 5 * N, dz);
    f[2] += deriv(sg + 2 * N, dz);
  }
  const gcptr<T> m = m0 + i;
  for (int s = 0; s < a.nsub; ++s) {
    if (!a.mel[s]) continue;
    const gcptr<T> ms = m + (long)s * 3 * N;
    T mv[3], g[3][3];  // g[j][c] = d_j m_c
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      mv[c] = ms[c * N];
      g[0][c] = deriv(ms + c * N, dx);
      g[1][c] = deriv(ms + c * N, dy);
      g[2][c] = T(0);
    }
    if (!flat) {
#pragma unroll
      for (int c = 0; c < 3; ++c) g[2][c] = deriv(ms + c * N, dz);
    }
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      T acc = T(2) * a.B1[s] * mv[r] * g[r][r];
#pragma unroll
      for (int j = 0; j < 3; ++j)
        if (j != r) acc += a.B2[s] * (mv[r] * g[j][j] + mv[j] * g[j][r]);
      f[r] += acc;
    }
  }
  const gcptr<T> v = v0 + i;
  T ku[3], kv[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    ku[c] = v[c * N];
    kv[c] = (f[c] - a.eta * ku[c]) * a.inv_rho;
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    KU0[i + c * N] = ku[c];
    KV0[i + c * N] = kv[c];
  }
  if (stage < ns) {
    T c[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) c[j] = (T)(rk.a[j] * h);
    T au[3], av[3];
    stage_sum_n<T>(nj, un, pu, c, i, N, au);
    stage_sum_n<T>(nj, vn, pv, c, i, N, av);
    T cs = T(0);   // weight of this stage's own slope
#pragma unroll
    for (int j = 0; j < 6; ++j) cs = j == nj ? (T)(rk.a[j] * h) : cs;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      uo0[i + q * N] = au[q] + cs * ku[q];
      vo0[i + q * N] = av[q] + cs * kv[q];
    }
  } else if (a.fuse2) {
    const T c21 = (T)(rk.a10 * h);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      uo0[i + c * N] = u0[i + c * N] + c21 * ku[c];
      vo0[i + c * N] = ku[c] + c21 * kv[c];
    }
  }
}

}  // namespace mmp
