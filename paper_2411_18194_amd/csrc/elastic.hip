// Elastodynamics on the magnet's grid (paper, Methods "Elasticity" and
// "Magnetoelasticity"): rho d2u/dt2 = div sigma + sum_s f_mel^(s) - eta v,
// integrated as (u, v) inside the same Runge-Kutta stages as m.
//
// Strain is the symmetrised gradient of u (schemes in elastic_dev.h), stress
// the cubic law plus the viscous stress beta C : eps(v) of
// stiffness-proportional Rayleigh damping; on each face of an axis with more
// than one cell the face cell's stress row along that axis is the traction
// (zero, i.e. traction-free), and the drive sigma_xz = A sin(w t) on x = 0
// is applied last.  The force is the divergence of that stress plus the
// magnetoelastic force of Eq. 8 per sublattice.
//
// A stage is two launches: strain and stress of a cell, both point-wise in
// the gradient, then the force (which needs its neighbours' stress) beside
// the magnetic field of the same stage, in one launch where the plain field
// kernel applies (field.hip).  At the sizes these grids have (a racetrack of
// 2048x64x1) every launch is latency: 40 us per stage in four launches
// before, 22 now.
#include "elastic_dev.h"

namespace mmp {

// Voigt slot of (row, col)
__device__ __forceinline__ int voigt(int r, int c) {
  if (r == c) return r;
  const int s = r + c;  // 1: xy, 2: xz, 3: yz
  return s == 1 ? 3 : (s == 2 ? 4 : 5);
}

// symmetrised gradient of the vector field f at the cell
template <typename T, bool ONE>
__device__ __forceinline__ void sym_grad(gcptr<T> f, long N, const Diff<T, ONE>& dx,
                                         const Diff<T, ONE>& dy, const Diff<T, false>& dz,
                                         bool flat, T* e) {
  T g[3][3];  // g[i][j] = d_i f_j
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    g[0][j] = deriv(f + j * N, dx);
    g[1][j] = deriv(f + j * N, dy);
    g[2][j] = T(0);
  }
  if (!flat) {
#pragma unroll
    for (int j = 0; j < 3; ++j) g[2][j] = deriv(f + j * N, dz);
  }
  e[0] = g[0][0];
  e[1] = g[1][1];
  e[2] = g[2][2];
  e[3] = T(0.5) * (g[0][1] + g[1][0]);
  e[4] = T(0.5) * (g[0][2] + g[2][0]);
  e[5] = T(0.5) * (g[1][2] + g[2][1]);
}

// cubic law
template <typename T>
__device__ __forceinline__ void cubic_stress(const ElasticArgs<T>& a, const T* e, T* s) {
  s[0] = a.C11 * e[0] + a.C12 * (e[1] + e[2]);
  s[1] = a.C11 * e[1] + a.C12 * (e[0] + e[2]);
  s[2] = a.C11 * e[2] + a.C12 * (e[0] + e[1]);
  s[3] = T(2) * a.C44 * e[3];
  s[4] = T(2) * a.C44 * e[4];
  s[5] = T(2) * a.C44 * e[5];
}

template <typename T, bool LIN, bool ONE>
__global__ __launch_bounds__(256) void k_strain(ElasticArgs<T> a, int ns, double cs, int eval) {
  const gcptr<T> u0 = u_in<T>(a.tbl, a.stage, ns), v0 = v_in<T>(a.tbl, a.stage, ns);
  if (ctrl_stopped(a.ctrl)) return;
  int x, y, z;
  const bool in = tile_cell<T, LIN>(a, (int)blockIdx.x, &x, &y, &z);
  double e_el = 0.0;
  if (in) {
    const long N = a.N;
    const long i = ((long)z * a.ny + y) * a.nx + x;
    const auto dx = diff_at<T, ONE>(x, a.nx, 1, a.dx), dy = diff_at<T, ONE>(y, a.ny, a.nx, a.dy);
    const auto dz = diff_at<T, false>(z, a.nz, a.nx * a.ny, a.dz);
    const bool flat = a.nz == 1;
    T e[6], s[6];
    sym_grad(u0 + i, N, dx, dy, dz, flat, e);
    cubic_stress<T>(a, e, s);
#pragma unroll
    for (int c = 0; c < 6; ++c) a.eps[c * N + i] = e[c];
    const gcptr<T> v = v0 + i;
    if (eval) {
      double w = 0.0;
      for (int c = 0; c < 3; ++c) w += (double)s[c] * e[c];
      for (int c = 3; c < 6; ++c) w += 2.0 * (double)s[c] * e[c];
      double kv = 0.0;
      for (int c = 0; c < 3; ++c) kv += (double)v[c * N] * v[c * N];
      e_el = (0.5 * w + 0.5 * a.rho * kv) * a.V;
    }
    if (a.beta != T(0)) {
      // viscous stress beta C : eps(v) (stiffness-proportional Rayleigh damping)
      T r[6], sr[6];
      sym_grad(v, N, dx, dy, dz, flat, r);
      cubic_stress<T>(a, r, sr);
#pragma unroll
      for (int c = 0; c < 6; ++c) s[c] += a.beta * sr[c];
    }
    const int pos[3] = {x, y, z};
    const int n[3] = {a.nx, a.ny, a.nz};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const bool face = n[k] > 1 && (pos[k] == 0 || pos[k] == n[k] - 1);
#pragma unroll
      for (int j = 0; j < 3; ++j) s[voigt(k, j)] = face ? T(0) : s[voigt(k, j)];
    }
    if (a.trac_amp != 0.0 && a.nx >= 2 && x == 0) {
      const double ts = a.ctrl ? a.ctrl->t + cs * a.ctrl->h : 0.0;
      s[4] = (T)(a.trac_amp * sin(a.trac_omega * ts));
    }
#pragma unroll
    for (int c = 0; c < 6; ++c) a.sig[c * N + i] = s[c];
  }
  if (eval && a.epart) {
    __shared__ double red[256];
    red[threadIdx.x] = e_el;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
      if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
      __syncthreads();
    }
    if (threadIdx.x == 0) a.epart[blockIdx.x] = red[0];
  }
}

template <typename T, bool LIN, bool ONE>
__global__ __launch_bounds__(256) void k_force(ElasticArgs<T> a, const RKStage rk) {
  force_block<T, LIN, ONE>(a, rk, (int)blockIdx.x);
}

template <typename T>
__global__ void k_elastic_combine2(const Table<T>* tbl, const Ctrl* ctrl, long n3) {
  if (ctrl_stopped(ctrl)) return;
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n3) return;
  const T c = (T)(RK::t[tbl->rk].a[1][0] * ctrl->h);
  tbl->usa[i] = tbl->un[i] + c * tbl->ku[0][i];
  tbl->vsa[i] = tbl->vn[i] + c * tbl->kv[0][i];
}

template <typename T>
static dim3 elastic_grid(const ElasticArgs<T>& a) {
  return dim3((unsigned)elastic_blocks(a.N, a.nbx, a.nby, a.nz));
}

template <typename T>
void launch_strain(const ElasticArgs<T>& a, bool eval, hipStream_t st, Prof* prof) {
  ProfScope ps(prof, P_ELASTIC, st);
  const RKTab& t = RK::t[a.rk];
  elastic_variant(a, [&](auto lin, auto one) {
    hipLaunchKernelGGL((k_strain<T, lin.value, one.value>), elastic_grid(a), dim3(256), 0, st, a,
                       t.ns, a.stage > 0 ? t.c[a.stage - 1] : 0.0, eval ? 1 : 0);
  });
}

template <typename T>
void launch_force(const ElasticArgs<T>& a, hipStream_t st, Prof* prof) {
  ProfScope ps(prof, P_ELASTIC, st);
  const RKStage rk = rk_stage(RK::t[a.rk], a.stage);
  elastic_variant(a, [&](auto lin, auto one) {
    hipLaunchKernelGGL((k_force<T, lin.value, one.value>), elastic_grid(a), dim3(256), 0, st, a,
                       rk);
  });
}

template <typename T>
void launch_elastic_combine2(const Table<T>* tbl, const Ctrl* ctrl, long N, hipStream_t st,
                             Prof* prof) {
  ProfScope ps(prof, P_COMBINE, st);
  hipLaunchKernelGGL(k_elastic_combine2<T>, dim3((unsigned)((3 * N + 255) / 256)), dim3(256), 0,
                     st, tbl, ctrl, 3 * N);
}

#define INST(T)                                                                        \
  template void launch_strain<T>(const ElasticArgs<T>&, bool, hipStream_t, Prof*);    \
  template void launch_force<T>(const ElasticArgs<T>&, hipStream_t, Prof*);           \
  template void launch_elastic_combine2<T>(const Table<T>*, const Ctrl*, long, hipStream_t, Prof*);
INST(float)
INST(double)

}  // namespace mmp
