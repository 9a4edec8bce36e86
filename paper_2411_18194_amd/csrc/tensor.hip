// FP64 demagnetising tensor of cuboid cells and its octant spectrum.
//
// The paper (Methods, "Magnetostatic field") uses the analytic cell-cell
// result of Newell, Williams and Dunlop below a cutoff radius and an
// asymptotic result beyond it.  With r = |R| / max(d):
//   r < 3        Newell: 27-point second difference of f (diagonal) / g
//                (off-diagonal), FP64;
//   3 <= r < 40  the same cell-pair average by Gauss-Legendre quadrature of
//                the point-dipole kernel over the triangle-distributed
//                offset (each half-axis an n-point rule, n = 8 for
//                near-cubic cells, 12 otherwise), where Newell's formula
//                loses digits to cancellation;
//   r >= 40      4th-moment asymptotic expansion (second and fourth moments
//                d^2/6, d^4/15 of the triangle density), with the
//                derivatives of 1/R from the Cartesian recurrence
//                n R^2 a_k = (2n-1) sum_i x_i a_{k-e_i} - (n-1) sum_i a_{k-2e_i},
//                a_k = (-1)^|k|/k! d^k (1/R).
// Along a periodic axis (x or y) the kernel is cyclic with the grid's period
// and holds, at each cyclic offset, the sum over the images k = -R..R (the
// mean of +n/2 and -n/2 at the half period); the transform then runs over
// the cyclic offsets only.
// Each component has a definite parity per axis, so its DFT on the padded
// grid is a product of cosine/sine sums: along x and y dense FP64 matrix
// products with the matrices of cosines or sines (exact integer phase
// indexes into FP64 trig tables), along z a short sum per column; then
// scaled by -mu0/(Px Py Pz) (and -1 for the odd-odd components, from
// (-i)^2).
#include <algorithm>

#include "demag.h"

namespace mmp {

constexpr double kRNear = 3.0;
constexpr double kRFar = 40.0;

// ------------------------------------------------------------- Newell --
__device__ double newell_f(double x, double y, double z) {
  x = fabs(x); y = fabs(y); z = fabs(z);
  const double x2 = x * x, y2 = y * y, z2 = z * z;
  const double R = sqrt(x2 + y2 + z2);
  double out = (2.0 * x2 - y2 - z2) * R / 6.0;
  double p = 0.5 * y * (z2 - x2);
  if (p != 0.0) out += p * asinh(y / sqrt(x2 + z2));
  p = 0.5 * z * (y2 - x2);
  if (p != 0.0) out += p * asinh(z / sqrt(x2 + y2));
  p = x * y * z;
  if (p != 0.0) out -= p * atan(y * z / (x * R));
  return out;
}

__device__ double newell_g(double x, double y, double z) {
  const double sgn = (x > 0 ? 1.0 : (x < 0 ? -1.0 : 0.0)) * (y > 0 ? 1.0 : (y < 0 ? -1.0 : 0.0));
  if (sgn == 0.0) return 0.0;
  x = fabs(x); y = fabs(y); z = fabs(z);
  const double x2 = x * x, y2 = y * y, z2 = z * z;
  const double R = sqrt(x2 + y2 + z2);
  double out = -x * y * R / 3.0;
  double p = x * y * z;
  if (p != 0.0) out += p * asinh(z / sqrt(x2 + y2));
  p = y * (3.0 * z2 - y2) / 6.0;
  if (p != 0.0) out += p * asinh(x / sqrt(y2 + z2));
  p = x * (3.0 * z2 - x2) / 6.0;
  if (p != 0.0) out += p * asinh(y / sqrt(x2 + z2));
  p = z2 * z / 6.0;
  if (p != 0.0) out -= p * atan(x * y / (z * R));
  p = 0.5 * z * y2;
  if (p != 0.0) out -= p * atan(x * z / (y * R));
  p = 0.5 * z * x2;
  if (p != 0.0) out -= p * atan(y * z / (x * R));
  return sgn * out;
}

// term t (0..26) of the second difference: weight times f or g at the cell
// pair's corner (a, b, c) = (t / 9, t / 3 % 3, t % 3) - 1
template <bool OFFDIAG>
__device__ double second_difference_term(int t, double X, double Y, double Z, double dx, double dy,
                                         double dz) {
  const int a = t / 9 - 1, b = t / 3 % 3 - 1, c = t % 3 - 1;
  const double w = (a == 0 ? 2.0 : -1.0) * (b == 0 ? 2.0 : -1.0) * (c == 0 ? 2.0 : -1.0);
  return w * (OFFDIAG ? newell_g(X + a * dx, Y + b * dy, Z + c * dz)
                      : newell_f(X + a * dx, Y + b * dy, Z + c * dz));
}

template <bool OFFDIAG>
__device__ double second_difference(double X, double Y, double Z, double dx, double dy, double dz) {
  double acc = 0.0;
  for (int t = 0; t < 27; ++t) acc += second_difference_term<OFFDIAG>(t, X, Y, Z, dx, dy, dz);
  return acc / (4.0 * kPi * dx * dy * dz);
}

// Offsets 0 <= X < nx, 0 <= Y < ny along x and y; vertical offset z0 + Z zs,
// Z < nz: the grid's own (0, dz), or a layer above it seen from layer Z (its
// height above layer 0, -dz).
struct TensorArgs {
  int nx, ny, nz;
  double dx, dy, dz, dmax;
  double z0, zs;
  double* n6;          // [6][nz][ny][nx]
  int bx, by, bz;      // box of offsets the launches cover
  long i0;             // first offset of this launch (near, middle regime)
  int nq;              // quadrature points per axis (2n)
  double qt[24], qw[24];
  int rx, ry;          // image repetitions along x and y (0: open axis)
};

// offset of this block in the box
__device__ __forceinline__ void box_offset(const TensorArgs& a, int* X, int* Y, int* Z) {
  const long i = a.i0 + blockIdx.x;
  const int r = (int)(i / a.bx);
  *X = (int)(i - (long)r * a.bx);
  *Y = r % a.by;
  *Z = r / a.by;
}

// Newell's formula: one block per offset of the box.  Each of the 6 x 27
// terms has its own thread (an evaluation takes microseconds of dependent
// FP64 logarithms and arctangents, so an offset per thread ran 162 of them
// back to back: 302 us for any grid, 10 now), summed in order by six threads.
constexpr int kNearThreads = 192;
__global__ __launch_bounds__(kNearThreads) void k_tensor_near(TensorArgs a) {
  int X, Y, Z;
  box_offset(a, &X, &Y, &Z);
  const double x = X * a.dx, y = Y * a.dy, z = a.z0 + Z * a.zs;
  const double r = sqrt(x * x + y * y + z * z) / a.dmax;
  if (r >= kRNear) return;
  __shared__ double term[6 * 27];
  const int t = threadIdx.x;
  if (t < 6 * 27) {
    const int c = t / 27, k = t % 27;
    // axes of the component: the formula is written for xx and xy
    const double p[3] = {x, y, z}, d[3] = {a.dx, a.dy, a.dz};
    const int i0 = c == 0 || c == 3 || c == 4 ? 0 : (c == 2 ? 2 : 1);
    const int i1 = c == 0 || c == 2 || c == 3 ? 1 : (c == 1 ? 0 : 2);
    const int i2 = 3 - i0 - i1;
    auto pick = [](const double* v, int j) { return j == 0 ? v[0] : (j == 1 ? v[1] : v[2]); };
    const double px = pick(p, i0), py = pick(p, i1), pz = pick(p, i2);
    const double ex = pick(d, i0), ey = pick(d, i1), ez = pick(d, i2);
    term[t] = c < 3 ? second_difference_term<false>(k, px, py, pz, ex, ey, ez)
                    : second_difference_term<true>(k, px, py, pz, ex, ey, ez);
  }
  __syncthreads();
  if (t < 6) {
    double acc = 0.0;
    for (int k = 0; k < 27; ++k) acc += term[t * 27 + k];
    const long N = (long)a.nx * a.ny * a.nz;
    a.n6[t * N + ((long)Z * a.ny + Y) * a.nx + X] =
        acc / (4.0 * kPi * a.dx * a.dy * a.dz);
  }
}

// The middle regime, one block per offset.  A thread takes points of one
// (x, y) node pair and sums w r^-5 times 1, sz and sz^2 over the z nodes:
// with sx and sy fixed these give all six components, so a point costs one
// reciprocal square root and a few multiplications (92 us for 41x41x4
// offsets with a division and six sums per point, 31 now).
constexpr int kQuadThreads = 256;
__global__ __launch_bounds__(kQuadThreads) void k_tensor_quad(TensorArgs a) {
  int X, Y, Z;
  box_offset(a, &X, &Y, &Z);
  const double x = X * a.dx, y = Y * a.dy, z = a.z0 + Z * a.zs;
  const double r = sqrt(x * x + y * y + z * z) / a.dmax;
  if (r < kRNear || r >= kRFar) return;
  const int nq = a.nq;
  __shared__ double node[24], wgt[24];
  if ((int)threadIdx.x < nq) {
    node[threadIdx.x] = a.qt[threadIdx.x];
    wgt[threadIdx.x] = a.qw[threadIdx.x];
  }
  __syncthreads();
  double acc[6] = {0, 0, 0, 0, 0, 0};
  for (int p = threadIdx.x; p < nq * nq; p += kQuadThreads) {
    const int ia = p % nq, ib = p / nq;
    const double sx = x + node[ia] * a.dx, sy = y + node[ib] * a.dy;
    const double rho2 = sx * sx + sy * sy;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    for (int ic = 0; ic < nq; ++ic) {
      const double sz = z + node[ic] * a.dz;
      const double q = rsqrt(rho2 + sz * sz), q2 = q * q;
      const double w5 = wgt[ic] * (q2 * q2 * q);
      s0 += w5;
      s1 += w5 * sz;
      s2 += w5 * sz * sz;
    }
    const double w = wgt[ia] * wgt[ib];
    acc[0] += w * ((2.0 * sx * sx - sy * sy) * s0 - s2);
    acc[1] += w * ((2.0 * sy * sy - sx * sx) * s0 - s2);
    acc[2] += w * (2.0 * s2 - rho2 * s0);
    acc[3] += w * (3.0 * sx * sy * s0);
    acc[4] += w * (3.0 * sx * s1);
    acc[5] += w * (3.0 * sy * s1);
  }
  __shared__ double red[6][kQuadThreads / 64];
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    double v = acc[c];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    if ((threadIdx.x & 63) == 0) red[c][threadIdx.x >> 6] = v;
  }
  __syncthreads();
  if (threadIdx.x < 6) {
    const int c = threadIdx.x;
    double v = 0.0;
    for (int k = 0; k < kQuadThreads / 64; ++k) v += red[c][k];
    const long N = (long)a.nx * a.ny * a.nz;
    a.n6[c * N + ((long)Z * a.ny + Y) * a.nx + X] = -(a.dx * a.dy * a.dz) / (4.0 * kPi) * v;
  }
}

// flat index of the multi-index (p, q, r), |k| = p+q+r <= 6: orders are stored
// consecutively, (p, q) ordered within an order (84 entries in all)
__device__ __forceinline__ int aidx(int p, int q, int r) {
  const int n = p + q + r;
  return n * (n + 1) * (n + 2) / 6 + p * (2 * n + 3 - p) / 2 + q;
}

// 4th-moment expansion at offset (x, y, z), |R| >= 40 max(d)
__device__ void tensor_far_at(double x, double y, double z, const TensorArgs& a, double* o6) {
  const double R2 = x * x + y * y + z * z;
  // a_k = (-1)^|k|/k! d^k (1/R) for |k| <= 6
  double A[84];
  A[aidx(0, 0, 0)] = 1.0 / sqrt(R2);
  for (int n = 1; n <= 6; ++n) {
    for (int p = 0; p <= n; ++p) {
      for (int q = 0; q <= n - p; ++q) {
        const int s = n - p - q;
        double acc = 0.0;
        if (p) acc += (2 * n - 1) * x * A[aidx(p - 1, q, s)];
        if (q) acc += (2 * n - 1) * y * A[aidx(p, q - 1, s)];
        if (s) acc += (2 * n - 1) * z * A[aidx(p, q, s - 1)];
        if (p >= 2) acc -= (n - 1) * A[aidx(p - 2, q, s)];
        if (q >= 2) acc -= (n - 1) * A[aidx(p, q - 2, s)];
        if (s >= 2) acc -= (n - 1) * A[aidx(p, q, s - 2)];
        A[aidx(p, q, s)] = acc / (n * R2);
      }
    }
  }
  const double fact[7] = {1, 1, 2, 6, 24, 120, 720};
  const double d[3] = {a.dx, a.dy, a.dz};
  const int comp_i[6] = {0, 1, 2, 0, 0, 1};
  const int comp_j[6] = {0, 1, 2, 1, 2, 2};
  const double pref = -(a.dx * a.dy * a.dz) / (4.0 * kPi);
  for (int c = 0; c < 6; ++c) {
    int base[3] = {0, 0, 0};
    base[comp_i[c]]++;
    base[comp_j[c]]++;
    auto D = [&](int e0, int e1, int e2) {
      const int p = base[0] + e0, q = base[1] + e1, s = base[2] + e2;
      const double sign = ((p + q + s) & 1) ? -1.0 : 1.0;
      return sign * fact[p] * fact[q] * fact[s] * A[aidx(p, q, s)];
    };
    double acc = D(0, 0, 0);
    acc += d[0] * d[0] / 12.0 * D(2, 0, 0) + d[1] * d[1] / 12.0 * D(0, 2, 0) +
           d[2] * d[2] / 12.0 * D(0, 0, 2);
    acc += d[0] * d[0] * d[0] * d[0] / 360.0 * D(4, 0, 0) +
           d[1] * d[1] * d[1] * d[1] / 360.0 * D(0, 4, 0) +
           d[2] * d[2] * d[2] * d[2] / 360.0 * D(0, 0, 4);
    acc += d[0] * d[0] * d[1] * d[1] / 144.0 * D(2, 2, 0) +
           d[0] * d[0] * d[2] * d[2] / 144.0 * D(2, 0, 2) +
           d[1] * d[1] * d[2] * d[2] / 144.0 * D(0, 2, 2);
    o6[c] = pref * acc;
  }
}

__global__ void k_tensor_far(TensorArgs a) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long N = (long)a.nx * a.ny * a.nz;
  if (i >= N) return;
  const int X = (int)(i % a.nx), Y = (int)((i / a.nx) % a.ny), Z = (int)(i / ((long)a.nx * a.ny));
  const double x = X * a.dx, y = Y * a.dy, z = a.z0 + Z * a.zs;
  const double r = sqrt(x * x + y * y + z * z) / a.dmax;
  if (r < kRFar) return;
  double o6[6];
  tensor_far_at(x, y, z, a, o6);
  for (int c = 0; c < 6; ++c) a.n6[c * N + i] = o6[c];
}

// The tensor at any offset, regime by distance; the middle regime's
// quadrature runs in the calling thread.
__device__ void tensor_at(double x, double y, double z, const TensorArgs& a, double* o6) {
  const double r = sqrt(x * x + y * y + z * z) / a.dmax;
  if (r < kRNear) {
    o6[0] = second_difference<false>(x, y, z, a.dx, a.dy, a.dz);
    o6[1] = second_difference<false>(y, x, z, a.dy, a.dx, a.dz);
    o6[2] = second_difference<false>(z, y, x, a.dz, a.dy, a.dx);
    o6[3] = second_difference<true>(x, y, z, a.dx, a.dy, a.dz);
    o6[4] = second_difference<true>(x, z, y, a.dx, a.dz, a.dy);
    o6[5] = second_difference<true>(y, z, x, a.dy, a.dz, a.dx);
  } else if (r < kRFar) {
    double acc[6] = {0, 0, 0, 0, 0, 0};
    const int nq = a.nq;
    for (int ic = 0; ic < nq; ++ic)
      for (int ib = 0; ib < nq; ++ib)
        for (int ia = 0; ia < nq; ++ia) {
          const double w = a.qw[ia] * a.qw[ib] * a.qw[ic];
          const double sx = x + a.qt[ia] * a.dx, sy = y + a.qt[ib] * a.dy,
                       sz = z + a.qt[ic] * a.dz;
          const double s2 = sx * sx + sy * sy + sz * sz;
          const double inv5 = w / (s2 * s2 * sqrt(s2));
          acc[0] += (3.0 * sx * sx - s2) * inv5;
          acc[1] += (3.0 * sy * sy - s2) * inv5;
          acc[2] += (3.0 * sz * sz - s2) * inv5;
          acc[3] += 3.0 * sx * sy * inv5;
          acc[4] += 3.0 * sx * sz * inv5;
          acc[5] += 3.0 * sy * sz * inv5;
        }
    const double pref = -(a.dx * a.dy * a.dz) / (4.0 * kPi);
    for (int c = 0; c < 6; ++c) o6[c] = pref * acc[c];
  } else {
    tensor_far_at(x, y, z, a, o6);
  }
}

// Periodic axes: the tensor at offsets 0 <= X <= nx/2 (and/or Y) summed over
// the images X + k nx, k = -rx..rx; at the half period (X = nx/2, nx even)
// the offsets +X and -X are one cyclic index holding their mean, so a
// component odd along that axis is zero there.  Open axes cover 0 <= X < n.
__global__ void k_tensor_images(TensorArgs a) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long nbox = (long)a.bx * a.by * a.bz;
  if (i >= nbox) return;
  const int X = (int)(i % a.bx), Y = (int)((i / a.bx) % a.by), Z = (int)(i / ((long)a.bx * a.by));
  double sum[6] = {0, 0, 0, 0, 0, 0};
  for (int ky = -a.ry; ky <= a.ry; ++ky)
    for (int kx = -a.rx; kx <= a.rx; ++kx) {
      double o6[6];
      tensor_at((X + (double)kx * a.nx) * a.dx, (Y + (double)ky * a.ny) * a.dy, Z * a.dz, a, o6);
      for (int c = 0; c < 6; ++c) sum[c] += o6[c];
    }
  const bool hx = a.rx > 0 && 2 * X == a.nx, hy = a.ry > 0 && 2 * Y == a.ny;
  const int oddx[6] = {0, 0, 0, 1, 1, 0}, oddy[6] = {0, 0, 0, 1, 0, 1};
  const long N = (long)a.nx * a.ny * a.nz;
  const long o = ((long)Z * a.ny + Y) * a.nx + X;
  for (int c = 0; c < 6; ++c)
    a.n6[c * N + o] = ((hx && oddx[c]) || (hy && oddy[c])) ? 0.0 : sum[c];
}

// --------------------------------------------------- trig transforms ----
__global__ void k_trig_table(double* cs, double* sn, int P) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= P) return;
  double s, c;
  sincospi(2.0 * (double)j / (double)P, &s, &c);
  cs[j] = c;
  sn[j] = s;
}

// parity per component (xx, yy, zz, xy, xz, yz): odd in x / y / z
__constant__ int kOddX[6] = {0, 0, 0, 1, 1, 0};
__constant__ int kOddY[6] = {0, 0, 0, 1, 0, 1};
__constant__ int kOddZ[6] = {0, 0, 0, 0, 1, 1};

// weight of offset X in a cosine/sine sum over X >= 0: offsets +X and -X
// both, except X = 0 and, on a periodic axis, the half period X = n/2
__device__ __forceinline__ double offset_weight(int X, int n, int per) {
  return (X == 0 || (per && 2 * X == n)) ? 1.0 : 2.0;
}

// ---- cosine and sine sums along x and y as FP64 matrix products --------
// C[m][n] = sum_k A(m, k) w_k trig(k n), n = 0..P/2.  Along x the rows m are
// the (Z, Y) rows of a component's tensor; along y they are the kx of one
// (component, Z) plane, read transposed, so that the result lies with ky
// contiguous as the kernel spectrum does.  A weight and a sign-free phase
// index per (k, n) cost far more than the multiplication they feed, so a
// block forms each tile of the trig matrix once for 64 rows and multiplies
// with the FP64 matrix instruction (16x16x4): 64x64 outputs per block, four
// waves of 32x32, 16 of the sum at a time through LDS.  Thread-per-output
// sums took 16.8 + 12.0 ms for 512x512x16 (1.5 TFLOP/s), this 1.0 + 1.2.
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int kTrigTile = 64, kTrigK = 16;

struct TrigArgs {
  const double* in;    // x: [6 planes][M][K]; y: [planes][K][M]
  double* out;         // [planes][M][N]
  const double* cs;
  const double* sn;
  int M, N, K;         // K offsets 0..K-1 enter the sum
  int ldk;             // stride of a plane's rows: x M rows of ldk, y ldk rows of M
  int P, per, nk;      // transform length, periodic axis, its cells
  int nz;              // planes per component
};

template <bool ALONG_Y>
__global__ __launch_bounds__(256) void k_trig_gemm(TrigArgs a) {
  // rows padded to 66 doubles: the four k of a fragment start 4 banks apart
  __shared__ double As[kTrigK][kTrigTile + 2], Bs[kTrigK][kTrigTile + 2];
  const int plane = blockIdx.z, c = plane / a.nz;
  const double* tab = (ALONG_Y ? kOddY[c] : kOddX[c]) ? a.sn : a.cs;
  const double* in = a.in + (long)plane * a.ldk * a.M;
  const int m0 = blockIdx.x * kTrigTile, n0 = blockIdx.y * kTrigTile;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave & 1) * 32, wn = (wave >> 1) * 32;
  const int li = lane & 15, lk = lane >> 4;
  f64x4 acc[2][2] = {};
  for (int k0 = 0; k0 < a.K; k0 += kTrigK) {
    for (int e = tid; e < kTrigK * kTrigTile; e += 256) {
      // consecutive threads read consecutive addresses of either layout
      const int kk = ALONG_Y ? e / kTrigTile : e % kTrigK;
      const int mm = ALONG_Y ? e % kTrigTile : e / kTrigK;
      const int k = k0 + kk, m = m0 + mm;
      const bool ok = k < a.K && m < a.M;
      const long o = ALONG_Y ? (long)k * a.M + m : (long)m * a.ldk + k;
      const double v = in[ok ? o : 0];
      As[kk][mm] = ok ? v * offset_weight(k, a.nk, a.per) : 0.0;
    }
    for (int e = tid; e < kTrigK * kTrigTile; e += 256) {
      const int kk = e / kTrigTile, nn = e % kTrigTile;
      Bs[kk][nn] = tab[(uint32_t)((k0 + kk) * (n0 + nn)) % (uint32_t)a.P];
    }
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < kTrigK; ks += 4) {
      double fa[2], fb[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        fa[i] = As[ks + lk][wm + 16 * i + li];
        fb[i] = Bs[ks + lk][wn + 16 * i + li];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[i], fb[j], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }
  double* out = a.out + (long)plane * a.M * a.N;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + wm + 16 * i + 4 * r + lk, n = n0 + wn + 16 * j + li;
        if (m < a.M && n < a.N) out[(long)m * a.N + n] = acc[i][j][r];
      }
}

// K[c][kz][kx][ky] = scale_c sum_Z w_Z F2[c][Z][kx][ky] trig(kz Z), kz <= Pz/2.
// A thread takes a (kx, ky) column of one component: its layers are read
// once (up to kTrigZ of them at a time) for all kz.
constexpr int kTrigZ = 16;
template <typename T>
__global__ __launch_bounds__(256) void k_trig_z(const double* f2, T* kout, const double* cs,
                                                const double* sn, int nz, int Pz, long plane,
                                                int Hz, double scale) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= plane) return;
  const int c = blockIdx.y;
  const double* tab = kOddZ[c] ? sn : cs;
  const double* in = f2 + (long)c * nz * plane + i;
  T* out = kout + (long)c * Hz * plane + i;
  const double sc = c >= 3 ? -scale : scale;
  if (nz <= kTrigZ) {
    double v[kTrigZ];
#pragma unroll
    for (int Z = 0; Z < kTrigZ; ++Z) v[Z] = Z < nz ? in[Z * plane] * (Z == 0 ? 1.0 : 2.0) : 0.0;
    for (int kz = 0; kz < Hz; ++kz) {
      double acc = 0.0;
#pragma unroll
      for (int Z = 0; Z < kTrigZ; ++Z)
        if (Z < nz) acc += v[Z] * tab[(uint32_t)(kz * Z) % (uint32_t)Pz];
      out[kz * plane] = (T)(sc * acc);
    }
  } else {
    for (int kz = 0; kz < Hz; ++kz) {
      double acc = 0.0;
      for (int Z = 0; Z < nz; ++Z)
        acc += (Z == 0 ? 1.0 : 2.0) * in[Z * plane] * tab[(uint32_t)(kz * Z) % (uint32_t)Pz];
      out[kz * plane] = (T)(sc * acc);
    }
  }
}

// ---------------------------------------------------------- host side --
static void gauss_legendre(int n, double* x, double* w) {
  for (int i = 0; i < n; ++i) {
    double z = std::cos(kPi * (i + 0.75) / (n + 0.5));
    double pp = 0.0;
    for (int it = 0; it < 100; ++it) {
      double p1 = 1.0, p2 = 0.0;
      for (int j = 1; j <= n; ++j) {
        const double p3 = p2;
        p2 = p1;
        p1 = ((2.0 * j - 1.0) * z * p2 - (j - 1.0) * p3) / j;
      }
      pp = n * (z * p1 - p2) / (z * z - 1.0);
      const double z1 = z;
      z = z1 - p1 / pp;
      if (std::fabs(z - z1) < 1e-16) {
        // one more evaluation of the derivative at the converged root
        p1 = 1.0; p2 = 0.0;
        for (int j = 1; j <= n; ++j) {
          const double p3 = p2;
          p2 = p1;
          p1 = ((2.0 * j - 1.0) * z * p2 - (j - 1.0) * p3) / j;
        }
        pp = n * (z * p1 - p2) / (z * z - 1.0);
        break;
      }
    }
    x[i] = z;
    w[i] = 2.0 / ((1.0 - z * z) * pp * pp);
  }
}

// nodes on [-1, 1] for the density (1 - |t|), 2n of them
static void triangle_rule(int n, double* t, double* w) {
  double x[12], gw[12];
  gauss_legendre(n, x, gw);
  for (int i = 0; i < n; ++i) {
    const double tp = 0.5 * (x[i] + 1.0);
    const double wp = 0.5 * gw[i] * (1.0 - tp);
    t[n + i] = tp;
    w[n + i] = wp;
    t[n - 1 - i] = -tp;
    w[n - 1 - i] = wp;
  }
}

static TensorArgs tensor_args(int nx, int ny, int nz, double dx, double dy, double dz, double z0,
                              double zs, double* n6) {
  TensorArgs a{};
  a.nx = nx; a.ny = ny; a.nz = nz;
  a.dx = dx; a.dy = dy; a.dz = dz;
  a.dmax = std::fmax(dx, std::fmax(dy, dz));
  const double dmin = std::fmin(dx, std::fmin(dy, dz));
  const int n = (a.dmax / dmin <= 1.25) ? 8 : 12;
  a.nq = 2 * n;
  triangle_rule(n, a.qt, a.qw);
  a.z0 = z0; a.zs = zs;
  a.n6 = n6;
  return a;
}

// The tensor at every offset of a, regime by regime (a block takes one
// offset of the boxes that hold the near and middle ones).
static int launch_tensor(TensorArgs a, hipStream_t st) {
  auto box = [&](double rcut, int nn, double d) {
    const int b = (int)std::ceil(rcut * a.dmax / d) + 1;
    return b < nn ? b : nn;
  };
  // layers of the box: from the offset nearest to zero upwards on the grid's
  // own offsets; a layer above the grid is nearest to the last one
  const bool own = a.z0 == 0.0;
  // a launch holds fewer than 2^32 threads, which the boxes of flat or tall
  // cells on a large grid exceed (40 dmax/d offsets per axis): in pieces
  constexpr long kPiece = 1L << 22;
  auto pieces = [&](auto kernel, int threads) {
    const long nb = (long)a.bx * a.by * a.bz;
    for (a.i0 = 0; a.i0 < nb; a.i0 += kPiece)
      hipLaunchKernelGGL(kernel, dim3((unsigned)std::min(kPiece, nb - a.i0)), dim3(threads), 0, st,
                         a);
  };
  a.bx = box(kRNear, a.nx, a.dx); a.by = box(kRNear, a.ny, a.dy);
  a.bz = own ? box(kRNear, a.nz, a.dz) : a.nz;
  pieces(k_tensor_near, kNearThreads);
  a.bx = box(kRFar, a.nx, a.dx); a.by = box(kRFar, a.ny, a.dy);
  a.bz = own ? box(kRFar, a.nz, a.dz) : a.nz;
  pieces(k_tensor_quad, kQuadThreads);
  const long N = (long)a.nx * a.ny * a.nz;
  hipLaunchKernelGGL(k_tensor_far, dim3((unsigned)((N + 127) / 128)), dim3(128), 0, st, a);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

static int fill_tensor(int nx, int ny, int nz, double dx, double dy, double dz, double* n6,
                       hipStream_t st) {
  return launch_tensor(tensor_args(nx, ny, nz, dx, dy, dz, 0.0, dz, n6), st);
}

int demag_tensor_only(int nx, int ny, int nz, double dx, double dy, double dz, double* n6,
                      hipStream_t st) {
  return fill_tensor(nx, ny, nz, dx, dy, dz, n6, st);
}

// The image-summed tensor of a grid periodic along x and/or y.
static int fill_tensor_images(int nx, int ny, int nz, double dx, double dy, double dz, int rx,
                              int ry, double* n6, hipStream_t st) {
  TensorArgs a = tensor_args(nx, ny, nz, dx, dy, dz, 0.0, dz, n6);
  a.rx = rx; a.ry = ry;
  a.bx = rx > 0 ? nx / 2 + 1 : nx;
  a.by = ry > 0 ? ny / 2 + 1 : ny;
  a.bz = nz;
  const long nb = (long)a.bx * a.by * a.bz;
  hipLaunchKernelGGL(k_tensor_images, dim3((unsigned)((nb + 63) / 64)), dim3(64), 0, st, a);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Tensor between a cell of a layer at height zt (centre, layer 0 of the grid
// centred at 0) and the cells of the grid at offsets (X dx, Y dy) >= 0:
// k6[c][z][Y][X] = N(X dx, Y dy, zt - z dz).
int stray_kernel_build(int nx, int ny, int nz, double dx, double dy, double dz, double zt,
                       double* k6, hipStream_t st) {
  return launch_tensor(tensor_args(nx, ny, nz, dx, dy, dz, zt, -dz, k6), st);
}

// scratch of demag_kernel_build: the tensor (and, once its x sums are formed,
// in its place the x-y sums), the x sums, trig tables
static void build_sizes(const DemagPlan& p, size_t* n0, size_t* n1, size_t* n2, size_t* nt) {
  *n0 = (size_t)6 * p.nx * p.ny * p.nz;
  *n1 = (size_t)6 * p.nz * p.ny * p.Hx;
  *n2 = (size_t)6 * p.nz * p.Hy * p.Hx;
  *nt = (size_t)2 * (p.Px + p.Py + p.Pz);
}
size_t demag_build_doubles(const DemagPlan& p) {
  size_t n0, n1, n2, nt;
  build_sizes(p, &n0, &n1, &n2, &nt);
  return std::max(n0, n2) + n1 + nt;
}

template <typename T>
int demag_kernel_build(const DemagPlan& p, double dx, double dy, double dz, double* scratch,
                       T* kout, hipStream_t st) {
  size_t n0, n1, n2, nt;
  build_sizes(p, &n0, &n1, &n2, &nt);
  double* n6 = scratch;
  double* f2 = scratch;
  double* f1 = scratch + std::max(n0, n2);
  double* tabs = f1 + n1;
  if (p.rep[0] > 0 || p.rep[1] > 0) {
    if (fill_tensor_images(p.nx, p.ny, p.nz, dx, dy, dz, p.rep[0], p.rep[1], n6, st)) return -1;
  } else if (fill_tensor(p.nx, p.ny, p.nz, dx, dy, dz, n6, st)) {
    return -1;
  }
  double* cx = tabs;            double* sx = cx + p.Px;
  double* cy = sx + p.Px;       double* sy = cy + p.Py;
  double* cz = sy + p.Py;       double* sz = cz + p.Pz;
  hipLaunchKernelGGL(k_trig_table, dim3((p.Px + 255) / 256), dim3(256), 0, st, cx, sx, p.Px);
  hipLaunchKernelGGL(k_trig_table, dim3((p.Py + 255) / 256), dim3(256), 0, st, cy, sy, p.Py);
  hipLaunchKernelGGL(k_trig_table, dim3((p.Pz + 255) / 256), dim3(256), 0, st, cz, sz, p.Pz);
  auto tiles = [](int v) { return (unsigned)((v + kTrigTile - 1) / kTrigTile); };
  TrigArgs x{};
  x.in = n6; x.out = f1; x.cs = cx; x.sn = sx;
  x.M = p.nz * p.ny; x.N = p.Hx; x.ldk = p.nx;
  x.per = p.rep[0] > 0 ? 1 : 0;
  x.K = x.per ? p.nx / 2 + 1 : p.nx;
  x.P = p.Px; x.nk = p.nx; x.nz = 1;
  hipLaunchKernelGGL(k_trig_gemm<false>, dim3(tiles(x.M), tiles(x.N), 6), dim3(256), 0, st, x);
  TrigArgs y{};
  y.in = f1; y.out = f2; y.cs = cy; y.sn = sy;
  y.M = p.Hx; y.N = p.Hy; y.ldk = p.ny;
  y.per = p.rep[1] > 0 ? 1 : 0;
  y.K = y.per ? p.ny / 2 + 1 : p.ny;
  y.P = p.Py; y.nk = p.ny; y.nz = p.nz;
  hipLaunchKernelGGL(k_trig_gemm<true>, dim3(tiles(y.M), tiles(y.N), 6 * p.nz), dim3(256), 0, st,
                     y);
  const double scale = -kMu0 / ((double)p.Px * p.Py * p.Pz);
  const long plane = (long)p.Hx * p.Hy;
  hipLaunchKernelGGL((k_trig_z<T>), dim3((unsigned)((plane + 255) / 256), 6), dim3(256), 0, st, f2,
                     kout, cz, sz, p.nz, p.Pz, plane, p.Hz, scale);
  return hipStreamSynchronize(st) == hipSuccess ? 0 : -1;
}

template int demag_kernel_build<float>(const DemagPlan&, double, double, double, double*, float*,
                                       hipStream_t);
template int demag_kernel_build<double>(const DemagPlan&, double, double, double, double*,
                                        double*, hipStream_t);

}  // namespace mmp
