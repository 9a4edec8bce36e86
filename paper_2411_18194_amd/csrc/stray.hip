// Stray field of the magnet in a layer of cells above it (paper: the
// out-of-plane stray field imaged at a height above a film, "Stray field
// imaging of the non-collinear antiferromagnet Mn3Sn"; the field itself is
// the magnetostatic field of "Magnetostatic field").
//
// B_t(x, y) = -mu0 sum_z sum_{x', y'} N(x - x', y - y', z_t - z) M(x', y', z),
// M = sum_s Ms_s m_s, with the cell-pair tensor table of stray_kernel_build.
// The table holds the offsets X, Y >= 0; the components odd along an axis
// change sign with the offset.  This is an output-time operation (one image
// per call), not part of a step.
//
// The sum as FP64 matrix products: for a fixed row offset dy the tensor
// between a row of 16 targets and 4 sources is a 16x4 slice of a Toeplitz
// matrix, and it serves 16 target rows y at once with the sources of rows
// y - dy (zero outside the grid).  So a wave owns 16x16 targets (three
// accumulators of the 16x16x4 FP64 matrix instruction) and per 4 sources
// loads six tensor and three moment values per lane for nine instructions of
// 2048 operations.  The (layer, dy) pairs are split over enough waves to fill
// the chip, whose partial sums a second kernel adds in order.
// Before, a block per 16x16 targets walked every source with nine LDS reads
// per pair: 1736 us for 128x96x2 (48 blocks on 256 CUs), 241 + 14 now.
#include <algorithm>
#include <mutex>

#include "stray.h"

namespace mmp {

typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int kST = 16;   // tile edge

// The state is read through its slot in the grid's device pointer table
// (the controller swaps that table after accepted steps), so a launch needs
// no host read-back of the table.
template <typename T>
__global__ __launch_bounds__(64) void k_stray(const T* const* __restrict__ mslot, int nsub,
                                             double ms0, double ms1, double ms2,
                                             const double* __restrict__ k6, int nx, int ny, int nz,
                                             double* __restrict__ part) {
  const gcptr<T> m = (gcptr<T>)*mslot;
  const int ntx = (nx + kST - 1) / kST;
  const int x0 = (int)(blockIdx.x % ntx) * kST, y0 = (int)(blockIdx.x / ntx) * kST;
  const int lane = threadIdx.x, li = lane & 15, lk = lane >> 4;
  const long N = (long)nx * ny * nz;
  // row offsets that pair a target row of the tile with a source row
  const int dlo = y0 - (ny - 1), dhi = min(y0 + kST - 1, ny - 1);
  const int nd = dhi - dlo + 1;
  const int units = nz * nd, ns = gridDim.y;
  const int u0 = (int)((long)units * blockIdx.y / ns);
  const int u1 = (int)((long)units * (blockIdx.y + 1) / ns);
  f64x4 acc[3] = {};
  for (int u = u0; u < u1; ++u) {
    const int z = u / nd, dy = dlo + (u - z * nd);
    const double sy = dy < 0 ? -1.0 : 1.0;
    const double* kr = k6 + ((long)z * ny + abs(dy)) * nx;
    const int ys = y0 + li - dy;
    const bool iny = ys >= 0 && ys < ny;
    const long mr = ((long)z * ny + (iny ? ys : 0)) * nx;
#pragma unroll 2
    for (int s = 0; s < nx; s += 4) {
      const int xs = s + lk;
      const bool in = iny && xs < nx;
      const long mi = mr + (xs < nx ? xs : 0);
      double v[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        v[c] = ms0 * (double)m[c * N + mi];
        if (nsub >= 2) v[c] += ms1 * (double)m[(3 + c) * N + mi];
        if (nsub == 3) v[c] += ms2 * (double)m[(6 + c) * N + mi];
        v[c] = in ? v[c] : 0.0;
      }
      // (targets and sources past the grid read a valid offset; their
      // results are not kept, their moments are zero)
      const int dx = x0 + li - xs, ax = min(abs(dx), nx - 1);
      const double sx = dx < 0 ? -1.0 : 1.0;
      const double txx = kr[ax], tyy = kr[N + ax], tzz = kr[2 * N + ax];
      const double txy = sx * sy * kr[3 * N + ax], txz = sx * kr[4 * N + ax],
                   tyz = sy * kr[5 * N + ax];
      acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(txx, v[0], acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(txy, v[0], acc[1], 0, 0, 0);
      acc[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(txz, v[0], acc[2], 0, 0, 0);
      acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(txy, v[1], acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(tyy, v[1], acc[1], 0, 0, 0);
      acc[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(tyz, v[1], acc[2], 0, 0, 0);
      acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(txz, v[2], acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(tyz, v[2], acc[1], 0, 0, 0);
      acc[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(tzz, v[2], acc[2], 0, 0, 0);
    }
  }
  // accumulator row (target x) 4 r + lane / 16, column (target y) lane % 16
  const long P = (long)nx * ny;
  double* out = part + (long)blockIdx.y * 3 * P;
  const int yt = y0 + li;
  if (yt < ny)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int xt = x0 + 4 * r + lk;
      if (xt < nx)
#pragma unroll
        for (int c = 0; c < 3; ++c) out[c * P + (long)yt * nx + xt] = acc[c][r];
    }
}

// out = -mu0 times the sum of the ns partial images (which may be out itself)
__global__ __launch_bounds__(256) void k_stray_sum(const double* part, int ns, long n,
                                                  double* out) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double acc = 0.0;
  for (int s = 0; s < ns; ++s) acc += part[s * n + i];
  out[i] = -kMu0 * acc;
}

// Waves per 16x16 targets: enough for four on every SIMD of the chip, at most
// one per (layer, row offset), and no more than the partial images that fit
// beside the tensor in the fixed table where the allocation-free call would
// use it (both calls take the same split, so they agree bitwise).
int stray_splits(int nx, int ny, int nz) {
  const long tiles = (long)((nx + kST - 1) / kST) * ((ny + kST - 1) / kST);
  long s = std::max<long>(1, std::min<long>(4096 / tiles, (long)nz * ny));
  if (6L * nz * (2L * nx - 1) * (2L * ny - 1) <= kStrayScratchDoubles)
    s = std::min(s, (kStrayScratchDoubles - 6L * nz * nx * ny) / (3L * nx * ny));
  return (int)std::max<long>(1, s);
}

template <typename T>
void launch_stray(const T* const* mslot, int nsub, double ms0, double ms1, double ms2,
                  const double* k6, double* part, int nx, int ny, int nz, double* out,
                  hipStream_t st) {
  const int ns = stray_splits(nx, ny, nz);
  const dim3 g((unsigned)(((nx + kST - 1) / kST) * ((ny + kST - 1) / kST)), (unsigned)ns);
  double* p = ns > 1 ? part : out;
  hipLaunchKernelGGL((k_stray<T>), g, dim3(64), 0, st, mslot, nsub, ms0, ms1, ms2, k6, nx, ny, nz,
                     p);
  const long n = 3L * nx * ny;
  hipLaunchKernelGGL(k_stray_sum, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, ns, n,
                     out);
}

template void launch_stray<float>(const float* const*, int, double, double, double,
                                  const double*, double*, int, int, int, double*, hipStream_t);
template void launch_stray<double>(const double* const*, int, double, double, double,
                                   const double*, double*, int, int, int, double*, hipStream_t);

// ------------------------------------------------ fixed tensor table --
// Tensor table of the allocation-free stray-field call: one array per GPU,
// held for the life of the process.  Host code must not pass the array's
// name to a kernel (in host code it only names a host-side stand-in); the
// device address comes from hipGetSymbolAddress, taken once per device
// with that device current.
static __device__ __align__(256) double scratch[kStrayScratchDoubles];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

int stray_scratch(int dev, double** out) {
  *out = nullptr;
  if (dev < 0 || dev >= kMaxDevices) return -1;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    int cur = -1;
    if (hipGetDevice(&cur) != hipSuccess) return -1;
    if (cur != dev && hipSetDevice(dev) != hipSuccess) return -1;
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (cur != dev) (void)hipSetDevice(cur);
    if (e != hipSuccess || !ptr) return -1;
    g_scratch_ptr[dev] = static_cast<double*>(ptr);
  }
  *out = g_scratch_ptr[dev];
  return 0;
}

}  // namespace mmp
