// Demagnetising field: zero-padded FFT convolution with the cell-averaged
// tensor (paper, Methods "Magnetostatic field"; the moment of a
// multi-sublattice cell is summed before the convolution).
//
// Pass structure (3-D grid):
//   x  forward  R2C of M (two real rows packed in one complex line), the
//               half spectrum stored transposed so y lines are contiguous
//   y  forward  zero-padded ny -> Py
//   z  fwd * K * inv  per (kx, ky) column, with the real octant kernel
//   y  inverse  Py -> crop ny
//   x  inverse  C2R (two rows per complex line), crop nx -> B_d
// The y, z and y passes are one pass where the lines of a kx column fit in
// LDS (2-D grids always do).
// Zero padding is never materialised in memory: the pads exist only in LDS.
#include "demag.h"
#include "demag4.h"

#include <algorithm>
#include <vector>

namespace mmp {

// largest blocks of the mixed-radix passes; the fused y-z pass holds the
// 3 PZ values of a column per thread and needs their registers (at most 96
// of 256 leave room for two waves per SIMD)
constexpr int kLineThreads = 256;
constexpr int yz_max_threads(int real_bytes, int pz) {
  return 3 * pz * 2 * (real_bytes / 4) <= 96 ? 512 : 256;
}
// complex elements of one block of the batched passes
constexpr long kMultiElems = 4096;

// ----------------------------------------------------------------- tables --
// Stage twiddles of a line transform and the places of its bins.
template <typename T>
__global__ void k_line_tables(LineFft f, cpx<T>* tw) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  for (int s = 0; s + 1 < f.n; ++s) {
    const LineStage t = f.stage(s);
    const int m = t.r * t.M;   // length of the sub-transform of this stage
    if (i < m) {
      const int q = i / t.M, lo = i - q * t.M;
      double sn, cs;
      sincospi(-2.0 * (double)(q * lo) / (double)m, &sn, &cs);
      tw[t.tw + i] = cmk<T>((T)cs, (T)sn);
    }
  }
  if (i < f.L) const_cast<uint16_t*>(line_places(f, tw))[i] = (uint16_t)f.place_of(i);
}

template <typename T>
void build_line_tables(const LineFft& f, cpx<T>* tw, hipStream_t st) {
  hipLaunchKernelGGL(k_line_tables<T>, dim3((f.L + 255) / 256), dim3(256), 0, st, f, tw);
}
template void build_line_tables<float>(const LineFft&, cpx<float>*, hipStream_t);
template void build_line_tables<double>(const LineFft&, cpx<double>*, hipStream_t);

// --------------------------------------------------------------- x pass --
template <typename T>
struct XArgs {
  const Table<T>* tbl;
  const Ctrl* ctrl;
  int src;    // table slot of the state to transform
  T ms0, ms1, ms2;
  int nsub;
  cpx<T>* S1;
  T* Bd;
  const cpx<T>* tw;
  int nx, ny, nz, Hx, ldy, ty;
  int lnl;    // log2(ty / 2)
  int half;   // the line is at least twice its data (an open axis)
  LineFft f;
};

// The pass bodies take the block's coordinates (and the stage) as
// arguments: the single-grid kernels pass blockIdx, the batched kernels
// the entry of their work table.
template <typename T>
__device__ __forceinline__ void fftx_fwd_body(const XArgs<T>& a, int zero, int src, int bx, int by,
                                              int bz) {
  using V = cpx<T>;
  const gcptr<T> m = (gcptr<T>)table_slot<T>(a.tbl, src + zero);
  if (ctrl_stopped(a.ctrl, zero)) return;
  extern __shared__ char smem_raw[];
  V* buf = reinterpret_cast<V*>(smem_raw);
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int c = bz, z = by, y0 = bx * a.ty;
  const int nl = a.ty >> 1;
  const long N = (long)a.nx * a.ny * a.nz;
  const gcptr<T> m0 = m + (long)c * N + (long)z * a.ny * a.nx;
  const gcptr<T> m1 = m0 + 3 * N;
  // rows past ny and cells past nx: a clamped load, zeroed afterwards
  auto ld = [&](int q, int x) -> V {
    const int ya = y0 + 2 * q, yb = ya + 1;
    const int xc = x < a.nx ? x : 0;
    const int ia = (ya < a.ny ? ya : 0) * a.nx + xc, ib = (yb < a.ny ? yb : 0) * a.nx + xc;
    T re = a.ms0 * m0[ia], im = a.ms0 * m0[ib];
    if (a.nsub >= 2) {
      re += a.ms1 * m1[ia];
      im += a.ms1 * m1[ib];
    }
    if (a.nsub == 3) {
      re += a.ms2 * m1[3 * N + ia];
      im += a.ms2 * m1[3 * N + ib];
    }
    const bool in = x < a.nx;
    return cmk<T>(in && ya < a.ny ? re : T(0), in && yb < a.ny ? im : T(0));
  };
  const V* twl = line_stage_tw<T>(a.f, buf, nl, a.tw, tid, nthr);
  line_fft_fwd<T>(a.f, buf, a.tw, twl, nl, a.half != 0, tid, nthr, ld);
  // unpack the two real spectra and store them transposed
  const uint16_t* place = line_places(a.f, twl);
  V* out = a.S1 + ((long)(c * a.nz + z) * a.Hx) * a.ldy + y0;
  for (int idx = tid; idx < nl * a.Hx; idx += nthr) {
    const int q = idx & (nl - 1), kx = idx >> a.lnl;
    const int km = kx == 0 ? 0 : a.f.L - kx;
    const V* b = buf + q * a.f.pitch;
    const V zk = b[place[kx]], zm = b[place[km]];
    const T h = T(0.5);
    store2<T>(out + (long)kx * a.ldy + 2 * q,
              cmk<T>(h * (zk.x + zm.x), h * (zk.y - zm.y)),
              cmk<T>(h * (zk.y + zm.y), h * (zm.x - zk.x)));
  }
}

template <typename T>
__global__ __launch_bounds__(kLineThreads) void k_fftx_fwd(XArgs<T> a) {
  const int zero = warm_args<XArgs<T>>();
  fftx_fwd_body<T>(a, zero, a.src, blockIdx.x, blockIdx.y, blockIdx.z);
}

template <typename T>
__device__ __forceinline__ void fftx_inv_body(const XArgs<T>& a, int zero, int bx, int by, int bz) {
  using V = cpx<T>;
  // (the spectrum is loaded beside the controller's flags, not behind them)
  const bool stop = ctrl_stopped(a.ctrl, zero);
  extern __shared__ char smem_raw[];
  V* buf = reinterpret_cast<V*>(smem_raw);
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int c = bz, z = by, y0 = bx * a.ty;
  const int nl = a.ty >> 1;
  const V* in = a.S1 + ((long)(c * a.nz + z) * a.Hx) * a.ldy + y0;
  const V* twl = line_stage_tw<T>(a.f, buf, nl, a.tw, tid, nthr);
  const uint16_t* place = line_places(a.f, a.tw);   // (from memory, with the data)
  for (int idx = tid; idx < nl * a.Hx; idx += nthr) {
    const int q = idx & (nl - 1), kx = idx >> a.lnl;
    const int pk = place[kx], pm = place[kx == 0 ? 0 : a.f.L - kx];
    V xa, xb;
    load2<T>(in + (long)kx * a.ldy + 2 * q, xa, xb);
    // past the last row S1 holds the forward pass's rounding of a zero row,
    // unscaled by the kernel: left in, it would leak into the row before
    if (y0 + 2 * q + 1 >= a.ny) xb = cmk<T>(T(0), T(0));
    V* b = buf + q * a.f.pitch;
    b[pk] = cmk<T>(xa.x - xb.y, xa.y + xb.x);
    if (kx > 0 && 2 * kx < a.f.L) b[pm] = cmk<T>(xa.x + xb.y, xb.x - xa.y);
  }
  lds_copies_done();
  if (stop) return;
  __syncthreads();
  const long N = (long)a.nx * a.ny * a.nz;
  T* out = a.Bd + (long)c * N + (long)z * a.ny * a.nx;
  line_fft_inv<T>(a.f, buf, twl, nl, a.half != 0, tid, nthr, [&](int q, int x, V v) {
    const int ya = y0 + 2 * q;
    if (x < a.nx) {
      if (ya < a.ny) out[ya * a.nx + x] = v.x;
      if (ya + 1 < a.ny) out[(ya + 1) * a.nx + x] = v.y;
    }
  });
}

template <typename T>
__global__ __launch_bounds__(kLineThreads) void k_fftx_inv(XArgs<T> a) {
  const int zero = warm_args<XArgs<T>>();
  fftx_inv_body<T>(a, zero, blockIdx.x, blockIdx.y, blockIdx.z);
}

// --------------------------------------------------------------- y pass --
template <typename T>
struct YArgs {
  const Ctrl* ctrl;
  const cpx<T>* in;
  cpx<T>* out;
  const cpx<T>* tw;
  int nlines, nvalid_in, ld_in, nvalid_out, ld_out, nl;
  int half;
  FastDiv dL;
  LineFft f;
};

template <typename T, bool INV>
__device__ __forceinline__ void ffty_body(const YArgs<T>& a, int zero, int bx) {
  using V = cpx<T>;
  if (ctrl_stopped(a.ctrl, zero)) return;
  extern __shared__ char smem_raw[];
  V* buf = reinterpret_cast<V*>(smem_raw);
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int l0 = bx * a.nl, L = a.f.L;
  const V* twl = line_stage_tw<T>(a.f, buf, a.nl, a.tw, tid, nthr);
  if constexpr (!INV) {
    line_fft_fwd<T>(a.f, buf, a.tw, twl, a.nl, a.half != 0, tid, nthr, [&](int l, int n) -> V {
      const bool in = l0 + l < a.nlines && n < a.nvalid_in;
      const V v = a.in[in ? (long)(l0 + l) * a.ld_in + n : 0];
      return in ? v : cmk<T>(T(0), T(0));
    });
    const uint16_t* place = line_places(a.f, twl);
    for (int idx = tid; idx < a.nl * L; idx += nthr) {
      const int l = a.dL.div(idx), k = idx - l * L;
      if (l0 + l < a.nlines) a.out[(long)(l0 + l) * a.ld_out + k] = buf[l * a.f.pitch + place[k]];
    }
  } else {
    const uint16_t* place = line_places(a.f, a.tw);
    for (int idx = tid; idx < a.nl * L; idx += nthr) {
      const int l = a.dL.div(idx), k = idx - l * L;
      const bool in = l0 + l < a.nlines;
      const V v = a.in[in ? (long)(l0 + l) * a.ld_in + k : 0];
      buf[l * a.f.pitch + place[k]] = v;
    }
    lds_copies_done();
    __syncthreads();
    line_fft_inv<T>(a.f, buf, twl, a.nl, a.half != 0, tid, nthr, [&](int l, int n, V v) {
      if (l0 + l < a.nlines && n < a.nvalid_out) a.out[(long)(l0 + l) * a.ld_out + n] = v;
    });
  }
}

template <typename T, bool INV>
__global__ __launch_bounds__(kLineThreads) void k_ffty(YArgs<T> a) {
  const int zero = warm_args<YArgs<T>>();
  ffty_body<T, INV>(a, zero, blockIdx.x);
}

// Symmetric 3x3 multiply with the octant kernel; sy/sz flip the odd parts
// (kxz = kyz = 0 on a 2-D grid).
template <typename T>
__device__ __forceinline__ void sym3(cpx<T>& mx, cpx<T>& my, cpx<T>& mz, T kxx, T kyy, T kzz,
                                     T kxy, T kxz, T kyz) {
  const cpx<T> x = mx, y = my, z = mz;
  mx = cmk<T>(kxx * x.x + kxy * y.x + kxz * z.x, kxx * x.y + kxy * y.y + kxz * z.y);
  my = cmk<T>(kxy * x.x + kyy * y.x + kyz * z.x, kxy * x.y + kyy * y.y + kyz * z.y);
  mz = cmk<T>(kxz * x.x + kyz * y.x + kzz * z.x, kxz * x.y + kyz * y.y + kzz * z.y);
}

// ------------------------------------------- fused y, z and multiply pass --
// One block carries nk kx columns of all 3 nz (component, layer) lines in
// LDS: y forward, then each ky column's z transform, kernel product and
// inverse z transform in the registers of one thread, then y inverse, in
// place in S1.  On a 2-D grid the column is the three components alone.
// Against separate y, z and y passes the padded spectrum never reaches
// memory (S2 is 2 (Py/ny) times S1, written twice and read twice) and two
// launches go.  Measured: 183x77x5 FP32 86.1 us in three passes -> 10.9 us;
// 64x64x4 FP32 15.1 (register kernels) -> 9.3 us; 333x130x1 FP64 57.1 ->
// 11.7 us.  One kx column per block: few grids have more than a few hundred.
template <typename T>
struct YzArgs {
  const Ctrl* ctrl;
  cpx<T>* S1;     // [3][nz][Hx][ldy]
  const T* K;     // [6][Hz][Hx][Hy]
  const cpx<T>* tw;
  int ny, nz, Pz, Hx, Hy, Hz, ldy, nk, lnk;
  int half;
  FastDiv dL;
  LineFft f;
};

// The kernel values of one column: 4 of the 2-D kernel, else 6 of each plane
// kz <= PZ/2.
template <typename T, int PZ>
struct YzKernel {
  T v[PZ == 1 ? 1 : PZ / 2 + 1][6];
};
// column idx of the block: its kx (columns past the spectrum: the first), ky
// and octant kernel column
template <typename T, int PZ>
__device__ __forceinline__ void yz_load_k(const YzArgs<T>& a, int kx0, int idx,
                                          YzKernel<T, PZ>& k) {
  const int L = a.f.L;
  const int j = a.dL.div(idx), ky = idx - j * L;
  const int kx = kx0 + j < a.Hx ? kx0 + j : 0, kyo = 2 * ky > L ? L - ky : ky;
  const long ks = (long)a.Hz * a.Hx * a.Hy, kzs = (long)a.Hx * a.Hy;
  const T* K = a.K + (long)kx * a.Hy + kyo;
  if constexpr (PZ == 1) {
#pragma unroll
    for (int c = 0; c < 4; ++c) k.v[0][c] = K[c * ks];
  } else {
#pragma unroll
    for (int kz = 0; kz <= PZ / 2; ++kz)
#pragma unroll
      for (int c = 0; c < 6; ++c) k.v[kz][c] = K[c * ks + kz * kzs];
  }
}

template <typename T, int PZ>
__device__ __forceinline__ void yz_column(const YzArgs<T>& a, cpx<T>* buf,
                                          const uint16_t* place, int kx0, int idx,
                                          const YzKernel<T, PZ>& k) {
  using V = cpx<T>;
  const int L = a.f.L;
  const int zl = a.nk * a.f.pitch, cl = a.nz * zl;   // LDS strides of layer, component
  const int j = a.dL.div(idx), ky = idx - j * L;
  if (kx0 + j >= a.Hx) return;
  const T sy = 2 * ky > L ? T(-1) : T(1);
  V* col = buf + j * a.f.pitch + place[ky];
  if constexpr (PZ == 1) {
    V mx = col[0], my = col[cl], mz = col[2 * cl];
    sym3<T>(mx, my, mz, k.v[0][0], k.v[0][1], k.v[0][2], sy * k.v[0][3], T(0), T(0));
    col[0] = mx;
    col[cl] = my;
    col[2 * cl] = mz;
  } else {
    V v[3][PZ];
#pragma unroll
    for (int z = 0; z < PZ / 2; ++z) {
      const bool in = z < a.nz;
      const int o = in ? z * zl : 0;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const V x = col[c * cl + o];
        v[c][z] = in ? x : cmk<T>(T(0), T(0));
      }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) dft_hz<T, PZ>(v[c]);
    // plane kz and its mirror PZ - kz share their kernel values, the
    // components odd along z with opposite signs
#pragma unroll
    for (int kz = 0; kz <= PZ / 2; ++kz) {
      const T* q = k.v[kz];
      const T kxy = sy * q[3], kyz = sy * q[5];
      sym3<T>(v[0][kz], v[1][kz], v[2][kz], q[0], q[1], q[2], kxy, q[4], kyz);
      if (kz > 0 && 2 * kz < PZ)
        sym3<T>(v[0][PZ - kz], v[1][PZ - kz], v[2][PZ - kz], q[0], q[1], q[2], kxy, -q[4], -kyz);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      dft<T, PZ, true>(v[c]);
#pragma unroll
      for (int z = 0; z < PZ / 2; ++z)
        if (z < a.nz) col[c * cl + z * zl] = v[c][z];
    }
  }
}

// z lengths the fused pass is built for (every pad up to 16 of a grid of
// up to 8 layers; longer columns would not fit a thread's registers beside
// enough waves)
#define MMP_YZ_SMALL(X) X(1) X(4) X(6) X(8)
#define MMP_YZ_LARGE(X) X(10) X(12) X(14) X(16)
#define MMP_YZ_LENGTHS(X) MMP_YZ_SMALL(X) MMP_YZ_LARGE(X)
constexpr int kYzClasses = 2;   // launches of a batch: short, long columns

// The first column's kernel values are asked for with the lines, two
// transforms before their use; blocks whose lines are longer than their
// threads load the later columns' at their turn.  The controller's flags come
// beside the lines, too, not before them.
template <typename T, int PZ>
__device__ __forceinline__ void yz_body(const YzArgs<T>& a, int zero, int bx) {
  using V = cpx<T>;
  const bool stop = ctrl_stopped(a.ctrl, zero);
  extern __shared__ char smem_raw[];
  V* buf = reinterpret_cast<V*>(smem_raw);
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int kx0 = bx * a.nk;
  const int lines = 3 * a.nz * a.nk, ncol = a.nk * a.f.L;
  const V* twl = line_stage_tw<T>(a.f, buf, lines, a.tw, tid, nthr);
  YzKernel<T, PZ> k;
  yz_load_k<T, PZ>(a, kx0, tid < ncol ? tid : 0, k);
  line_fft_fwd<T>(a.f, buf, a.tw, twl, lines, a.half != 0, tid, nthr, [&](int l, int n) -> V {
    const int kx = kx0 + (l & (a.nk - 1));
    const bool in = kx < a.Hx && n < a.ny;
    const V v = a.S1[in ? ((long)(l >> a.lnk) * a.Hx + kx) * a.ldy + n : 0];
    return in ? v : cmk<T>(T(0), T(0));
  });
  if (stop) return;
  for (int idx = tid; idx < ncol; idx += nthr) {
    if (idx != tid) yz_load_k<T, PZ>(a, kx0, idx, k);
    yz_column<T, PZ>(a, buf, line_places(a.f, twl), kx0, idx, k);
  }
  __syncthreads();
  line_fft_inv<T>(a.f, buf, twl, lines, a.half != 0, tid, nthr, [&](int l, int n, V v) {
    const int kx = kx0 + (l & (a.nk - 1));
    if (kx < a.Hx && n < a.ny) a.S1[((long)(l >> a.lnk) * a.Hx + kx) * a.ldy + n] = v;
  });
}

template <typename T, int PZ>
__global__ __launch_bounds__(yz_max_threads((int)sizeof(T), PZ)) void k_yz(YzArgs<T> a) {
  const int zero = warm_args<YzArgs<T>>();
  yz_body<T, PZ>(a, zero, blockIdx.x);
}

// ---------------------------------------------------------------- z pass --
// 3-D grids whose lines do not fit the fused pass: z forward, multiply, z
// inverse for tk ky values of one kx, lines in LDS.
template <typename T>
struct ZArgs {
  const Ctrl* ctrl;
  cpx<T>* S2;     // [3][nz][Hx][Py]
  const T* K;     // [6][Hz][Hx][Hy]
  const cpx<T>* tw;
  int nz, Hx, Py, Hy, Hz, tk, ltk;
  LineFft f;
};

template <typename T>
__device__ __forceinline__ void fftz_mul_body(const ZArgs<T>& a, int zero, int bx, int by) {
  using V = cpx<T>;
  if (ctrl_stopped(a.ctrl, zero)) return;
  extern __shared__ char smem_raw[];
  V* buf = reinterpret_cast<V*>(smem_raw);
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int kx = by, ky0 = bx * a.tk;
  const int L = a.f.L, pitch = a.f.pitch, tk = a.tk;
  const long zstride = (long)a.Hx * a.Py;
  const long cstride = (long)a.nz * zstride;
  V* base = a.S2 + (long)kx * a.Py + ky0;
  const V* twl = line_stage_tw<T>(a.f, buf, 3 * tk, a.tw, tid, nthr);
  // planes in natural order, columns fastest (coalesced along ky)
  for (int c = 0; c < 3; ++c)
    for (int idx = tid; idx < tk * L; idx += nthr) {
      const int j = idx & (tk - 1), z = idx >> a.ltk;
      const bool in = z < a.nz && ky0 + j < a.Py;
      const V v = base[in ? c * cstride + z * zstride + j : 0];
      buf[(c * tk + j) * pitch + z + a.f.drl.div(z) * a.f.pad] = in ? v : cmk<T>(T(0), T(0));
    }
  lds_copies_done();
  __syncthreads();
  line_fft_fwd_lds<T>(a.f, buf, twl, 3 * tk, tid, nthr);
  const long ks = (long)a.Hz * a.Hx * a.Hy;
  for (int idx = tid; idx < tk * L; idx += nthr) {
    const int j = idx & (tk - 1), kz = idx >> a.ltk;
    const int ky = ky0 + j;
    if (ky >= a.Py) continue;
    const int kyo = ky <= a.Py / 2 ? ky : a.Py - ky;
    const T sy = ky <= a.Py / 2 ? T(1) : T(-1);
    const int kzo = kz <= L / 2 ? kz : L - kz;
    const T sz = kz <= L / 2 ? T(1) : T(-1);
    V* p = buf + j * pitch + line_places(a.f, twl)[kz];
    const int cl = tk * pitch;
    const T* K = a.K + ((long)kzo * a.Hx + kx) * a.Hy + kyo;
    V mx = p[0], my = p[cl], mz = p[2 * cl];
    sym3<T>(mx, my, mz, K[0], K[ks], K[2 * ks], sy * K[3 * ks], sz * K[4 * ks],
            sy * sz * K[5 * ks]);
    p[0] = mx;
    p[cl] = my;
    p[2 * cl] = mz;
  }
  __syncthreads();
  line_fft_inv_lds<T>(a.f, buf, twl, 3 * tk, tid, nthr);
  for (int c = 0; c < 3; ++c)
    for (int idx = tid; idx < tk * a.nz; idx += nthr) {
      const int j = idx & (tk - 1), z = idx >> a.ltk;
      if (ky0 + j < a.Py)
        base[c * cstride + z * zstride + j] =
            buf[(c * tk + j) * pitch + z + a.f.drl.div(z) * a.f.pad];
    }
}

template <typename T>
__global__ __launch_bounds__(kLineThreads) void k_fftz_mul(ZArgs<T> a) {
  const int zero = warm_args<ZArgs<T>>();
  fftz_mul_body<T>(a, zero, blockIdx.x, blockIdx.y);
}

// --------------------------------------------------------- batched passes --
// One launch of a pass for many grids: block b runs the pass body of grid
// work[b].x at block coordinates (work[b].y, .z, .w) with that grid's
// arguments.  256 threads per block; the dynamic LDS is the largest any
// grid's block needs.
constexpr int kMultiThreads = 256;

template <typename T>
__global__ __launch_bounds__(kMultiThreads) void k_fftx_fwd_multi(
    const XArgs<T>* __restrict__ args, const int4* __restrict__ work, int src) {
  const int4 w = work[blockIdx.x];
  fftx_fwd_body<T>(args[w.x], warm_lines((const uint32_t*)&args[w.x], (int)sizeof(XArgs<T>)), src, w.y, w.z, w.w);
}

template <typename T>
__global__ __launch_bounds__(kMultiThreads) void k_fftx_inv_multi(
    const XArgs<T>* __restrict__ args, const int4* __restrict__ work) {
  const int4 w = work[blockIdx.x];
  fftx_inv_body<T>(args[w.x], warm_lines((const uint32_t*)&args[w.x], (int)sizeof(XArgs<T>)), w.y, w.z, w.w);
}

template <typename T, bool INV>
__global__ __launch_bounds__(kMultiThreads) void k_ffty_multi(const YArgs<T>* __restrict__ args,
                                                              const int4* __restrict__ work) {
  const int4 w = work[blockIdx.x];
  ffty_body<T, INV>(args[w.x], 0, w.y);
}

template <typename T>
__global__ __launch_bounds__(kMultiThreads) void k_fftz_mul_multi(
    const ZArgs<T>* __restrict__ args, const int4* __restrict__ work) {
  const int4 w = work[blockIdx.x];
  fftz_mul_body<T>(args[w.x], 0, w.y, w.z);
}

// LARGE: the members with z pads of 10..16 (one launch for them and one for
// the others, so that the short columns do not hold the long ones' registers)
template <typename T, bool LARGE>
__global__ __launch_bounds__(kMultiThreads) void k_yz_multi(const YzArgs<T>* __restrict__ args,
                                                            const int4* __restrict__ work) {
  const int4 w = work[blockIdx.x];
  const YzArgs<T>& a = args[w.x];
  const int zero = warm_lines((const uint32_t*)&a, (int)sizeof(YzArgs<T>));
#define X(P) case P: yz_body<T, P>(a, zero, w.y); break;
  if constexpr (LARGE) {
    switch (a.Pz) { MMP_YZ_LARGE(X) }
  } else {
    switch (a.Pz) { MMP_YZ_SMALL(X) }
  }
#undef X
}

// ------------------------------------------------------------------ plan --
constexpr long kMixedTarget = 2048;
constexpr size_t kLdsMax = 65536;   // dynamic LDS of one block of the register z pass

// complex elements one block may hold in LDS (64 KiB before row padding)
static long lds_cap(int real_bytes) { return 65536 / (2 * real_bytes); }

// threads of a block of `lines` mixed-radix line transforms: one butterfly
// of the longest stage each, at most `most`
static int line_threads(const LineFft& f, long lines, int most) {
  int nb = 1;
  for (const LineStage* t : {&f.s0, &f.s1, &f.s2, &f.s3})
    if (t->nb > nb) nb = t->nb;
  const long t = (lines * nb + 63) / 64 * 64;
  return (int)std::min<long>(t, most);
}

// The fused y-z pass takes a 3-D grid when its z length is one it is built
// for and the 3 nz lines of a kx column fit the LDS of a block (128 of the
// 160 KiB of a CU; a block that size still moves a quarter of what the
// separate passes move through memory).  This is the default, not a rule for
// every grid: up to about 90 KiB it wins (steps in one pass / two, default
// shapes, FP32: 128x128x8 195 / 223 us, 200x240x8 357 / 423), from about 100
// KiB, one block per CU, it wins or loses by the number of blocks (FP32
// 256x256x8 463 / 441, 512x512x4 663 / 647; FP64 256x128x8 502 / 436, 128x128x8
// 299 / 299, 1024x256x4 1694 / 1779), which the tuner finds out.
static constexpr long kYzLds = 131072;
static bool yz_built(int Pz) {
  switch (Pz) {
#define X(P) case P: return true;
    MMP_YZ_LENGTHS(X)
#undef X
  }
  return false;
}
static bool yz_fits(int nz, int Pz, const LineFft& fy, int real_bytes) {
  return nz > 1 && Pz > 1 && yz_built(Pz) && (long)line_lds_elems(fy, 3L * nz, 2 * real_bytes) * 2 * real_bytes <= kYzLds;
}

// An open axis is zero-padded to P >= 2n - 1; a periodic one is cyclic
// with P = n.  P is 1 or even and 7-smooth, at most 4096.
static bool pad_ok(int n, int P, bool periodic = false) {
  if (n == 1) return P == 1;
  if (periodic ? P != n : P < 2 * n - 1) return false;
  if ((P & 1) || P > 4096) return false;
  int r[kMaxStages];
  return line_radices(P, r) > 0;
}

// threads of each pass for the plan's shapes
static int x_threads(const DemagPlan& p, int ty) {
  return p.p2x ? (ty / 2) * split_l2(p.Px) : line_threads(p.fx, ty / 2, kLineThreads);
}
static int y_threads(const DemagPlan& p, int nl) {
  return p.p2y ? nl * split_l2(p.Py) : line_threads(p.fy, nl, kLineThreads);
}
static int m2_threads(const DemagPlan& p, int real_bytes) {
  return p.p2y ? 3 * p.nk * split_l2(p.Py)
               : line_threads(p.fy, 3L * p.nk, yz_max_threads(real_bytes, 1));
}
static int z_threads(const DemagPlan& p) { return line_threads(p.fz, 3L * p.tk, kLineThreads); }

static bool pow2_in(int v, int lo, int hi) { return v >= lo && v <= hi && is_pow2(v); }

int demag_plan_check(const DemagPlan& p, int real_bytes) {
  const long cap = lds_cap(real_bytes);
  for (int ty : {p.tyf, p.tyi}) {
    if (!pow2_in(ty, 2, 16) || (long)(ty / 2) * p.Px > cap) return -1;
    if (p.p2x && x_threads(p, ty) > 256) return -1;
  }
  if (p.nz == 1) {
    if (!pow2_in(p.nk, 1, 64) || (long)3 * p.nk * p.Py > cap) return -1;
    if (p.p2y && m2_threads(p, real_bytes) > 256) return -1;
  } else {
    for (int nl : {p.nlyf, p.nlyi}) {
      if (!pow2_in(nl, 1, 64) || (long)nl * p.Py > cap) return -1;
      if (p.p2y && y_threads(p, nl) > 256) return -1;
    }
    if (p.p2z) {
      if (!zreg_waves_ok(real_bytes, p.Pz, p.zq, p.zw)) return -1;
      if (p.zt != 64 && p.zt != 128 && p.zt != 256) return -1;
      if (p.zmode < 0 || p.zmode > 1) return -1;
      if (p.zmode == 1 &&
          (real_bytes != 4 || p.zw != 1 || zk_lds_bytes(p.Pz, p.zq, p.zt) > (long)kLdsMax))
        return -1;
    } else {
      if (!pow2_in(p.tk, 1, 64) || (long)3 * p.tk * (p.Pz + 1) > cap) return -1;
    }
  }
  return 0;
}

int demag_plan(int nx, int ny, int nz, int real_bytes, const int* pads, DemagPlan* p,
               const int* rep) {
  DemagPlan d;
  d.nx = nx; d.ny = ny; d.nz = nz;
  if (rep)
    for (int a = 0; a < 3; ++a) d.rep[a] = rep[a];
  if (d.rep[2] != 0) return -1;
  const bool px = d.rep[0] > 0, py = d.rep[1] > 0;
  if (pads) {
    if (!pad_ok(nx, pads[0], px) || !pad_ok(ny, pads[1], py) || !pad_ok(nz, pads[2])) return -1;
    d.Px = pads[0]; d.Py = pads[1]; d.Pz = pads[2];
  } else {
    d.Px = px ? nx : smooth_pad(nx);
    d.Py = py ? ny : smooth_pad(ny);
    d.Pz = smooth_pad(nz);
    if (!pad_ok(nx, d.Px, px) || !pad_ok(ny, d.Py, py) || !pad_ok(nz, d.Pz)) return -1;
  }
  d.Hx = d.Px / 2 + 1; d.Hy = d.Py / 2 + 1; d.Hz = d.Pz / 2 + 1;
  if (!make_line_fft(d.Px, &d.fx) || !make_line_fft(d.Py, &d.fy) || !make_line_fft(d.Pz, &d.fz))
    return -1;
  // power-of-two axes: register four-step kernels (FP64 lines up to 2048
  // points); the register z pass spreads a column over zq lanes
  const int lmax = real_bytes == 8 ? 2048 : 4096;
  d.p2x = is_pow2(d.Px) && d.Px <= lmax;
  d.p2y = is_pow2(d.Py) && d.Py <= lmax;
  d.p2z = is_pow2(d.Pz) && d.Pz <= 64;
  d.ldy = round_up(ny, 16);
  const long cap = lds_cap(real_bytes);
  // the mixed-radix LDS passes are latency-bound: at most kMixedTarget
  // complex elements per block, so that even small grids launch many
  // blocks (the power-of-two register passes take as many as fit)
  const long mcap = std::min<long>(cap, kMixedTarget);
  // x passes: the most rows per block that the LDS, the block size and the
  // grid (no more rows than it has) allow
  int ty = 2;
  const long xcap = d.p2x ? cap : mcap;
  while (ty < 16 && (long)ty * d.Px <= xcap && ty < ny + (ny & 1)) ty *= 2;
  while (ty > 2 && ((long)(ty / 2) * d.Px > cap || (d.p2x && x_threads(d, ty) > 256)))
    ty /= 2;
  d.tyf = d.tyi = ty;
  // y passes: lines per block
  {
    int n = 1;
    if (d.p2y) {
      // one wavefront per block: its lines wait at no barrier for another's
      // (1024-point lines, 2 per block instead of 4, forward and inverse:
      // FP32 56.2 -> 54.2 and 70.6 -> 67.0 us, FP64 113 -> 109 and 135 ->
      // 129 us on a 512x512x16 film; 128 to 512 points: within 4 %)
      const int l2 = split_l2(d.Py);
      while (n < 64 && (long)(2 * n) * d.Py <= cap && 2 * n * l2 <= 64) n *= 2;
    } else {
      while (n < 8 && (long)(2 * n) * d.Py <= mcap) n *= 2;
    }
    d.nlyf = d.nlyi = n;
  }
  // 2-D fused pass: kx columns per block
  {
    int k = 1;
    if (d.p2y) {
      const int l2 = split_l2(d.Py);
      while (k < 64 && (long)3 * (2 * k) * d.Py <= cap && 3 * (2 * k) * l2 <= 256) k *= 2;
    } else {
      while (k < 64 && (long)3 * (2 * k) * d.Py <= mcap) k *= 2;
    }
    d.nk = k;
  }
  // z pass: mixed-radix ky per block; register lanes per column
  {
    int tk = 64;
    while (tk > 1 && (long)3 * tk * (d.Pz + 1) > mcap) tk /= 2;
    d.tk = tk;
    // FP32 columns of up to 32 points: one lane per column, two waves per
    // SIMD (the column's 192 registers and the transform's temporaries fit
    // the 256 of a wave); otherwise the fewest lanes whose share of a
    // column takes at most 96 registers, one wave's worth of the rest
    int q = 1, w = 1;
    if (real_bytes == 4 && zreg_waves_ok(real_bytes, d.Pz, 1, 2)) {
      w = 2;
    } else {
      while (q < 4 &&
             (!zreg_ok(real_bytes, d.Pz, q) || zreg_data_vgprs(real_bytes, d.Pz, q) > 96))
        q *= 2;
      if (!zreg_ok(real_bytes, d.Pz, q)) q = 1;
    }
    d.zq = q;
    d.zw = w;
    d.zt = 128;
    if (d.p2z && !zreg_ok(real_bytes, d.Pz, d.zq)) d.p2z = false;
  }
  d.s1_elems = (size_t)3 * nz * d.Hx * d.ldy;
  d.fuse = yz_fits(nz, d.Pz, d.fy, real_bytes);
  d.s2_elems = nz > 1 && !d.fuse ? (size_t)3 * nz * d.Hx * d.Py : 0;
  d.k_elems = (size_t)6 * d.Hz * d.Hx * d.Hy;
  if (demag_plan_check(d, real_bytes) != 0) return -1;
  *p = d;
  return 0;
}

void demag_plan_separate(DemagPlan* p) {
  p->fuse = false;
  p->nk = 0;
  p->s2_elems = (size_t)3 * p->nz * p->Hx * p->Py;
}

// --------------------------------------------------------------- passes --
static int log2i(int v) {
  int l = 0;
  while ((1 << l) < v) ++l;
  return l;
}

// argument blocks of the mixed-radix passes
template <typename T>
static XArgs<T> x_args(const DemagPlan& p, const DemagBufs<T>& b, const Table<T>* tbl, int stage,
                       const Ctrl* ctrl, T ms0, T ms1, T ms2, int nsub, int ty) {
  XArgs<T> a{};
  a.tbl = tbl; a.ctrl = ctrl; a.src = slot_in(stage, b.ns);
  a.ms0 = ms0; a.ms1 = ms1; a.ms2 = ms2; a.nsub = nsub;
  a.S1 = b.S1; a.Bd = b.Bd; a.tw = b.twx;
  a.nx = p.nx; a.ny = p.ny; a.nz = p.nz; a.Hx = p.Hx; a.ldy = p.ldy;
  a.ty = ty; a.lnl = log2i(ty / 2); a.half = p.rep[0] > 0 || p.Px == 1 ? 0 : 1; a.f = p.fx;
  return a;
}

template <typename T>
static YzArgs<T> yz_args(const DemagPlan& p, const DemagBufs<T>& b, const Ctrl* ctrl, int nk) {
  YzArgs<T> a{};
  a.ctrl = ctrl; a.S1 = b.S1; a.K = b.K; a.tw = b.twy;
  a.ny = p.ny; a.nz = p.nz; a.Pz = p.Pz; a.Hx = p.Hx; a.Hy = p.Hy; a.Hz = p.Hz; a.ldy = p.ldy;
  a.nk = nk; a.lnk = log2i(nk); a.half = p.rep[1] > 0 || p.Py == 1 ? 0 : 1;
  a.dL = make_div(p.Py); a.f = p.fy;
  return a;
}

template <typename T>
static ZArgs<T> z_args(const DemagPlan& p, const DemagBufs<T>& b, const Ctrl* ctrl, int tk) {
  ZArgs<T> a{};
  a.ctrl = ctrl; a.S2 = b.S2; a.K = b.K; a.tw = b.twz;
  a.nz = p.nz; a.Hx = p.Hx; a.Py = p.Py; a.Hy = p.Hy; a.Hz = p.Hz;
  a.tk = tk; a.ltk = log2i(tk); a.f = p.fz;
  return a;
}

template <typename T>
void demag_pass(int pass, const DemagPlan& p, const DemagBufs<T>& b, const Table<T>* tbl,
                int stage, const Ctrl* ctrl, T ms0, T ms1, int nsub, hipStream_t st, T ms2) {
  using V = cpx<T>;
  switch (pass) {
    case DP_XF:
    case DP_XI: {
      const bool inv = pass == DP_XI;
      const int ty = inv ? p.tyi : p.tyf;
      const dim3 g((p.ny + ty - 1) / ty, p.nz, 3);
      if (p.p2x) {
        const size_t lds4 = x4_lds_bytes(p.Px, ty / 2, inv, (int)sizeof(V));
        X4Args<T> a;
        a.tbl = tbl; a.ctrl = ctrl; a.src = slot_in(stage, b.ns); a.ms0 = ms0; a.ms1 = ms1; a.nsub = nsub;
        a.ms2 = ms2;
        a.S1 = b.S1; a.Bd = b.Bd; a.tw4 = b.tw4x;
        a.nx = p.nx; a.ny = p.ny; a.nz = p.nz; a.Hx = p.Hx; a.ldy = p.ldy; a.ty = ty;
        a.lnl = 0;
        while ((2 << a.lnl) < ty) ++a.lnl;
        launch_x4<T>(p.Px, inv, p.rep[0] > 0, g, x_threads(p, ty), lds4, st, a);
      } else {
        const XArgs<T> a = x_args<T>(p, b, tbl, stage, ctrl, ms0, ms1, ms2, nsub, ty);
        const dim3 blk(x_threads(p, ty));
        const size_t lds = line_lds_elems(p.fx, ty / 2, sizeof(V)) * sizeof(V);
        if (inv) hipLaunchKernelGGL((k_fftx_inv<T>), g, blk, lds, st, a);
        else hipLaunchKernelGGL((k_fftx_fwd<T>), g, blk, lds, st, a);
      }
      break;
    }
    case DP_M2: {
      const size_t lds = (size_t)3 * p.nk * p.Py * sizeof(V);
      const dim3 g((p.Hx + p.nk - 1) / p.nk);
      if (p.p2y) {
        M4Args<T> a;
        a.ctrl = ctrl; a.S1 = b.S1; a.K = b.K; a.tw4 = b.tw4y;
        a.ny = p.ny; a.Hx = p.Hx; a.Hy = p.Hy; a.ldy = p.ldy; a.nk = p.nk;
        launch_m4<T>(p.Py, p.rep[1] > 0, g, m2_threads(p, (int)sizeof(T)), lds, st, a);
      } else {
        hipLaunchKernelGGL((k_yz<T, 1>), g, dim3(m2_threads(p, (int)sizeof(T))),
                           line_lds_elems(p.fy, 3L * p.nk, sizeof(V)) * sizeof(V), st,
                           yz_args<T>(p, b, ctrl, p.nk));
      }
      break;
    }
    case DP_YZ: {
      const dim3 g(p.Hx);
      const dim3 blk(line_threads(p.fy, 3L * p.nz, yz_max_threads((int)sizeof(T), p.Pz)));
      const size_t lds = line_lds_elems(p.fy, 3L * p.nz, sizeof(V)) * sizeof(V);
      const YzArgs<T> a = yz_args<T>(p, b, ctrl, 1);
      switch (p.Pz) {
#define X(P) case P: hipLaunchKernelGGL((k_yz<T, P>), g, blk, lds, st, a); break;
        MMP_YZ_LENGTHS(X)
#undef X
      }
      break;
    }
    case DP_YF:
    case DP_YI: {
      const bool inv = pass == DP_YI;
      const int nl = inv ? p.nlyi : p.nlyf;
      const int nlines = 3 * p.nz * p.Hx;
      const dim3 g((nlines + nl - 1) / nl);
      const size_t lds = (size_t)nl * p.Py * sizeof(V);
      const cpx<T>* in = inv ? b.S2 : b.S1;
      cpx<T>* out = inv ? b.S1 : b.S2;
      const int nvi = inv ? p.Py : p.ny, ldi = inv ? p.Py : p.ldy;
      const int nvo = inv ? p.ny : p.Py, ldo = inv ? p.ldy : p.Py;
      if (p.p2y) {
        Y4Args<T> a;
        a.ctrl = ctrl; a.in = in; a.out = out; a.tw4 = b.tw4y;
        a.nlines = nlines; a.nvalid_in = nvi; a.ld_in = ldi; a.nvalid_out = nvo; a.ld_out = ldo;
        a.nl = nl;
        launch_y4<T>(p.Py, inv, p.rep[1] > 0, g, y_threads(p, nl), lds, st, a);
      } else {
        YArgs<T> a{};
        a.ctrl = ctrl; a.in = in; a.out = out; a.tw = b.twy;
        a.nlines = nlines; a.nvalid_in = nvi; a.ld_in = ldi; a.nvalid_out = nvo; a.ld_out = ldo;
        a.nl = nl; a.half = p.rep[1] > 0 || p.Py == 1 ? 0 : 1; a.dL = make_div(p.Py); a.f = p.fy;
        const dim3 blk(y_threads(p, nl));
        const size_t ldm = line_lds_elems(p.fy, nl, sizeof(V)) * sizeof(V);
        if (inv) hipLaunchKernelGGL((k_ffty<T, true>), g, blk, ldm, st, a);
        else hipLaunchKernelGGL((k_ffty<T, false>), g, blk, ldm, st, a);
      }
      break;
    }
    case DP_Z: {
      if (p.p2z) {
        Z4Args<T> a;
        a.ctrl = ctrl; a.S2 = b.S2; a.K = b.K;
        a.nz = p.nz; a.Hx = p.Hx; a.Py = p.Py; a.Hy = p.Hy; a.Hz = p.Hz; a.tk = p.zt;
        const int cpb = p.zt / p.zq;
        const int nblk = ((p.Py + cpb - 1) / cpb) * p.Hx;
        a.nb_pad = round_up(nblk, 8);
        launch_z4<T>(p.Pz, p.zq, p.zw, p.zmode, dim3(a.nb_pad), p.zt, st, a);
      } else {
        const dim3 g((p.Py + p.tk - 1) / p.tk, p.Hx), blk(z_threads(p));
        hipLaunchKernelGGL((k_fftz_mul<T>), g, blk, line_lds_elems(p.fz, 3L * p.tk, sizeof(V)) * sizeof(V), st,
                           z_args<T>(p, b, ctrl, p.tk));
      }
      break;
    }
  }
}

// ------------------------------------------------------ batched driver --
template <typename T>
struct DemagMulti<T>::Impl {
  // host copies (kept until the next build) and one device allocation
  std::vector<XArgs<T>> xf;
  std::vector<YArgs<T>> yf, yi;
  std::vector<ZArgs<T>> z;
  std::vector<YzArgs<T>> yz;
  std::vector<int4> wxf, wxi, wyf, wyi, wz, wyz[kYzClasses];
  const XArgs<T>* d_xf = nullptr;
  const XArgs<T>* d_xi = nullptr;
  const YArgs<T>* d_yf = nullptr;
  const YArgs<T>* d_yi = nullptr;
  const ZArgs<T>* d_z = nullptr;
  const YzArgs<T>* d_yz = nullptr;
  const int4 *d_wxf = nullptr, *d_wxi = nullptr, *d_wyf = nullptr, *d_wyi = nullptr,
             *d_wz = nullptr, *d_wyz[kYzClasses] = {};
  size_t lds_x = 0, lds_y = 0, lds_z = 0, lds_yz[kYzClasses] = {};
};

template <typename T>
void DemagMulti<T>::release() {
  if (mem_) {
    DeviceLock lk(device_mutex());
    (void)hipFree(mem_);
  }
  mem_ = nullptr;
  cap_ = 0;
  delete impl;
  impl = nullptr;
}

// largest power of two <= cap (>= 1), at most hi
static int pow2_floor(long cap, int hi) {
  int v = 1;
  while (v < hi && 2L * v <= cap) v *= 2;
  return v;
}

bool demag_multi_fits(const DemagPlan& p) {
  // a block takes at least one line
  const long cap = kMultiElems;
  if (p.Px > cap || p.Py > cap) return false;
  if (p.nz == 1) return 3L * p.Py <= cap;
  return 3L * p.Pz <= cap;
}

template <typename T>
int DemagMulti<T>::build(const std::vector<DemagMember<T>>& members, hipStream_t st) {
  using V = cpx<T>;
  delete impl;
  impl = nullptr;
  if (members.empty()) return 0;
  for (const auto& mb : members)
    if (!demag_multi_fits(*mb.plan)) {
      set_error("batched demag: a pad is too long for one block's lines");
      return MMP_E_ARG;
    }
  impl = new Impl();
  Impl& I = *impl;
  const long cap = kMultiElems;   // complex elements per block
  for (size_t g = 0; g < members.size(); ++g) {
    const DemagMember<T>& mb = members[g];
    const DemagPlan& p = *mb.plan;
    const int gi = (int)g;
    // x passes: the most rows per block (<= 16) that fit
    int ty = 2;
    while (ty < 16 && (long)ty * p.Px <= cap && ty < p.ny + (p.ny & 1)) ty *= 2;
    I.xf.push_back(x_args<T>(p, mb.bufs, mb.tbl, 0, mb.ctrl, mb.ms0, mb.ms1, mb.ms2, mb.nsub, ty));
    for (int c = 0; c < 3; ++c)
      for (int z = 0; z < p.nz; ++z)
        for (int b = 0; b < (p.ny + ty - 1) / ty; ++b) {
          I.wxf.push_back(make_int4(gi, b, z, c));
          I.wxi.push_back(make_int4(gi, b, z, c));
        }
    I.lds_x = std::max(I.lds_x, line_lds_elems(p.fx, ty / 2, sizeof(V)) * sizeof(V));
    if (p.nz == 1 || p.fuse) {
      const int nk = p.fuse ? 1 : pow2_floor(cap / (3L * p.Py), 64);
      I.yz.push_back(yz_args<T>(p, mb.bufs, mb.ctrl, nk));
      const int idx = (int)I.yz.size() - 1, cls = p.Pz >= 10 ? 1 : 0;
      for (int b = 0; b < (p.Hx + nk - 1) / nk; ++b)
        I.wyz[cls].push_back(make_int4(idx, b, 0, 0));
      I.lds_yz[cls] =
          std::max(I.lds_yz[cls], line_lds_elems(p.fy, 3L * p.nz * nk, sizeof(V)) * sizeof(V));
    } else {
      const int nl = pow2_floor(cap / p.Py, 64);
      const int nlines = 3 * p.nz * p.Hx;
      YArgs<T> a{};
      a.ctrl = mb.ctrl; a.tw = mb.bufs.twy; a.nlines = nlines; a.nl = nl;
      a.half = p.rep[1] > 0 || p.Py == 1 ? 0 : 1; a.dL = make_div(p.Py); a.f = p.fy;
      YArgs<T> f = a, i = a;
      f.in = mb.bufs.S1; f.out = mb.bufs.S2;
      f.nvalid_in = p.ny; f.ld_in = p.ldy; f.nvalid_out = p.Py; f.ld_out = p.Py;
      i.in = mb.bufs.S2; i.out = mb.bufs.S1;
      i.nvalid_in = p.Py; i.ld_in = p.Py; i.nvalid_out = p.ny; i.ld_out = p.ldy;
      I.yf.push_back(f);
      I.yi.push_back(i);
      const int idx = (int)I.yf.size() - 1;
      for (int b = 0; b < (nlines + nl - 1) / nl; ++b) {
        I.wyf.push_back(make_int4(idx, b, 0, 0));
        I.wyi.push_back(make_int4(idx, b, 0, 0));
      }
      I.lds_y = std::max(I.lds_y, line_lds_elems(p.fy, nl, sizeof(V)) * sizeof(V));
      const int tk = pow2_floor(cap / (3L * p.Pz), 64);
      I.z.push_back(z_args<T>(p, mb.bufs, mb.ctrl, tk));
      const int zi = (int)I.z.size() - 1;
      for (int kx = 0; kx < p.Hx; ++kx)
        for (int b = 0; b < (p.Py + tk - 1) / tk; ++b) I.wz.push_back(make_int4(zi, b, kx, 0));
      I.lds_z = std::max(I.lds_z, line_lds_elems(p.fz, 3L * tk, sizeof(V)) * sizeof(V));
    }
  }
  // one device allocation, 256-byte aligned segments
  size_t off = 0;
  auto seg = [&](size_t bytes) {
    const size_t o = off;
    off += (bytes + 255) / 256 * 256;
    return o;
  };
  const size_t o_xf = seg(I.xf.size() * sizeof(XArgs<T>));
  const size_t o_yf = seg(I.yf.size() * sizeof(YArgs<T>));
  const size_t o_yi = seg(I.yi.size() * sizeof(YArgs<T>));
  const size_t o_z = seg(I.z.size() * sizeof(ZArgs<T>));
  const size_t o_yz = seg(I.yz.size() * sizeof(YzArgs<T>));
  const size_t o_wxf = seg(I.wxf.size() * sizeof(int4));
  const size_t o_wxi = seg(I.wxi.size() * sizeof(int4));
  const size_t o_wyf = seg(I.wyf.size() * sizeof(int4));
  const size_t o_wyi = seg(I.wyi.size() * sizeof(int4));
  const size_t o_wz = seg(I.wz.size() * sizeof(int4));
  size_t o_wyz[kYzClasses];
  for (int i = 0; i < kYzClasses; ++i) o_wyz[i] = seg(I.wyz[i].size() * sizeof(int4));
  // the block only grows: freeing it waits for every stream of the device
  if (off > cap_) {
    DeviceLock lk(device_mutex());
    if (mem_) (void)hipFree(mem_);
    mem_ = nullptr;
    cap_ = 0;
    if (!device_alloc(&mem_, 2 * off)) {
      release();
      set_error("device allocation failed (batched demag tables)");
      return MMP_E_NOMEM;
    }
    cap_ = 2 * off;
  }
  auto put = [&](size_t o, const void* src, size_t bytes) {
    return bytes ? hipMemcpyAsync(mem_ + o, src, bytes, hipMemcpyHostToDevice, st) : hipSuccess;
  };
  hipError_t e = hipSuccess;
  for (auto r : {put(o_xf, I.xf.data(), I.xf.size() * sizeof(XArgs<T>)),
                 put(o_yf, I.yf.data(), I.yf.size() * sizeof(YArgs<T>)),
                 put(o_yi, I.yi.data(), I.yi.size() * sizeof(YArgs<T>)),
                 put(o_z, I.z.data(), I.z.size() * sizeof(ZArgs<T>)),
                 put(o_yz, I.yz.data(), I.yz.size() * sizeof(YzArgs<T>)),
                 put(o_wxf, I.wxf.data(), I.wxf.size() * sizeof(int4)),
                 put(o_wxi, I.wxi.data(), I.wxi.size() * sizeof(int4)),
                 put(o_wyf, I.wyf.data(), I.wyf.size() * sizeof(int4)),
                 put(o_wyi, I.wyi.data(), I.wyi.size() * sizeof(int4)),
                 put(o_wz, I.wz.data(), I.wz.size() * sizeof(int4))})
    if (r != hipSuccess) e = r;
  for (int i = 0; i < kYzClasses; ++i) {
    const hipError_t r = put(o_wyz[i], I.wyz[i].data(), I.wyz[i].size() * sizeof(int4));
    if (r != hipSuccess) e = r;
  }
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) {
    release();
    set_error(std::string("batched demag tables: ") + hipGetErrorString(e));
    return MMP_E_HIP;
  }
  // the x inverse pass reads the same arguments as the forward one
  I.d_xf = reinterpret_cast<const XArgs<T>*>(mem_ + o_xf);
  I.d_xi = I.d_xf;
  I.d_yf = reinterpret_cast<const YArgs<T>*>(mem_ + o_yf);
  I.d_yi = reinterpret_cast<const YArgs<T>*>(mem_ + o_yi);
  I.d_z = reinterpret_cast<const ZArgs<T>*>(mem_ + o_z);
  I.d_yz = reinterpret_cast<const YzArgs<T>*>(mem_ + o_yz);
  I.d_wxf = reinterpret_cast<const int4*>(mem_ + o_wxf);
  I.d_wxi = reinterpret_cast<const int4*>(mem_ + o_wxi);
  I.d_wyf = reinterpret_cast<const int4*>(mem_ + o_wyf);
  I.d_wyi = reinterpret_cast<const int4*>(mem_ + o_wyi);
  I.d_wz = reinterpret_cast<const int4*>(mem_ + o_wz);
  for (int i = 0; i < kYzClasses; ++i)
    I.d_wyz[i] = reinterpret_cast<const int4*>(mem_ + o_wyz[i]);
  return 0;
}

template <typename T>
void DemagMulti<T>::launch(int stage, hipStream_t st) const {
  if (!impl) return;
  const Impl& I = *impl;
  const dim3 b(kMultiThreads);
  hipLaunchKernelGGL((k_fftx_fwd_multi<T>), dim3((unsigned)I.wxf.size()), b, I.lds_x, st, I.d_xf,
                     I.d_wxf, slot_in(stage, RK::t[RK_DP45].ns));
  if (!I.wyz[0].empty())
    hipLaunchKernelGGL((k_yz_multi<T, false>), dim3((unsigned)I.wyz[0].size()), b, I.lds_yz[0], st,
                       I.d_yz, I.d_wyz[0]);
  if (!I.wyz[1].empty())
    hipLaunchKernelGGL((k_yz_multi<T, true>), dim3((unsigned)I.wyz[1].size()), b, I.lds_yz[1], st,
                       I.d_yz, I.d_wyz[1]);
  if (!I.wyf.empty()) {
    hipLaunchKernelGGL((k_ffty_multi<T, false>), dim3((unsigned)I.wyf.size()), b, I.lds_y, st,
                       I.d_yf, I.d_wyf);
    hipLaunchKernelGGL((k_fftz_mul_multi<T>), dim3((unsigned)I.wz.size()), b, I.lds_z, st, I.d_z,
                       I.d_wz);
    hipLaunchKernelGGL((k_ffty_multi<T, true>), dim3((unsigned)I.wyi.size()), b, I.lds_y, st,
                       I.d_yi, I.d_wyi);
  }
  hipLaunchKernelGGL((k_fftx_inv_multi<T>), dim3((unsigned)I.wxi.size()), b, I.lds_x, st, I.d_xi,
                     I.d_wxi);
}

template class DemagMulti<float>;
template class DemagMulti<double>;

static const int kPassProf[DP_COUNT] = {P_FFTX_FWD, P_FFTY_FWD, P_FFTZ_MUL,  P_FFTY_INV,
                                        P_FFTX_INV, P_FFTY_MUL2D, P_FFTZ_MUL};

static int demag_passes(const DemagPlan& p, int* out) {
  int n = 0;
  out[n++] = DP_XF;
  if (p.nz == 1) {
    out[n++] = DP_M2;
  } else if (p.fuse) {
    out[n++] = DP_YZ;
  } else {
    out[n++] = DP_YF;
    out[n++] = DP_Z;
    out[n++] = DP_YI;
  }
  out[n++] = DP_XI;
  return n;
}

// --------------------------------------------------------------- driver --
template <typename T>
void demag_field(const DemagPlan& p, const DemagBufs<T>& b, const Table<T>* tbl, int stage,
                 const Ctrl* ctrl, T ms0, T ms1, int nsub, hipStream_t st, Prof* prof, T ms2) {
  int passes[DP_COUNT];
  const int n = demag_passes(p, passes);
  for (int i = 0; i < n; ++i) {
    ProfScope ps(prof, kPassProf[passes[i]], st);
    demag_pass<T>(passes[i], p, b, tbl, stage, ctrl, ms0, ms1, nsub, st, ms2);
  }
}

// ------------------------------------------------------------ autotuner --
// Mean time of `reps` launches of the passes in seq[0..ns) after one warm-up
// launch of the last; negative when a launch fails. The tuner times each
// candidate of a pass right after the pass before it in an evaluation, so the
// candidate meets the caches as it does there (the pair's time ranks the
// candidates as their own would), and the first pass's in whole evaluations.
template <typename T>
static double time_passes(const int* seq, int ns, const DemagPlan& p, const DemagBufs<T>& b,
                          const Table<T>* tbl, T ms0, T ms1, int nsub, hipStream_t st, int reps,
                          T ms2) {
  hipEvent_t e0, e1;
  if (hipEventCreate(&e0) != hipSuccess) return -1.0;
  if (hipEventCreate(&e1) != hipSuccess) {
    (void)hipEventDestroy(e0);
    return -1.0;
  }
  double ms = -1.0;
  demag_pass<T>(seq[ns - 1], p, b, tbl, 1, nullptr, ms0, ms1, nsub, st, ms2);
  if (hipGetLastError() == hipSuccess && hipEventRecord(e0, st) == hipSuccess) {
    for (int r = 0; r < reps; ++r)
      for (int j = 0; j < ns; ++j) demag_pass<T>(seq[j], p, b, tbl, 1, nullptr, ms0, ms1, nsub, st, ms2);
    float f = 0.f;
    if (hipGetLastError() == hipSuccess && hipEventRecord(e1, st) == hipSuccess &&
        hipEventSynchronize(e1) == hipSuccess && hipEventElapsedTime(&f, e0, e1) == hipSuccess)
      ms = (double)f / reps;
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  return ms;
}

template <typename T>
double demag_tune(DemagPlan* pp, const DemagBufs<T>& b, const Table<T>* tbl, T ms0, T ms1,
                  int nsub, hipStream_t st, T ms2, double give_up) {
  constexpr int rb = (int)sizeof(T);
  DemagPlan best = *pp;
  int passes[DP_COUNT];
  const int n = demag_passes(best, passes);
  // launches per timing: enough to average out launch jitter on small grids
  // and run-to-run spread of a few percent on large ones
  const long work = (long)best.Hx * best.Py * best.Pz;
  const int reps = work >= (1L << 22) ? 8 : work >= (1L << 16) ? 10 : 30;
  if (give_up > 0.0) {
    const double t = time_passes<T>(passes, n, best, b, tbl, ms0, ms1, nsub, st, reps, ms2);
    if (t < 0.0 || t > give_up) return t;
  }
  for (int i = 0; i < n; ++i) {
    const int pass = passes[i];
    std::vector<DemagPlan> cand;
    auto add = [&](DemagPlan c) {
      if (demag_plan_check(c, rb) == 0) cand.push_back(c);
    };
    switch (pass) {
      case DP_XF:
      case DP_XI:
        for (int ty = 2; ty <= 16; ty *= 2) {
          DemagPlan c = best;
          (pass == DP_XF ? c.tyf : c.tyi) = ty;
          add(c);
        }
        break;
      case DP_YF:
      case DP_YI:
        for (int nl = 1; nl <= 64; nl *= 2) {
          DemagPlan c = best;
          (pass == DP_YF ? c.nlyf : c.nlyi) = nl;
          add(c);
        }
        break;
      case DP_M2:
        for (int k = 1; k <= 64; k *= 2) {
          DemagPlan c = best;
          c.nk = k;
          add(c);
        }
        break;
      case DP_YZ:   // one shape
        add(best);
        break;
      case DP_Z:
        if (best.p2z) {
          for (int q = 1; q <= 4; q *= 2)
            for (int w = 1; w <= 4; w *= 2)
              for (int t = 64; t <= 256; t *= 2)
                for (int k = 0; k <= 1; ++k) {
                  DemagPlan c = best;
                  c.zq = q; c.zw = w; c.zt = t; c.zmode = k;
                  add(c);
                }
        } else {
          for (int tk = 1; tk <= 64; tk *= 2) {
            DemagPlan c = best;
            c.tk = tk;
            add(c);
          }
        }
        break;
    }
    double bt = -1.0;
    for (const DemagPlan& c : cand) {
      // the x forward pass by whole evaluations: what its narrower stores (8
      // rows are half a line of S1 in FP32) cost shows under the y and z
      // passes' traffic only (512x512x16 FP32: 8 and 16 rows tie after the x
      // inverse pass, and take 47 and 36 us in a step)
      const int pair[2] = {passes[i > 0 ? i - 1 : n - 1], pass};
      const double t = pass == DP_XF
                           ? time_passes<T>(passes, n, c, b, tbl, ms0, ms1, nsub, st, reps, ms2)
                           : time_passes<T>(pair, n > 1 ? 2 : 1, c, b, tbl, ms0, ms1, nsub, st,
                                            reps, ms2);
      if (t < 0.0) continue;
      if (bt < 0.0 || t < bt) {
        bt = t;
        best = c;
      }
    }
    if (bt < 0.0) return -1.0;
  }
  // the reported estimate: one whole evaluation with the chosen plan
  const double total = time_passes<T>(passes, n, best, b, tbl, ms0, ms1, nsub, st, reps, ms2);
  if (total < 0.0) return -1.0;
  *pp = best;
  return total;
}

#define INST(T)                                                                                 \
  template void demag_field<T>(const DemagPlan&, const DemagBufs<T>&, const Table<T>*, int,      \
                               const Ctrl*, T, T, int, hipStream_t, Prof*, T);                  \
  template void demag_pass<T>(int, const DemagPlan&, const DemagBufs<T>&, const Table<T>*, int,  \
                              const Ctrl*, T, T, int, hipStream_t, T);                          \
  template double demag_tune<T>(DemagPlan*, const DemagBufs<T>&, const Table<T>*, T, T, int,    \
                                hipStream_t, T, double);
INST(float)
INST(double)
#undef INST

}  // namespace mmp
