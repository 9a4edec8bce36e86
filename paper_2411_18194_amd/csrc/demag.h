// Demagnetising-field convolution on the GPU: plan, buffers, launchers.
#pragma once

#include <vector>

#include "common.h"
#include "fft_lines.h"
#include "prof.h"

namespace mmp {

// Geometry of the padded convolution.  Spectra are stored with the y axis
// contiguous:  S1[c][z][kx][y] (y < ny, line stride ldy)  after the x pass,
// S2[c][z][kx][ky] (ky < Py) after the forward y pass (3-D grids only).
// The kernel spectrum is real and stored on one octant:
// K[comp][kz <= Pz/2][kx < Hx][ky <= Py/2], comp = xx, yy, zz, xy, xz, yz.
//
// The pads and the launch shapes below are the tunable part of the plan;
// every valid choice computes the same convolution (the launch shapes only
// regroup identical per-line transforms, except zq, which changes the
// factorisation of the z transform).
struct DemagPlan {
  int nx = 0, ny = 0, nz = 0;
  int Px = 0, Py = 0, Pz = 0, Hx = 0, Hy = 0, Hz = 0;
  int ldy = 0;                      // multiple of 16, so any x block shape fits
  LineFft fx{}, fy{}, fz{};         // mixed-radix line transforms of the axes
  // 3-D grids: y, z and multiply as one pass over the layers of a kx column
  // in LDS (see yz_fits); S2 is then not used.  The default wherever it fits;
  // nk = 0 stands for the separate passes there (demag_plan_separate)
  bool fuse = false;
  // power-of-two axes use the register four-step kernels
  bool p2x = false, p2y = false, p2z = false;
  // launch shapes
  int tyf = 0, tyi = 0;             // x passes: rows (even, <= 16) per block, fwd / inv
  int nlyf = 0, nlyi = 0;           // y passes: lines per block, fwd / inv
  int nk = 0;                       // 2-D fused y pass: kx columns per block (3-D: see fuse)
  int tk = 0;                       // mixed-radix z pass: ky columns per block
  int zq = 1, zw = 1, zt = 0;       // register z pass: lanes per column, waves hint, threads
  int zmode = 0;                    // register z pass: 1 = kernel values staged through LDS
  // image repetitions per axis; > 0 makes the axis periodic (x and y only):
  // P = n, no zero padding, the kernel summed over the images
  int rep[3] = {0, 0, 0};
  // axes (bits 0/1/2 = x/y/z) forced onto the mixed-radix LDS kernels
  // although their pads are powers of two
  int force_lds = 0;
  size_t s1_elems = 0, s2_elems = 0, k_elems = 0;
};

// Plan with the default launch shapes for the given pads (nullptr: the
// smallest even 7-smooth pads, n on a periodic axis) and image repetitions
// rep (nullptr: open boundaries).  Returns 0, or -1 for an unsupported pad.
int demag_plan(int nx, int ny, int nz, int real_bytes, const int* pads, DemagPlan* p,
               const int* rep = nullptr);
// The same pads with y and z as separate passes.
void demag_plan_separate(DemagPlan* p);
// 0 if every launch shape of p is within the kernels' limits.
int demag_plan_check(const DemagPlan& p, int real_bytes);

enum DemagPass { DP_XF = 0, DP_YF, DP_Z, DP_YI, DP_XI, DP_M2, DP_YZ, DP_COUNT };

template <typename T>
struct DemagBufs {
  cpx<T>* S1 = nullptr;
  cpx<T>* S2 = nullptr;
  T* K = nullptr;           // octant spectrum, scaled by -mu0/(Px Py Pz)
  cpx<T>* twx = nullptr;    // stage twiddles of the line transforms
  cpx<T>* twy = nullptr;
  cpx<T>* twz = nullptr;
  cpx<T>* tw4x = nullptr;   // four-step tables [k1][t] = exp(-2 pi i t k1/L)
  cpx<T>* tw4y = nullptr;
  T* Bd = nullptr;          // output field [3][N]
  int ns = 7;               // stages of the pair in use (where stage inputs are)
};

// B_d for the input of stage `stage` (0 and 1: the accepted state).
// M = Ms0 m0 + Ms1 m1 (+ Ms2 m2 for three sublattices).
template <typename T>
void demag_field(const DemagPlan& p, const DemagBufs<T>& b, const Table<T>* tbl, int stage,
                 const Ctrl* ctrl, T ms0, T ms1, int nsub, hipStream_t st, Prof* prof,
                 T ms2 = T(0));

// One pass of demag_field on its own (the autotuner times them one by one).
template <typename T>
void demag_pass(int pass, const DemagPlan& p, const DemagBufs<T>& b, const Table<T>* tbl,
                int stage, const Ctrl* ctrl, T ms0, T ms1, int nsub, hipStream_t st,
                T ms2 = T(0));

// Times the candidate launch shapes of every pass for the pads of *p on the
// buffers b and keeps the fastest in *p.  Returns the time of one demag
// evaluation with the chosen shapes in ms (< 0 on a HIP error).  With give_up
// > 0 an evaluation with the shapes of *p is timed first, and returned, *p
// unchanged, where it takes longer than that.
template <typename T>
double demag_tune(DemagPlan* p, const DemagBufs<T>& b, const Table<T>* tbl, T ms0, T ms1,
                  int nsub, hipStream_t st, T ms2 = T(0), double give_up = 0.0);

// FP64 tensor on the non-negative offsets and its transformed octant
// spectrum: kout receives the scaled spectrum (k_elems values of type T,
// device); scratch holds demag_build_doubles(p) doubles (device).  Returns
// after the build has finished.
size_t demag_build_doubles(const DemagPlan& p);
template <typename T>
int demag_kernel_build(const DemagPlan& p, double dx, double dy, double dz, double* scratch,
                       T* kout, hipStream_t st);

// The tensor from the cells of the grid to a layer of cells centred at
// height zt (layer 0 of the grid centred at 0), at the offsets X, Y >= 0:
// 6*nz*ny*nx doubles [c][z][Y][X] (device).
int stray_kernel_build(int nx, int ny, int nz, double dx, double dy, double dz, double zt,
                       double* k6, hipStream_t st);
int demag_tensor_only(int nx, int ny, int nz, double dx, double dy, double dz, double* n6,
                      hipStream_t st);

// One grid of a batched demag evaluation: its plan (pads; its launch
// shapes are not used), buffers, state table, controller and moments.
template <typename T>
struct DemagMember {
  const DemagPlan* plan;
  DemagBufs<T> bufs;
  const Table<T>* tbl;
  const Ctrl* ctrl;
  T ms0, ms1, ms2;
  int nsub;
};

// The demag passes of many grids of any pads, each pass one launch for all
// of them over a device work table of (grid, block) entries, through the
// mixed-radix LDS kernels with 256-thread blocks.  A grid's field does not
// depend on the other members, and is the one its own plan gives with every axis
// on those kernels (force_lds = 7) up to rounding: the same arithmetic per
// line, however lines are grouped into blocks, in kernels of its own.
// Whether a grid with plan p can join a batched demag evaluation (its lines
// fit one 256-thread block of the LDS kernels).
bool demag_multi_fits(const DemagPlan& p);

template <typename T>
class DemagMulti {
 public:
  DemagMulti() = default;
  DemagMulti(const DemagMulti&) = delete;
  DemagMulti& operator=(const DemagMulti&) = delete;
  ~DemagMulti() { release(); }
  // device tables for the members (synchronous); 0, or MMP_E_NOMEM /
  // MMP_E_HIP
  int build(const std::vector<DemagMember<T>>& members, hipStream_t st);
  // B_d of every member for the stage input of `stage`
  void launch(int stage, hipStream_t st) const;
  bool empty() const { return impl == nullptr; }
  void release();

 private:
  struct Impl;
  Impl* impl = nullptr;
  char* mem_ = nullptr;   // device tables, cap_ bytes
  size_t cap_ = 0;
};

// line_tw_elems(L) twiddles of one axis
template <typename T>
void build_line_tables(const LineFft& f, cpx<T>* tw, hipStream_t st);
template <typename T>
void build_twiddles4(cpx<T>* tw, int L, hipStream_t st);
int split_l2(int L);

}  // namespace mmp
