// LDS-resident line transforms of any 7-smooth length for gfx950.
//
// A line of L = r0 r1 ... points (radices up to 16, the fewest and most even
// that multiply to L) is transformed in place: stage s of the forward
// transform takes r_s-point butterflies over digit s of the element index
// e = (d0, d1, ...), d0 most significant, and multiplies output q of the
// butterfly at inner index lo by exp(-2 pi i q lo / (r_s M_s)), M_s the
// length below digit s.  Digit s then holds frequency digit s, so the
// spectrum sits at permuted places: bin k = d0 + r0 d1 + r0 r1 d2 + ... at
// a place of its own (place_of).  The inverse runs the stages backwards from there to
// natural order.  Nothing is reordered in between: what works on the
// spectrum (the unpacking of two real lines, the kernel products, the z
// transforms) looks its places up.
//
// What bounds these transforms on the grids they serve is latency and LDS
// passes, not flops: hence few large radices instead of many small ones
// (378 = 6 7 9 is three passes, 160 = 10 16 two), butterflies that read and
// write the same places (one barrier per pass), first and last passes that
// move their data between global memory and registers directly, and index
// arithmetic by multiplication with reciprocals.  The rows of r_last elements
// are padded to an odd pitch, so that the last pass (each thread on its own
// row) spreads over the LDS banks.
// Measured (MI355X, one launch): x forward / inverse of 183x77x5 FP32 cells
// (lines of 378) 28.4 / 21.8 -> 6.9 / 7.0 us, of 333x130x1 FP64 (lines of
// 672) 24.2 / 22.3 -> 9.5 / 9.0 us against passes of radix 2-8 with
// autosorting stages, two barriers each and integer divisions.
#pragma once

#include "common.h"

namespace mmp {

// ------------------------------------------------- constants of the DFTs --
// cos and sin of 2 pi j/n for the compile-time twiddles: the angle is brought
// into [0, pi/4] exactly, in units of 1/(8n) turns, then a Taylor series.
constexpr double ct_series(double x, bool sine) {
  double t = sine ? x : 1.0, sum = 0.0, terms[16] = {};
  int k = 0;
  for (; k < 14; ++k) {
    terms[k] = t;
    const double a = 2.0 * k + (sine ? 2.0 : 1.0);
    t *= -x * x / (a * (a + 1.0));
  }
  for (k = 13; k >= 0; --k) sum += terms[k];   // small terms first
  return sum;
}
constexpr double ct_cs(int j, int n, bool sine) {
  // angle = 2 pi j/n = pi/4 (8j/n); octant o and remainder r/n in [0, 1)
  j %= n;
  int a = 8 * j;
  const int o = a / n, r = a - o * n;
  const double quarter = kPi / 4.0;
  // odd octants measure back from their upper end
  const bool back = (o & 1) != 0;
  const double x = quarter * (double)(back ? n - r : r) / (double)n;
  // cos, sin of the first-octant angle, then of the full angle
  const double c = ct_series(x, false), s = ct_series(x, true);
  double cc = 0.0, ss = 0.0;
  switch (o) {
    case 0: cc = c; ss = s; break;
    case 1: cc = s; ss = c; break;
    case 2: cc = -s; ss = c; break;
    case 3: cc = -c; ss = s; break;
    case 4: cc = -c; ss = -s; break;
    case 5: cc = -s; ss = -c; break;
    case 6: cc = s; ss = -c; break;
    default: cc = c; ss = -s; break;
  }
  return sine ? ss : cc;
}

// x times exp(-/+ 2 pi i J/N), trivial angles without a multiplication
template <int J, int N, bool INV, typename V>
__device__ __forceinline__ V ct_twiddle(V x) {
  constexpr int j = J % N;
  V r;
  if constexpr (j == 0) {
    return x;
  } else if constexpr (4 * j == N) {
    r.x = INV ? -x.y : x.y;
    r.y = INV ? x.x : -x.x;
  } else if constexpr (2 * j == N) {
    r.x = -x.x;
    r.y = -x.y;
  } else if constexpr (4 * j == 3 * N) {
    r.x = INV ? x.y : -x.y;
    r.y = INV ? -x.x : x.x;
  } else {
    using T = decltype(x.x);
    constexpr double c = ct_cs(j, N, false), s = ct_cs(j, N, true);
    const T cc = T(c), ss = T(INV ? s : -s);
    r.x = x.x * cc - x.y * ss;
    r.y = x.x * ss + x.y * cc;
  }
  return r;
}

// f(integral_constant<int, I>) for I = B .. E-1, unrolled at compile time
template <int V>
struct IntC { static constexpr int value = V; };
template <int I, int E, typename F>
__device__ __forceinline__ void ct_for(F&& f) {
  if constexpr (I < E) {
    f(IntC<I>{});
    ct_for<I + 1, E>(f);
  }
}

// The split R = A B of a composite transform (A first): A = 1 for the ones
// done directly (2, 3, 4, 5, 7, 8).
constexpr int dft_first(int R) {
  return R <= 5 || R == 7 || R == 8 ? 1
         : R % 4 == 0              ? 4
         : R % 2 == 0              ? 2
         : R % 3 == 0              ? 3
                                   : 5;
}

template <typename T, int R, bool INV>
__device__ __forceinline__ void dft(cpx<T>* v);

// two passes, n = B n1 + n2, k = k1 + A k2
template <typename T, int A, int B, bool INV>
__device__ __forceinline__ void dft_two(cpx<T>* v) {
  using V = cpx<T>;
  V u[B][A];
#pragma unroll
  for (int n2 = 0; n2 < B; ++n2) {
#pragma unroll
    for (int n1 = 0; n1 < A; ++n1) u[n2][n1] = v[B * n1 + n2];
    dft<T, A, INV>(u[n2]);
  }
  ct_for<0, A>([&](auto kc) {
    constexpr int k1 = decltype(kc)::value;
    V w[B];
    ct_for<0, B>([&](auto nc) {
      constexpr int n2 = decltype(nc)::value;
      w[n2] = ct_twiddle<n2 * k1, A * B, INV>(u[n2][k1]);
    });
    dft<T, B, INV>(w);
#pragma unroll
    for (int k2 = 0; k2 < B; ++k2) v[k1 + A * k2] = w[k2];
  });
}

// R-point transform in registers, natural order in and out; forward uses
// exp(-2 pi i n k/R), the inverse is unnormalised.
template <typename T, int R, bool INV>
__device__ __forceinline__ void dft(cpx<T>* v) {
  using V = cpx<T>;
  if constexpr (R == 1) {
  } else if constexpr (R == 2) {
    const V a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  } else if constexpr (R == 4) {
    const V s02 = cadd(v[0], v[2]), d02 = csub(v[0], v[2]);
    const V s13 = cadd(v[1], v[3]), d13 = csub(v[1], v[3]);
    const V jd = INV ? cmk<T>(-d13.y, d13.x) : cmk<T>(d13.y, -d13.x);
    v[0] = cadd(s02, s13);
    v[2] = csub(s02, s13);
    v[1] = cadd(d02, jd);
    v[3] = csub(d02, jd);
  } else if constexpr (R == 8) {
    const T h = T(0.70710678118654752440);
    V a[4], b[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      a[r] = cadd(v[r], v[r + 4]);
      b[r] = csub(v[r], v[r + 4]);
    }
    if (!INV) {
      b[1] = cmk<T>(h * (b[1].x + b[1].y), h * (b[1].y - b[1].x));
      b[2] = cmk<T>(b[2].y, -b[2].x);
      b[3] = cmk<T>(h * (b[3].y - b[3].x), -h * (b[3].x + b[3].y));
    } else {
      b[1] = cmk<T>(h * (b[1].x - b[1].y), h * (b[1].y + b[1].x));
      b[2] = cmk<T>(-b[2].y, b[2].x);
      b[3] = cmk<T>(-h * (b[3].x + b[3].y), h * (b[3].x - b[3].y));
    }
    dft<T, 4, INV>(a);
    dft<T, 4, INV>(b);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[2 * k] = a[k];
      v[2 * k + 1] = b[k];
    }
  } else if constexpr (dft_first(R) == 1) {
    // odd prime: sums and differences of the pairs n, R - n carry the real
    // and the imaginary roots
    constexpr int H = R / 2;
    V s[H], d[H], o[R];
    o[0] = v[0];
#pragma unroll
    for (int n = 1; n <= H; ++n) {
      s[n - 1] = cadd(v[n], v[R - n]);
      d[n - 1] = csub(v[n], v[R - n]);
      o[0] = cadd(o[0], s[n - 1]);
    }
    ct_for<1, H + 1>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      V p = v[0], q = cmk<T>(T(0), T(0));
      ct_for<1, H + 1>([&](auto nc) {
        constexpr int n = decltype(nc)::value;
        constexpr double c = ct_cs(n * k, R, false), sn = ct_cs(n * k, R, true);
        p.x += T(c) * s[n - 1].x;
        p.y += T(c) * s[n - 1].y;
        q.x += T(sn) * d[n - 1].x;
        q.y += T(sn) * d[n - 1].y;
      });
      // forward: X_k = p - i q, X_{R-k} = p + i q
      const V a = cmk<T>(p.x + q.y, p.y - q.x), b = cmk<T>(p.x - q.y, p.y + q.x);
      o[k] = INV ? b : a;
      o[R - k] = INV ? a : b;
    });
#pragma unroll
    for (int k = 0; k < R; ++k) v[k] = o[k];
  } else {
    constexpr int A = dft_first(R);
    // the inverse takes the even factor last, so that a caller that keeps
    // only the first half of the outputs leaves half of that pass out
    if constexpr (INV) dft_two<T, R / A, A, INV>(v);
    else dft_two<T, A, R / A, INV>(v);
  }
}

// The forward transform of an input whose upper half is zero (not read), R
// even: the first pass over the even factor works on half its inputs.
template <typename T, int R>
__device__ __forceinline__ void dft_hz(cpx<T>* v) {
  using V = cpx<T>;
  static_assert(R % 2 == 0, "half-zero transforms of even length");
  constexpr int A = R % 4 == 0 ? 4 : 2, B = R / A;
  ct_for<0, B>([&](auto nc) {
    constexpr int n2 = decltype(nc)::value;
    if constexpr (A == 2) {
      v[B + n2] = ct_twiddle<n2, R, false>(v[n2]);
    } else {
      const V a = v[n2], b = v[B + n2];
      const V jb = cmk<T>(b.y, -b.x);
      v[n2] = cadd(a, b);
      v[B + n2] = ct_twiddle<n2, R, false>(cadd(a, jb));
      v[2 * B + n2] = ct_twiddle<2 * n2, R, false>(csub(a, b));
      v[3 * B + n2] = ct_twiddle<3 * n2, R, false>(csub(a, jb));
    }
  });
  V o[R];
#pragma unroll
  for (int k1 = 0; k1 < A; ++k1) {
    dft<T, B, false>(v + B * k1);
#pragma unroll
    for (int k2 = 0; k2 < B; ++k2) o[k1 + A * k2] = v[B * k1 + k2];
  }
#pragma unroll
  for (int k = 0; k < R; ++k) v[k] = o[k];
}

// ------------------------------------------------------------- geometry --
constexpr int kMaxStages = 4;

// x / d for 0 <= x, d < 2^16: x times the rounded-up reciprocal (m = 0
// stands for d = 1)
struct FastDiv {
  uint32_t m;
  __device__ __forceinline__ int div(int x) const {
    return m ? (int)__umulhi((uint32_t)x, m) : x;
  }
};
inline FastDiv make_div(int d) {
  FastDiv f;
  f.m = d <= 1 ? 0u : (uint32_t)((1ull << 32) / (uint32_t)d) + 1u;
  return f;
}

// One stage: radix r, inner length M (natural elements below the digit) and
// its padded stride PM, padded stride HP of the index above the digit,
// butterflies per line nb, offset of the stage's twiddles.
struct LineStage {
  int r, M, PM, HP, nb, tw;
  FastDiv dM, dnb;
};

// The stages are separate members, picked by a uniform index with scalar
// selects: an indexed array in a kernel argument would be copied to private
// memory.
struct LineFft {
  int L, n, pitch;   // points, stages, padded elements per line
  int ntw, nst;      // twiddles of all stages but the last; with the bins' places
  int rl, pad;       // last radix, padding per row of rl elements
  FastDiv drl;
  LineStage s0, s1, s2, s3;
  __device__ __forceinline__ LineStage stage(int s) const {
    LineStage o;
    auto pick = [&](int a, int b, int c, int d) { return s == 0 ? a : s == 1 ? b : s == 2 ? c : d; };
    o.r = pick(s0.r, s1.r, s2.r, s3.r);
    o.M = pick(s0.M, s1.M, s2.M, s3.M);
    o.PM = pick(s0.PM, s1.PM, s2.PM, s3.PM);
    o.HP = pick(s0.HP, s1.HP, s2.HP, s3.HP);
    o.nb = pick(s0.nb, s1.nb, s2.nb, s3.nb);
    o.tw = pick(s0.tw, s1.tw, s2.tw, s3.tw);
    o.dM.m = (uint32_t)pick((int)s0.dM.m, (int)s1.dM.m, (int)s2.dM.m, (int)s3.dM.m);
    o.dnb.m = (uint32_t)pick((int)s0.dnb.m, (int)s1.dnb.m, (int)s2.dnb.m, (int)s3.dnb.m);
    return o;
  }
  // LDS place of bin k: its digits, least significant first, are the digits
  // of the element index, most significant first
  __host__ __device__ int place_of(int k) const {
    int e = 0;
    const LineStage* st[kMaxStages] = {&s0, &s1, &s2, &s3};
    for (int s = 0; s < n; ++s) {
      e += (k % st[s]->r) * st[s]->M;
      k /= st[s]->r;
    }
    return e + e / rl * pad;
  }
};

// Radices (of those built) of a 7-smooth L <= 4096: the fewest, then the
// most even ones; the first even where L is even (its butterflies then
// skip the zero half of a padded line as whole inputs).  Returns the count,
// 0 if L has another prime factor.
inline int line_radices(int L, int* out) {
  static const int R[] = {16, 15, 14, 12, 10, 9, 8, 7, 6, 5, 4, 3, 2};
  if (L == 1) {
    out[0] = 1;
    return 1;
  }
  struct Rec {
    int best_n = kMaxStages + 1, best_max = 99, best_min = 0, best[kMaxStages] = {},
        cur[kMaxStages] = {};
    void go(int left, int n, int from, const int* R) {
      if (left == 1) {
        const int mx = cur[0], mn = cur[n - 1];   // radices descend
        if (n < best_n || (n == best_n && (mx < best_max || (mx == best_max && mn > best_min)))) {
          best_n = n;
          best_max = mx;
          best_min = mn;
          for (int i = 0; i < n; ++i) best[i] = cur[i];
        }
        return;
      }
      if (n >= kMaxStages) return;
      for (int i = from; i < 13; ++i)
        if (left % R[i] == 0) {
          cur[n] = R[i];
          go(left / R[i], n + 1, i, R);
        }
    }
  } rec;
  rec.go(L, 0, 0, R);
  if (rec.best_n > kMaxStages) return 0;
  // an even radix first (the largest even one), the others as they are
  int first = 0;
  for (int i = 0; i < rec.best_n; ++i)
    if (rec.best[i] % 2 == 0) {
      first = i;
      break;
    }
  int k = 0;
  out[k++] = rec.best[first];
  for (int i = 0; i < rec.best_n; ++i)
    if (i != first) out[k++] = rec.best[i];
  return rec.best_n;
}

inline bool make_line_fft(int L, LineFft* f) {
  int r[kMaxStages] = {};
  const int n = line_radices(L, r);
  if (n == 0) return false;
  LineFft o{};
  o.L = L;
  o.n = n;
  o.rl = r[n - 1];
  o.pad = o.rl % 2 == 0 ? 1 : 0;
  o.drl = make_div(o.rl);
  o.pitch = L / o.rl * (o.rl + o.pad);
  LineStage* st[kMaxStages] = {&o.s0, &o.s1, &o.s2, &o.s3};
  int M = L, tw = 0;
  for (int s = 0; s < n; ++s) {
    LineStage& t = *st[s];
    M /= r[s];
    t.r = r[s];
    t.M = M;
    const bool last = s == n - 1;
    t.PM = last ? 1 : M / o.rl * (o.rl + o.pad);
    t.HP = last ? o.rl + o.pad : r[s] * t.PM;
    t.nb = L / r[s];
    t.tw = tw;
    t.dM = make_div(M);
    t.dnb = make_div(t.nb);
    if (!last) tw += r[s] * M;
  }
  o.ntw = tw;
  o.nst = (tw + 1) / 2 * 2 + (L + 3) / 4;
  *f = o;
  return true;
}

// Table of one axis, in complex elements: the twiddles of all stages but the
// last (fewer than 1.6 L), then, from an even element on, the places of the
// bins as 16-bit values (four or eight to an element; nst counts four).
inline int line_tw_elems(int L) { return 2 * L + 256; }
template <typename V>
__host__ __device__ inline const uint16_t* line_places(const LineFft& f, const V* tw) {
  return reinterpret_cast<const uint16_t*>(tw + (f.ntw + 1) / 2 * 2);
}
// LDS elements of `lines` lines (to an even number of elements) and, behind
// them, the axis' table in whole kilobytes (line_stage_tw)
__host__ __device__ inline int line_tw_at(const LineFft& f, int lines) {
  return (lines * f.pitch + 1) & ~1;
}
inline size_t line_lds_elems(const LineFft& f, long lines, size_t elem_bytes) {
  const size_t kb = 1024 / elem_bytes;
  return line_tw_at(f, (int)lines) + (f.nst + kb - 1) / kb * kb;
}

// --------------------------------------------------------------- passes --
// The radices a line may have, one code path each.
#define MMP_RADICES(X) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(12) X(14) X(15) X(16)

// places of butterfly b of a stage: LDS element of its first input, inner
// index lo (its twiddles)
__device__ __forceinline__ int line_place(const LineFft& f, const LineStage& t, int b, int* lo) {
  const int hi = t.M > 1 ? t.dM.div(b) : b;
  const int l = b - hi * t.M;
  *lo = l;
  return hi * t.HP + l + f.drl.div(l) * f.pad;
}

// Copies the axis' table behind the lines in LDS: every stage but the first
// forward one reads its twiddles there, and whatever works on the spectrum
// the places (a trip to L2 per stage is longer than the stage).  The copy goes to LDS without registers, 16 bytes per lane and 1 KiB
// per wave, and nothing waits for it before lds_copies_done() and a barrier;
// a copy through registers would hold up the data loads behind it.
template <typename T>
__device__ __forceinline__ const cpx<T>* line_stage_tw(const LineFft& f, cpx<T>* buf, int lines,
                                                       const cpx<T>* __restrict__ tw, int tid,
                                                       int nthr) {
  constexpr int PER = 16 / (int)sizeof(cpx<T>), CH = 64 * PER;
  cpx<T>* d = buf + line_tw_at(f, lines);
  const int wave = uni(tid >> 6), lane = tid & 63, last = (f.nst - 1) / PER * PER;
  for (int i = wave * CH; i < f.nst; i += (nthr >> 6) * CH) {
    const int e = i + lane * PER;
    // (the table has room behind nst: its last 16 bytes may reach past it)
    const cpx<T>* src = tw + (e < f.nst ? e : last);
    __builtin_amdgcn_global_load_lds(
        (__attribute__((address_space(1))) void*)const_cast<cpx<T>*>(src),
        (__attribute__((address_space(3))) void*)(d + i), 16, 0, 0);
  }
  return d;
}
__device__ __forceinline__ void lds_copies_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// First forward stage of `lines` lines: element n of line l comes from
// ld(l, n) (which loads a clamped address where it must return zero), goes
// through the butterfly and to its place in LDS.  half: elements n >= L/2
// are zero (radix even).
template <typename T, int R, typename LD>
__device__ __forceinline__ void line_fwd_first_r(const LineFft& f, cpx<T>* buf,
                                                 const cpx<T>* __restrict__ tw, int lines,
                                                 bool half, int tid, int nthr, LD&& ld) {
  using V = cpx<T>;
  const LineStage t = f.s0;
  const int total = lines * t.nb;
  for (int w = tid; w < total; w += nthr) {
    const int l = t.dnb.div(w), b = w - l * t.nb;
    V v[R];
    constexpr int RH = R % 2 == 0 ? R / 2 : R;
#pragma unroll
    for (int q = 0; q < RH; ++q) v[q] = ld(l, q * t.M + b);
    if constexpr (R % 2 == 0) {
      if (half) {
#pragma unroll
        for (int q = RH; q < R; ++q) v[q] = cmk<T>(T(0), T(0));
      } else {
#pragma unroll
        for (int q = RH; q < R; ++q) v[q] = ld(l, q * t.M + b);
      }
    }
    // (the stage's twiddles come with the data, from memory)
    int lo;
    V* p = buf + l * f.pitch + line_place(f, t, b, &lo);
    V t1[R];
#pragma unroll
    for (int q = 1; q < R; ++q) t1[q] = tw[f.n > 1 ? t.tw + q * t.M + lo : 0];
    dft<T, R, false>(v);
    if (f.n > 1) {
#pragma unroll
      for (int q = 1; q < R; ++q) v[q] = cmul(v[q], t1[q]);
    }
#pragma unroll
    for (int q = 0; q < R; ++q) p[q * t.PM] = v[q];
  }
}

template <typename T, int R, bool INV>
__device__ __forceinline__ void line_inner_r(const LineFft& f, const LineStage& t, bool twid,
                                             cpx<T>* buf, const cpx<T>* tw,
                                             int lines, int tid, int nthr) {
  using V = cpx<T>;
  const int total = lines * t.nb;
  for (int w = tid; w < total; w += nthr) {
    const int l = t.dnb.div(w), b = w - l * t.nb;
    int lo;
    V* p = buf + l * f.pitch + line_place(f, t, b, &lo);
    V v[R];
#pragma unroll
    for (int q = 0; q < R; ++q) v[q] = p[q * t.PM];
    if (INV && twid) {
#pragma unroll
      for (int q = 1; q < R; ++q) v[q] = cmul(v[q], cconj(tw[t.tw + q * t.M + lo]));
    }
    dft<T, R, INV>(v);
    if (!INV && twid) {
#pragma unroll
      for (int q = 1; q < R; ++q) v[q] = cmul(v[q], tw[t.tw + q * t.M + lo]);
    }
#pragma unroll
    for (int q = 0; q < R; ++q) p[q * t.PM] = v[q];
  }
}

// Last inverse stage: element n of line l goes to st(l, n, value); half:
// elements n >= L/2 are not wanted (radix even).
template <typename T, int R, typename ST>
__device__ __forceinline__ void line_inv_last_r(const LineFft& f, const cpx<T>* buf,
                                                const cpx<T>* tw, int lines,
                                                bool half, int tid, int nthr, ST&& st) {
  using V = cpx<T>;
  const LineStage t = f.s0;
  const int total = lines * t.nb;
  for (int w = tid; w < total; w += nthr) {
    const int l = t.dnb.div(w), b = w - l * t.nb;
    int lo;
    const V* p = buf + l * f.pitch + line_place(f, t, b, &lo);
    V v[R];
#pragma unroll
    for (int q = 0; q < R; ++q) v[q] = p[q * t.PM];
    if (f.n > 1) {
#pragma unroll
      for (int q = 1; q < R; ++q) v[q] = cmul(v[q], cconj(tw[t.tw + q * t.M + lo]));
    }
    dft<T, R, true>(v);
    constexpr int RH = R % 2 == 0 ? R / 2 : R;
#pragma unroll
    for (int q = 0; q < RH; ++q) st(l, q * t.M + b, v[q]);
    if constexpr (R % 2 == 0) {
      if (!half) {
#pragma unroll
        for (int q = RH; q < R; ++q) st(l, q * t.M + b, v[q]);
      }
    }
  }
}

// Forward transform of `lines` lines into LDS (bin k at line_places()[k] of
// each line); tw: the table in memory, twl: in LDS (line_stage_tw, no barrier
// needed in between).  Ends with a barrier.
template <typename T, typename LD>
__device__ __forceinline__ void line_fft_fwd(const LineFft& f, cpx<T>* buf,
                                             const cpx<T>* __restrict__ tw, const cpx<T>* twl,
                                             int lines, bool half, int tid, int nthr, LD&& ld) {
  switch (f.s0.r) {
#define X(R) case R: line_fwd_first_r<T, R>(f, buf, tw, lines, half, tid, nthr, ld); break;
    MMP_RADICES(X)
#undef X
  }
  lds_copies_done();
  __syncthreads();
  for (int s = 1; s < f.n; ++s) {
    const LineStage t = f.stage(s);
    const bool twid = s < f.n - 1;
    switch (t.r) {
#define X(R) case R: line_inner_r<T, R, false>(f, t, twid, buf, twl, lines, tid, nthr); break;
      MMP_RADICES(X)
#undef X
    }
    __syncthreads();
  }
}

// Inverse transform (unnormalised) of `lines` spectra in LDS, twiddles in
// LDS; the caller's writes to both are behind a barrier.
template <typename T, typename ST>
__device__ __forceinline__ void line_fft_inv(const LineFft& f, cpx<T>* buf, const cpx<T>* twl,
                                             int lines, bool half, int tid, int nthr, ST&& st) {
  for (int s = f.n - 1; s > 0; --s) {
    const LineStage t = f.stage(s);
    const bool twid = s < f.n - 1;
    switch (t.r) {
#define X(R) case R: line_inner_r<T, R, true>(f, t, twid, buf, twl, lines, tid, nthr); break;
      MMP_RADICES(X)
#undef X
    }
    __syncthreads();
  }
  switch (f.s0.r) {
#define X(R) case R: line_inv_last_r<T, R>(f, buf, twl, lines, half, tid, nthr, st); break;
    MMP_RADICES(X)
#undef X
  }
}

// The same on lines already in LDS (natural element e at e + (e / rl) pad),
// each ending with a barrier.
template <typename T, bool INV>
__device__ __forceinline__ void line_stage_lds(const LineFft& f, int s, cpx<T>* buf,
                                               const cpx<T>* tw, int lines, int tid,
                                               int nthr) {
  const LineStage t = f.stage(s);
  const bool twid = s < f.n - 1;
  switch (t.r) {
#define X(R) case R: line_inner_r<T, R, INV>(f, t, twid, buf, tw, lines, tid, nthr); break;
    MMP_RADICES(X)
#undef X
  }
  __syncthreads();
}
template <typename T>
__device__ __forceinline__ void line_fft_fwd_lds(const LineFft& f, cpx<T>* buf,
                                                 const cpx<T>* __restrict__ tw, int lines,
                                                 int tid, int nthr) {
  for (int s = 0; s < f.n; ++s) line_stage_lds<T, false>(f, s, buf, tw, lines, tid, nthr);
}
template <typename T>
__device__ __forceinline__ void line_fft_inv_lds(const LineFft& f, cpx<T>* buf,
                                                 const cpx<T>* __restrict__ tw, int lines,
                                                 int tid, int nthr) {
  for (int s = f.n - 1; s >= 0; --s) line_stage_lds<T, true>(f, s, buf, tw, lines, tid, nthr);
}

inline bool is_pow2(int L) { return L > 0 && (L & (L - 1)) == 0; }

}  // namespace mmp
