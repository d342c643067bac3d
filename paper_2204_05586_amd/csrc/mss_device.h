// Device-side building blocks of the solver: small complex matrices held in
// registers, the two exponentiators, the field-program interpreter and one
// CF4 fine step.  gfx950 only: FP64 on the vector ALUs (a 3x3 complex
// product is 108 FP64 FMAs and not a dense contraction worth MFMA).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mss.h"

namespace mss {

// ---------------------------------------------------------------------------
// constants (IEEE double values of the printed closed forms)
// ---------------------------------------------------------------------------
// Gauss-Legendre nodes (1 -/+ 1/sqrt 3) / 2 and CF4 weights (3 +/- 2 sqrt 3) / 12
// (Sec. "Unitary time evolution and the Magnus expansion", eqs. cf4_sample_1/2).
constexpr double kNode1 = 0x1.b0cb174df99c6p-3;
constexpr double kNode2 = 0x1.93cd3a2c8198ep-1;
constexpr double kWPlus = 0x1.13cd3a2c8198ep-1;
constexpr double kWMinus = -0x1.3cd3a2c8198e0p-5;
constexpr double kTwoPi = 0x1.921fb54442d18p+2;
constexpr double kRsqrt2 = 0x1.6a09e667f3bccp-1;

// Field program as a kernel argument (scalar-loaded, uniform across a wave).
// The first n_varying terms are those of components that depend on time, in
// list order; the others belong to components all of whose terms are
// constant and always on (program_order).
struct FieldProgram {
  int32_t n_terms;
  int32_t n_varying;
  mss_term t[MSS_MAX_TERMS];
};

// Does a field source provide the full su(3) basis (the field-program
// interpreter does; a user field function gives four components)?
template <class T, class = void>
struct has_full_basis {
  static constexpr bool value = false;
};
template <class T>
struct has_full_basis<T, decltype((void)T::kFullBasis)> {
  static constexpr bool value = T::kFullBasis;
};

// Memory that no kernel writes while this one runs (descriptors, term tables,
// parameters): read through the constant address space, a wave-uniform
// address is a scalar load whatever the kernel stores in between.  Through
// an ordinary pointer the compiler must assume that a store or atomic has
// changed it, and every read inside a work loop becomes a vector load.
template <class T>
using Constant = const T __attribute__((address_space(4)));
template <class T>
__device__ __forceinline__ Constant<T>* as_constant(const T* p) {
  return (Constant<T>*)(uint64_t)p;
}
// A whole structure of 8-byte words.
template <class T>
__device__ __forceinline__ T load_constant(const T* p) {
  static_assert(sizeof(T) % 8 == 0, "8-byte words");
  Constant<uint64_t>* src = (Constant<uint64_t>*)(uint64_t)p;
  uint64_t w[sizeof(T) / 8];
#pragma unroll
  for (unsigned i = 0; i < sizeof(T) / 8; ++i) w[i] = src[i];
  T v;
  __builtin_memcpy(&v, w, sizeof(T));
  return v;
}

// Term sources for the interpreter: the kernel-argument program of a single
// simulation, or a slice of a term table in device memory (batches).
struct ArgTerms {
  static constexpr bool kFullBasis = true;  // field programs may use all eight components
  const FieldProgram& fp;
  __device__ __forceinline__ int size() const { return fp.n_terms; }
  __device__ __forceinline__ int varying() const { return fp.n_varying; }
  __device__ __forceinline__ const mss_term& operator[](int i) const { return fp.t[i]; }
};
struct TableTerms {
  static constexpr bool kFullBasis = true;
  const mss_term* t;
  int n, n_varying;
  __device__ __forceinline__ int size() const { return n; }
  __device__ __forceinline__ int varying() const { return n_varying; }
  __device__ __forceinline__ Constant<mss_term>& operator[](int i) const {
    return as_constant(t)[i];
  }
};

template <int N>
struct Mat {
  double r[N][N];
  double i[N][N];
};

template <int N>
__device__ __forceinline__ void set_identity(Mat<N>& m) {
#pragma unroll
  for (int a = 0; a < N; ++a)
#pragma unroll
    for (int b = 0; b < N; ++b) {
      m.r[a][b] = (a == b) ? 1.0 : 0.0;
      m.i[a][b] = 0.0;
    }
}

// C = A * B (complex, N x N), 4 real FMAs per complex multiply-add.
template <int N>
__device__ __forceinline__ void matmul(const Mat<N>& A, const Mat<N>& B, Mat<N>& C) {
#pragma unroll
  for (int a = 0; a < N; ++a)
#pragma unroll
    for (int b = 0; b < N; ++b) {
      double re = A.r[a][0] * B.r[0][b];
      double im = A.r[a][0] * B.i[0][b];
      re = fma(-A.i[a][0], B.i[0][b], re);
      im = fma(A.i[a][0], B.r[0][b], im);
#pragma unroll
      for (int k = 1; k < N; ++k) {
        re = fma(A.r[a][k], B.r[k][b], re);
        re = fma(-A.i[a][k], B.i[k][b], re);
        im = fma(A.r[a][k], B.i[k][b], im);
        im = fma(A.i[a][k], B.r[k][b], im);
      }
      C.r[a][b] = re;
      C.i[a][b] = im;
    }
}

// M <- A * M
template <int N>
__device__ __forceinline__ void premultiply(const Mat<N>& A, Mat<N>& M) {
  Mat<N> t;
  matmul<N>(A, M, t);
  M = t;
}

// The running product of an integration.
//
// Full su(3) basis: the whole operator (its squarings at low tau are not
// unitary).
//
// Spin-1: the outer two columns (72 FMAs an exponential instead of 108); the
// middle one of a unitary matrix of determinant 1 is the conjugate cross
// product of the two, taken once per interval.  Rounding makes the columns'
// norms drift, and the cross product's norm would drift by the sum of
// theirs; it is scaled to their mean.  Against the scheme in extended
// precision, 28 simulations drawn over 2e3 to 3e5 intervals and 5 to 40 fine
// steps are off by 2.10e-12 in the geometric mean and 7.1e-12 in the mean
// square (the squarings with whole operators: 2.15e-12 and 7.3e-12).  A
// running U - I would drift a tenth as much, but is then further from a
// solver that rounds U than the 1e-10 the two are held to over 1e7 steps.
// 4.5e7 intervals of 10 fine steps, chained: 9.20 ms with three columns, 7.96
// with two.
//
// Spin-1/2: the first column, less that of I, and exponentials less I
// (20 instructions instead of 32); the second column mirrors the first.
// Against the same scheme in extended precision the states of 1e4 intervals
// of 100 fine steps are 4.6e-14 off, and were 8.5e-13 off with the identity
// inside.
template <int N, bool FULL> struct Running;
template <> struct Running<3, true> {
  Mat<3> u;
  __device__ __forceinline__ void clear() { set_identity<3>(u); }
  __device__ __forceinline__ void multiply(const Mat<3>& E) { premultiply<3>(E, u); }
  __device__ __forceinline__ void whole(Mat<3>& U) const { U = u; }
};
template <> struct Running<3, false> {
  double r[3][2], i[3][2];  // columns 0 and 2
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        r[a][b] = a == 2 * b ? 1.0 : 0.0;
        i[a][b] = 0.0;
      }
  }
  __device__ __forceinline__ void multiply(const Mat<3>& E) {
    double nr[3][2], ni[3][2];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        double re = E.r[a][0] * r[0][b];
        double im = E.r[a][0] * i[0][b];
        re = fma(-E.i[a][0], i[0][b], re);
        im = fma(E.i[a][0], r[0][b], im);
#pragma unroll
        for (int k = 1; k < 3; ++k) {
          re = fma(E.r[a][k], r[k][b], re);
          re = fma(-E.i[a][k], i[k][b], re);
          im = fma(E.r[a][k], i[k][b], im);
          im = fma(E.i[a][k], r[k][b], im);
        }
        nr[a][b] = re;
        ni[a][b] = im;
      }
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        r[a][b] = nr[a][b];
        i[a][b] = ni[a][b];
      }
  }
  __device__ __forceinline__ void whole(Mat<3>& U) const {
#pragma clang fp contract(off)
    double n2 = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const int j = (a + 1) % 3, k = (a + 2) % 3;
      U.r[a][0] = r[a][0];
      U.i[a][0] = i[a][0];
      U.r[a][2] = r[a][1];
      U.i[a][2] = i[a][1];
      // conj(y_j x_k - y_k x_j), x and y the first and last column
      double re = r[j][1] * r[k][0], im = r[j][1] * i[k][0];
      re = fma(-i[j][1], i[k][0], re);
      im = fma(i[j][1], r[k][0], im);
      re = fma(-r[k][1], r[j][0], re);
      im = fma(-r[k][1], i[j][0], im);
      re = fma(i[k][1], i[j][0], re);
      im = fma(-i[k][1], r[j][0], im);
      U.r[a][1] = re;
      U.i[a][1] = -im;
      n2 = fma(re, re, fma(im, im, n2));
    }
    const double scale = 1.0 - 0.25 * (n2 - 1.0);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      U.r[a][1] *= scale;
      U.i[a][1] *= scale;
    }
  }
};
template <> struct Running<2, false> {
  double r[2], i[2];
  __device__ __forceinline__ void clear() { r[0] = r[1] = i[0] = i[1] = 0.0; }
  // I + x <- (I + A) (I + x): x <- A x + (A + x), the first column
  __device__ __forceinline__ void multiply(const Mat<2>& A) {
    double nr[2], ni[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      double re = A.r[a][0] + r[a], im = A.i[a][0] + i[a];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        re = fma(A.r[a][k], r[k], re);
        re = fma(-A.i[a][k], i[k], re);
        im = fma(A.r[a][k], i[k], im);
        im = fma(A.i[a][k], r[k], im);
      }
      nr[a] = re;
      ni[a] = im;
    }
    r[0] = nr[0];
    r[1] = nr[1];
    i[0] = ni[0];
    i[1] = ni[1];
  }
  // columns (u, v) and (-conj v, conj u)
  __device__ __forceinline__ void whole(Mat<2>& U) const {
    const double ur = 1.0 + r[0];
    U.r[0][0] = ur;     U.i[0][0] = i[0];
    U.r[1][0] = r[1];   U.i[1][0] = i[1];
    U.r[0][1] = -r[1];  U.i[0][1] = i[1];
    U.r[1][1] = ur;     U.i[1][1] = -i[0];
  }
};

// y = M x for a complex N x N matrix and an N-vector (re / im parts apart).
template <int N>
__device__ __forceinline__ void matvec(const Mat<N>& M, const double* xr, const double* xi,
                                       double* yr, double* yi) {
#pragma unroll
  for (int a = 0; a < N; ++a) {
    double re = 0.0, im = 0.0;
#pragma unroll
    for (int b = 0; b < N; ++b) {
      re = fma(M.r[a][b], xr[b], re);
      re = fma(-M.i[a][b], xi[b], re);
      im = fma(M.r[a][b], xi[b], im);
      im = fma(M.i[a][b], xr[b], im);
    }
    yr[a] = re;
    yi[a] = im;
  }
}

template <int N>
__device__ __forceinline__ Mat<N> shfl_down_mat(const Mat<N>& m, int d) {
  Mat<N> o;
#pragma unroll
  for (int a = 0; a < N; ++a)
#pragma unroll
    for (int b = 0; b < N; ++b) {
      o.r[a][b] = __shfl_down(m.r[a][b], d, 64);
      o.i[a][b] = __shfl_down(m.i[a][b], d, 64);
    }
  return o;
}

template <int N>
__device__ __forceinline__ Mat<N> shfl_up_mat(const Mat<N>& m, int d) {
  Mat<N> o;
#pragma unroll
  for (int a = 0; a < N; ++a)
#pragma unroll
    for (int b = 0; b < N; ++b) {
      o.r[a][b] = __shfl_up(m.r[a][b], d, 64);
      o.i[a][b] = __shfl_up(m.i[a][b], d, 64);
    }
  return o;
}

template <int N>
__device__ __forceinline__ void load_mat(const double* __restrict__ p, Mat<N>& m) {
#pragma unroll
  for (int a = 0; a < N; ++a)
#pragma unroll
    for (int b = 0; b < N; ++b) {
      m.r[a][b] = p[2 * (a * N + b)];
      m.i[a][b] = p[2 * (a * N + b) + 1];
    }
}

template <int N>
__device__ __forceinline__ void store_mat(double* __restrict__ p, const Mat<N>& m) {
#pragma unroll
  for (int a = 0; a < N; ++a)
#pragma unroll
    for (int b = 0; b < N; ++b) {
      p[2 * (a * N + b)] = m.r[a][b];
      p[2 * (a * N + b) + 1] = m.i[a][b];
    }
}

// ---------------------------------------------------------------------------
// sine and cosine
// ---------------------------------------------------------------------------
// sincos_cw: Cody-Waite reduction x = k pi/2 + r with pi/2 split into three
// doubles (P1 and P2 of 32 significant bits, P3 the rest).  x - k P1 is a
// multiple of 2^-31 or of x's last place and at most 2 in size, so the first
// step is exact for every k; the other two round at the size of r.  Then
// minimax polynomials of sin r and cos r on |r| <= pi/4, rotated by the
// quadrant k mod 4.  The polynomials are from a Remez exchange in 60 digits:
// sin r = r + r y S(y) and cos r = 1 - y / 2 + y^2 C(y), y = r^2, S and C of
// degree 5 (with the coefficients rounded as below, sine and cosine to 2^-57
// and 2^-59 relative).  4e6 arguments in each
// of |x| < 3, 1e3, 4e5, 1e7 and 1e9 are off by at most 1.7e-16, 3.5e-17 in the
// mean square, as with the Taylor series to r^17 and r^16 before them, in 3
// steps less.  (One odd polynomial on |r| <= pi/2 would do without the
// second: 2.1e-16 and 4.2e-17.)  From |x| = 2^30 on, where k would leave an
// int's range, ocml's sincos is used, out of line.
constexpr double kTwoOverPi = 0x1.45f306dc9c883p-1;
constexpr double kPio2_1 = 0x1.921fb54400000p+0;
constexpr double kPio2_2 = 0x1.0b4611a600000p-34;
constexpr double kPio2_3 = 0x1.3198a2e037073p-69;

// NaN: no
__device__ __forceinline__ bool sincos_in_range(double x) { return fabs(x) < 0x1p+30; }

struct SinCos {
  double s, c;
};
__device__ __attribute__((noinline)) SinCos sincos_far(double x) {
  SinCos r;
  sincos(x, &r.s, &r.c);
  return r;
}

// A constant as a scalar operand.  Left to itself the compiler forms each
// step of a Horner chain in place of its constant (a two-operand multiply-
// add), which takes a vector move per coefficient: 15 of the 48 instructions
// of a sine and cosine.  A scalar constant is moved beside the vector work
// and serves every chain that uses it.
__device__ __forceinline__ double scalar_constant(double c) {
  asm("" : "+s"(c));
  return c;
}

// The reduction and series for M arguments in range, the chains side by side.
template <int M>
__device__ __forceinline__ void sincos_reduced(const double (&x)[M], double (&s)[M],
                                               double (&c)[M]) {
  constexpr double kSin[6] = {0x1.5d932f4b3062ep-33, -0x1.ae5e66d4cdfebp-26,
                              0x1.71de357874087p-19, -0x1.a01a019c126a4p-13,
                              0x1.111111110f880p-7,  -0x1.5555555555549p-3};
  constexpr double kCos[7] = {-0x1.8faecfa48eeadp-37, 0x1.1ee9ec48989bcp-29,
                              -0x1.27e4f80a77ac2p-22, 0x1.a01a019cb270cp-16,
                              -0x1.6c16c16c15184p-10, 0x1.555555555554cp-5, -0.5};
  double k[M], r[M], r2[M], ps[M], pc[M];
  const double over = scalar_constant(kTwoOverPi);
  const double p1 = scalar_constant(kPio2_1), p2 = scalar_constant(kPio2_2),
               p3 = scalar_constant(kPio2_3);
#pragma unroll
  for (int i = 0; i < M; ++i) {
    k[i] = rint(x[i] * over);
    r[i] = fma(-k[i], p1, x[i]);
    r[i] = fma(-k[i], p2, r[i]);
    r[i] = fma(-k[i], p3, r[i]);
    r2[i] = r[i] * r[i];
    ps[i] = kSin[0];
    pc[i] = kCos[0];
  }
#pragma unroll
  for (int j = 1; j < 6; ++j) {
    const double a = scalar_constant(kSin[j]), b = scalar_constant(kCos[j]);
#pragma unroll
    for (int i = 0; i < M; ++i) {
      ps[i] = fma(ps[i], r2[i], a);
      pc[i] = fma(pc[i], r2[i], b);
    }
  }
#pragma unroll
  for (int i = 0; i < M; ++i) {
    const double sn = fma(r[i] * r2[i], ps[i], r[i]);
    const double cn = fma(r2[i], fma(pc[i], r2[i], kCos[6]), 1.0);
    const int q = ((int)k[i]) & 3;
    const double s1 = (q & 1) ? cn : sn;
    const double c1 = (q & 1) ? sn : cn;
    s[i] = (q & 2) ? -s1 : s1;
    c[i] = ((q + 1) & 2) ? -c1 : c1;
  }
}

// Of M arguments at once: one branch for all (ocml's sincos for all of them
// when one is out of range).
template <int M>
__device__ __forceinline__ void sincos_cw(const double (&x)[M], double (&s)[M], double (&c)[M]) {
  bool all = true;
#pragma unroll
  for (int i = 0; i < M; ++i) all = all && sincos_in_range(x[i]);
  if (all) {
    sincos_reduced(x, s, c);
  } else {
#pragma unroll
    for (int i = 0; i < M; ++i) {
      const SinCos far = sincos_far(x[i]);
      s[i] = far.s;
      c[i] = far.c;
    }
  }
}

__device__ __forceinline__ void sincos_cw(double x, double* s, double* c) {
  if (sincos_in_range(x)) {
    const double xi[1] = {x};
    double si[1], ci[1];
    sincos_reduced(xi, si, ci);
    *s = si[0];
    *c = ci[0];
  } else {
    const SinCos far = sincos_far(x);
    *s = far.s;
    *c = far.c;
  }
}

// Tiny angles inside the exponentiators: below 2^-10 the Taylor series to
// x^5 (sin) and x^6 (cos) is exact to far below one ulp (next terms
// < 2e-22 relative); above it, sincos_cw, with LEAF without a call for far
// arguments.
template <bool LEAF = false>
__device__ __forceinline__ void sincos_small(double x, double* s, double* c) {
  if (fabs(x) < 0x1p-10) {
    const double x2 = x * x;
    *s = fma(x * x2, fma(x2, 1.0 / 120.0, -1.0 / 6.0), x);
    *c = fma(x2, fma(x2, fma(x2, -1.0 / 720.0, 1.0 / 24.0), -0.5), 1.0);
  } else if (LEAF && !sincos_in_range(x)) {
    sincos(x, s, c);
  } else {
    sincos_cw(x, s, c);
  }
}

// ---------------------------------------------------------------------------
// spin-1/2 exponential: exp(-i theta . sigma / 2)
// = cos(|theta|/2) I - i sin(|theta|/2) (theta/|theta|) . sigma, less I
// ---------------------------------------------------------------------------
// u = |theta|^2 / 4, c = cos(|theta|/2) - 1 and S = sin(|theta|/2) / |theta|.
__device__ __forceinline__ void half_coefficients(const double th[4], double& u, double& c,
                                                  double& S) {
  // cos and sin(x) / x are even in x = |theta| / 2: up to x = 1 their series
  // in x^2 need no square root, division or range reduction
  const double t2 = fma(th[0], th[0], fma(th[1], th[1], th[2] * th[2]));
  u = 0.25 * t2;
  if (u <= 0x1p-8) {  // next terms below 2^-61
    c = u * fma(u, fma(u, fma(u, 1.0 / 40320, -1.0 / 720), 1.0 / 24), -0.5);
    S = fma(u, fma(u, fma(u, fma(u, 0.5 / 362880, -0.5 / 5040), 0.5 / 120), -0.5 / 6), 0.5);
  } else if (u <= 1.0) {  // next terms below 2^-61
    double pc = 1.0 / 6402373705728000.0, ps = 0.5 / 121645100408832000.0;  // 18!, 19!
    pc = fma(-pc, u, 1.0 / 20922789888000.0);      // 16!
    ps = fma(-ps, u, 0.5 / 355687428096000.0);     // 17!
    pc = fma(-pc, u, 1.0 / 87178291200.0);
    ps = fma(-ps, u, 0.5 / 1307674368000.0);
    pc = fma(-pc, u, 1.0 / 479001600.0);
    ps = fma(-ps, u, 0.5 / 6227020800.0);
    pc = fma(-pc, u, 1.0 / 3628800.0);
    ps = fma(-ps, u, 0.5 / 39916800.0);
    pc = fma(-pc, u, 1.0 / 40320.0);
    ps = fma(-ps, u, 0.5 / 362880.0);
    pc = fma(-pc, u, 1.0 / 720.0);
    ps = fma(-ps, u, 0.5 / 5040.0);
    pc = fma(-pc, u, 1.0 / 24.0);
    ps = fma(-ps, u, 0.5 / 120.0);
    pc = fma(-pc, u, 0.5);
    ps = fma(-ps, u, 0.5 / 6.0);
    c = -pc * u;
    S = fma(-ps, u, 0.5);
  } else {
    const double big = sqrt(t2);
    double s, co;
    sincos_cw(0.5 * big, &s, &co);
    c = co - 1.0;
    S = s / big;
  }
}

__device__ __forceinline__ void exp_half(const double th[4], int /*tau*/, Mat<2>& E) {
  double u, c, S;
  half_coefficients(th, u, c, S);
  E.r[0][0] = c;           E.i[0][0] = -S * th[2];
  E.r[0][1] = -S * th[1];  E.i[0][1] = -S * th[0];
  E.r[1][0] = S * th[1];   E.i[1][0] = -S * th[0];
  E.r[1][1] = c;           E.i[1][1] = S * th[2];
}

// ---------------------------------------------------------------------------
// spin-1 Lie-Trotter exponential (Sec. "Lie-Trotter based exponentiator")
// ---------------------------------------------------------------------------
// T = exp(-iD/2) exp(-i Phi J_phi) exp(-iD/2) with z = theta_z / n,
// q = theta_q / n, Phi = |theta_xy| / n, n = 2^tau (the symmetric split of
// the spin-1 Lie-Trotter step).  With P = diag(e^{-i phi}, 1, e^{i phi}),
// exp(-i Phi J_phi) = P exp(-i Phi J_x) P^H and P commutes with D, so
// T = P T' P^H where T' is the same split at phi = 0.  T' is complex
// symmetric (J_x real symmetric, D diagonal), and so is every residual
// squaring of it (a polynomial in the residual); T^(2^tau) = P T'^(2^tau) P^H.
// The squarings therefore run on the six entries on and above the diagonal
// and the phases e^{-i phi (m_j - m_k)}, m = (1, 0, -1), are put back once.
//
// Complex symmetric 3x3 residual: entries 0..2 the diagonal, 3 = (0,1),
// 4 = (0,2), 5 = (1,2).
struct Sym3 {
  double r[6], i[6];
};

// Residual a' = T' - I, written entry by entry (element-wise form of the
// paper at phi = 0, the T_13 and T_22 misprints corrected); diagonals as
// (e^{i b} - 1) - k S^2 e^{i b} with e^{i b} - 1 = -2 sin^2(b/2) + i sin b,
// so nothing cancels.  Returns e^{i phi} = (theta_x + i theta_y) / rho.
template <bool LEAF = false>
__device__ __forceinline__ void lie_trotter_residual(const double th[4], int tau, Sym3& a,
                                                     double* ep_r, double* ep_i) {
  const double ninv = ldexp(1.0, -tau);
  const double z = th[2] * ninv;
  const double q = th[3] * ninv;
  const double rho = sqrt(fma(th[0], th[0], th[1] * th[1]));  // angles are far from overflow
  const double Phi = rho * ninv;
  double epr = 1.0, epi = 0.0;
  if (rho > 0.0) {
    const double inv = 1.0 / rho;
    epr = th[0] * inv;
    epi = th[1] * inv;
  }
  *ep_r = epr;
  *ep_i = epi;
  double S, C;
  sincos_small<LEAF>(0.5 * Phi, &S, &C);
  const double S2 = S * S;
  const double rs = kRsqrt2 * (2.0 * S * C);  // sin(Phi) / sqrt 2
  double sz, cz, sq, cq;
  sincos_small<LEAF>(0.5 * z, &sz, &cz);           // e^{i z/2}
  sincos_small<LEAF>(q * (1.0 / 6.0), &sq, &cq);   // e^{i q/6}
  // g = e^{iq/6} e^{-iz/2}, h = e^{iq/6} e^{iz/2}
  const double gr = fma(cq, cz, sq * sz), gi = fma(sq, cz, -cq * sz);
  const double hr = fma(cq, cz, -sq * sz), hi = fma(sq, cz, cq * sz);
  // T'_12 = -i rs g, T'_23 = -i rs h; (-i rs) (x + i y) = rs y - i rs x
  a.r[3] = rs * gi;  a.i[3] = -rs * gr;
  a.r[5] = rs * hi;  a.i[5] = -rs * hr;
  // T'_13 = -S^2 e^{-iq/3}
  const double e3r = fma(cq, cq, -sq * sq), e3i = -2.0 * sq * cq;
  a.r[4] = -S2 * e3r;
  a.i[4] = -S2 * e3i;
  // diagonals, b1 = -z - q/3, b2 = 2q/3, b3 = z - q/3: the half-angle
  // exponentials e^{i b_j / 2} are conj(h), conj(e^{-iq/3}) and conj(g)
  const double shv[3] = {-hi, -e3i, -gi};  // sin(b_j / 2)
  const double chv[3] = {hr, e3r, gr};     // cos(b_j / 2)
  const double k[3] = {S2, 2.0 * S2, S2};
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const double sh = shv[j], ch = chv[j];
    const double mr = -2.0 * sh * sh;  // Re(e^{ib} - 1)
    const double mi = 2.0 * sh * ch;   // Im = sin b
    a.r[j] = fma(-k[j], 1.0 + mr, mr);
    a.i[j] = fma(-k[j], mi, mi);
  }
}

// One residual squaring y = (x + 2I) x of a complex symmetric x:
//   y_jj = (x_jj + 2) x_jj + x_jk^2 + x_jl^2
//   y_jk = x_jk (x_jj + 2 + x_kk) + x_jl x_kl        ({j, k, l} = {0, 1, 2})
// 63 instructions where the general 3x3 product takes 111.
__device__ __forceinline__ void residual_square(const Sym3& x, Sym3& y) {
  const double b0 = x.r[0] + 2.0, b1 = x.r[1] + 2.0, b2 = x.r[2] + 2.0;
  // squares of the off-diagonal entries
  double sr[3], si[3];
#pragma unroll
  for (int o = 0; o < 3; ++o) {
    const double xr = x.r[3 + o], xi = x.i[3 + o];
    const double t = xr * xi;
    sr[o] = fma(xr, xr, -xi * xi);
    si[o] = t + t;
  }
  // diagonal j adds the squares of the two off-diagonal entries in its row:
  // row 0: (0,1), (0,2); row 1: (0,1), (1,2); row 2: (0,2), (1,2)
  {
    const double ar = sr[0] + sr[1], ai = si[0] + si[1];
    y.r[0] = fma(b0, x.r[0], fma(-x.i[0], x.i[0], ar));
    y.i[0] = fma(b0, x.i[0], fma(x.i[0], x.r[0], ai));
  }
  {
    const double ar = sr[0] + sr[2], ai = si[0] + si[2];
    y.r[1] = fma(b1, x.r[1], fma(-x.i[1], x.i[1], ar));
    y.i[1] = fma(b1, x.i[1], fma(x.i[1], x.r[1], ai));
  }
  {
    const double ar = sr[1] + sr[2], ai = si[1] + si[2];
    y.r[2] = fma(b2, x.r[2], fma(-x.i[2], x.i[2], ar));
    y.i[2] = fma(b2, x.i[2], fma(x.i[2], x.r[2], ai));
  }
  // (0,1) = x01 (x00 + 2 + x11) + x02 x12
  {
    const double cr = b0 + x.r[1], ci = x.i[0] + x.i[1];
    y.r[3] = fma(x.r[3], cr, fma(-x.i[3], ci, fma(x.r[4], x.r[5], -x.i[4] * x.i[5])));
    y.i[3] = fma(x.r[3], ci, fma(x.i[3], cr, fma(x.r[4], x.i[5], x.i[4] * x.r[5])));
  }
  // (0,2) = x02 (x00 + 2 + x22) + x01 x12
  {
    const double cr = b0 + x.r[2], ci = x.i[0] + x.i[2];
    y.r[4] = fma(x.r[4], cr, fma(-x.i[4], ci, fma(x.r[3], x.r[5], -x.i[3] * x.i[5])));
    y.i[4] = fma(x.r[4], ci, fma(x.i[4], cr, fma(x.r[3], x.i[5], x.i[3] * x.r[5])));
  }
  // (1,2) = x12 (x11 + 2 + x22) + x01 x02
  {
    const double cr = b1 + x.r[2], ci = x.i[1] + x.i[2];
    y.r[5] = fma(x.r[5], cr, fma(-x.i[5], ci, fma(x.r[3], x.r[4], -x.i[3] * x.i[4])));
    y.i[5] = fma(x.r[5], ci, fma(x.i[5], cr, fma(x.r[3], x.i[4], x.i[3] * x.r[4])));
  }
}

// M = P (s + d I) P^H for a complex symmetric s: the off-diagonal entries
// take the phases e^{-i phi (m_j - m_k)}, m = (1, 0, -1), of
// e^{i phi} = (epr, epi); d is added to the real diagonal.
__device__ __forceinline__ void sym_to_full(const Sym3& s, double d, double epr, double epi,
                                            Mat<3>& M) {
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    M.r[j][j] = s.r[j] + d;
    M.i[j][j] = s.i[j];
  }
  // (0,1), (1,2) carry e^{-i phi}, (1,0), (2,1) carry e^{i phi}
  M.r[0][1] = fma(s.r[3], epr, s.i[3] * epi);
  M.i[0][1] = fma(s.i[3], epr, -s.r[3] * epi);
  M.r[1][0] = fma(s.r[3], epr, -s.i[3] * epi);
  M.i[1][0] = fma(s.i[3], epr, s.r[3] * epi);
  M.r[1][2] = fma(s.r[5], epr, s.i[5] * epi);
  M.i[1][2] = fma(s.i[5], epr, -s.r[5] * epi);
  M.r[2][1] = fma(s.r[5], epr, -s.i[5] * epi);
  M.i[2][1] = fma(s.i[5], epr, s.r[5] * epi);
  // (0,2) carries e^{-2i phi}, (2,0) carries e^{2i phi}
  const double e2r = fma(epr, epr, -epi * epi), e2i = 2.0 * epr * epi;
  M.r[0][2] = fma(s.r[4], e2r, s.i[4] * e2i);
  M.i[0][2] = fma(s.i[4], e2r, -s.r[4] * e2i);
  M.r[2][0] = fma(s.r[4], e2r, -s.i[4] * e2i);
  M.i[2][0] = fma(s.i[4], e2r, s.r[4] * e2i);
}

// tau residual squarings a' <- (a' + 2I) a' (two per trip, alternating
// between two register sets, so nothing is copied): E = P (I + a') P^H.  Any
// tau and any angles; exp_one takes it only where the split at n = 2^tau can
// be told from the exponential itself.  Entries j of a' at 2j and 2j + 1, then
// e^{i phi}.
using SplitPower = double __attribute__((ext_vector_type(16)));
__device__ __forceinline__ SplitPower split_power(const double th[4], int tau) {
  Sym3 a, b;
  double epr, epi;
  lie_trotter_residual<true>(th, tau, a, &epr, &epi);
  for (int s = 0; s + 2 <= tau; s += 2) {
    residual_square(a, b);
    residual_square(b, a);
  }
  if (tau & 1) {
    residual_square(a, b);
    a = b;
  }
  SplitPower v;
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    v[2 * j] = a.r[j];
    v[2 * j + 1] = a.i[j];
  }
  v[12] = epr;
  v[13] = epi;
  return v;
}
// As a call, so that the code is there once and its registers bind no caller.
// Arguments and result pass in registers (a structure of 14 doubles would come
// back through memory), and nothing is called from it, so that its return
// address stays in registers too: 1e5 spin-1 intervals of 10 fine steps at
// tau = 0, 12 and 22, all angles by the squarings: 65, 115 and 148 us with a
// structure and a call inside, 35, 93 and 133 now; without a call (integrators
// that knew nothing but squarings) 32, 83 and 128.
__device__ __attribute__((noinline)) SplitPower split_power_call(double x, double y, double z,
                                                                 double q, int tau) {
  const double th[4] = {x, y, z, q};
  return split_power(th, tau);
}

// The spin-1 exponential in closed form.
//
// The generator G = theta_x J_x + theta_y J_y + theta_z J_z + theta_q Q is
// traceless Hermitian, so G^3 = p G + d with p = tr G^2 / 2 and d = det G,
// and exp(-i G) = C - i S with C = cos G and S = sin G both real
// combinations of I, G and G^2.  Horner's rule on the Taylor series keeps
// three real coefficients (a, b, c) of a I + b G + c G^2; one more factor G
// maps them to (d c, a + p c, b): two FMAs a degree and part.
//
// The tau-fold squaring of the split T computes T^n, n = 2^tau, and
// T^n = exp(-i (G + G_3 / n^2 + ...)) with G_3 the Strang splitting's double
// commutators, |G_3| <= v^2 r / 24 + r^2 (|theta_z| + 4 |theta_q|) / 12 with
// v = |theta_z| + |theta_q| and r = |theta_xy|, at most 0.3 p^{3/2}.  Where
// p <= 2^(2 tau - 53) the difference from G is below 2^-54 |G|, less than
// the rounding of the angles themselves, and the closed form gives the
// scheme's exponential to rounding (with some 20 roundings where the
// squarings take some 10 tau).  tau = 28 allows p <= 8 and tau = 24
// p <= 2^-5; lower tau or larger angles take the squarings.
struct Gen3 {
  double a[3];    // diagonal of G
  double wr, wi;  // G_01 = G_12 = w = (theta_x - i theta_y) / sqrt 2; G_02 = 0
  double h;       // |w|^2
  double p, d;
};

__device__ __forceinline__ void generator(const double th[4], Gen3& g) {
#pragma clang fp contract(off)
  const double z = th[2], q3 = th[3] * (1.0 / 3.0);
  g.a[0] = z + q3;
  g.a[1] = -2.0 * q3;
  g.a[2] = q3 - z;
  g.wr = kRsqrt2 * th[0];
  g.wi = -kRsqrt2 * th[1];
  g.h = fma(g.wr, g.wr, g.wi * g.wi);
  const double z2 = z * z;
  g.p = fma(2.0, g.h, fma(3.0 * q3, q3, z2));
  // det G = a_0 a_1 a_2 - h (a_0 + a_2) = 2 q3 (z^2 - q3^2 - h)
  g.d = (2.0 * q3) * (fma(-q3, q3, z2) - g.h);
}

// 1 / k!
constexpr double kInvFact[20] = {
    1.0, 1.0, 1.0 / 2, 1.0 / 6, 1.0 / 24, 1.0 / 120, 1.0 / 720, 1.0 / 5040, 1.0 / 40320,
    1.0 / 362880, 1.0 / 3628800, 1.0 / 39916800, 1.0 / 479001600, 1.0 / 6227020800.0,
    1.0 / 87178291200.0, 1.0 / 1307674368000.0, 1.0 / 20922789888000.0,
    1.0 / 355687428096000.0, 1.0 / 6402373705728000.0, 1.0 / 121645100408832000.0};

// One part's coefficients over (I, G, G^2), the series to G^M without its
// constant term: x, and with TANGENT dx, their derivative along a direction
// (dp, dd) of (p, d).
template <int M, bool TANGENT>
__device__ __forceinline__ void series_part(double p, double d, double dp, double dd, double x[3],
                                            double dx[3]) {
  static_assert(M >= 6, "");
  constexpr double sign = (M / 2) % 2 ? -1.0 : 1.0;  // of G^M
  // The top powers are (c_{M-2}, 0, c_M); two factors G lead to
  // (c_{M-4}, d c_M, c_{M-2} + p c_M), without the products with 0.
  double a = sign * kInvFact[M - 4];
  double b = d * (sign * kInvFact[M]);
  double e = fma(p, sign * kInvFact[M], -sign * kInvFact[M - 2]);
  double ta = 0.0, tb = 0.0, te = 0.0;
  if constexpr (TANGENT) {
    tb = dd * (sign * kInvFact[M]);
    te = dp * (sign * kInvFact[M]);
  }
#pragma unroll
  for (int k = M - 5; k >= 0; --k) {
    if constexpr (TANGENT) {
      const double na = fma(dd, e, d * te);
      const double nb = k == M - 5 ? fma(dp, e, p * te) : fma(dp, e, fma(p, te, ta));
      te = tb;
      ta = na;
      tb = nb;
    }
    const bool term = k % 2 == M % 2 && k > 0;
    const double na = term ? fma(d, e, ((k / 2) % 2 ? -1.0 : 1.0) * kInvFact[k]) : d * e;
    const double nb = fma(p, e, a);
    e = b;
    a = na;
    b = nb;
  }
  x[0] = a;
  x[1] = b;
  x[2] = e;
  if constexpr (TANGENT) {
    dx[0] = ta;
    dx[1] = tb;
    dx[2] = te;
  }
}

// Coefficients of C - I (series to G^MC) and of S (to G^MS).
template <int MC, int MS>
__device__ __forceinline__ void series(double p, double d, double c[3], double s[3]) {
  static_assert(MC % 2 == 0 && MS % 2 == 1, "");
  series_part<MC, false>(p, d, 0.0, 0.0, c, nullptr);
  series_part<MS, false>(p, d, 0.0, 0.0, s, nullptr);
}

// E = I + (c_0 + c_1 G + c_2 G^2) - i (s_0 + s_1 G + s_2 G^2).  With a
// traceless diagonal G^2 has the entries (a_j^2 + h, a_1^2 + 2 h, ...) on the
// diagonal, -a_2 w and -a_0 w beside it, and w^2 in the corner.
__device__ __forceinline__ void assemble(const Gen3& g, const double c[3], const double s[3],
                                         Mat<3>& E) {
#pragma clang fp contract(off)
  const double sq[3] = {fma(g.a[0], g.a[0], g.h), fma(g.a[1], g.a[1], 2.0 * g.h),
                        fma(g.a[2], g.a[2], g.h)};
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    E.r[j][j] = 1.0 + fma(c[2], sq[j], fma(c[1], g.a[j], c[0]));
    E.i[j][j] = -fma(s[2], sq[j], fma(s[1], g.a[j], s[0]));
  }
  // beside the diagonal: (kr - i ki) w above, (kr - i ki) conj w below
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const double other = g.a[2 - 2 * j];
    const double kr = fma(-c[2], other, c[1]), ki = fma(-s[2], other, s[1]);
    const double rr = kr * g.wr, ii = ki * g.wi, ri = kr * g.wi, ir = ki * g.wr;
    E.r[j][j + 1] = rr + ii;
    E.i[j][j + 1] = ri - ir;
    E.r[j + 1][j] = rr - ii;
    E.i[j + 1][j] = -ri - ir;
  }
  const double vr = fma(g.wr, g.wr, -(g.wi * g.wi)), vi = 2.0 * (g.wr * g.wi);  // w^2
  const double rr = c[2] * vr, ii = s[2] * vi, ri = c[2] * vi, ir = s[2] * vr;
  E.r[0][2] = rr + ii;
  E.i[0][2] = ri - ir;
  E.r[2][0] = rr - ii;
  E.i[2][0] = -ri - ir;
}

// Bounds on p = tr G^2 / 2 (the eigenvalues of G are at most sqrt(4 p / 3)):
// to the first, |lambda| <= 2^-6, the series to G^6 and G^7 is exact to
// 2^-63 and 2^-66 relative; to the second, |lambda| <= 1, to G^18 and G^17
// to 2^-61 and 2^-56.
constexpr double kShortSeries = 0x1.8p-13;
constexpr double kLongSeries = 0.75;

// E = exp(-i G) of the step angles: the closed form where it is the
// scheme's exponential to rounding (above), else the squarings.  About 75
// instructions against 1,830 at tau = 28 (62 a squaring), and a third of
// the error (angles of 3e-4: E - I off by 7.1e-20 against 2.1e-19).
// 4096 spin-1 simulations, 4.5e7 intervals of 10 fine steps in one chained
// launch: 54.2 ms with the squarings, 9.0 ms with the series (7.0 with two
// columns of the product besides); one of 2e5 intervals, scan included: 298 and
// 91 us (79).
template <bool INLINE = false>
__device__ __forceinline__ void exp_one(const double th[4], int tau, Mat<3>& E) {
  Gen3 g;
  generator(th, g);
  const double most = ldexp(1.0, 2 * tau - 53);
  double c[3], s[3];
  if (g.p <= fmin(most, kShortSeries)) {
    series<6, 7>(g.p, g.d, c, s);
  } else if (g.p <= fmin(most, kLongSeries)) {
    series<18, 17>(g.p, g.d, c, s);
  } else {  // also angles that are not finite
    SplitPower v;
    if constexpr (INLINE) v = split_power(th, tau);
    else v = split_power_call(th[0], th[1], th[2], th[3], tau);
    Sym3 a;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      a.r[j] = v[2 * j];
      a.i[j] = v[2 * j + 1];
    }
    sym_to_full(a, 1.0, v[12], v[13], E);
    return;
  }
  assemble(g, c, s, E);
}

template <int N> struct Exponentiator;
template <> struct Exponentiator<2> {
  template <bool INLINE = false>
  static __device__ __forceinline__ void apply(const double th[4], int tau, Mat<2>& E) {
    exp_half(th, tau, E);
  }
};
template <> struct Exponentiator<3> {
  template <bool INLINE = false>
  static __device__ __forceinline__ void apply(const double th[4], int tau, Mat<3>& E) {
    exp_one<INLINE>(th, tau, E);
  }
};

// ---------------------------------------------------------------------------
// field program interpreter and node arithmetic.  Multiply-adds are kept
// unfused here, so node times and phase arguments (up to ~1e6 rad) round
// exactly as the plain definition t_k = t_start + k Dt,
// tau_i = (l + c_i) dt, phase = 2 pi (f t) + phi prescribes.
// ---------------------------------------------------------------------------
// The field over C components (4, or 8 in the full basis) comes in two parts.
// field_constant: the components whose terms are all constant, once per
// interval; the others 0.
template <int C, class Terms>
__device__ __forceinline__ void field_constant(const Terms& fp, const double* __restrict__ params,
                                               double (&fc)[C]) {
#pragma clang fp contract(off)
#pragma unroll
  for (int j = 0; j < C; ++j) fc[j] = 0.0;
  const int nt = fp.size();
  for (int n = fp.varying(); n < nt; ++n) {
    const auto& tm = fp[n];
    const double v = tm.a_slot >= 0 ? as_constant(params)[tm.a_slot] : tm.a;
    const int comp = tm.comp;
#pragma unroll
    for (int j = 0; j < C; ++j)
      if (comp == j) fc[j] = fc[j] + v;  // uniform across the wave
  }
}

template <int M>
__device__ __forceinline__ bool any_of(const bool (&on)[M]) {
  bool any = false;
#pragma unroll
  for (int i = 0; i < M; ++i) any = any || on[i];
  return any;
}

// field_at: the whole field at M times, the constant part given: one walk
// over the varying terms for all of them (each term is read once, and the M
// chains of dependent operations run side by side).  only >= 0: no other
// component is wanted.  Terms of one component are summed in list order.
// What bounds the interpreter is the latency of its scalar loads and
// branches between the sines: 1e6 spin-1 intervals of 10 fine steps, sensing
// drive, took 391 us with a walk over all terms at every node and take 220
// (156 with the field compiled in); 3e5 spin-1/2 intervals of 20, 103 and 73.
template <int C, int M, class Terms>
__device__ __forceinline__ void field_at(const Terms& fp, const double* __restrict__ params,
                                         const double (&fc)[C], const double (&t)[M],
                                         double (&f)[M][C], int only = -1) {
#pragma clang fp contract(off)
#pragma unroll
  for (int i = 0; i < M; ++i)
#pragma unroll
    for (int j = 0; j < C; ++j) f[i][j] = fc[j];
  const int nt = fp.varying();
  for (int n = 0; n < nt; ++n) {
    const auto& tm = fp[n];
    const int comp = tm.comp, kind = tm.kind;
    if (only >= 0 && comp != only) continue;
    const double t_on = tm.t_on, t_off = tm.t_off;
    bool on[M];
#pragma unroll
    for (int i = 0; i < M; ++i) on[i] = t_on < t[i] && t[i] < t_off;
    if (!any_of(on)) continue;
    const double a = tm.a_slot >= 0 ? as_constant(params)[tm.a_slot] : tm.a;
    double amp[M], v[M];
#pragma unroll
    for (int i = 0; i < M; ++i) amp[i] = a;
    int seg[M];
    if (kind >= MSS_TERM_PWC) {
      const double t0 = tm.seg_t0, len = tm.seg_len;
      const int last = tm.n_seg - 1;
#pragma unroll
      for (int i = 0; i < M; ++i) {
        const double x = (t[i] - t0) / len;
        const double fl = floor(x);
        seg[i] = fl < 0.0 ? 0 : (fl > (double)last ? last : (int)fl);
        if (tm.seg_a_slot >= 0) amp[i] = params[tm.seg_a_slot + seg[i]];
      }
    }
    if (kind == MSS_TERM_CONST || kind == MSS_TERM_PWC) {
#pragma unroll
      for (int i = 0; i < M; ++i) v[i] = amp[i];
    } else {
      const double fr = tm.f_slot >= 0 ? as_constant(params)[tm.f_slot] : tm.f;
      const double phi = tm.phi_slot >= 0 ? as_constant(params)[tm.phi_slot] : tm.phi;
      double arg[M], sn[M], cs[M];
#pragma unroll
      for (int i = 0; i < M; ++i) {
        double ph = phi;
        if (kind >= MSS_TERM_PWC && tm.seg_phi_slot >= 0) ph = params[tm.seg_phi_slot + seg[i]];
        const double ft = fr * t[i];
        const double x = kTwoPi * ft;
        arg[i] = x + ph;
      }
      sincos_cw(arg, sn, cs);
      const bool is_cos = kind == MSS_TERM_COS || kind == MSS_TERM_PWC_COS;
#pragma unroll
      for (int i = 0; i < M; ++i) v[i] = amp[i] * (is_cos ? cs[i] : sn[i]);
    }
#pragma unroll
    for (int j = 0; j < C; ++j)
      if (comp == j) {
#pragma unroll
        for (int i = 0; i < M; ++i) f[i][j] = on[i] ? f[i][j] + v[i] : f[i][j];
      }
  }
}

// Frame rotations of the two CF4 nodes of a run of fine steps: cos and sin
// of wr tau_i at tau_i = (l + c_i) dt, taken directly at the run's first
// step and advanced by the rotation over one fine step (angle addition),
// so a step costs two complex products instead of two sines and cosines.
struct NodeRotations {
  double c[2], s[2];  // cos, sin of wr tau_i for the current step
  double cd, sd;      // cos, sin of wr dt
  __device__ __forceinline__ void start(double wr, int l, double dt) {
#pragma clang fp contract(off)
    const double x[3] = {wr * (((double)l + kNode1) * dt), wr * (((double)l + kNode2) * dt),
                         wr * dt};
    double sn[3], cs[3];
    sincos_cw(x, sn, cs);
    s[0] = sn[0];
    s[1] = sn[1];
    sd = sn[2];
    c[0] = cs[0];
    c[1] = cs[1];
    cd = cs[2];
  }
  __device__ __forceinline__ void advance() {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const double cn = fma(c[i], cd, -s[i] * sd);
      const double sn = fma(s[i], cd, c[i] * sd);
      c[i] = cn;
      s[i] = sn;
    }
  }
  // to the step before
  __device__ __forceinline__ void retreat() {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const double cn = fma(c[i], cd, s[i] * sd);
      const double sn = fma(s[i], cd, -(c[i] * sd));
      c[i] = cn;
      s[i] = sn;
    }
  }
};

// Node i of the fine step starting at t_k + l dt: its offset from t_k.
__device__ __forceinline__ double node_offset(int i, int l, double dt) {
#pragma clang fp contract(off)
  return ((double)l + (i == 0 ? kNode1 : kNode2)) * dt;
}

// Angular rates w of a node from its field f, in the frame rotating at wr
// about z whose angle there has cosine c and sine s (wr = 0: lab frame; c
// and s are then not read).
__device__ __forceinline__ void node_rates(const double f[4], double wr, double c, double s,
                                           double w[4]) {
#pragma clang fp contract(off)
#pragma unroll
  for (int j = 0; j < 4; ++j) w[j] = kTwoPi * f[j];
  if (wr != 0.0) {
    // (w_x + i w_y) e^{-i wr tau_i}
    const double xr = w[0] * c + w[1] * s;
    const double xi = w[1] * c - w[0] * s;
    w[0] = xr;
    w[1] = xi;
    w[2] = w[2] - wr;
  }
}

// The two exponentials' angles from the rates of both nodes.
__device__ __forceinline__ void cf4_combine(const double w[2][4], double dt, double th1[4],
                                            double th2[4]) {
#pragma clang fp contract(off)
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    th1[j] = (kWPlus * w[0][j] + kWMinus * w[1][j]) * dt;
    th2[j] = (kWMinus * w[0][j] + kWPlus * w[1][j]) * dt;
  }
}

// Angles theta_{1,2} = omega_bar_{1,2} dt of one CF4 fine step starting at
// t_k + l dt, in the frame rotating at wr about z (wr = 0: lab frame; then
// rot is not read).
template <class Terms>
__device__ __forceinline__ void cf4_angles(const Terms& fp, const double* __restrict__ params,
                                           const double (&fc)[4], double tk, int l, double dt,
                                           double wr, const NodeRotations& rot, double th1[4],
                                           double th2[4]) {
#pragma clang fp contract(off)
  const double t[2] = {tk + node_offset(0, l, dt), tk + node_offset(1, l, dt)};
  double f[2][4], w[2][4];
  field_at(fp, params, fc, t, f);
#pragma unroll
  for (int i = 0; i < 2; ++i) node_rates(f[i], wr, rot.c[i], rot.s[i], w[i]);
  cf4_combine(w, dt, th1, th2);
}

// Angles of one Euler-family step (one exponential): H sampled at the
// midpoint (method 1) or averaged over both ends of the step (method 2).
template <class Terms>
__device__ __forceinline__ void euler_angles(const Terms& fp, const double* __restrict__ params,
                                             const double (&fc)[4], double tk, int l, double dt,
                                             double wr, int method, double th[4]) {
#pragma clang fp contract(off)
  const int nn = method == 1 ? 1 : 2;
  double w[2][4];
  for (int i = 0; i < nn; ++i) {
    const double c = method == 1 ? 0.5 : (i == 0 ? 0.0 : 1.0);
    const double tau_i = ((double)l + c) * dt;
    const double t[1] = {tk + tau_i};
    double f[1][4], s = 0.0, cs = 1.0;
    field_at(fp, params, fc, t, f);
    if (wr != 0.0) sincos_cw(wr * tau_i, &s, &cs);
    node_rates(f[0], wr, cs, s, w[i]);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) th[j] = (method == 1 ? w[0][j] : (w[0][j] + w[1][j]) / 2.0) * dt;
}

// Start time of interval k and the frame rate omega_r = 2 pi f_z(t_k + Dt/2)
// (fc: the constant part of the field).
template <int C, class Terms>
__device__ __forceinline__ void interval_setup(const Terms& fp, const double* __restrict__ params,
                                               const double (&fc)[C], double t_start, double Dt,
                                               int64_t k, int frame, double* tk_out,
                                               double* wr_out) {
#pragma clang fp contract(off)
  const double tk = t_start + (double)k * Dt;
  double wr = 0.0;
  if (frame) {
    const double t[1] = {tk + Dt / 2.0};
    double f[1][C];
    field_at(fp, params, fc, t, f, MSS_Z);
    wr = kTwoPi * f[0][MSS_Z];
  }
  *tk_out = tk;
  *wr_out = wr;
}

// U <- diag(exp(-i m wr Dt)) U, m = +s ... -s  (eq. exit_rotating_frame)
template <int N>
__device__ __forceinline__ void exit_frame(double wr, double Dt, Mat<N>& U) {
  if (wr == 0.0) return;
  const double beta = wr * Dt;
  // the two outer levels turn by opposite angles
  double s0, c;
  sincos_cw((N == 2 ? -0.5 : -1.0) * beta, &s0, &c);
#pragma unroll
  for (int a = 0; a < N; ++a) {
    if (N == 3 && a == 1) continue;
    const double s = a == 0 ? s0 : -s0;
#pragma unroll
    for (int b = 0; b < N; ++b) {
      const double xr = U.r[a][b], xi = U.i[a][b];
      U.r[a][b] = fma(c, xr, -s * xi);
      U.i[a][b] = fma(c, xi, s * xr);
    }
  }
}

// ---------------------------------------------------------------------------
// spin-1 in the full su(3) basis: components x, y, z, q, u1, u2, v1, v2 of
// H = 2 pi (f_x J_x + f_y J_y + f_z J_z + f_q Q + f_u1 U_1 + f_u2 U_2 + f_v1 V_1
// + f_v2 V_2), with U_1 = J_x^2 - J_y^2, U_2 = J_x J_y + J_y J_x (Delta m = 2)
// and V_1 = J_z J_x + J_x J_z, V_2 = J_y J_z + J_z J_y (Delta m = 1).  A
// spin-1 problem takes this path when a term is on u1, u2, v1 or v2.
// ---------------------------------------------------------------------------
constexpr int kFullComps = 8;

// Node field in the rotating frame: (x + i y) and (v1 + i v2) times
// e^{-i wr tau}, (u1 + i u2) times e^{-2i wr tau} (Delta m = 1 and 2 under
// rotations about z), z - wr; (c, s) = (cos, sin)(wr tau).
__device__ __forceinline__ void frame_full(double w[kFullComps], double c, double s, double wr) {
#pragma clang fp contract(off)
  const double c2 = c * c - s * s, s2 = 2.0 * (c * s);
  const double xr = w[0] * c + w[1] * s, xi = w[1] * c - w[0] * s;
  const double ur = w[4] * c2 + w[5] * s2, ui = w[5] * c2 - w[4] * s2;
  const double vr = w[6] * c + w[7] * s, vi = w[7] * c - w[6] * s;
  w[0] = xr;
  w[1] = xi;
  w[2] = w[2] - wr;
  w[4] = ur;
  w[5] = ui;
  w[6] = vr;
  w[7] = vi;
}

template <class Terms>
__device__ __forceinline__ void cf4_angles_full(const Terms& fp, const double* __restrict__ params,
                                                const double (&fc)[kFullComps], double tk, int l,
                                                double dt, double wr, const NodeRotations& rot,
                                                double th1[kFullComps], double th2[kFullComps]) {
#pragma clang fp contract(off)
  const double t[2] = {tk + node_offset(0, l, dt), tk + node_offset(1, l, dt)};
  double w[2][kFullComps];
  field_at(fp, params, fc, t, w);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
#pragma unroll
    for (int j = 0; j < kFullComps; ++j) w[i][j] = kTwoPi * w[i][j];
    if (wr != 0.0) frame_full(w[i], rot.c[i], rot.s[i], wr);
  }
#pragma unroll
  for (int j = 0; j < kFullComps; ++j) {
    th1[j] = (kWPlus * w[0][j] + kWMinus * w[1][j]) * dt;
    th2[j] = (kWMinus * w[0][j] + kWPlus * w[1][j]) * dt;
  }
}

template <class Terms>
__device__ __forceinline__ void euler_angles_full(const Terms& fp,
                                                  const double* __restrict__ params,
                                                  const double (&fc)[kFullComps], double tk, int l,
                                                  double dt, double wr, int method,
                                                  double th[kFullComps]) {
#pragma clang fp contract(off)
  const int nn = method == 1 ? 1 : 2;
  double w[2][kFullComps] = {};
#pragma unroll
  for (int i = 0; i < 2; ++i) {  // a fixed trip count keeps w in registers
    if (i >= nn) break;
    const double c = method == 1 ? 0.5 : (i == 0 ? 0.0 : 1.0);
    const double tau_i = ((double)l + c) * dt;
    const double t[1] = {tk + tau_i};
    double f[1][kFullComps];
    field_at(fp, params, fc, t, f);
#pragma unroll
    for (int j = 0; j < kFullComps; ++j) w[i][j] = kTwoPi * f[0][j];
    if (wr != 0.0) {
      double s, cs;
      sincos_cw(wr * tau_i, &s, &cs);
      frame_full(w[i], cs, s, wr);
    }
  }
#pragma unroll
  for (int j = 0; j < kFullComps; ++j)
    th[j] = (method == 1 ? w[0][j] : (w[0][j] + w[1][j]) / 2.0) * dt;
}

// One general residual squaring y = (x + 2I) x.
__device__ __forceinline__ void residual_square_full(const Mat<3>& x, Mat<3>& y) {
  Mat<3> b = x;
  b.r[0][0] += 2.0;
  b.r[1][1] += 2.0;
  b.r[2][2] += 2.0;
  matmul<3>(b, x, y);
}

// exp(-i G), G = sum_j theta_j A_j over the full basis, by scaling and
// squaring: X = -i G / n with n = 2^tau, the residual of exp(X) from its
// degree-4 Taylor polynomial in Horner form, X (I + X/2 (I + X/3 (I + X/4)))
// (no identity term, nothing cancels), then tau residual squarings, I + a.
__device__ __attribute__((noinline)) void exp_full_squarings(const double th[kFullComps],
                                                             int tau, Mat<3>& E) {
  const double ninv = ldexp(1.0, -tau);
  // G entry by entry: J_x, J_y, V_1, V_2 couple neighbouring levels (1/sqrt 2),
  // U_1, U_2 the outer pair; J_z and Q on the diagonal.
  const double g00 = th[2] + th[3] * (1.0 / 3.0);
  const double g11 = th[3] * (-2.0 / 3.0);
  const double g22 = -th[2] + th[3] * (1.0 / 3.0);
  const double g01r = kRsqrt2 * (th[0] + th[6]), g01i = -kRsqrt2 * (th[1] + th[7]);
  const double g12r = kRsqrt2 * (th[0] - th[6]), g12i = -kRsqrt2 * (th[1] - th[7]);
  const double g02r = th[4], g02i = -th[5];
  // X = -i G / n: -i (gr + i gi) = gi - i gr; the lower triangle holds conj(G)
  Mat<3> X;
  X.r[0][0] = 0.0;  X.i[0][0] = -g00 * ninv;
  X.r[1][1] = 0.0;  X.i[1][1] = -g11 * ninv;
  X.r[2][2] = 0.0;  X.i[2][2] = -g22 * ninv;
  X.r[0][1] = g01i * ninv;   X.i[0][1] = -g01r * ninv;
  X.r[1][0] = -g01i * ninv;  X.i[1][0] = -g01r * ninv;
  X.r[1][2] = g12i * ninv;   X.i[1][2] = -g12r * ninv;
  X.r[2][1] = -g12i * ninv;  X.i[2][1] = -g12r * ninv;
  X.r[0][2] = g02i * ninv;   X.i[0][2] = -g02r * ninv;
  X.r[2][0] = -g02i * ninv;  X.i[2][0] = -g02r * ninv;
  Mat<3> a, t;
#pragma unroll
  for (int p = 0; p < 3; ++p)
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      a.r[p][q] = X.r[p][q] * 0.25 + (p == q ? 1.0 : 0.0);
      a.i[p][q] = X.i[p][q] * 0.25;
    }
  const double inv_k[2] = {1.0 / 3.0, 0.5};
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    matmul<3>(X, a, t);
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        a.r[p][q] = t.r[p][q] * inv_k[h] + (p == q ? 1.0 : 0.0);
        a.i[p][q] = t.i[p][q] * inv_k[h];
      }
  }
  matmul<3>(X, a, t);
  for (int s = 0; s + 2 <= tau; s += 2) {
    residual_square_full(t, a);
    residual_square_full(a, t);
  }
  if (tau & 1) {
    residual_square_full(t, a);
    t = a;
  }
  E = t;
  E.r[0][0] += 1.0;
  E.r[1][1] += 1.0;
  E.r[2][2] += 1.0;
}

// exp(-i G) of the full basis: the closed form of exp_one with all of G's
// entries, where the squarings' starting polynomial can't be told from the
// exponential: their result is exp(-i G (1 + e)), |e| <= |lambda|^4 /
// (120 n^4), below 2^-56 for p <= 2^(2 tau - 25).  Else the squarings.
__device__ __forceinline__ void exp_full(const double th[kFullComps], int tau, Mat<3>& E) {
#pragma clang fp contract(off)
  const double q3 = th[3] * (1.0 / 3.0);
  const double a0 = th[2] + q3, a1 = -2.0 * q3, a2 = q3 - th[2];
  const double xr = kRsqrt2 * (th[0] + th[6]), xi = -kRsqrt2 * (th[1] + th[7]);  // G_01
  const double yr = kRsqrt2 * (th[0] - th[6]), yi = -kRsqrt2 * (th[1] - th[7]);  // G_12
  const double ur = th[4], ui = -th[5];                                          // G_02
  const double hx = fma(xr, xr, xi * xi), hy = fma(yr, yr, yi * yi), hu = fma(ur, ur, ui * ui);
  const double xyr = fma(xr, yr, -(xi * yi)), xyi = fma(xr, yi, xi * yr);  // G_01 G_12
  const double p = fma(q3, 3.0 * q3, fma(th[2], th[2], hx + hy + hu));
  // a_0 a_1 a_2 + 2 Re(G_01 G_12 conj G_02) - a_0 |G_12|^2 - a_1 |G_02|^2 - a_2 |G_01|^2
  const double d = fma(a0, fma(a1, a2, -hy),
                       fma(2.0, fma(xyr, ur, xyi * ui), -fma(a1, hu, a2 * hx)));
  const double most = ldexp(1.0, 2 * tau - 25);
  double c[3], s[3];
  if (p <= fmin(most, kShortSeries)) {
    series<6, 7>(p, d, c, s);
  } else if (p <= fmin(most, kLongSeries)) {
    series<18, 17>(p, d, c, s);
  } else {  // also angles that are not finite
    double angles[kFullComps];  // copies, so that the caller's stay in registers
    Mat<3> F;
#pragma unroll
    for (int j = 0; j < kFullComps; ++j) angles[j] = th[j];
    exp_full_squarings(angles, tau, F);
    E = F;
    return;
  }
  const double a[3] = {a0, a1, a2};
  const double sq[3] = {fma(a0, a0, hx + hu), fma(a1, a1, hx + hy), fma(a2, a2, hy + hu)};
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    E.r[j][j] = 1.0 + fma(c[2], sq[j], fma(c[1], a[j], c[0]));
    E.i[j][j] = -fma(s[2], sq[j], fma(s[1], a[j], s[0]));
  }
  // above the diagonal G and G^2 have the entries (0,1): G_01, -a_2 G_01 +
  // G_02 conj G_12; (1,2): G_12, -a_0 G_12 + conj G_01 G_02; (0,2): G_02,
  // -a_1 G_02 + G_01 G_12; below it their conjugates
  const double gr[3] = {xr, yr, ur}, gi[3] = {xi, yi, ui};
  const double tr[3] = {fma(-a2, xr, fma(ur, yr, ui * yi)), fma(-a0, yr, fma(xr, ur, xi * ui)),
                        fma(-a1, ur, xyr)};
  const double ti[3] = {fma(-a2, xi, fma(ui, yr, -(ur * yi))), fma(-a0, yi, fma(xr, ui, -(xi * ur))),
                        fma(-a1, ui, xyi)};
  const int row[3] = {0, 1, 0}, col[3] = {1, 2, 2};
#pragma unroll
  for (int o = 0; o < 3; ++o) {
    const double cr = fma(c[2], tr[o], c[1] * gr[o]), ci = fma(c[2], ti[o], c[1] * gi[o]);
    const double sr = fma(s[2], tr[o], s[1] * gr[o]), si = fma(s[2], ti[o], s[1] * gi[o]);
    // (cr + i ci) - i (sr + i si), and with both conjugated below
    E.r[row[o]][col[o]] = cr + si;
    E.i[row[o]][col[o]] = ci - sr;
    E.r[col[o]][row[o]] = cr - si;
    E.i[col[o]][row[o]] = -ci - sr;
  }
}

// The wave's issue priority, rotated with a wave-uniform count: the hardware
// slot number offsets the rotation, so waves sharing a SIMD take turns at
// the highest of the four levels and advance at the same rate.  (Among waves
// of equal priority the arbiter prefers the older one, which in a
// persistent launch with two blocks per CU runs the first block's waves
// about 2.4 times as fast as the second's for the whole launch.)
__device__ __forceinline__ void rotate_priority(int count, int slot) {
  switch (__builtin_amdgcn_readfirstlane(count + slot) & 3) {
    case 0: __builtin_amdgcn_s_setprio(0); break;
    case 1: __builtin_amdgcn_s_setprio(1); break;
    case 2: __builtin_amdgcn_s_setprio(2); break;
    default: __builtin_amdgcn_s_setprio(3); break;
  }
}

// The wave's slot on its SIMD (HW_ID bits 3:0).
__device__ __forceinline__ int wave_slot() {
  return (int)(__builtin_amdgcn_s_getreg(4 | (3 << 11)) & 15u);
}

// The fine steps l0 .. l1 of an interval, into R.  INLINE: with the
// squarings in the loop instead of a call.
template <int N, bool INLINE, class Terms>
__device__ __forceinline__ void integrate_slice(const Terms& terms, const double* __restrict__ params,
                                                const double (&fc)[4], double tk, int l0, int l1,
                                                double dt, double wr, int tau, int method,
                                                Running<N, false>& R) {
  if (method == 0) {
    NodeRotations rot;
    if (wr != 0.0) rot.start(wr, l0, dt);
    for (int l = l0; l < l1; ++l) {
      double th1[4], th2[4];
      cf4_angles(terms, params, fc, tk, l, dt, wr, rot, th1, th2);
      if (wr != 0.0) rot.advance();
      Mat<N> E;
      Exponentiator<N>::template apply<INLINE>(th1, tau, E);
      R.multiply(E);
      Exponentiator<N>::template apply<INLINE>(th2, tau, E);
      R.multiply(E);
    }
  } else {
    for (int l = l0; l < l1; ++l) {
      double th[4];
      euler_angles(terms, params, fc, tk, l, dt, wr, method, th);
      Mat<N> E;
      Exponentiator<N>::template apply<INLINE>(th, tau, E);
      R.multiply(E);
    }
  }
}

// Below this tau most angles take the squarings (2 pi 2 kHz over 50 ns, the
// sensing drive's largest, from tau = 16 on none), and the integrator of a
// compiled field has them in its loop: 31.5 us at tau = 0 and 88 at 12 against
// 35 and 93 with the call.  Not the others: the interpreter gains 2 us of 44 and
// 101, a chained run nothing, and every copy of a compiled field's loop is
// compiled at run time.
constexpr int kOftenSquared = 16;

// Operator of one interval (rows a1-a9) computed by S = 2^sl cooperating
// lanes: slice s integrates fine steps [s L / S, (s + 1) L / S) and the
// partial products are combined in order with wave shuffles; the full
// U_k (frame exit applied) ends up in the lane with s == 0.  Every lane of
// the wave must call this (the shuffles need the whole wave).
template <int N, bool FULL = false, bool OFTEN = false, class Terms>
__device__ __forceinline__ void interval_operator(const Terms& terms, const double* __restrict__ params,
                                                  double t_start, double Dt, double dt, int L,
                                                  int tau, int frame, int method, int64_t k, int s,
                                                  int sl, bool active, Mat<N>& U, double* tk_out) {
  static_assert(!FULL || N == 3, "the full basis is spin-1 only");
  Running<N, FULL> R;
  R.clear();
  double tk = 0.0, wr = 0.0;
  if (active) {
    constexpr int C = FULL ? kFullComps : 4;
    double fc[C];
    field_constant(terms, params, fc);
    interval_setup(terms, params, fc, t_start, Dt, k, frame, &tk, &wr);
    const int l0 = (int)(((int64_t)s * L) >> sl);
    const int l1 = (int)(((int64_t)(s + 1) * L) >> sl);
    if constexpr (FULL) {
      if (method == 0) {
        NodeRotations rot;
        if (wr != 0.0) rot.start(wr, l0, dt);
        for (int l = l0; l < l1; ++l) {
          double th1[kFullComps], th2[kFullComps];
          cf4_angles_full(terms, params, fc, tk, l, dt, wr, rot, th1, th2);
          if (wr != 0.0) rot.advance();
          Mat<3> E;
          exp_full(th1, tau, E);
          R.multiply(E);
          exp_full(th2, tau, E);
          R.multiply(E);
        }
      } else {
        for (int l = l0; l < l1; ++l) {
          double th[kFullComps];
          euler_angles_full(terms, params, fc, tk, l, dt, wr, method, th);
          Mat<3> E;
          exp_full(th, tau, E);
          R.multiply(E);
        }
      }
    } else if (OFTEN && N == 3 && tau < kOftenSquared) {
      integrate_slice<N, true>(terms, params, fc, tk, l0, l1, dt, wr, tau, method, R);
    } else {
      integrate_slice<N, false>(terms, params, fc, tk, l0, l1, dt, wr, tau, method, R);
    }
  }
  R.whole(U);
  for (int d = 1; d < (1 << sl); d <<= 1) {
    const Mat<N> o = shfl_down_mat<N>(U, d);
    if ((s & (2 * d - 1)) == 0) premultiply<N>(o, U);
  }
  if (active && s == 0) exit_frame<N>(wr, Dt, U);
  *tk_out = tk;
}

// Time grid, outputs and options of one simulation's integrator launch
// (everything but the field source): lane g of the grid has slice g mod 2^sl
// of interval g >> sl.
struct IntervalGrid {
  const double* params;  // the simulation's parameter vector (may be null)
  double* U;             // [K][N][N] complex
  double* time;          // [K] interval start times, or null
  double t_start;
  double dt_out;         // Dt
  double dt;             // Dt / L
  int64_t K;
  int32_t L;
  int32_t tau;
  int32_t frame;
  int32_t method;
  int32_t sl;            // log2 of the lane-slices per interval
  int32_t full;          // spin-1 in the full su(3) basis
};

// Lane body of the single-simulation integrator: one lane per (interval k,
// slice s), the S = 2^sl slices of an interval in consecutive lanes of one
// wave; the whole wave must call it.  `terms` is any field source
// field_at accepts.
template <int N, class Terms>
__device__ __forceinline__ void integrate_lanes(const Terms& terms, const IntervalGrid& g) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int sl = g.sl;
  const int64_t k = gid >> sl;
  const int s = (int)(gid & ((1 << sl) - 1));
  const bool active = k < g.K;
  Mat<N> U;
  double tk;
  bool done = false;
  if constexpr (N == 3 && has_full_basis<Terms>::value) {
    if (g.full) {
      interval_operator<3, true>(terms, g.params, g.t_start, g.dt_out, g.dt, g.L, g.tau, g.frame,
                                 g.method, k, s, sl, active, U, &tk);
      done = true;
    }
  }
  if (!done)
    interval_operator<N, false, !has_full_basis<Terms>::value>(
        terms, g.params, g.t_start, g.dt_out, g.dt, g.L, g.tau, g.frame, g.method, k, s, sl, active,
        U, &tk);
  if (active && s == 0) {
    store_mat<N>(g.U + (size_t)k * 2 * N * N, U);
    if (g.time) g.time[k] = tk;
  }
}

}  // namespace mss
